// Shared host/device helpers for the ARRoL HIP library (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include <tuple>
#include <type_traits>
#include <utility>
#include "arrol.h"

#define ARROL_WAVE 64

// 16-byte native vector (the nontemporal builtins need a native vector, not HIP's uint4 class)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Kernel launches go through arrol_launch(), which keeps the runtime's OWN return value of each launch
// (hipLaunchKernel) in a per-thread slot: an error some earlier, unrelated HIP call of the caller left in
// the thread's sticky error state is neither reported as a failure of this library nor cleared from the
// caller's view.  arrol_launch_failed() peeks at the slot between the launches of one entry point;
// arrol_launch_status() turns it into the entry point's return code and empties it.
inline hipError_t& arrol_launch_error_slot() {
    static thread_local hipError_t err = hipSuccess;
    return err;
}
template <class Tuple, size_t... I>
static inline hipError_t arrol_launch_packed(const void* fn, dim3 grid, dim3 block, size_t lds, hipStream_t st,
                                             Tuple& vals, std::index_sequence<I...>) {
    void* ptrs[] = {static_cast<void*>(&std::get<I>(vals))..., nullptr};
    return hipLaunchKernel(fn, grid, block, ptrs, lds, st);
}
template <class... KArgs, class... Args>
static inline void arrol_launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t st,
                                Args&&... args) {
    static_assert(sizeof...(KArgs) == sizeof...(Args), "one argument per kernel parameter");
    hipError_t& slot = arrol_launch_error_slot();
    if (slot != hipSuccess) return;   // an earlier launch of this entry point failed: enqueue nothing more
    std::tuple<std::remove_cv_t<KArgs>...> vals(static_cast<KArgs>(args)...);
    slot = arrol_launch_packed(reinterpret_cast<const void*>(kernel), grid, block, lds, st, vals,
                               std::index_sequence_for<KArgs...>{});
}
static inline bool arrol_launch_failed() { return arrol_launch_error_slot() != hipSuccess; }
static inline int arrol_launch_status() {
    hipError_t& slot = arrol_launch_error_slot();
    const bool ok = slot == hipSuccess;
    slot = hipSuccess;
    return ok ? ARROL_OK : ARROL_EHIP;
}

// Raises a kernel's dynamic-LDS limit once per device (function attributes are per device); `bytes` is the
// most the kernel is ever launched with.  Safe to call from several host threads.
typedef std::atomic<bool> arrol_device_flags[64];
template <class K>
static inline bool arrol_allow_lds(K kernel, int bytes, arrol_device_flags& done) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
    if (done[dev].load(std::memory_order_acquire)) return true;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
        return false;
    done[dev].store(true, std::memory_order_release);
    return true;
}

static inline bool arrol_aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// The value of lane `src` (the same in every lane) in all lanes, by way of a scalar register.
__device__ __forceinline__ int wave_bcast(int v, int src) { return __builtin_amdgcn_readlane(v, __builtin_amdgcn_readfirstlane(src)); }
__device__ __forceinline__ int64_t wave_bcast(int64_t v, int src) {
    const uint32_t lo = static_cast<uint32_t>(wave_bcast(static_cast<int>(v & 0xffffffffll), src));
    return (static_cast<int64_t>(wave_bcast(static_cast<int>(v >> 32), src)) << 32) | lo;
}

// Between the LDS writes of one wavefront's lanes and the reads of its other lanes: the hardware completes one wavefront's
// LDS accesses in order, the fences hold the compiler to it (the barrier alone does not order memory for it).  No instructions.
__device__ __forceinline__ void wave_lds_exchange() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- wave-wide reductions: the butterfly 32, 16, 8, 4, 2, 1 without the LDS --------------------------------------
// __shfl_xor goes through the LDS pipe (some 100 cycles of latency a step, twice for 64 bits); here steps 32 and 16 are
// the lane-swapping moves of gfx950 and the others DPP moves, a few cycles each.  wave_pair_* returns a value and its
// partner's - steps 32 and 16 in the order (lower lane's, upper lane's), the others (own, partner's) - so the operation has
// to be commutative; the pairs and so the results are the shuffle butterfly's, bit for bit.  Rotations by 4 within a row of 16 stand for xor 4 because after
// step 8 the row repeats every 8 lanes (every 4 after step 4 for the rotation by 2).  All 64 lanes must be active.
struct wave_pair32 { uint32_t a, b; };
template <int STEP>
__device__ __forceinline__ wave_pair32 wave_pair_u32(uint32_t v) {
    static_assert(STEP == 32 || STEP == 16 || STEP == 8 || STEP == 4 || STEP == 2 || STEP == 1, "butterfly step");
    if constexpr (STEP == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return {r[0], r[1]};
    } else if constexpr (STEP == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return {r[0], r[1]};
    } else {
        constexpr int ctrl = STEP == 8 ? 0x128 : STEP == 4 ? 0x124 : STEP == 2 ? 0x4E : 0xB1;   // row_ror:8, :4, quad_perm
        return {v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), ctrl, 0xF, 0xF, false))};
    }
}
template <int STEP, class T, class Op>
__device__ __forceinline__ T wave_step(T v, Op op) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "32- or 64-bit values");
    if constexpr (sizeof(T) == 4) {
        const wave_pair32 p = wave_pair_u32<STEP>(__builtin_bit_cast(uint32_t, v));
        return op(__builtin_bit_cast(T, p.a), __builtin_bit_cast(T, p.b));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const wave_pair32 lo = wave_pair_u32<STEP>(static_cast<uint32_t>(u)), hi = wave_pair_u32<STEP>(static_cast<uint32_t>(u >> 32));
        return op(__builtin_bit_cast(T, (static_cast<uint64_t>(hi.a) << 32) | lo.a), __builtin_bit_cast(T, (static_cast<uint64_t>(hi.b) << 32) | lo.b));
    }
}
template <class T, class Op>
__device__ __forceinline__ T wave_reduce(T v, Op op) {
    v = wave_step<32>(v, op);
    v = wave_step<16>(v, op);
    v = wave_step<8>(v, op);
    v = wave_step<4>(v, op);
    v = wave_step<2>(v, op);
    return wave_step<1>(v, op);
}
__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) { return wave_reduce(v, [](int64_t a, int64_t b) { return a + b; }); }
__device__ __forceinline__ int64_t wave_min_i64(int64_t v) { return wave_reduce(v, [](int64_t a, int64_t b) { return a < b ? a : b; }); }
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v) { return wave_reduce(v, [](uint64_t a, uint64_t b) { return a < b ? a : b; }); }
__device__ __forceinline__ int64_t wave_max_i64(int64_t v) { return wave_reduce(v, [](int64_t a, int64_t b) { return a > b ? a : b; }); }
__device__ __forceinline__ float wave_sum_f32(float v) { return wave_reduce(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ double wave_sum_f64(double v) { return wave_reduce(v, [](double a, double b) { return a + b; }); }

// Inclusive prefix sum over the lanes, four steps within each row of 16 and two that hand a row's total on (DPP moves, as
// above; 0 comes in where there is no lower lane).  All 64 lanes must be active.
template <int CTRL, int ROWS, class T>
__device__ __forceinline__ T wave_scan_step(T v) {
    static_assert(sizeof(T) == 8, "64-bit values");
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(u), CTRL, ROWS, 0xF, true));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), CTRL, ROWS, 0xF, true));
    return v + __builtin_bit_cast(T, (static_cast<uint64_t>(hi) << 32) | lo);
}
template <class T>
__device__ __forceinline__ T wave_scan_sum(T v) {
    v = wave_scan_step<0x111, 0xF>(v);   // row_shr:1, :2, :4, :8
    v = wave_scan_step<0x112, 0xF>(v);
    v = wave_scan_step<0x114, 0xF>(v);
    v = wave_scan_step<0x118, 0xF>(v);
    v = wave_scan_step<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    return wave_scan_step<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }
// fp32 -> bf16, round to nearest even (NaN stays a quiet NaN)
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

// Sum over p of partial[p*stride + col]: 32 columns (threadIdx.x & 31) x G groups of rows (threadIdx.x >> 5), workgroups of
// 32*G.  Every group adds its rows in index order, eight at a time, the eight and the groups by a fixed tree:
// bit-reproducible.  Bound by the latency of its loads, so eight are in flight per thread (501 x 2048: 20.3 us with 8 groups
// and one load at a time, 5.1 us with 32 groups and eight).  The sum is valid where threadIdx.x < 32; red: [G][32].
template <int N>
__device__ __forceinline__ float tree_sum(const float* x) {
    if constexpr (N == 1) return x[0];
    else return tree_sum<N / 2>(x) + tree_sum<N / 2>(x + N / 2);
}
template <int G>
__device__ __forceinline__ float reduce_rows_column(const float* __restrict__ partial, int n_partials, int64_t stride,
                                                    int64_t col, bool valid, float (*red)[32]) {
    constexpr int kInFlight = 8;
    const int cx = threadIdx.x & 31, ry = threadIdx.x >> 5;
    float s = 0.f;
    if (valid)
        for (int p = ry; p < n_partials; p += kInFlight * G) {
            float x[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {   // past the end the group's first row again, so that no load waits on a branch
                const int q = p + u * G;
                x[u] = partial[static_cast<int64_t>(q < n_partials ? q : p) * stride + col];
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) x[u] = p + u * G < n_partials ? x[u] : 0.f;
            s += tree_sum<kInFlight>(x);
        }
    red[ry][cx] = s;
    __syncthreads();
    float t[G];
    if (ry != 0) return 0.f;
#pragma unroll
    for (int k = 0; k < G; ++k) t[k] = red[k][cx];
    return tree_sum<G>(t);
}

// out[c] = scale * sum_p partial[p*stride + c] for c < width; n_partials == 0 writes zeros.
// Launch with (width + 31) / 32 workgroups of 32*G.
template <int G>
__global__ __launch_bounds__(32 * G) void reduce_rows_f32_kernel(const float* __restrict__ partial, int n_partials,
                                                                 int64_t stride, int64_t width, float scale,
                                                                 float* __restrict__ out) {
    __shared__ float red[G][32];
    const int64_t col = static_cast<int64_t>(blockIdx.x) * 32 + (threadIdx.x & 31);
    const float t = reduce_rows_column<G>(partial, n_partials, stride, col, col < width, red);
    if (threadIdx.x < 32 && col < width) out[col] = t * scale;
}
