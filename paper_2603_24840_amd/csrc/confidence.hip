// Trace confidence (Sec. 3 "Trace Confidence"): token confidence H_t = -sum_j log P_t(j) and its trace-level
// aggregates (trace mean, sliding-window means, their minimum and the mean of the lowest share of windows).
//
// With z_t = W h_t and lse_t = logsumexp_j z_t[j] (an output of the fused log-prob kernel):
//     H_t = V * lse_t - sum_j z_t[j] = V * lse_t - <h_t, sum_j W_j>
// so beside the log-prob pass the token confidence costs one column sum of the LM head (HBM stream over W,
// once per weight version) and one dot product per token (HBM stream over the hidden states): no second
// [T, V] contraction.  The aggregates run one workgroup per trace in fp64.
#include "common.h"

namespace {

constexpr int kColThreads = 256;
constexpr int kColRows = 256;      // LM-head rows per workgroup of the column-sum pass
constexpr int kColUnroll = 8;
constexpr int kColUnits = 256;     // compute units

// partial[b][c] = sum of W[v][c] over the `rows` rows v of block b.  Thread -> (row group, 16-byte chunk of a row): `lanes` chunks (a power of
// two) and 256 / lanes groups, which take every so many-th row and meet in LDS in a fixed order.  Bound by HBM where all units have loads
// in flight, and by the unit with most rows (colsum_plan).  us a confidence call, one group a block of 256 rows with all chunks in turn -> now:
// 128,256 x 256 36 -> 15, x 512 40 -> 25, 32,000 x 2048 42 -> 26, x 4096 76 -> 47, 151,936 x 2048 107 -> 99, x 4096 241 -> 196 (6.4 TB/s).
// Error against 64 bits of 7.1e-8 in both.
__global__ __launch_bounds__(kColThreads) void colsum_partial_kernel(
    const u32x4* __restrict__ lm_head, int V, int d_vec, int lanes, int rows, float* __restrict__ partial) {
    __shared__ float4 sums[2][kColThreads];
    const int groups = kColThreads / lanes, group = threadIdx.x / lanes, lane = threadIdx.x % lanes;
    const int v0 = blockIdx.x * rows, n = V - v0 < rows ? V - v0 : rows;
    float* out = partial + static_cast<int64_t>(blockIdx.x) * d_vec * 8;
    const int c = blockIdx.y * lanes + lane;
    float acc[2][8] = {};            // two sums a column: none of more than 200 rows, where one had 256
    if (c < d_vec) {
        const u32x4* p = lm_head + static_cast<int64_t>(v0) * d_vec + c;
        for (int r = group; r < n; r += kColUnroll * groups) {
            u32x4 x[kColUnroll];
#pragma unroll
            for (int u = 0; u < kColUnroll; ++u)
                x[u] = r + u * groups < n ? __builtin_nontemporal_load(p + static_cast<int64_t>(r + u * groups) * d_vec)
                                          : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int u = 0; u < kColUnroll; ++u) {
                float* a = acc[u & 1];
                a[0] += bf16_lo(x[u].x); a[1] += bf16_hi(x[u].x);
                a[2] += bf16_lo(x[u].y); a[3] += bf16_hi(x[u].y);
                a[4] += bf16_lo(x[u].z); a[5] += bf16_hi(x[u].z);
                a[6] += bf16_lo(x[u].w); a[7] += bf16_hi(x[u].w);
            }
        }
    }
    for (int k = 0; k < 8; ++k) acc[0][k] += acc[1][k];
    float4 lo = make_float4(acc[0][0], acc[0][1], acc[0][2], acc[0][3]), hi = make_float4(acc[0][4], acc[0][5], acc[0][6], acc[0][7]);
    if (groups > 1) {
        sums[0][threadIdx.x] = lo;
        sums[1][threadIdx.x] = hi;
        __syncthreads();
        for (int g = 1; group == 0 && g < groups; ++g) {
            const float4 a = sums[0][g * lanes + lane], b = sums[1][g * lanes + lane];
            lo.x += a.x; lo.y += a.y; lo.z += a.z; lo.w += a.w;
            hi.x += b.x; hi.y += b.y; hi.z += b.z; hi.w += b.w;
        }
    }
    if (group == 0 && c < d_vec) {
        *reinterpret_cast<float4*>(out + c * 8) = lo;
        *reinterpret_cast<float4*>(out + c * 8 + 4) = hi;
    }
}

constexpr int kConfThreads = 512;
constexpr int kConfWaves = kConfThreads / ARROL_WAVE;
constexpr int kConfUnroll = 4;

// one wavefront per token: conf[t] = V * lse[t] - <h_t, colsum>.  CH > 0: lane l owns chunks c*64 + l (c < CH) of
// every row and keeps its slice of colsum in registers (d <= 512*CH); CH == 0: colsum staged in LDS, any d.
template <int CH>
__global__ __launch_bounds__(kConfThreads) void token_conf_kernel(
    const u32x4* __restrict__ hidden, const float* __restrict__ colsum, const float* __restrict__ lse,
    int64_t T, int V, int d_vec, float* __restrict__ conf) {
    extern __shared__ float c_lds[];
    const int lane = threadIdx.x & (ARROL_WAVE - 1);
    const int wave = threadIdx.x / ARROL_WAVE;
    constexpr int NR = CH > 0 ? CH : 1;
    float4 wa[NR], wb[NR];
    if (CH > 0) {
#pragma unroll
        for (int c = 0; c < NR; ++c) {
            const int v = c * ARROL_WAVE + lane;
            wa[c] = v < d_vec ? *reinterpret_cast<const float4*>(colsum + v * 8) : make_float4(0.f, 0.f, 0.f, 0.f);
            wb[c] = v < d_vec ? *reinterpret_cast<const float4*>(colsum + v * 8 + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    } else {
        for (int i = threadIdx.x; i < d_vec * 8; i += kConfThreads) c_lds[i] = colsum[i];
        __syncthreads();
    }
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kConfWaves;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kConfWaves + wave; t < T; t += stride) {
        const u32x4* p = hidden + t * d_vec;
        float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f, acc3 = 0.f;
        if (CH > 0) {
            u32x4 x[NR];
#pragma unroll
            for (int c = 0; c < NR; ++c) {
                const int v = c * ARROL_WAVE + lane;
                x[c] = v < d_vec ? __builtin_nontemporal_load(p + v) : u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int c = 0; c < NR; ++c) {
                acc0 = fmaf(bf16_lo(x[c].x), wa[c].x, acc0); acc1 = fmaf(bf16_hi(x[c].x), wa[c].y, acc1);
                acc2 = fmaf(bf16_lo(x[c].y), wa[c].z, acc2); acc3 = fmaf(bf16_hi(x[c].y), wa[c].w, acc3);
                acc0 = fmaf(bf16_lo(x[c].z), wb[c].x, acc0); acc1 = fmaf(bf16_hi(x[c].z), wb[c].y, acc1);
                acc2 = fmaf(bf16_lo(x[c].w), wb[c].z, acc2); acc3 = fmaf(bf16_hi(x[c].w), wb[c].w, acc3);
            }
        } else {
            for (int v0 = 0; v0 < d_vec; v0 += kConfUnroll * ARROL_WAVE) {
                u32x4 x[kConfUnroll];
#pragma unroll
                for (int u = 0; u < kConfUnroll; ++u) {
                    const int v = v0 + u * ARROL_WAVE + lane;
                    x[u] = v < d_vec ? __builtin_nontemporal_load(p + v) : u32x4{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int u = 0; u < kConfUnroll; ++u) {
                    const int v = v0 + u * ARROL_WAVE + lane;
                    if (v < d_vec) {
                        const float4 la = *reinterpret_cast<const float4*>(c_lds + v * 8);
                        const float4 lb = *reinterpret_cast<const float4*>(c_lds + v * 8 + 4);
                        acc0 = fmaf(bf16_lo(x[u].x), la.x, acc0); acc1 = fmaf(bf16_hi(x[u].x), la.y, acc1);
                        acc2 = fmaf(bf16_lo(x[u].y), la.z, acc2); acc3 = fmaf(bf16_hi(x[u].y), la.w, acc3);
                        acc0 = fmaf(bf16_lo(x[u].z), lb.x, acc0); acc1 = fmaf(bf16_hi(x[u].z), lb.y, acc1);
                        acc2 = fmaf(bf16_lo(x[u].w), lb.z, acc2); acc3 = fmaf(bf16_hi(x[u].w), lb.w, acc3);
                    }
                }
            }
        }
        const float dot = wave_sum_f32((acc0 + acc1) + (acc2 + acc3));
        if (lane == 0)
            conf[t] = static_cast<float>(static_cast<double>(V) * static_cast<double>(lse[t]) -
                                         static_cast<double>(dot));
    }
}

// ---- trace-level aggregates -------------------------------------------------------------------------------
// Bound by the chain of steps of one workgroup (a trace is a few thousand numbers), so the steps are few: the prefix sums
// of a trace that one round of the scan covers stay in LDS, every thread keeps up to ITEMS window keys in registers, and the m-th
// smallest key is found eight bits at a time from LDS counts, from the highest bit in which the keys differ on and only
// until one key is left (two or three rounds for windows that differ; deciding one bit a round took 64 rounds with a
// barrier each).  256 traces of 256 to 2,048 tokens, window 1,024: 46.1 -> 8.7 us under the profiler (7.3 in a graph of
// such calls, the measure of the launch's rule).
constexpr int kAggBits = 8;        // bits of the key decided per round
constexpr int kAggBins = 1 << kAggBits;

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) { return wave_reduce(v, [](uint64_t a, uint64_t b) { return a > b ? a : b; }); }
// order-preserving map of a double onto unsigned integers
__device__ __forceinline__ uint64_t key_of(double v) {
    const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double value_of(uint64_t k) {
    const uint64_t b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
    return __longlong_as_double(static_cast<int64_t>(b));
}

// One workgroup per trace.  prefix and keys are per-trace slices of the workspace: trace i owns entries
// [cu[i] + i, cu[i+1] + i + 1) of each (L+1 prefix sums, up to L window keys); they are used only as far as the LDS array
// and the registers do not reach.
// ITEMS: tokens per thread and round of the scan, and window keys per thread in registers.
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void trace_conf_kernel(
    const float* __restrict__ conf, const int64_t* __restrict__ cu, int64_t T, int window, int bottom_percent,
    double* __restrict__ prefix_all, uint64_t* __restrict__ keys_all, double* __restrict__ mean_out,
    double* __restrict__ min_out, double* __restrict__ bottom_out) {
    constexpr int kWaves = THREADS / ARROL_WAVE;
    constexpr int64_t kRound = static_cast<int64_t>(ITEMS) * THREADS;   // tokens whose prefix sums fit the LDS array, windows whose keys are in registers
    __shared__ double sh_prefix[kRound + 1];
    __shared__ double sh_d[2][kWaves];
    __shared__ unsigned long long sh_u[2][kWaves];
    __shared__ unsigned long long sh_bin[3][kAggBins];
    __shared__ unsigned long long sh_key;
    const int i = blockIdx.x;
    const int lane = threadIdx.x & (ARROL_WAVE - 1), wave = threadIdx.x / ARROL_WAVE;
    int64_t lo = cu[i], hi = cu[i + 1];
    lo = lo < 0 ? 0 : (lo > T ? T : lo);
    hi = hi < lo ? lo : (hi > T ? T : hi);
    const int64_t L = hi - lo;
    const double nan = __longlong_as_double(0x7ff8000000000000ll);
    if (L == 0) {
        if (threadIdx.x == 0) { mean_out[i] = nan; min_out[i] = nan; bottom_out[i] = nan; }
        return;
    }
    const bool in_lds = L <= kRound;                    // uniform over the workgroup
    double* prefix = prefix_all + lo + i;
    uint64_t* keys = keys_all + lo + i;
    const float* x = conf + lo;
    const auto prefix_at = [&](int64_t k) { return in_lds ? sh_prefix[k] : prefix[k]; };

    // ---- inclusive prefix sums in fp64, ITEMS * THREADS tokens per round
    double carry = 0.0;
    if (threadIdx.x == 0) { if (in_lds) sh_prefix[0] = 0.0; else prefix[0] = 0.0; }
    for (int b = threadIdx.x; b < 3 * kAggBins; b += THREADS) sh_bin[b / kAggBins][b % kAggBins] = 0;
    int par = 0;
    for (int64_t base = 0; base < L; base += THREADS * ITEMS, par ^= 1) {
        const int64_t first = base + static_cast<int64_t>(threadIdx.x) * ITEMS;
        double v[ITEMS];
        double run = 0.0;
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            run += first + k < L ? static_cast<double>(x[first + k]) : 0.0;
            v[k] = run;
        }
        const double incl = wave_scan_sum(run);
        if (lane == ARROL_WAVE - 1) sh_d[par][wave] = incl;
        __syncthreads();
        double before = carry, total = carry;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const double s = sh_d[par][w];
            if (w < wave) before += s;
            total += s;
        }
        const double offset = before + (incl - run);
#pragma unroll
        for (int k = 0; k < ITEMS; ++k)
            if (first + k < L) {
                if (in_lds) sh_prefix[first + k + 1] = offset + v[k];
                else prefix[first + k + 1] = offset + v[k];
            }
        carry = total;
    }
    __syncthreads();                                    // the prefix sums of this trace are complete and visible

    // ---- window means, their keys, the smallest and the largest
    const int64_t w_eff = window < L ? window : L;
    const int64_t n_w = L - w_eff + 1;
    const double inv_w = 1.0 / static_cast<double>(w_eff);
    const auto window_key = [&](int64_t k) { return key_of((prefix_at(k + w_eff) - prefix_at(k)) * inv_w); };
    uint64_t held[ITEMS];
    uint64_t kmin = ~0ull, kmax = 0ull;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t k = threadIdx.x + static_cast<int64_t>(j) * THREADS;
        held[j] = k < n_w ? window_key(k) : 0ull;
        if (k < n_w) {
            kmin = held[j] < kmin ? held[j] : kmin;
            kmax = held[j] > kmax ? held[j] : kmax;
        }
    }
    for (int64_t k = kRound + threadIdx.x; k < n_w; k += THREADS) {   // written and read back by the same thread
        const uint64_t key = window_key(k);
        keys[k] = key;
        kmin = key < kmin ? key : kmin;
        kmax = key > kmax ? key : kmax;
    }
    const auto each_key = [&](auto&& f) {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (threadIdx.x + static_cast<int64_t>(j) * THREADS < n_w) f(held[j]);
        for (int64_t k = kRound + threadIdx.x; k < n_w; k += THREADS) f(keys[k]);
    };
    kmin = wave_min_u64(kmin);
    kmax = wave_max_u64(kmax);
    if (lane == 0) { sh_u[0][wave] = kmin; sh_u[1][wave] = kmax; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        kmin = sh_u[0][w] < kmin ? sh_u[0][w] : kmin;
        kmax = sh_u[1][w] > kmax ? sh_u[1][w] : kmax;
    }

    // ---- X = the m-th smallest window key.  The bits above `open` are decided and the same in X and in every key that
    // still counts; `rank` is X's place among those.  The counts rotate over three arrays, so that one barrier a round is
    // enough: the array of the next round was last read in the round before the one that ended with the last barrier.
    const int64_t m_low = (n_w * bottom_percent + 99) / 100 < 1 ? 1 : (n_w * bottom_percent + 99) / 100;
    uint64_t X = kmin;
    int open = m_low == 1 || kmin == kmax ? 0 : 64 - __clzll(static_cast<long long>(kmin ^ kmax));
    if (open > 0) X = open == 64 ? 0ull : (kmin >> open) << open;
    uint64_t rank = static_cast<uint64_t>(m_low);
    for (int round = 0; open > 0; ++round) {
        const int bits = open < kAggBits ? open : kAggBits, shift = open - bits;
        unsigned long long* bin = sh_bin[round % 3];
        if (round > 0)                                  // the first round's successor is still zero
            for (int b = threadIdx.x; b < kAggBins; b += THREADS) sh_bin[(round + 1) % 3][b] = 0;
        each_key([&](uint64_t key) {
            if (open == 64 || ((key ^ X) >> open) == 0)
                atomicAdd(&bin[(key >> shift) & ((1u << bits) - 1u)], 1ull);
        });
        __syncthreads();
        // every wavefront finds the bin of the rank for itself: four bins per lane, inclusive scan over the lanes
        constexpr int kPer = kAggBins / ARROL_WAVE;
        uint64_t c[kPer], own = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) { c[k] = bin[lane * kPer + k]; own += c[k]; }
        const uint64_t incl = wave_scan_sum(own);
        uint64_t below = incl - own;
        const int src = __builtin_ctzll(__ballot(incl >= rank));   // counts sum up to at least the rank: some lane has it
        int digit = lane * kPer;
        uint64_t in_bin = c[0];
#pragma unroll
        for (int k = 1; k < kPer; ++k)
            if (below + in_bin < rank) { below += in_bin; in_bin = c[k]; digit = lane * kPer + k; }
        digit = wave_bcast(digit, src);
        rank -= static_cast<uint64_t>(wave_bcast(static_cast<int64_t>(below), src));
        const uint64_t left = static_cast<uint64_t>(wave_bcast(static_cast<int64_t>(in_bin), src));
        X |= static_cast<uint64_t>(digit) << shift;
        open = shift;
        if (left == 1 && open > 0) {                    // one key has these leading bits: its owner publishes it
            each_key([&](uint64_t key) { if (((key ^ X) >> open) == 0) sh_key = key; });
            __syncthreads();
            X = sh_key;
            open = 0;
        }
    }
    // sum of the values below X, then as many copies of X as are still missing
    double s_low = 0.0;
    int64_t c_low = 0;
    each_key([&](uint64_t key) { if (key < X) { s_low += value_of(key); ++c_low; } });
    s_low = wave_sum_f64(s_low);
    c_low = wave_sum_i64(c_low);
    __syncthreads();                                    // sh_u still held the smallest and largest keys
    if (lane == 0) { sh_d[0][wave] = s_low; sh_u[0][wave] = static_cast<unsigned long long>(c_low); }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        unsigned long long c = 0;
        for (int w = 0; w < kWaves; ++w) { s += sh_d[0][w]; c += sh_u[0][w]; }
        s += static_cast<double>(m_low - static_cast<int64_t>(c)) * value_of(X);
        mean_out[i] = prefix_at(L) / static_cast<double>(L);
        min_out[i] = value_of(kmin);
        bottom_out[i] = s / static_cast<double>(m_low);
    }
}

int colsum_blocks(int V) { return (V + kColRows - 1) / kColRows; }

// The column sum's workgroups: blocks of `rows` rows x slabs of `lanes` chunks.
struct ColsumPlan { int lanes, slabs, rows, blocks; };

ColsumPlan colsum_plan(int V, int d_vec) {
    ColsumPlan p = {kColThreads, 1, kColRows, colsum_blocks(V)};
    // Chunks of a row side by side: as many as a row has, but 64 to 128 rather than 256 where there would be fewer than 1.5 workgroups
    // to a compute unit (32,000 x 4096: 55 us a call with 64, 84 with 256; 80,000 x 2048 64 with 128, 65 with 256; but of more workgroups
    // whole kilobytes read side by side count: 128,256 x 2048 83 with 256, 88 with 128, 101 with 64).
    while (p.lanes > 1 && p.lanes / 2 >= d_vec) p.lanes /= 2;
    while (p.lanes > ARROL_WAVE && static_cast<int64_t>(p.blocks) * ((d_vec + p.lanes - 1) / p.lanes) < 384) p.lanes /= 2;
    p.slabs = (d_vec + p.lanes - 1) / p.lanes;
    // As many workgroups to each unit, from two on: what would be a last round for some of them goes into longer blocks.  us a call with
    // blocks of 256 rows and so: 100,000 x 3072 110 -> 100, x 3584 130 -> 116, x 4096 145 -> 128, x 8192 299 -> 277, 140,000 x 1024
    // 56 -> 49, x 4096 192 -> 184; of 2.9 rounds 96,000 x 4096 128 -> 121, but 64,000 x 5120 108 -> 113; of 1.96 rounds 128,256 x 2048 83 -> 86:
    // a unit needs two workgroups.  A last slab of less than half its chunks does not count: 128,256 x 2056 89 -> 92 if it did.
    const int rest = d_vec % p.lanes, full = p.slabs - (p.slabs > 1 && rest && 2 * rest < p.lanes ? 1 : 0);
    const int rounds = static_cast<int>(static_cast<int64_t>(p.blocks) * full / kColUnits);
    if (rounds >= 2) {
        const int blocks = static_cast<int>(static_cast<int64_t>(rounds) * kColUnits / full);
        p.rows = (V - 1) / blocks + 1;
        p.blocks = (V - 1) / p.rows + 1;
    }
    return p;
}

}  // namespace

extern "C" size_t arrol_token_confidence_workspace_bytes(int32_t V, int32_t d) {
    if (V < 1 || d < 8) return 0;
    return (static_cast<size_t>(colsum_blocks(V)) + 1) * static_cast<size_t>(d) * sizeof(float);
}

extern "C" int arrol_token_confidence(const void* hidden, const void* lm_head, const float* lse, int64_t T,
                                      int32_t V, int32_t d, float* conf_out, void* workspace,
                                      size_t workspace_bytes, void* stream) {
    if (T < 0 || V < 1 || d < 8 || (d & 7) || d > 16384) return ARROL_EINVAL;
    if (T == 0) return ARROL_OK;
    if (!hidden || !lm_head || !lse || !conf_out || !arrol_aligned16(hidden) || !arrol_aligned16(lm_head))
        return ARROL_EINVAL;
    if (!workspace || !arrol_aligned16(workspace) || workspace_bytes < arrol_token_confidence_workspace_bytes(V, d))
        return ARROL_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const ColsumPlan p = colsum_plan(V, d / 8);
    float* colsum = static_cast<float*>(workspace);
    float* partial = colsum + d;
    arrol_launch(colsum_partial_kernel, dim3(p.blocks, p.slabs), dim3(kColThreads), 0, st,
                       static_cast<const u32x4*>(lm_head), V, d / 8, p.lanes, p.rows, partial);
    arrol_launch(reduce_rows_f32_kernel<32>, dim3((d + 31) / 32), dim3(1024), 0, st, partial, p.blocks,
                       static_cast<int64_t>(d), static_cast<int64_t>(d), 1.f, colsum);
    const int64_t blocks_needed = (T + kConfWaves - 1) / kConfWaves;
    const int grid = static_cast<int>(blocks_needed < 256 * 8 ? blocks_needed : 256 * 8);
    const u32x4* h = static_cast<const u32x4*>(hidden);
    const int chunks = (d / 8 + ARROL_WAVE - 1) / ARROL_WAVE;
#define ARROL_CONF(CH, LDS) arrol_launch(token_conf_kernel<CH>, dim3(grid), dim3(kConfThreads), LDS, st, h, colsum, lse, T, V, d / 8, conf_out)
    if (chunks <= 1) ARROL_CONF(1, 0);
    else if (chunks <= 2) ARROL_CONF(2, 0);
    else if (chunks <= 4) ARROL_CONF(4, 0);
    else if (chunks <= 8) ARROL_CONF(8, 0);
    else {
        static arrol_device_flags lds_ok;
        if (!arrol_allow_lds(token_conf_kernel<0>, static_cast<int>(sizeof(float) * 16384), lds_ok)) return ARROL_EHIP;
        ARROL_CONF(0, sizeof(float) * d);
    }
#undef ARROL_CONF
    return arrol_launch_status();
}

extern "C" size_t arrol_trace_confidence_workspace_bytes(int64_t T, int32_t n_seq) {
    if (T < 0 || n_seq < 0) return 0;
    return 2 * (static_cast<size_t>(T) + static_cast<size_t>(n_seq)) * sizeof(double);
}

extern "C" int arrol_trace_confidence(const float* conf, const int64_t* cu_seqlens, int64_t T, int32_t n_seq,
                                      int32_t window, int32_t bottom_percent, double* mean_out,
                                      double* min_out, double* bottom_out, void* workspace,
                                      size_t workspace_bytes, void* stream) {
    if (T < 0 || n_seq < 0 || window < 1 || bottom_percent < 1 || bottom_percent > 100) return ARROL_EINVAL;
    if (n_seq == 0) return ARROL_OK;
    if (!cu_seqlens || !mean_out || !min_out || !bottom_out || (T > 0 && !conf)) return ARROL_EINVAL;
    if (!workspace || !arrol_aligned16(workspace) || workspace_bytes < arrol_trace_confidence_workspace_bytes(T, n_seq))
        return ARROL_EWORKSPACE;
    double* prefix = static_cast<double*>(workspace);
    uint64_t* keys = reinterpret_cast<uint64_t*>(prefix + T + n_seq);
    // Threads by the mean length and the number of traces: a wide workgroup needs fewer rounds for a long trace, but its
    // barriers and scans cost more and fewer of them fit a compute unit.  256 / 512 / 1,024 threads: 256 traces of 64 to 512
    // tokens 4.7 / 5.1 / 6.9 us, of 256 to 2,048 8.2 / 7.3 / 9.6, of 512 to 4,096 16.2 / 11.9 / 11.3, of 4,096 to 8,192
    // 39.9 / 26.0 / 21.1; 1,024 traces of 256 to 2,048 12.2 / 12.6 / 29.9.
    const int64_t mean = T / n_seq;
#define ARROL_TRACE(N, ITEMS) arrol_launch(trace_conf_kernel<N, ITEMS>, dim3(n_seq), dim3(N), 0, static_cast<hipStream_t>(stream), conf, cu_seqlens, T, window, bottom_percent, prefix, keys, mean_out, min_out, bottom_out)
    if (mean > 4096 && n_seq <= 256) ARROL_TRACE(1024, 4);
    else if (mean > 512 && n_seq <= 512) ARROL_TRACE(512, 4);
    else ARROL_TRACE(256, 4);
#undef ARROL_TRACE
    return arrol_launch_status();
}
