// arrol_score_mlp: quality head as a 2-layer MLP (Sec. 4.2 allows a small two-layer MLP as the
// rollout quality head), followed by the sigmoid normalisation (App. A.4):
//     a = relu(W1 h + b1),  s = <w2, a> + b2,  q = sigmoid(s)
// One fused kernel: bf16 MFMA for W1 h (transposed, A^T = W1 H^T, so that a lane's accumulator values
// belong to one rollout and the reduction over hidden units is lane-local), bias + ReLU + the dot with w2
// on the accumulators in registers; the [N, m] activations never reach memory.
// Tile: 256 hidden units x 128 rollouts per workgroup pass, 4 wavefronts, each 2 x (32 units) x 128
// rollouts; K chunks of 64 in XOR-swizzled 16-byte chunks, loaded global -> LDS directly into three stages
// when d is a multiple of 64, else staged global -> registers -> LDS (two stages).
//
// arrol_score_mlp_grad: cross-entropy training gradient of the same head (Sec. 4.2, Sec. 4.3 (iii)).  The same
// tile loop runs in two more modes:
//   delta   (d not a multiple of 64; else the blocked forward passes keep the activations, which mlp_score_delta_kernel or, of
//           larger batches, mlp_delta_kernel reads) recomputes the pre-activations and, instead of the w2 dot, writes delta^T[u][i] =
//           r_i * w2[u] * [pre > 0] (bf16, unit-major) and the per-workgroup sums for dL/dw2 and dL/db1;
//   wgrad   the contraction over rollouts dL/dW1 = delta^T . H as the same "A rows x B rows over a shared
//           contiguous K" product, with A = delta^T [m, N] and B = H^T [d, N] (transposed once into the
//           workspace), fp32 tile stores, optionally split over K with partial slabs added in a fixed order.
#include "common.h"
#include "ring_nt.h"

namespace {

using ring_nt::bf16x8;
using ring_nt::f32x4;
typedef float f32x16 __attribute__((ext_vector_type(16)));   // 32x32x16 accumulators of the tile kernel

constexpr int kThreads = 256;
constexpr int BU = 256;   // hidden units per pass
constexpr int BR = 128;   // rollouts per workgroup
constexpr int BK = 64;
constexpr int TU = 2;     // 32-unit blocks per wave (unit rows c*128 + wave*32 + ...)
constexpr int TR = 4;     // 32-rollout blocks per wave
constexpr int kStageBytes = (BU + BR) * BK * 2;
constexpr int kLdsBytes = 2 * kStageBytes;          // register-staged path: two stages
constexpr int kRingStages = 3;                      // direct-to-LDS path: three stages, two of them in flight
constexpr int kRingLdsBytes = kRingStages * kStageBytes;
constexpr int kRingLoadsA = BU / 8 / 4;             // load instructions (8 rows x 128 bytes) per wave and stage
constexpr int kRingLoadsB = BR / 8 / 4;
constexpr int kRingLoads = kRingLoadsA + kRingLoadsB;
constexpr int kPassA = BU * (BK / 8) / kThreads;   // 16-byte loads per thread for the W1 tile
constexpr int kPassB = BR * (BK / 8) / kThreads;

__device__ __forceinline__ int chunk_offset(int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); }

enum MlpMode { kForward = 0, kDelta = 1, kWgrad = 2, kForwardKeep = 3 };   // kForwardKeep: ring kernel only

// The tile loop multiplies A rows (w1, a_stride elements apart, m of them) with B rows (hidden, n_rows of
// them) over a contiguous K extent of d elements.
struct MlpArgs {
    const uint16_t* hidden; int64_t row_stride; const int64_t* row_index;
    const uint16_t* w1; int64_t a_stride; const float* b1; const float* w2; float b2;
    int n_rows, d, m;
    float* score_out; float* prob_out;
    // delta mode
    const float* resid;          // [n_rows] r_i = (q_i - y_i) / N
    uint16_t* delta_t;           // [m][delta_stride] bf16
    uint16_t* delta_lo;          // NULL, or [m][delta_stride] bf16: bf16(delta - float(delta_t)), the second term
    int64_t delta_stride;
    float* unit_partial;         // [gridDim.x][2][m]: sums over the workgroup's rollouts for dL/dw2, dL/db1
    // wgrad mode: blockIdx.y = K split, blockIdx.z = group of 256 A rows
    float* c_out;                // [gridDim.y][m][c_stride] fp32
    int64_t c_stride;
    int kc_per_split;            // K chunks (of 64) per split
};

template <int N>
__device__ __forceinline__ void mlp_wait_vmcnt() {  // s_waitcnt vmcnt(N) only (gfx9 encoding: bits 3:0 and 15:14), N <= 63
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Units past the last one fill up a block; they repeat its row of W1, so their pre-activations may be infinite, and infinity
// times their zero weight would be NaN.  With this bias they are -inf, or NaN, and fmaxf(pre, 0) is 0 for both.  (Loads from
// a clamped address: one that may be skipped is waited for before the next.)
__device__ __forceinline__ float unit_bias(const float* b1, int u, bool live) {
    const float b = b1 ? b1[live ? u : 0] : 0.f;
    return live ? b : -__builtin_inff();
}
__device__ __forceinline__ float unit_weight(const float* w2, int u, bool live) {
    const float w = w2[live ? u : 0];
    return live ? w : 0.f;
}

// RING = false: any d (multiple of 8), K chunks staged global -> registers -> LDS, one chunk ahead.
// RING = true (d a multiple of 64): K chunks go global -> LDS directly (no staging registers) into three
// stages, two chunks ahead, so that a workgroup that is alone on its CU (few rollouts) still hides the
// memory latency.  One instruction moves 8 tile rows x 128 bytes; lane l writes physical chunk l%8 of row
// l/8, and fetches the logical chunk that the XOR swizzle stores there.
template <int MODE, bool RING>
__global__ __launch_bounds__(kThreads) void score_mlp_kernel(MlpArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    typedef __attribute__((address_space(3))) void* lds_ptr_t;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, lh = lane >> 5;
    const int row0 = blockIdx.x * BR;

    // staging geometry: thread -> (tile row tid/8 (+32 per pass), 16-byte chunk tid%8)
    const int ld_c = tid & 7, ld_r = tid >> 3;
    const int ld_lds = chunk_offset(ld_r, ld_c);
    const uint16_t* h_row[kPassB];
#pragma unroll
    for (int p = 0; p < kPassB; ++p) {
        int r = row0 + ld_r + p * 32;
        r = r < a.n_rows ? r : a.n_rows - 1;
        const int64_t src = a.row_index ? a.row_index[r] : r;
        h_row[p] = a.hidden + src * a.row_stride;
    }
    const int n_kc_all = (a.d + BK - 1) / BK;
    // forward / delta: every K chunk, every group of 256 units in turn; wgrad: one K split, one group
    const int kc0 = MODE == kWgrad ? static_cast<int>(blockIdx.y) * a.kc_per_split : 0;
    const int kc1 = MODE == kWgrad ? (kc0 + a.kc_per_split < n_kc_all ? kc0 + a.kc_per_split : n_kc_all) : n_kc_all;
    const int n_kc = kc1 - kc0;
    const int g0 = MODE == kWgrad ? static_cast<int>(blockIdx.z) : 0;
    const int n_groups = MODE == kWgrad ? 1 : (a.m + BU - 1) / BU;
    const int total_it = n_groups * n_kc;

    float resid[TR] = {0.f, 0.f, 0.f, 0.f};
    if (MODE == kDelta) {
#pragma unroll
        for (int j = 0; j < TR; ++j) {
            const int r = row0 + j * 32 + l31;
            resid[j] = r < a.n_rows ? a.resid[r] : 0.f;
        }
    }

    constexpr int NSTAGE_REGS = RING ? 1 : kPassA + kPassB;
    uint4 stage[NSTAGE_REGS];
    int ld_g = g0, ld_kc = 0;
    auto issue_loads = [&]() {
        const int k = (kc0 + ld_kc) * BK + ld_c * 8;
        const bool k_ok = k < a.d;
#pragma unroll
        for (int p = 0; p < kPassA; ++p) {
            int u = ld_g * BU + ld_r + p * 32;
            u = u < a.m ? u : a.m - 1;
            stage[p] = k_ok ? *reinterpret_cast<const uint4*>(a.w1 + static_cast<int64_t>(u) * a.a_stride + k) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < kPassB; ++p)
            stage[kPassA + p] = k_ok ? *reinterpret_cast<const uint4*>(h_row[p] + k) : make_uint4(0, 0, 0, 0);
        if (++ld_kc == n_kc) { ld_kc = 0; ++ld_g; }
    };
    auto store_stage = [&](int buf) {
        unsigned char* sa = lds + buf * kStageBytes + ld_lds;
        unsigned char* sb = sa + BU * BK * 2;
#pragma unroll
        for (int p = 0; p < kPassA; ++p) *reinterpret_cast<uint4*>(sa + p * 32 * 128) = stage[p];
#pragma unroll
        for (int p = 0; p < kPassB; ++p) *reinterpret_cast<uint4*>(sb + p * 32 * 128) = stage[kPassA + p];
    };

    // ---- direct-to-LDS loader (RING) ---------------------------------------------------------------------
    // wave w fetches A groups w*8 .. w*8+7 and B groups w*4 .. w*4+3 of every stage (a group = 8 tile rows)
    const int rl_row = lane >> 3;                                     // row inside the group
    constexpr int NPTR_A = RING ? kRingLoadsA : 1, NPTR_B = RING ? kRingLoadsB : 1;
    const uint16_t* ring_a[NPTR_A];                                   // per lane: row base + logical chunk, k = 0
    const uint16_t* ring_b[NPTR_B];
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((lds_ptr_t)lds));
    auto ring_point_a = [&](int grp) {                                // A rows of unit group `grp`
#pragma unroll
        for (int q = 0; q < NPTR_A; ++q) {
            const int r = (wave * kRingLoadsA + q) * 8 + rl_row;      // tile row 0 .. 255
            int u = grp * BU + r;
            u = u < a.m ? u : a.m - 1;
            const int logical = (lane & 7) ^ ((r >> 1) & 7);
            ring_a[q] = a.w1 + static_cast<int64_t>(u) * a.a_stride + logical * 8;
        }
    };
    if (RING) {
#pragma unroll
        for (int q = 0; q < NPTR_B; ++q) {
            const int r = (wave * kRingLoadsB + q) * 8 + rl_row;      // tile row 0 .. 127
            int row = row0 + r;
            row = row < a.n_rows ? row : a.n_rows - 1;
            const int64_t src = a.row_index ? a.row_index[row] : row;
            const int logical = (lane & 7) ^ ((r >> 1) & 7);
            ring_b[q] = a.hidden + src * a.row_stride + logical * 8;
        }
        ring_point_a(g0);
    }
    int ring_g = g0, ring_kc = 0, ring_buf = 0;
    auto ring_issue = [&]() {                                         // the next chunk -> stage ring_buf
        const int64_t k = static_cast<int64_t>(kc0 + ring_kc) * BK;
        const unsigned dst_a = lds0 + ring_buf * kStageBytes + wave * kRingLoadsA * 1024;
        const unsigned dst_b = lds0 + ring_buf * kStageBytes + BU * BK * 2 + wave * kRingLoadsB * 1024;
#pragma unroll
        for (int q = 0; q < NPTR_A; ++q) {
            const uint16_t* src = ring_a[q] + k;
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(dst_a + q * 1024) : "memory");
        }
#pragma unroll
        for (int q = 0; q < NPTR_B; ++q) {
            const uint16_t* src = ring_b[q] + k;
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(dst_b + q * 1024) : "memory");
        }
        ring_buf = ring_buf + 1 == kRingStages ? 0 : ring_buf + 1;
        if (++ring_kc == n_kc) {
            ring_kc = 0;
            ++ring_g;
            ring_point_a(ring_g);        // rows of the next unit group (clamped: harmless past the last group)
        }
    };

    f32x16 acc[TU][TR];
#pragma unroll
    for (int c = 0; c < TU; ++c)
#pragma unroll
        for (int j = 0; j < TR; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[c][j][v] = 0.f;
    float part[TR] = {0.f, 0.f, 0.f, 0.f};   // this lane's share of s for rollout row0 + j*32 + l31

    const int swz = (l31 >> 1) & 7;
    if (RING) {
        ring_issue();
        if (total_it > 1) ring_issue();
    } else {
        issue_loads();
        store_stage(0);
        __syncthreads();
    }
    int g = g0, kc = 0, buf = 0;
    for (int it = 0; it < total_it; ++it) {
        const bool more = it + 1 < total_it;
        if (RING) {
            // this wave's share of chunk `it` has landed (only the chunk after it may still be in flight) ...
            if (more) mlp_wait_vmcnt<kRingLoads>(); else mlp_wait_vmcnt<0>();
            // ... then so has everybody's, and nobody still reads the stage of chunk it-1, which chunk it+2 refills
            __syncthreads();
            if (it + 2 < total_it) ring_issue();
        } else if (more) {
            issue_loads();
        }
        const unsigned char* sa = lds + buf * kStageBytes;
        const unsigned char* sb = sa + BU * BK * 2;
        buf = buf + 1 == (RING ? kRingStages : 2) ? 0 : buf + 1;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            const int coff = ((kk * 2 + lh) ^ swz) << 4;
            bf16x8 fa[TU], fb[TR];
#pragma unroll
            for (int c = 0; c < TU; ++c)
                fa[c] = *reinterpret_cast<const bf16x8*>(sa + (c * 128 + wave * 32 + l31) * 128 + coff);
#pragma unroll
            for (int j = 0; j < TR; ++j)
                fb[j] = *reinterpret_cast<const bf16x8*>(sb + (j * 32 + l31) * 128 + coff);
#pragma unroll
            for (int c = 0; c < TU; ++c)
#pragma unroll
                for (int j = 0; j < TR; ++j)
                    acc[c][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[c], fb[j], acc[c][j], 0, 0, 0);
        }
        if (!RING) {
            if (more) store_stage(buf);
            __syncthreads();
        }
        if (++kc == n_kc) {
            // acc[c][j][v] belongs to A row (unit) g*BU + c*128 + wave*32 + (v/4)*8 + lh*4 + v%4 and B row
            // (rollout) row0 + j*32 + l31
#pragma unroll
            for (int c = 0; c < TU; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int u = g * BU + c * 128 + wave * 32 + (v >> 2) * 8 + lh * 4 + (v & 3);
                    const bool live = u < a.m;
                    if (MODE == kWgrad) {
                        float* crow = a.c_out + (static_cast<int64_t>(blockIdx.y) * a.m + u) * a.c_stride;
#pragma unroll
                        for (int j = 0; j < TR; ++j) {
                            const int col = row0 + j * 32 + l31;
                            if (live && col < a.n_rows) crow[col] = acc[c][j][v];
                            acc[c][j][v] = 0.f;
                        }
                    } else {
                        const float bias = unit_bias(a.b1, u, live);
                        const float w = unit_weight(a.w2, u, live);
                        if (MODE == kForward) {
#pragma unroll
                            for (int j = 0; j < TR; ++j) {
                                part[j] = fmaf(fmaxf(acc[c][j][v] + bias, 0.f), w, part[j]);
                                acc[c][j][v] = 0.f;
                            }
                        } else {
                            float gw = 0.f, gb = 0.f;
                            uint16_t* drow = a.delta_t + static_cast<int64_t>(live ? u : 0) * a.delta_stride + row0 + l31;
#pragma unroll
                            for (int j = 0; j < TR; ++j) {
                                const float pre = acc[c][j][v] + bias;
                                const float dl = pre > 0.f ? resid[j] * w : 0.f;
                                gw = fmaf(resid[j], fmaxf(pre, 0.f), gw);
                                gb += dl;
                                if (live) {
                                    const uint16_t hi = f32_to_bf16_rne(dl);
                                    drow[j * 32] = hi;
                                    if (a.delta_lo) (a.delta_lo + (drow - a.delta_t))[j * 32] = f32_to_bf16_rne(dl - bf16_lo(hi));
                                }
                                acc[c][j][v] = 0.f;
                            }
                            // sum over the 32 rollout lanes of this half-wave (both halves run the same steps)
#pragma unroll
                            for (int msk = 16; msk >= 1; msk >>= 1) {
                                gw += __shfl_xor(gw, msk, ARROL_WAVE);
                                gb += __shfl_xor(gb, msk, ARROL_WAVE);
                            }
                            if (live && l31 == 0) {
                                float* up = a.unit_partial + static_cast<int64_t>(blockIdx.x) * 2 * a.m;
                                up[u] = gw;
                                up[a.m + u] = gb;
                            }
                        }
                    }
                }
            kc = 0;
            ++g;
        }
    }
    if (MODE != kForward) return;
    // lane halves hold different units of the same rollout; then the four waves
#pragma unroll
    for (int j = 0; j < TR; ++j) part[j] += __shfl_xor(part[j], 32, ARROL_WAVE);
    if (RING) __syncthreads();                    // every wave has finished reading the last stage
    float* red = reinterpret_cast<float*>(lds);   // [4 waves][BR]
    if (lh == 0) {
#pragma unroll
        for (int j = 0; j < TR; ++j) red[wave * BR + j * 32 + l31] = part[j];
    }
    __syncthreads();
    if (tid < BR && row0 + tid < a.n_rows) {
        const float s = red[tid] + red[BR + tid] + red[2 * BR + tid] + red[3 * BR + tid] + a.b2;
        float q;
        if (s >= 0.f) {
            q = 1.f / (1.f + expf(-s));
        } else {
            const float e = expf(s);
            q = e / (1.f + e);
        }
        if (a.score_out) a.score_out[row0 + tid] = s;
        a.prob_out[row0 + tid] = q;
    }
}

// ---------------------------------------------------------------------------------------------------------
// Batches below the ring kernels' size, and gathered rows of any number: BM units x BN rollouts per workgroup of KG groups of
// WM x WN wavefronts, K64 steps of both operands direct to LDS, NS stages deep, one barrier per stage.  What bounds it is a
// step's chain of barrier, fragment reads and MFMAs while few workgroups run, and each workgroup's (BM + BN) rows of K
// through its compute unit's L1 path when the chip is full; pick_forward takes the block that makes the sum smallest.
// Where a compute unit has no second workgroup to fill the chain, the groups do: group g takes the steps g, g + KG, ... of the
// block, a stage is KG steps, and the groups' sums are added in the LDS at the end.  512 x 2048 x 512 with 32 x 32 blocks: 7.7 us
// with one group, 6.9 with four; 1,024 x 2048 x 512 with 64 x 64: 10.9, 10.4 with two; 4,096 x 4096 x 512 with 128 x 64: 27.1, 25.7.
// (Of 4,096 x 2048 x 512's 16.7 us the steps take 9.6, the activations kept for the gradient 2.2, an empty launch 2.2.  Under the profiler it
// is 16.5, with the loads alone 14.6, without them 15.4, with neither, barriers and all else in place, 10.0: the two are even.)
// Stage layout: 16-byte chunk c of row r at position c ^ (r & 6) of its 128-byte row, which keeps the fragment reads
// (lane -> row lane % 16, chunk lane / 16) free of bank conflicts by the serving rule given in ring_nt.h.
template <int BM_, int BN_, int WM_, int WN_, int KG_, int NS_>
struct MidTile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KG = KG_, NS = NS_;
    static constexpr int GW = WM * WN, NT = KG * GW * ARROL_WAVE;                  // wavefronts per group
    static constexpr int TI = BM / WM / 16, TJ = BN / WN / 16;
    static constexpr int SUB_BYTES = (BM + BN) * 128, STAGE_BYTES = KG * SUB_BYTES;
    static constexpr int LA = BM / 8 / GW, LB = BN / 8 / GW, LOADS = LA + LB;      // load instructions (8 rows) per wave and stage
    static constexpr int RED_BYTES = KG > 1 ? KG * BM * BN * 4 : 0, PART_BYTES = KG * WM * BN * 4;
    static constexpr int LDS_BYTES = NS * STAGE_BYTES > RED_BYTES + PART_BYTES ? NS * STAGE_BYTES : RED_BYTES + PART_BYTES;
    static_assert(LDS_BYTES <= 163840 && BM % (8 * GW) == 0 && BN % (8 * GW) == 0, "tile");
};

struct MlpMidArgs {
    const uint16_t* hidden; int64_t row_stride; const int64_t* row_index;
    const uint16_t* w1; const float* b1; const float* w2;
    int n_rows, d, m;
    float* partial;                          // [gridDim.y][n_rows]
    float* act_t; int64_t act_stride;        // NULL, or relu(pre) for the gradient call, [m][act_stride]
};

template <class C>
__global__ __launch_bounds__(C::NT, 2) void mlp_mid_kernel(MlpMidArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    typedef __attribute__((address_space(3))) void* lds_ptr_t;
    constexpr int BM = C::BM, BN = C::BN, NS = C::NS, TI = C::TI, TJ = C::TJ, KG = C::KG, GW = C::GW;
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / GW, wq = wave % GW, wm = wq / C::WN, wn = wq % C::WN;
    const int u0 = blockIdx.y * BM, r0 = blockIdx.x * BN;
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((lds_ptr_t)lds)) + kg * C::SUB_BYTES;
    const int n_k64 = a.d / 64, n_st = (n_k64 + KG - 1) / KG;
    // loader: lane -> (row lane/8 of an 8-row group, position lane%8); rows past the end repeat the last one
    const uint16_t* src[C::LOADS];
#pragma unroll
    for (int q = 0; q < C::LOADS; ++q) {
        const bool is_a = q < C::LA;
        const int r = (is_a ? wq * C::LA + q : wq * C::LB + q - C::LA) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ (r & 6);
        if (is_a) {
            const int u = u0 + r < a.m ? u0 + r : a.m - 1;
            src[q] = a.w1 + static_cast<int64_t>(u) * a.d + c * 8;
        } else {
            const int row = r0 + r < a.n_rows ? r0 + r : a.n_rows - 1;
            src[q] = a.hidden + (a.row_index ? a.row_index[row] : row) * a.row_stride + c * 8;
        }
    }
    int ld_k = kg < n_k64 ? kg : 0, ld_slot = 0;
    auto issue = [&]() {                     // the next stage; past the last one its lines again
        const int64_t k = static_cast<int64_t>(ld_k) * 64;
        const unsigned dst = lds0 + ld_slot * C::STAGE_BYTES;
#pragma unroll
        for (int q = 0; q < C::LOADS; ++q) {
            const unsigned to = dst + (q < C::LA ? (wq * C::LA + q) * 1024 : BM * 128 + (wq * C::LB + q - C::LA) * 1024);
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src[q] + k), "s"(to) : "memory");
        }
        ld_slot = ld_slot + 1 == NS ? 0 : ld_slot + 1;
        if (ld_k + KG < n_k64) ld_k += KG;
    };
    f32x4 acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int a_off = kg * C::SUB_BYTES + (wm * (BM / C::WM) + l15) * 128, b_off = kg * C::SUB_BYTES + (BM + wn * (BN / C::WN) + l15) * 128;
    const int pos[2] = {(lq ^ (l15 & 6)) * 16, ((lq + 4) ^ (l15 & 6)) * 16};
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue();
    // bias and weight of the units this lane finishes, fetched here: at the end their latency would be bare, and once for
    // every store of an activation
    float bias[TI][4], wgt[TI][4];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int u = u0 + wm * (BM / C::WM) + i * 16 + lq * 4 + v;
            bias[i][v] = unit_bias(a.b1, u, u < a.m);
            wgt[i][v] = unit_weight(a.w2, u, u < a.m);
        }
    int slot = 0;
    for (int s = 0; s < n_st; ++s) {
        // this stage has landed (the NS - 2 after it may fly), for every wavefront, and all have read the one before
        mlp_wait_vmcnt<(NS - 2) * C::LOADS>();
        __syncthreads();
        issue();
        const unsigned char* st = lds + slot * C::STAGE_BYTES;
        slot = slot + 1 == NS ? 0 : slot + 1;
        if (KG > 1 && s * KG + kg >= n_k64) continue;
        bf16x8 fa[2][TI], fb[2][TJ];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int i = 0; i < TI; ++i) fa[h][i] = *reinterpret_cast<const bf16x8*>(st + a_off + i * 2048 + pos[h]);
#pragma unroll
            for (int j = 0; j < TJ; ++j) fb[h][j] = *reinterpret_cast<const bf16x8*>(st + b_off + j * 2048 + pos[h]);
        }
        __builtin_amdgcn_sched_barrier(0);   // all reads first
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][i], fb[h][j], acc[i][j], 0, 0, 0);
    }
    // the groups' sums: block (i, j) of a wavefront position is finished by the group (i TJ + j) % KG, added in group order
    mlp_wait_vmcnt<0>();
    __syncthreads();                         // every stage has been read and every load into LDS has landed
    f32x4* red = reinterpret_cast<f32x4*>(lds);   // [group][position][TI TJ][lane]
    if (KG > 1) {
#pragma unroll
        for (int b = 0; b < TI * TJ; ++b) red[(wave * TI * TJ + b) * 64 + lane] = acc[b / TJ][b % TJ];
        __syncthreads();
    }
    float part[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) part[j] = 0.f;
#pragma unroll
    for (int b = 0; b < TI * TJ; ++b) {
        if (b % KG != kg) continue;
        const int i = b / TJ, j = b % TJ;
        f32x4 s = acc[i][j];
        if (KG > 1) s = red[(wq * TI * TJ + b) * 64 + lane];
#pragma unroll
        for (int g = 1; g < KG; ++g) s += red[((g * GW + wq) * TI * TJ + b) * 64 + lane];
        // s[v]: unit wm * BM/WM + i*16 + lq*4 + v, rollout wn * BN/WN + j*16 + l15 of the block
        const int col = r0 + wn * (BN / C::WN) + j * 16 + l15;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int u = u0 + wm * (BM / C::WM) + i * 16 + lq * 4 + v;
            const float act = fmaxf(s[v] + bias[i][v], 0.f);
            part[j] = fmaf(act, wgt[i][v], part[j]);
            if (a.act_t && u < a.m && col < a.n_rows) a.act_t[static_cast<int64_t>(u) * a.act_stride + col] = act;
        }
    }
    float* sums = reinterpret_cast<float*>(lds + C::RED_BYTES);   // [group][wm][BN]
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        part[j] += __shfl_xor(part[j], 16, ARROL_WAVE);
        part[j] += __shfl_xor(part[j], 32, ARROL_WAVE);
        if (lq == 0) sums[(kg * C::WM + wm) * BN + wn * (BN / C::WN) + j * 16 + l15] = part[j];
    }
    __syncthreads();
    if (tid < BN && r0 + tid < a.n_rows) {
        float s = sums[tid];
#pragma unroll
        for (int q = 1; q < KG * C::WM; ++q) s += sums[q * BN + tid];
        a.partial[static_cast<int64_t>(blockIdx.y) * a.n_rows + r0 + tid] = s;
    }
}

template <class C>
int launch_mlp_mid(const MlpMidArgs& a, hipStream_t st) {
    static arrol_device_flags ok;
    if (!arrol_allow_lds(&mlp_mid_kernel<C>, C::LDS_BYTES, ok)) return ARROL_EHIP;
    arrol_launch(mlp_mid_kernel<C>, dim3((a.n_rows + C::BN - 1) / C::BN, (a.m + C::BM - 1) / C::BM), dim3(C::NT), C::LDS_BYTES, st, a);
    return ARROL_OK;
}

// The unit blocks' partial scores of rollout i in index order, eight loads in flight.
__device__ __forceinline__ float sum_unit_blocks(const float* __restrict__ partial, int n_ub, int n_rows, int i) {
    float s = 0.f;
    for (int ub0 = 0; ub0 < n_ub; ub0 += 8) {
        float x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) x[q] = ub0 + q < n_ub ? partial[static_cast<int64_t>(ub0 + q) * n_rows + i] : 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) s += x[q];
    }
    return s;
}

__global__ __launch_bounds__(256) void score_mlp_finish_kernel(const float* __restrict__ partial, int n_ub,
                                                                     int n_rows, float b2, float* __restrict__ score_out,
                                                                     float* __restrict__ prob_out) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n_rows) return;
    const float s = sum_unit_blocks(partial, n_ub, n_rows, i) + b2;
    float q;
    if (s >= 0.f) {
        q = 1.f / (1.f + expf(-s));
    } else {
        const float e = expf(s);
        q = e / (1.f + e);
    }
    if (score_out) score_out[i] = s;
    prob_out[i] = q;
}

// ---------------------------------------------------------------------------------------------------------
// Large batches (d a multiple of 64, rows addressed without row_index; pick_forward): the contractions on the 8-wavefront
// direct-to-LDS ring pipeline of ring_nt.h (v_mfma_f32_16x16x32_bf16), one 256 x 256 accumulator tile per workgroup:
// grid = (blocks of 256 B rows, tiles of 256 A rows, K splits).
//   forward  A = W1 [m, d], B = hidden [N, d]: bias + ReLU + w2 dot per rollout (lane-local over the
//            units), partial scores [unit tile][rollout] to the workspace, summed by the finish kernel;
//            for the gradient call the same pass also keeps the activations a = relu(pre) in fp32, unit-major
//            (the accumulator's own layout: 16 lanes = 16 consecutive rollouts), so that nothing is recomputed:
//            delta^T = r w2 [a > 0] and the per-unit sums are then one streaming pass (mlp_delta_kernel);
//   wgrad    A = delta^T [m, n_pad], B = the hidden states themselves, [N, d] = K-major (ring_nt's TN form, no
//            transposed copy), over K = rollouts (split): fp32 tile stores.
using RingCfg = ring_nt::RingTile<256, 256, 2, 4>;

struct MlpRingArgs {
    const uint16_t* a; unsigned a_stride;   // A rows (bytes between rows), a_rows of them
    const uint16_t* b; unsigned b_stride;   // B rows, b_rows of them; wgrad: k-rows of b_rows values, b_k_rows of them
    int a_rows, b_rows, b_k_rows, n_k64, k64_per_split;
    const float* b1; const float* w2;
    float* partial;              // forward: [gridDim.y][b_rows]
    float* act_t; int64_t act_stride;       // forward for the gradient: relu(pre), [a_rows][act_stride] fp32
    float* c_out; int64_t c_stride;         // wgrad: [gridDim.z][a_rows][c_stride]
};

template <int MODE>
__global__ __launch_bounds__(RingCfg::NT) void mlp_ring_kernel(MlpRingArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    using C = RingCfg;
    constexpr int BM = C::BM, BN = C::BN, TI = C::TI, TJ = C::TJ;
    const int tb = blockIdx.x, vt = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int l15 = lane & 15, lq = lane >> 4;
    const int k64_lo = MODE == kWgrad ? static_cast<int>(blockIdx.z) * a.k64_per_split : 0;
    const int k64_hi = MODE == kWgrad ? (k64_lo + a.k64_per_split < a.n_k64 ? k64_lo + a.k64_per_split : a.n_k64) : a.n_k64;

    ring_nt::Walk w;
    w.a_base = reinterpret_cast<const char*>(a.a) + static_cast<int64_t>(vt) * BM * a.a_stride + static_cast<int64_t>(k64_lo) * 128;
    w.b_base = MODE == kWgrad
                   ? reinterpret_cast<const char*>(a.b) + static_cast<int64_t>(k64_lo) * 64 * a.b_stride + static_cast<int64_t>(tb) * BN * 2
                   : reinterpret_cast<const char*>(a.b) + static_cast<int64_t>(tb) * BN * a.b_stride + static_cast<int64_t>(k64_lo) * 128;
    w.a_stride = a.a_stride;
    w.b_stride = a.b_stride;
    w.a_rows = a.a_rows - vt * BM;
    w.b_rows = a.b_rows - tb * BN < BN ? a.b_rows - tb * BN : BN;
    w.n_k64 = k64_hi > k64_lo ? k64_hi - k64_lo : 0;
    w.b_k_rows = a.b_k_rows - k64_lo * 64;

    const int unit0 = vt * BM + wm * (BM / C::WM);           // first A row of this wavefront
    const int row0 = tb * BN + wn * (BN / C::WN);            // first B row of this wavefront
    float part[TJ] = {0.f, 0.f, 0.f, 0.f};
    ring_nt::f32x4 acc[TI][TJ];
    ring_nt::walk<C, MODE == kWgrad>(w, lds, acc);
    {
        // acc[i][j][v]: A row unit0 + i*16 + lq*4 + v, B row row0 + j*16 + l15
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int u = unit0 + i * 16 + lq * 4 + v;
                const bool live = u < a.a_rows;
                if (MODE == kWgrad) {
                    float* crow = a.c_out + (static_cast<int64_t>(blockIdx.z) * a.a_rows + u) * a.c_stride;
#pragma unroll
                    for (int j = 0; j < TJ; ++j) {
                        const int col = row0 + j * 16 + l15;
                        if (live && col < a.b_rows) crow[col] = acc[i][j][v];
                    }
                } else {
                    const float bias = unit_bias(a.b1, u, live);
                    const float wu = unit_weight(a.w2, u, live);
                    float* arow = MODE == kForwardKeep ? a.act_t + static_cast<int64_t>(live ? u : 0) * a.act_stride : nullptr;
#pragma unroll
                    for (int j = 0; j < TJ; ++j) {
                        const float act = fmaxf(acc[i][j][v] + bias, 0.f);
                        part[j] = fmaf(act, wu, part[j]);
                        if (MODE == kForwardKeep) {
                            const int col = row0 + j * 16 + l15;
                            if (live && col < a.b_rows) arow[col] = act;
                        }
                    }
                }
            }
    }
    if (MODE == kWgrad) return;
    // the four lane quarters and the two wavefront rows hold different units of the same rollouts
    float* red = reinterpret_cast<float*>(lds);   // [WM][BN]
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        part[j] += __shfl_xor(part[j], 16, ARROL_WAVE);
        part[j] += __shfl_xor(part[j], 32, ARROL_WAVE);
    }
    if (lq == 0) {
#pragma unroll
        for (int j = 0; j < TJ; ++j) red[wm * BN + wn * (BN / C::WN) + j * 16 + l15] = part[j];
    }
    __syncthreads();
    for (int col = tid; col < BN; col += C::NT) {
        const int r = tb * BN + col;
        if (r < a.b_rows) a.partial[static_cast<int64_t>(vt) * a.b_rows + r] = red[col] + red[BN + col];
    }
}

template <int MODE>
int launch_mlp_ring(const MlpRingArgs& a, dim3 grid, hipStream_t st) {
    static arrol_device_flags ok;
    if (!arrol_allow_lds(&mlp_ring_kernel<MODE>, RingCfg::LDS_BYTES, ok)) return ARROL_EHIP;
    arrol_launch(mlp_ring_kernel<MODE>, grid, dim3(RingCfg::NT), RingCfg::LDS_BYTES, st, a);
    return ARROL_OK;
}

// ---------------------------------------------------------------------------------------------------------
// What mlp_score_delta_kernel left to be added up (unit_partial NULL: nothing): [n_blocks][2][m] parts of dL/dw2 and dL/db1,
// [2][n_blocks] of the loss and dL/db2.  Added in block order, whoever does it.
struct MlpSums {
    const float* unit_partial; const float* block_sums;
    int n_blocks, n_rows, m;
    float* grad_w2; float* grad_b1; float* loss; float* grad_b2;      // the last two may be NULL
};
// In 64 bits: up to 40 parts one after the other cost a bit in 32 (16,384 x 1024 x 64: dL/dw2 9.5e-8 off, 2.7e-8 so).
__device__ __forceinline__ void finish_unit(const MlpSums& f, int u, int which) {
    const float* part = f.unit_partial + static_cast<int64_t>(which) * f.m + u;
    double sum = 0.0;
    for (int b0 = 0; b0 < f.n_blocks; b0 += 8) {
        float x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)     // past the end the first one again, so that no load waits on a branch
            x[q] = part[static_cast<int64_t>(b0 + q < f.n_blocks ? b0 + q : b0) * 2 * f.m];
#pragma unroll
        for (int q = 0; q < 8; ++q) sum += b0 + q < f.n_blocks ? x[q] : 0.f;
    }
    (which ? f.grad_b1 : f.grad_w2)[u] = static_cast<float>(sum);
}
__device__ __forceinline__ void finish_loss(const MlpSums& f, int lane) {   // by a whole wavefront
    double l = 0.0, r = 0.0;
    for (int b = lane; b < f.n_blocks; b += ARROL_WAVE) { l += f.block_sums[b]; r += f.block_sums[f.n_blocks + b]; }
    if (f.n_blocks > 1) {
        l = wave_sum_f64(l);
        r = wave_sum_f64(r);
    }
    if (lane == 0 && f.loss) *f.loss = static_cast<float>(l) / static_cast<float>(f.n_rows);
    if (lane == 0 && f.grad_b2) *f.grad_b2 = static_cast<float>(r);
}
__global__ __launch_bounds__(256) void mlp_sums_kernel(MlpSums f) {   // where mlp_wgrad_mid_kernel does not do it
    const int v = blockIdx.x * 256 + threadIdx.x;
    if (v < f.m) finish_unit(f, v, blockIdx.y);
    if (v < ARROL_WAVE && blockIdx.y == 0) finish_loss(f, v);
}

// dL/dW1 = delta^T . H over the rollouts where the ring form has too few 256 x 256 tiles to fill the chip: BM rows of
// delta^T x 64 columns per workgroup of KG groups of WM x WN wavefronts.  Group g takes the K64 steps g, g + KG, ... of the
// tile, so two wavefronts share a SIMD and a barrier stands for KG steps, and the groups' sums are added in the LDS at the
// end.  Where tiles are too few, K (rollouts) is also split over gridDim.z into slabs.  Of two-term deltas both terms of a K64
// step come next to each other, into the same sums, while its hidden states are near: one term's steps behind the other's read
// them from memory twice (131,072 x 1024 x 128, whole call: 298 us, so 251).  The hidden states are read in place: a step holds
// 64 rollouts x 128 bytes, and the B fragments come out through the transposing LDS read (lane layout as in ring_nt.h).  16-byte
// chunk c of rollout row r sits at position c ^ 2 ((r / 2) % 2) ^ 4 ((r / 8) % 2): the 32 lanes of a half-wave fall on 32 different
// 8-byte bank pairs.
// Bound by the loads into LDS (16 KB a step at 73 bytes per nanosecond and compute unit with 64 x 64; 4,096 x 2048 x 512 under the profiler 18.7 us,
// with the loads alone 16.5, without them 14.0, with neither 6.9).  4,096 x 2048 x 512,
// 256 tiles of 64 x 64: 17.4 us; before, one group of four wavefronts, 128 x 64, 2 splits and the sum of their slabs: 20.0.
// 1,024: 9.2 -> 7.3; 4,096 x 4096 x 512 with 128 x 64: 26.6 -> 25.6.
template <int BM_, int WM_, int WN_, int KG_, int NS_>
struct WgradTile {
    static constexpr int BM = BM_, BN = 64, WM = WM_, WN = WN_, KG = KG_, NS = NS_, GW = WM * WN, NT = KG * GW * ARROL_WAVE;
    static constexpr int TI = BM / WM / 16, TJ = BN / WN / 16;
    static constexpr int SUB_BYTES = (BM + BN) * 128, STAGE_BYTES = KG * SUB_BYTES;
    static constexpr int LA = BM / 8 / GW, LB = BN / 8 / GW, LOADS = LA + LB;
    static constexpr int RED_BYTES = KG * BM * BN * 4, LDS_BYTES = NS * STAGE_BYTES > RED_BYTES ? NS * STAGE_BYTES : RED_BYTES;
    static_assert(LDS_BYTES <= 163840 && BM % (8 * GW) == 0 && BN % (8 * GW) == 0, "tile");
};

template <class C>
__global__ __launch_bounds__(C::NT, 2) void mlp_wgrad_mid_kernel(MlpRingArgs a, int terms, bool strips, MlpSums f) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    typedef __attribute__((address_space(3))) void* lds_ptr_t;
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4_t;
    constexpr int NS = C::NS, TI = C::TI, TJ = C::TJ, KG = C::KG, GW = C::GW, BM = C::BM, BN = C::BN;
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, lq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / GW, wq = wave % GW, wm = wq / C::WN, wn = wq % C::WN;
    // tile (unit block, column): blockIdx.y, .x or, in strips of 8 columns (wgrad_strips), blockIdx.x / 8 and 8 blockIdx.y + blockIdx.x % 8
    const int ub = strips ? blockIdx.x / 8 : blockIdx.y, cb = strips ? blockIdx.y * 8 + blockIdx.x % 8 : blockIdx.x;
    const int u0 = ub * BM, c0 = cb * BN;
    if (c0 >= a.b_rows) return;              // the last strip's missing columns
    // steps of this split: of each K64 all terms, one or two, so that the hidden states come from memory once
    const int k64_lo = static_cast<int>(blockIdx.z) * a.k64_per_split;
    const int k64_hi = k64_lo + a.k64_per_split < a.n_k64 ? k64_lo + a.k64_per_split : a.n_k64;   // > k64_lo (host)
    const int per = k64_hi - k64_lo, n_steps = per * terms, n_st = (n_steps + KG - 1) / KG;
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((lds_ptr_t)lds)) + kg * C::SUB_BYTES;
    // loader: lane -> (row lane/8 of an 8-row group, position lane%8); rows and columns past the end repeat the last ones
    const uint16_t* src_a[C::LA];
#pragma unroll
    for (int q = 0; q < C::LA; ++q) {
        const int r = (wq * C::LA + q) * 8 + (lane >> 3);
        const int u = u0 + r < a.a_rows ? u0 + r : a.a_rows - 1;
        src_a[q] = a.a + static_cast<int64_t>(u) * (a.a_stride / 2) + ((lane & 7) ^ (r & 6)) * 8;
    }
    const int64_t term = static_cast<int64_t>(a.a_rows) * (a.a_stride / 2);
    int b_row[C::LB];                        // rollout of the step and first column of this lane's chunk
    int64_t b_col[C::LB];
#pragma unroll
    for (int q = 0; q < C::LB; ++q) {
        const int r = (wq * C::LB + q) * 8 + (lane >> 3);
        const int c = c0 + ((lane & 7) ^ (((r >> 1) & 1) << 1) ^ (((r >> 3) & 1) << 2)) * 8;
        b_row[q] = r;
        b_col[q] = c < a.b_rows ? c : a.b_rows - 8;      // (d % 64 == 0)
    }
    // the group's next step: number, first rollout, offset in src_a, LDS slot
    int ld_s = kg < n_steps ? kg : 0, ld_row = (k64_lo + (ld_s >> (terms - 1))) * 64;
    int64_t ld_a = (ld_s & (terms - 1)) * term + ld_row;
    const int move = 64 * KG / terms;        // of a group that stays with one term
    unsigned ld_dst = lds0;
    auto issue = [&]() {                     // past the last step its lines again
        int64_t ak = ld_a;
        if (KG == 1) asm("" : "+s"(ak));     // one scalar: the compiler makes two vector additions a load of the sum (38.9 -> 37.1 us at
                                             // 4,096 x 3072 x 768; two groups 1 % slower with it)
#pragma unroll
        for (int q = 0; q < C::LA; ++q)
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src_a[q] + ak), "s"(ld_dst + (wq * C::LA + q) * 1024) : "memory");
#pragma unroll
        for (int q = 0; q < C::LB; ++q) {
            int k = ld_row + b_row[q];                   // rollouts past the last one repeat it: delta^T is zero there
            k = k < a.b_k_rows ? k : a.b_k_rows - 1;
            asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(a.b + static_cast<int64_t>(k) * (a.b_stride / 2) + b_col[q]),
                         "s"(ld_dst + BM * 128 + (wq * C::LB + q) * 1024) : "memory");
        }
        ld_dst = ld_dst == lds0 + (NS - 1) * C::STAGE_BYTES ? lds0 : ld_dst + C::STAGE_BYTES;
        if (ld_s + KG < n_steps) {
            ld_s += KG;
            if (KG == 1 && terms == 2) {     // the other term of the same rollouts, then the first of the next
                ld_a += ld_s & 1 ? term : 64 - term;
                ld_row += ld_s & 1 ? 0 : 64;
            } else {
                ld_a += move;
                ld_row += move;
            }
        }
    };
    f32x4 acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int a_off = kg * C::SUB_BYTES + (wm * (BM / C::WM) + l15) * 128;
    const int pos[2] = {(lq ^ (l15 & 6)) * 16, ((lq + 4) ^ (l15 & 6)) * 16};
    // lane 16 lq + 4 e + q addresses rollout 32 h + 8 lq + 4 h2 + e, columns wn * 16 TJ + 16 j + 4 q .. + 3
    const int e = l15 >> 2, cq = l15 & 3;
    int bt[2];
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
        const int chunk = (wn * 2 * TJ + (cq >> 1)) ^ ((e >> 1) << 1) ^ ((lq & 1) << 2);
        bt[h2] = kg * C::SUB_BYTES + BM * 128 + (8 * lq + 4 * h2 + e) * 128 + chunk * 16 + (cq & 1) * 8;
    }
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue();
    if (f.unit_partial && cb == 0 && blockIdx.z == 0) {   // while the first steps are on their way
        for (int v = tid; v < 2 * BM; v += C::NT)
            if (u0 + v % BM < f.m) finish_unit(f, u0 + v % BM, v / BM);
        if (ub == 0 && wave == GW * KG - 1) finish_loss(f, lane);
    }
    int slot = 0;
    for (int s = 0; s < n_st; ++s) {
        // these steps have landed (the NS - 2 after them may fly), for every wavefront, and all have read the ones before
        mlp_wait_vmcnt<(NS - 2) * C::LOADS>();
        __syncthreads();
        issue();
        const unsigned char* st = lds + slot;
        slot = slot == (NS - 1) * C::STAGE_BYTES ? 0 : slot + C::STAGE_BYTES;
        if (KG > 1 && s * KG + kg >= n_steps) continue;
        bf16x8 fa[2][TI], fb[2][TJ];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int i = 0; i < TI; ++i) fa[h][i] = *reinterpret_cast<const bf16x8*>(st + a_off + i * 2048 + pos[h]);
#pragma unroll
            for (int j = 0; j < TJ; ++j) {               // block j is two chunks on: an XOR (they commute with the swizzle)
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t)(st + h * 4096 + (bt[0] ^ (j << 5))));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t)(st + h * 4096 + (bt[1] ^ (j << 5))));
                fb[h][j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // all reads first
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][i], fb[h][j], acc[i][j], 0, 0, 0);
    }
    mlp_wait_vmcnt<0>();
    __syncthreads();                         // every stage has been read and every load into LDS has landed
    // block b = (i, j) of a wavefront's tile is finished by group b % KG, the sums added in group order
    f32x4* red = reinterpret_cast<f32x4*>(lds);   // [group][position][TI TJ][lane]
    if (KG > 1) {
#pragma unroll
        for (int b = 0; b < TI * TJ; ++b) red[(wave * TI * TJ + b) * 64 + lane] = acc[b / TJ][b % TJ];
        __syncthreads();
    }
#pragma unroll
    for (int b = 0; b < TI * TJ; ++b) {
        if (b % KG != kg) continue;
        f32x4 s = acc[b / TJ][b % TJ];
        if (KG > 1) s = red[(wq * TI * TJ + b) * 64 + lane];
#pragma unroll
        for (int g = 1; g < KG; ++g) s += red[((g * GW + wq) * TI * TJ + b) * 64 + lane];
        const int col = c0 + wn * (BN / C::WN) + (b % TJ) * 16 + l15;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int u = u0 + wm * (BM / C::WM) + (b / TJ) * 16 + lq * 4 + v;
            if (u < a.a_rows && col < a.b_rows) a.c_out[(static_cast<int64_t>(blockIdx.z) * a.a_rows + u) * a.c_stride + col] = s[v];
        }
    }
}

// one group of wavefronts, two workgroups to a compute unit, and two or four groups, one workgroup to a unit
using Mid32 = MidTile<32, 32, 2, 2, 1, 8>;
using Mid64 = MidTile<64, 64, 2, 2, 1, 4>;
using Mid128 = MidTile<128, 64, 2, 2, 1, 3>;
using Mid32Groups = MidTile<32, 32, 2, 1, 4, 3>;
using Mid64Groups = MidTile<64, 64, 2, 2, 2, 4>;
using Mid128Groups = MidTile<128, 64, 2, 2, 2, 3>;
using Wgrad64 = WgradTile<64, 2, 2, 2, 4>;
using Wgrad128 = WgradTile<128, 2, 2, 2, 3>;
using Wgrad128Two = WgradTile<128, 2, 2, 1, 3>;      // two workgroups to a compute unit

// Ids congruent mod 8 are on one XCD.  Strips of 8 columns keep all unit blocks of a column on the same XCD, whose L2 then holds
// their hidden states once, where the columns are no multiple of 8 and a whole row at a time would spread them (7,426 x 4032 x 256,
// 63 columns x 4 unit blocks, whole call: 72.2 us, in strips 62.4; 4,096 x 896 x 512 31.3, 29.8) - unless the columns that the last strip
// lacks leave some XCDs a round more than all have together (4,097 x 768 x 512 with two terms, 12 columns: 39.8, in strips 47.5) or
// are more than a fifth of the strips (65,536 x 64 x 128, whose one column would be all on one XCD: 57.9, in strips 67.2).
template <class C>
bool wgrad_strips(int n_cb, int n_ub, int splits) {
    constexpr int kPerXcd = C::LDS_BYTES > 81920 ? 32 : 64;       // workgroups that run together
    const int64_t fullest = static_cast<int64_t>((n_cb + 7) / 8) * n_ub * splits, all = static_cast<int64_t>(n_cb) * n_ub * splits;
    return n_ub > 65535 ||
           (4 * 8 * ((n_cb + 7) / 8) <= 5 * n_cb && (fullest + kPerXcd - 1) / kPerXcd == (all + 8 * kPerXcd - 1) / (8 * kPerXcd));
}

template <class C>
int launch_wgrad_mid(const MlpRingArgs& g, int terms, int splits, const MlpSums& f, hipStream_t st) {
    static arrol_device_flags ok;
    if (!arrol_allow_lds(&mlp_wgrad_mid_kernel<C>, C::LDS_BYTES, ok)) return ARROL_EHIP;
    const int n_cb = (g.b_rows + C::BN - 1) / C::BN, n_ub = (g.a_rows + C::BM - 1) / C::BM;
    const bool strips = wgrad_strips<C>(n_cb, n_ub, splits);
    arrol_launch(mlp_wgrad_mid_kernel<C>, strips ? dim3(8 * n_ub, (n_cb + 7) / 8, splits) : dim3(n_cb, n_ub, splits), dim3(C::NT),
                 C::LDS_BYTES, st, g, terms, strips, f);
    return ARROL_OK;
}

enum ForwardPath { kPathTile, kPathMid32, kPathMid64, kPathMid128, kPathRing };

int64_t n_blocks(int n_rows, int m, int bn, int bm) { return static_cast<int64_t>((n_rows + bn - 1) / bn) * ((m + bm - 1) / bm); }

// Which forward pass a batch takes: the smallest of the measured times (microseconds at d = 2048, all proportional to d)
// for up to 256 workgroups and for every 512 (the mid kernels, two workgroups per compute unit) or 256 (ring) beyond.
// m = 512: 32 x 32 blocks up to some 700 rollouts, 64 x 64 up to 2,048, 128 x 64 up to 10,000, then the ring (at 8,192
// rollouts 28 us against 43 of the ring; at 16,384 49 against 45).
ForwardPath pick_forward(int n_rows, int d, int m, int64_t row_stride_elems, bool gathered) {
    if (d % 64) return kPathTile;
    constexpr int kMaxGridY = 65535;         // unit blocks are blockIdx.y
    auto mid = [&](int bn, int bm, double one, double two) {
        const int64_t n = n_blocks(n_rows, m, bn, bm);
        if ((m + bm - 1) / bm > kMaxGridY) return 1e30;
        return n <= 256 ? one : two * static_cast<double>((n + 511) / 512);
    };
    const double t32 = mid(32, 32, 5.0, 8.3), t64 = mid(64, 64, 7.8, 15.5), t128 = mid(64, 128, 12.5, 22.5);
    ForwardPath best = kPathTile;
    double t = 1e29;
    if (t32 < t) { t = t32; best = kPathMid32; }
    if (t64 < t) { t = t64; best = kPathMid64; }
    if (t128 < t) { t = t128; best = kPathMid128; }
    // the ring kernel addresses a lane's row with a 32-bit byte offset inside a 256-row tile
    if (!gathered && row_stride_elems * 2 * 256 < (1ll << 31) && (m + 255) / 256 <= kMaxGridY) {
        const int64_t n = n_blocks(n_rows, m, 256, 256);
        const double tr = n <= 192 ? 38.0 : 50.0 * static_cast<double>((n + 255) / 256);
        // Up to 128 units two and more rounds of 128 x 64 blocks cost more than their share next to the ring (65,536 rollouts x
        // 64 / 512 / 2048: 12.6 / 21.3 / 56.2 us against 9.6 / 19.9 / 50.2), until the rows outgrow the last-level cache
        // (65,536 x 4096: 132 against 139).
        const bool crowded = best == kPathMid128 && n_blocks(n_rows, m, 64, 128) > 512 && 2.0 * n_rows * d <= 384e6;
        if (tr < (crowded ? 1.13 * t : t)) best = kPathRing;
    }
    return best;
}
// 128 x 64 blocks read every rollout's row once per 128 units, the tile kernel reads it once; where rows are narrow or
// there are very many of them and the ring form is not to be had (gathered rows), it is the faster one for a forward pass
// that keeps no activations.  Microseconds measured over 300 to 131,072 gathered rollouts, d of 64 to 4096, 32 to 1,024
// units; beyond the last-level cache (256 MB) the repeated reads come from memory.  Tile and 128 x 64: 20,000 x 64 x 512
// 12.1 and 16.5, 32,768 x 1024 x 512 55.0 and 57.5, 131,072 x 2048 x 512 401 and 525, but 32,768 x 2048 x 512 100 and 95,
// 20,000 x 1024 x 256 29.2 and 26.2.
bool tile_beats_mid128(int n_rows, int d, int m) {
    const double rounds = static_cast<double>((n_blocks(n_rows, 1, 128, 1) + 255) / 256);
    const double tile = 2.0 + rounds * (1.5 + ((m + 255) / 256) * (2.8 + 0.0222 * d));
    const int64_t blocks = n_blocks(n_rows, m, 64, 128), last = blocks % 512;
    double mid = 7.6 + 0.0055 * d;
    if (blocks > 256) mid = 3.5 + (static_cast<double>(blocks / 512) + (last == 0 ? 0.0 : last <= 256 ? 0.75 : 1.0)) * (3.9 + 0.0095 * d);
    const double bytes = 2.0 * n_rows * d, reads = ((m + 127) / 128) * bytes / 4.0e6;
    if (bytes > 384e6 && reads > mid) mid = reads;
    return tile < mid;
}
ForwardPath pick_score(int n_rows, int d, int m, int64_t row_stride_elems, bool gathered) {   // no activations kept
    const ForwardPath p = pick_forward(n_rows, d, m, row_stride_elems, gathered);
    return p == kPathMid128 && gathered && tile_beats_mid128(n_rows, d, m) ? kPathTile : p;
}
int unit_block(ForwardPath p) { return p == kPathMid32 ? 32 : p == kPathMid64 ? 64 : p == kPathMid128 ? 128 : 256; }

// Wavefront groups that share a block's K: several where a compute unit has one workgroup anyhow and K is long enough to pay for
// adding them up (d = 320: 6.7 against 7.1 us with 300 rollouts x 1,000, d = 512 even); 64 x 64 blocks of 129 to 256 are not
// faster for it.
int forward_groups(ForwardPath path, int n_rows, int d, int m) {
    if (d < 768) return 1;
    if (path == kPathMid32) return n_blocks(n_rows, m, 32, 32) <= 256 ? Mid32Groups::KG : 1;
    if (path == kPathMid64) return n_blocks(n_rows, m, 64, 64) <= 128 ? Mid64Groups::KG : 1;
    if (path == kPathMid128) return n_blocks(n_rows, m, 64, 128) <= 256 ? Mid128Groups::KG : 1;
    return 1;
}

// Partial scores of every unit block to `partial`, with act_t also the activations (kPathTile: not for this).
int enqueue_forward(ForwardPath path, const void* hidden, int64_t row_stride_elems, const int64_t* row_index, const void* w1,
                    const float* b1, const float* w2, int n_rows, int d, int m, float* partial, float* act_t,
                    int64_t act_stride, hipStream_t st) {
    if (path == kPathRing) {
        MlpRingArgs r = {};
        r.a = static_cast<const uint16_t*>(w1); r.a_stride = static_cast<unsigned>(d) * 2; r.a_rows = m;
        r.b = static_cast<const uint16_t*>(hidden); r.b_stride = static_cast<unsigned>(row_stride_elems * 2); r.b_rows = n_rows;
        r.n_k64 = d / 64; r.b1 = b1; r.w2 = w2; r.partial = partial;
        r.act_t = act_t; r.act_stride = act_stride;
        const dim3 grid((n_rows + 255) / 256, (m + 255) / 256);
        return act_t ? launch_mlp_ring<kForwardKeep>(r, grid, st) : launch_mlp_ring<kForward>(r, grid, st);
    }
    MlpMidArgs a = {static_cast<const uint16_t*>(hidden), row_stride_elems, row_index, static_cast<const uint16_t*>(w1), b1, w2,
                    n_rows, d, m, partial, act_t, act_stride};
    const bool groups = forward_groups(path, n_rows, d, m) > 1;
    if (path == kPathMid32) return groups ? launch_mlp_mid<Mid32Groups>(a, st) : launch_mlp_mid<Mid32>(a, st);
    if (path == kPathMid64) return groups ? launch_mlp_mid<Mid64Groups>(a, st) : launch_mlp_mid<Mid64>(a, st);
    return groups ? launch_mlp_mid<Mid128Groups>(a, st) : launch_mlp_mid<Mid128>(a, st);
}

// dL/dW1 on the ring pipeline's K-major B form: any batch size, rows addressed in place
bool wgrad_in_place(int d, int64_t row_stride_elems, bool gathered) {
    return d % 64 == 0 && !gathered && row_stride_elems * 2 * 256 < (1ll << 31);
}

// r_i = (q_i - y_i) / N and the loss: one workgroup per 1024 rows writes its two partial sums, the second
// kernel adds them in block order (fixed summation order, bit-reproducible)
__global__ __launch_bounds__(1024) void mlp_residual_kernel(const float* __restrict__ score,
                                                            const float* __restrict__ prob,
                                                            const float* __restrict__ labels, int n_rows,
                                                            float* __restrict__ resid, float* __restrict__ block_sums) {
    __shared__ float red[2][16];
    const float inv_n = 1.f / static_cast<float>(n_rows);
    float loss = 0.f, rs = 0.f;
    const int i = blockIdx.x * 1024 + threadIdx.x;
    if (i < n_rows) {
        const float s = score[i], y = labels[i];
        const float r = (prob[i] - y) * inv_n;
        resid[i] = r;
        rs = r;
        loss = fmaxf(s, 0.f) - y * s + log1pf(expf(-fabsf(s)));
    }
    loss = wave_sum_f32(loss);
    rs = wave_sum_f32(rs);
    const int lane = threadIdx.x & (ARROL_WAVE - 1), wave = threadIdx.x / ARROL_WAVE;
    if (lane == 0) { red[0][wave] = loss; red[1][wave] = rs; }
    __syncthreads();
    if (threadIdx.x == 0) {
        float a = 0.f, b = 0.f;
        for (int w = 0; w < 16; ++w) { a += red[0][w]; b += red[1][w]; }
        block_sums[blockIdx.x] = a;
        block_sums[gridDim.x + blockIdx.x] = b;
    }
}

// The gradient call after a forward pass that leaves partial scores (partial[unit block][rollout]):
// score_mlp_finish_kernel and mlp_residual_kernel in one launch - score = sum over the unit blocks in index
// order + b2, then r_i and the loss terms as above; neither scores nor probabilities go to memory.
__global__ __launch_bounds__(1024) void mlp_finish_residual_kernel(const float* __restrict__ partial, int n_ub,
                                                                   float b2, const float* __restrict__ labels,
                                                                   int n_rows, float* __restrict__ resid,
                                                                   float* __restrict__ block_sums) {
    __shared__ float red[2][16];
    const float inv_n = 1.f / static_cast<float>(n_rows);
    float loss = 0.f, rs = 0.f;
    const int i = blockIdx.x * 1024 + threadIdx.x;
    if (i < n_rows) {
        const float s = sum_unit_blocks(partial, n_ub, n_rows, i) + b2;
        float q;
        if (s >= 0.f) {
            q = 1.f / (1.f + expf(-s));
        } else {
            const float e = expf(s);
            q = e / (1.f + e);
        }
        const float y = labels[i];
        const float r = (q - y) * inv_n;
        resid[i] = r;
        rs = r;
        loss = fmaxf(s, 0.f) - y * s + log1pf(expf(-fabsf(s)));
    }
    loss = wave_sum_f32(loss);
    rs = wave_sum_f32(rs);
    const int lane = threadIdx.x & (ARROL_WAVE - 1), wave = threadIdx.x / ARROL_WAVE;
    if (lane == 0) { red[0][wave] = loss; red[1][wave] = rs; }
    __syncthreads();
    if (threadIdx.x == 0) {
        float a = 0.f, b = 0.f;
        for (int w = 0; w < 16; ++w) { a += red[0][w]; b += red[1][w]; }
        block_sums[blockIdx.x] = a;
        block_sums[gridDim.x + blockIdx.x] = b;
    }
}

__global__ void mlp_residual_finish_kernel(const float* __restrict__ block_sums, int n_blocks, int n_rows,
                                           float* __restrict__ loss_out, float* __restrict__ grad_b2) {
    float a = 0.f, b = 0.f;
    for (int k = 0; k < n_blocks; ++k) { a += block_sums[k]; b += block_sums[n_blocks + k]; }
    if (loss_out) *loss_out = a / static_cast<float>(n_rows);
    if (grad_b2) *grad_b2 = b;
}

// delta^T and the per-unit sums from the kept activations: one workgroup per unit u streams its row
//   delta^T[u][i] = r_i w2_u [a_ui > 0] (bf16, 0 for n_rows <= i < n_pad; optionally the bf16 remainder too),
//   dL/dw2_u = sum_i r_i a_ui,  dL/db1_u = sum_i r_i w2_u [a_ui > 0],
// each lane over its own columns in ascending order, then lanes, then wavefronts: a fixed summation order.
// Workgroup 0 also finishes the loss and dL/db2 from the residual pass's block sums.
constexpr int kDeltaThreads = 1024;
__global__ __launch_bounds__(kDeltaThreads) void mlp_delta_kernel(const float* __restrict__ act_t, int64_t act_stride,
                                                                  const float* __restrict__ resid,
                                                                  const float* __restrict__ w2, int n_rows, int n_pad,
                                                                  uint16_t* __restrict__ delta_t,
                                                                  uint16_t* __restrict__ delta_lo,
                                                                  float* __restrict__ grad_w2,
                                                                  float* __restrict__ grad_b1,
                                                                  const float* __restrict__ block_sums, int n_blocks,
                                                                  float* __restrict__ loss_out,
                                                                  float* __restrict__ grad_b2) {
    __shared__ float red[2][kDeltaThreads / ARROL_WAVE];
    const int u = blockIdx.x;
    if (u == 0 && threadIdx.x == 0) {   // loss and dL/db2: the residual pass's block sums, added in block order
        float a = 0.f, b = 0.f;
        for (int k = 0; k < n_blocks; ++k) { a += block_sums[k]; b += block_sums[n_blocks + k]; }
        if (loss_out) *loss_out = a / static_cast<float>(n_rows);
        if (grad_b2) *grad_b2 = b;
    }
    const float wu = w2[u];
    const float* arow = act_t + static_cast<int64_t>(u) * act_stride;
    uint16_t* drow = delta_t + static_cast<int64_t>(u) * n_pad;
    float gw = 0.f, gb = 0.f;
    for (int i = threadIdx.x * 4; i < n_pad; i += kDeltaThreads * 4) {   // n_pad is a multiple of 4
        float av[4] = {0.f, 0.f, 0.f, 0.f}, rv[4] = {0.f, 0.f, 0.f, 0.f};
        if (i + 3 < n_rows) {
            const float4 a4 = *reinterpret_cast<const float4*>(arow + i);
            const float4 r4 = *reinterpret_cast<const float4*>(resid + i);
            av[0] = a4.x; av[1] = a4.y; av[2] = a4.z; av[3] = a4.w;
            rv[0] = r4.x; rv[1] = r4.y; rv[2] = r4.z; rv[3] = r4.w;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (i + q < n_rows) { av[q] = arow[i + q]; rv[q] = resid[i + q]; }
        }
        uint16_t dq[4], lq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float dl = av[q] > 0.f ? rv[q] * wu : 0.f;
            gw = fmaf(rv[q], av[q], gw);
            gb += dl;
            dq[q] = f32_to_bf16_rne(dl);
            lq[q] = f32_to_bf16_rne(dl - bf16_lo(dq[q]));
        }
        uint2 o;
        o.x = static_cast<uint32_t>(dq[0]) | (static_cast<uint32_t>(dq[1]) << 16);
        o.y = static_cast<uint32_t>(dq[2]) | (static_cast<uint32_t>(dq[3]) << 16);
        *reinterpret_cast<uint2*>(drow + i) = o;
        if (delta_lo) {     // second term of the two-term form: what bf16 rounding left of delta
            o.x = static_cast<uint32_t>(lq[0]) | (static_cast<uint32_t>(lq[1]) << 16);
            o.y = static_cast<uint32_t>(lq[2]) | (static_cast<uint32_t>(lq[3]) << 16);
            *reinterpret_cast<uint2*>(delta_lo + static_cast<int64_t>(u) * n_pad + i) = o;
        }
    }
    gw = wave_sum_f32(gw);
    gb = wave_sum_f32(gb);
    const int lane = threadIdx.x & (ARROL_WAVE - 1), wave = threadIdx.x / ARROL_WAVE;
    if (lane == 0) { red[0][wave] = gw; red[1][wave] = gb; }
    __syncthreads();
    if (threadIdx.x == 0) {
        float a = 0.f, b = 0.f;
        for (int w = 0; w < kDeltaThreads / ARROL_WAVE; ++w) { a += red[0][w]; b += red[1][w]; }
        grad_w2[u] = a;
        grad_b1[u] = b;
    }
}

// The two in one: workgroup (b, g) forms the residuals of rows 512 b .. itself, into the LDS, and then, one unit a wavefront,
// delta^T of those rows and their parts of dL/dw2 and dL/db1; those with g = 0 also of the loss and dL/db2.  The parts are added
// in block order by the dL/dW1 kernel that follows, or by mlp_sums_kernel.
// What bounds it is a chain of dependent loads and a launch, beyond the activations' bytes; a row's residual is formed m / 8
// times, which costs less than the launch that formed it once: 4,096 x 512 6.2 us against 4.4 + 4.9, 1,024 x 512 4.8 against
// 3.9 + 4.4; with 1,024 rows a workgroup 7.2, with 256 7.1.
// The line, by whole calls, one launch over the pair (d of 512 to 3072): where the dL/dW1 kernel adds the parts 0.85 - 0.98 up to 3
// million activations of up to 20,000 rows (4,096 x 768 53.1 us against 55.5), 0.98 - 1.02 of 4 million, 1.01 - 1.05 of 65,536 rows.  Where
// another launch adds them 0.92 - 1.00 up to 2,048 rows, 1.00 - 1.01 of 4,096 and 1.01 - 1.04 beyond.
constexpr int kFusedRows = 20000, kFusedRowsAlone = 2048, kFusedSize = 3 << 20;
constexpr int kPartRows = 512;
__global__ __launch_bounds__(kPartRows) void mlp_score_delta_kernel(const float* __restrict__ partial, int n_ub, float b2,
                                                                    const float* __restrict__ labels,
                                                                    const float* __restrict__ act_t, int64_t act_stride,
                                                                    const float* __restrict__ w2, int n_rows, int n_pad, int m,
                                                                    int n_groups,
                                                                    uint16_t* __restrict__ delta_t, uint16_t* __restrict__ delta_lo,
                                                                    float* __restrict__ unit_partial, float* __restrict__ block_sums) {
    constexpr int kWaves = kPartRows / ARROL_WAVE, kSteps = kPartRows / (4 * ARROL_WAVE);
    __shared__ __attribute__((aligned(16))) float resid[kPartRows];
    __shared__ float red[2][kWaves];
    const int lane = threadIdx.x & (ARROL_WAVE - 1), wave = threadIdx.x / ARROL_WAVE;
    const int block = blockIdx.x / n_groups, group = blockIdx.x - block * n_groups, n_blocks = gridDim.x / n_groups;
    const int row0 = block * kPartRows;
    const int unit = group * kWaves + wave, u = unit < m ? unit : m - 1;
    // the unit's activations are on their way while the residuals are formed (n_pad is a multiple of 4; the columns from n_rows
    // on hold whatever the workspace held and are masked below)
    const float* arow = act_t + static_cast<int64_t>(u) * act_stride;
    float4 a4[kSteps];
#pragma unroll
    for (int k = 0; k < kSteps; ++k) {
        const int i = row0 + (k * ARROL_WAVE + lane) * 4;
        a4[k] = *reinterpret_cast<const float4*>(arow + (i < n_pad ? i : 0));
    }
    const float wu = w2[u];
    {
        const int i = row0 + threadIdx.x;
        float r = 0.f, loss = 0.f;
        if (i < n_rows) {
            const float y = labels[i];
            const float s = sum_unit_blocks(partial, n_ub, n_rows, i) + b2;
            float q;
            if (s >= 0.f) {
                q = 1.f / (1.f + expf(-s));
            } else {
                const float e = expf(s);
                q = e / (1.f + e);
            }
            r = (q - y) * (1.f / static_cast<float>(n_rows));
            if (group == 0) loss = fmaxf(s, 0.f) - y * s + log1pf(expf(-fabsf(s)));
        }
        resid[threadIdx.x] = r;
        if (group == 0) {
            loss = wave_sum_f32(loss);
            r = wave_sum_f32(r);
            if (lane == 0) { red[0][wave] = loss; red[1][wave] = r; }
        }
    }
    __syncthreads();
    if (group == 0 && threadIdx.x == 0) {
        float a = 0.f, b = 0.f;
        for (int w = 0; w < kWaves; ++w) { a += red[0][w]; b += red[1][w]; }
        block_sums[block] = a;
        block_sums[n_blocks + block] = b;
    }
    if (unit >= m) return;
    uint16_t* drow = delta_t + static_cast<int64_t>(u) * n_pad;
    float gw = 0.f, gb = 0.f;
#pragma unroll
    for (int k = 0; k < kSteps; ++k) {
        const int c = (k * ARROL_WAVE + lane) * 4, i = row0 + c;
        if (i >= n_pad) continue;
        const float4 r4 = *reinterpret_cast<const float4*>(resid + c);
        const float av[4] = {a4[k].x, a4[k].y, a4[k].z, a4[k].w}, rv[4] = {r4.x, r4.y, r4.z, r4.w};
        uint16_t dq[4], lq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool live = i + q < n_rows;
            const float dl = live && av[q] > 0.f ? rv[q] * wu : 0.f;
            gw = live ? fmaf(rv[q], av[q], gw) : gw;
            gb += dl;
            dq[q] = f32_to_bf16_rne(dl);
            lq[q] = f32_to_bf16_rne(dl - bf16_lo(dq[q]));
        }
        uint2 o;
        o.x = static_cast<uint32_t>(dq[0]) | (static_cast<uint32_t>(dq[1]) << 16);
        o.y = static_cast<uint32_t>(dq[2]) | (static_cast<uint32_t>(dq[3]) << 16);
        *reinterpret_cast<uint2*>(drow + i) = o;
        if (delta_lo) {     // second term of the two-term form: what bf16 rounding left of delta
            o.x = static_cast<uint32_t>(lq[0]) | (static_cast<uint32_t>(lq[1]) << 16);
            o.y = static_cast<uint32_t>(lq[2]) | (static_cast<uint32_t>(lq[3]) << 16);
            *reinterpret_cast<uint2*>(delta_lo + static_cast<int64_t>(u) * n_pad + i) = o;
        }
    }
    gw = wave_sum_f32(gw);
    gb = wave_sum_f32(gb);
    if (lane == 0) {
        float* out = unit_partial + static_cast<int64_t>(block) * 2 * m;
        out[u] = gw;
        out[m + u] = gb;
    }
}

// out[c][i] = hidden[row(i)][c] for i < n_rows, 0 for n_rows <= i < n_pad: 64 x 64 tiles through LDS, 16 bytes
// per lane on both sides (8 lanes cover the 128 bytes a tile row has in the source and in the destination)
__global__ __launch_bounds__(256) void mlp_transpose_kernel(const uint16_t* __restrict__ hidden, int64_t row_stride,
                                                            const int64_t* __restrict__ row_index, int n_rows,
                                                            int d, int n_pad, uint16_t* __restrict__ out) {
    __shared__ __attribute__((aligned(16))) uint16_t tile_t[64][72];   // [column][rollout], 144-byte pitch
    const int i0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
    const int chunk = threadIdx.x & 7, r8 = threadIdx.x >> 3;           // 32 rows x 8 chunks per pass
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int r = r8 + p * 32, i = i0 + r, c = c0 + chunk * 8;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (i < n_rows && c < d) {      // d is a multiple of 8: a chunk is inside the row or outside it
            const int64_t src = row_index ? row_index[i] : i;
            v = *reinterpret_cast<const uint4*>(hidden + src * row_stride + c);
        }
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            tile_t[chunk * 8 + 2 * q][r] = static_cast<uint16_t>(w[q] & 0xffffu);
            tile_t[chunk * 8 + 2 * q + 1][r] = static_cast<uint16_t>(w[q] >> 16);
        }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int cr = r8 + p * 32, c = c0 + cr, i = i0 + chunk * 8;
        if (c < d && i < n_pad)          // n_pad is a multiple of 64: whole chunks
            *reinterpret_cast<uint4*>(out + static_cast<int64_t>(c) * n_pad + i) =
                *reinterpret_cast<const uint4*>(&tile_t[cr][chunk * 8]);
    }
}

struct GradPlan {
    int n_rb, n_pad, n_cb, n_groups, n_kc, splits, kc_per_split;
    int r_cb, r_gt, r_splits, r_k64_per_split;
    int w_rows, w_groups;              // dL/dW1 of rows read in place: rows of the mid kernel's tile, 64 or 128, and wavefront groups; 256: the ring form
    bool w_stacked;                    // the mid kernel takes two terms as rows of their own, as the ring form does, not into the same sums
    size_t off_score, off_prob, off_resid, off_bsum, off_ht, off_dt, off_unit, off_slab, off_small, off_rslab, off_act, total;
};

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

GradPlan make_grad_plan(int n_rows, int d, int m, int terms) {
    GradPlan p;
    p.n_rb = (n_rows + BR - 1) / BR;
    p.n_pad = p.n_rb * BR;
    p.n_cb = (d + BR - 1) / BR;              // wgrad: 128 columns of dL/dW1 per workgroup
    // dL/dW1 contracts [hi; lo] (terms * m rows) with H and leaves one partial per term and K split
    const int mt = terms * m;
    p.n_groups = (mt + BU - 1) / BU;
    p.n_kc = p.n_pad / BK;
    // split K so that about 256 workgroups run, each with at least 8 chunks; at most 8 partial slabs
    int s = 256 / (p.n_cb * p.n_groups);
    if (s > p.n_kc / 8) s = p.n_kc / 8;
    if (s > 8) s = 8;
    if (s < 1) s = 1;
    p.kc_per_split = (p.n_kc + s - 1) / s;
    p.splits = (p.n_kc + p.kc_per_split - 1) / p.kc_per_split;
    size_t o = 0;
    p.off_score = o; o = align256(o + sizeof(float) * n_rows);
    p.off_prob = o;  o = align256(o + sizeof(float) * n_rows);
    p.off_resid = o; o = align256(o + sizeof(float) * n_rows);
    p.off_bsum = o;  o = align256(o + sizeof(float) * 2 * ((n_rows + kPartRows - 1) / kPartRows));
    p.off_ht = o;    o = align256(o + sizeof(uint16_t) * static_cast<size_t>(d) * p.n_pad);
    p.off_dt = o;    o = align256(o + sizeof(uint16_t) * static_cast<size_t>(mt) * p.n_pad);
    // per-unit partial sums of the tile kernel: one row per 128 rollouts
    p.off_unit = o;  o = align256(o + sizeof(float) * static_cast<size_t>(p.n_rb) * 2 * m);
    p.off_slab = o;
    if (p.splits * terms > 1) o = align256(o + sizeof(float) * static_cast<size_t>(p.splits) * mt * d);
    p.off_small = o;                      // partial scores of the mid / ring forward pass
    if (d % 64 == 0) {
        const size_t blocks = (m + 31) / 32;          // of the forward pass with the smallest ones
        o = align256(o + sizeof(float) * blocks * n_rows);
    }
    // rows read in place: kernel and K split with the smallest estimate (microseconds: the measured time per K64 step of
    // a workgroup when the chip is full, a start of 5 or 7, and the partial slabs written and read once at 4.5 TB/s).  First the
    // ring form (a slab per split and term) against 128 x 64 tiles of four wavefronts, two workgroups to a compute unit.
    p.r_cb = (d + 255) / 256;
    p.r_gt = (mt + 255) / 256;         // dL/dW1
    const int n_k64 = (n_rows + 63) / 64;
    const double slab_us = static_cast<double>(mt) * d * 8.0 / 4.5e6;
    const int64_t ring_tiles = static_cast<int64_t>(p.r_cb) * p.r_gt;
    const int64_t mid_tiles = static_cast<int64_t>((d + Wgrad128::BN - 1) / Wgrad128::BN) * ((mt + Wgrad128::BM - 1) / Wgrad128::BM);
    constexpr int kMaxSplits = 16;
    constexpr double kRingStep = 1.45, kRingStart = 7.0, kMidStep = 0.68, kMidStart = 5.0, kSlabStart = 2.5;
    double best = -1.0, one = 0.0;
    for (int s = 1; s <= kMaxSplits && (s == 1 || n_k64 / s >= 4); ++s) {
        const int per = (n_k64 + s - 1) / s, used = (n_k64 + per - 1) / per;
        const double slabs = used * terms > 1 ? kSlabStart + used * slab_us : 0.0;
        const int64_t nr = ring_tiles * used, nm = mid_tiles * used;
        const double ring = static_cast<double>((nr + 255) / 256) * (per * kRingStep + kRingStart) + slabs;
        const double mid = (mt + Wgrad128::BM - 1) / Wgrad128::BM > 65535 ? 1e30
                           : (nm <= 256 ? per * 0.38 + kMidStart : static_cast<double>((nm + 511) / 512) * (per * kMidStep + kMidStart)) + slabs;
        const double t = mid < ring ? mid : ring;
        if (s == 1) one = t;
        if (best < 0.0 || t < best) { best = t; p.w_rows = mid < ring ? 128 : 256; p.r_k64_per_split = per; p.r_splits = used; }
    }
    // The split count can fall from one batch to the next larger one, but a workspace sized for the largest batch is to
    // serve every smaller one.  Room is made for the most splits that a batch up to this one can take: s of them are only
    // chosen where their slabs and the work on a full chip, which no estimate is below, come to less than one split's
    // estimate.  What is left of that estimate after the work grows with the batch, and so does the room.
    int room = 1, room_mid = 1;
    const double ring_work = static_cast<double>(ring_tiles) / 256.0 * kRingStep, mid_work = static_cast<double>(mid_tiles) / 512.0 * kMidStep;
    const double work = n_k64 * (ring_work < mid_work ? ring_work : mid_work) + kMidStart;
    for (int s = 2; s <= kMaxSplits && n_k64 / s >= 4; ++s)
        if (kSlabStart + s * slab_us + work <= one + 1e-6) room = s;
    if (room < p.r_splits) room = p.r_splits;
    // Then, where the tiles won, which ones and how many splits, all terms in one sum: 64 x 64 or 128 x 64 with K split over two
    // groups of wavefronts and one workgroup to a compute unit (4,096 x 2048 x 512: 17.4 / 23.2 us without a split, 19.2 with two
    // of 128 x 64), or four wavefronts, two workgroups to a unit, where there are more tiles than compute units (2,048 x 4096 x 1,024: 35.8 / 28.5 /
    // 25.9; 4,096 x 3072 x 768: 47.9 / 45.5 / 31.2).
    const double mid_slab_us = static_cast<double>(m) * d * 8.0 / 4.5e6;
    const int64_t tiles64 = static_cast<int64_t>((d + 63) / 64) * ((m + 63) / 64), tiles128 = static_cast<int64_t>((d + 63) / 64) * ((m + 127) / 128);
    // Of a last round of more than 256 workgroups the pairs on some units set the time (288: 0.5 us a step, 512: 0.68); with their
    // share of 512 for it 8,192 x 2048 x 257 took 288 workgroups, 26.3 us, instead of 480, 20.5.
    const auto one_group_us = [&](int64_t n, int steps) {
        const double last = n % 512 <= 256 ? 0.38 : 0.5 + (kMidStep - 0.5) * static_cast<double>(n % 512 - 256) / 256.0;
        return static_cast<double>(n / 512) * (steps * kMidStep + kMidStart) + (n % 512 ? steps * last + kMidStart : 0.0);
    };
    constexpr double kStep64 = 0.205, kStep128 = 0.31, kRound64 = 4.3, kRound128 = 5.5;
    struct Blocks { double us; int rows, groups; };
    const auto blocks_us = [&](int64_t n64, int64_t n128, int steps) {        // the three forms, of that many tiles
        const double t64 = static_cast<double>((n64 + 255) / 256) * (steps * kStep64 + kRound64);
        const double t128 = static_cast<double>((n128 + 255) / 256) * (steps * kStep128 + kRound128), two = one_group_us(n128, steps);
        if (two < t64 && two < t128) return Blocks{two, 128, 1};
        return t64 <= t128 ? Blocks{t64, 64, 2} : Blocks{t128, 128, 2};
    };
    double best_mid = -1.0, one_mid = 0.0;
    p.w_stacked = false;
    for (int s = 1; s <= kMaxSplits && (s == 1 || n_k64 / s >= 4); ++s) {
        const int per = (n_k64 + s - 1) / s, used = (n_k64 + per - 1) / per;
        const Blocks b = blocks_us(tiles64 * used, tiles128 * used, per * terms);
        const double t = b.us + (used > 1 ? kSlabStart + used * mid_slab_us : 0.0);
        if (s == 1) one_mid = t;
        if (best_mid < 0.0 || t < best_mid) {
            best_mid = t;
            if (p.w_rows != 256) { p.w_rows = b.rows; p.w_groups = b.groups; p.r_k64_per_split = per; p.r_splits = used; }
        }
    }
    // Two terms as rows of their own cost a slab more each, but no more time in a tile that they leave room in or on units that
    // would be idle: whole calls of 21,203 x 2176 x 5 52.8 us in the same sums, 47.9 so, 33,986 x 128 x 128 58.2 and 50.8.  Where the
    // estimates are close the same sums are faster, since they read the hidden states once (30,014 x 192 x 256, 0.89 by the
    // estimates: 60.8 and 66.8): a fifth less or nothing.
    const int64_t st64 = static_cast<int64_t>((d + 63) / 64) * ((mt + 63) / 64), st128 = static_cast<int64_t>((d + 63) / 64) * ((mt + 127) / 128);
    for (int s = 1; terms == 2 && p.w_rows != 256 && s <= room && (s == 1 || n_k64 / s >= 4); ++s) {
        const int per = (n_k64 + s - 1) / s, used = (n_k64 + per - 1) / per;
        const Blocks b = blocks_us(st64 * used, st128 * used, per);
        const double t = (b.us + kSlabStart + used * slab_us) / 0.8;
        if (t < best_mid) { best_mid = t; p.w_stacked = true; p.w_rows = b.rows; p.w_groups = b.groups; p.r_k64_per_split = per; p.r_splits = used; }
    }
    // the same room for their splits (whichever form this batch takes: a smaller one may take the other)
    double step_mid = static_cast<double>(tiles64) * kStep64 / 256.0;
    step_mid = tiles128 * kStep128 / 256.0 < step_mid ? tiles128 * kStep128 / 256.0 : step_mid;
    step_mid = tiles128 * kMidStep / 512.0 < step_mid ? tiles128 * kMidStep / 512.0 : step_mid;
    for (int s = 2; s <= kMaxSplits && n_k64 / s >= 4; ++s)
        if (kSlabStart + s * mid_slab_us + n_k64 * terms * step_mid + kRound64 <= one_mid + 1e-6) room_mid = s;
    const int room_slabs = room * terms > room_mid ? room * terms : room_mid;
    p.off_rslab = o;
    if (d % 64 == 0 && room_slabs > 1) o = align256(o + sizeof(float) * static_cast<size_t>(room_slabs) * m * d);
    p.off_act = o;                        // mid / ring forward pass: kept activations, fp32 [m][n_pad]
    if (d % 64 == 0) o = align256(o + sizeof(float) * static_cast<size_t>(m) * p.n_pad);
    p.total = o;
    return p;
}

// out = the slabs' sum in slab order; 16 bytes per lane where the caller's output allows it (the slabs always do: m * d
// is a multiple of 8).  9 slabs of 4 MB (4,096 x 2048 x 512 with 8 splits): 15 us at 4 bytes per lane in 128-byte rows.
template <int VEC>
__global__ __launch_bounds__(256) void reduce_slabs_kernel(const float* __restrict__ slabs, int n_slabs, int64_t width,
                                                           float* __restrict__ out) {
    const int64_t c = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * VEC;
    if (c >= width) return;
    float s[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) s[v] = 0.f;
    for (int p0 = 0; p0 < n_slabs; p0 += 4) {
        float x[4][VEC];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float* src = slabs + static_cast<int64_t>(p0 + q < n_slabs ? p0 + q : p0) * width + c;
            if constexpr (VEC == 4) {
                const float4 f = *reinterpret_cast<const float4*>(src);
                x[q][0] = f.x; x[q][1] = f.y; x[q][2] = f.z; x[q][3] = f.w;
            } else {
                x[q][0] = src[0];
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (p0 + q < n_slabs) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) s[v] += x[q][v];
            }
    }
    if constexpr (VEC == 4) *reinterpret_cast<float4*>(out + c) = make_float4(s[0], s[1], s[2], s[3]);
    else out[c] = s[0];
}
void launch_reduce_slabs(const float* slabs, int n_slabs, int64_t width, float* out, hipStream_t st) {
    if (arrol_aligned16(out))
        arrol_launch(reduce_slabs_kernel<4>, dim3(static_cast<unsigned>((width / 4 + 255) / 256)), dim3(256), 0, st, slabs, n_slabs, width, out);
    else
        arrol_launch(reduce_slabs_kernel<1>, dim3(static_cast<unsigned>((width + 255) / 256)), dim3(256), 0, st, slabs, n_slabs, width, out);
}

template <int MODE>
int launch_mlp(const MlpArgs& a, dim3 grid, hipStream_t st) {
    static arrol_device_flags lds_ok, ring_ok;
    // direct-to-LDS path; the delta mode only runs where the forward pass keeps no activations: other d, or more units than
    // a launch of the blocked forward passes can number
    if constexpr (MODE != kDelta) {
        if (a.d % BK == 0) {
            if (!arrol_allow_lds(&score_mlp_kernel<MODE, true>, kRingLdsBytes, ring_ok)) return ARROL_EHIP;
            arrol_launch((score_mlp_kernel<MODE, true>), grid, dim3(kThreads), kRingLdsBytes, st, a);
            return arrol_launch_status();
        }
    }
    if (!arrol_allow_lds(&score_mlp_kernel<MODE, false>, kLdsBytes, lds_ok)) return ARROL_EHIP;
    arrol_launch((score_mlp_kernel<MODE, false>), grid, dim3(kThreads), kLdsBytes, st, a);
    return arrol_launch_status();
}

}  // namespace

extern "C" size_t arrol_score_mlp_workspace_bytes(int32_t n_rows, int32_t d, int32_t m) {
    if (n_rows < 1 || d < 8 || m < 1) return 0;
    if (d % 64) return 0;   // the one-launch tile kernel needs no scratch
    return align256(sizeof(float) * static_cast<size_t>((m + 31) / 32) * n_rows);   // smallest unit blocks of the forward passes
}

extern "C" int arrol_score_mlp(const void* hidden, int64_t row_stride_elems, const int64_t* row_index,
                               const void* w1, const float* b1, const float* w2, float b2, int32_t n_rows,
                               int32_t d, int32_t m, float* score_out, float* prob_out, void* workspace,
                               size_t workspace_bytes, void* stream) {
    if (n_rows < 0 || d < 8 || (d & 7) || m < 1 || row_stride_elems < d || (row_stride_elems & 7)) return ARROL_EINVAL;
    if (n_rows == 0) return ARROL_OK;
    if (!hidden || !w1 || !w2 || !prob_out || !arrol_aligned16(hidden) || !arrol_aligned16(w1)) return ARROL_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t need = arrol_score_mlp_workspace_bytes(n_rows, d, m);
    const ForwardPath path = pick_score(n_rows, d, m, row_stride_elems, row_index != nullptr);
    if (path != kPathTile && workspace && arrol_aligned16(workspace) && workspace_bytes >= need) {
        float* partial = static_cast<float*>(workspace);
        const int rc = enqueue_forward(path, hidden, row_stride_elems, row_index, w1, b1, w2, n_rows, d, m, partial, nullptr, 0, st);
        if (rc != ARROL_OK) return rc;
        if (arrol_launch_failed()) return arrol_launch_status();
        const int ub = unit_block(path);
        arrol_launch(score_mlp_finish_kernel, dim3((n_rows + 255) / 256), dim3(256), 0, st, partial, (m + ub - 1) / ub,
                     n_rows, b2, score_out, prob_out);
        return arrol_launch_status();
    }
    MlpArgs a = {};
    a.hidden = static_cast<const uint16_t*>(hidden); a.row_stride = row_stride_elems; a.row_index = row_index;
    a.w1 = static_cast<const uint16_t*>(w1); a.a_stride = d; a.b1 = b1; a.w2 = w2; a.b2 = b2;
    a.n_rows = n_rows; a.d = d; a.m = m; a.score_out = score_out; a.prob_out = prob_out;
    return launch_mlp<kForward>(a, dim3((n_rows + BR - 1) / BR), st);
}

extern "C" size_t arrol_score_mlp_grad_workspace_bytes(int32_t n_rows, int32_t d, int32_t m, int32_t delta_terms) {
    if (n_rows < 1 || d < 8 || m < 1 || delta_terms < 1 || delta_terms > 2) return 0;
    return make_grad_plan(n_rows, d, m, delta_terms).total;
}

extern "C" int arrol_score_mlp_grad(const void* hidden, int64_t row_stride_elems, const int64_t* row_index,
                                    const void* w1, const float* b1, const float* w2, float b2,
                                    const float* labels, int32_t n_rows, int32_t d, int32_t m, float* loss_out,
                                    float* grad_w1, float* grad_b1, float* grad_w2, float* grad_b2,
                                    int32_t delta_terms, void* workspace, size_t workspace_bytes, void* stream) {
    if (n_rows < 0 || d < 8 || (d & 7) || m < 1 || row_stride_elems < d || (row_stride_elems & 7)) return ARROL_EINVAL;
    if (delta_terms < 1 || delta_terms > 2 || m > INT32_MAX / 2) return ARROL_EINVAL;
    if (!grad_w1 || !grad_b1 || !grad_w2) return ARROL_EINVAL;
    if (n_rows == 0) {   // empty batch: zero loss and gradients
        hipStream_t s0 = static_cast<hipStream_t>(stream);
        const int64_t width = static_cast<int64_t>(m) * d;
        arrol_launch(reduce_rows_f32_kernel<8>, dim3(static_cast<unsigned>((width + 31) / 32)), dim3(256), 0, s0,
                           nullptr, 0, width, width, 0.f, grad_w1);
        arrol_launch(reduce_rows_f32_kernel<8>, dim3((m + 31) / 32), dim3(256), 0, s0, nullptr, 0,
                           static_cast<int64_t>(m), static_cast<int64_t>(m), 0.f, grad_b1);
        arrol_launch(reduce_rows_f32_kernel<8>, dim3((m + 31) / 32), dim3(256), 0, s0, nullptr, 0,
                           static_cast<int64_t>(m), static_cast<int64_t>(m), 0.f, grad_w2);
        if (loss_out) arrol_launch(reduce_rows_f32_kernel<8>, dim3(1), dim3(256), 0, s0, nullptr, 0, 1, 1, 0.f, loss_out);
        if (grad_b2) arrol_launch(reduce_rows_f32_kernel<8>, dim3(1), dim3(256), 0, s0, nullptr, 0, 1, 1, 0.f, grad_b2);
        return arrol_launch_status();
    }
    if (!hidden || !w1 || !w2 || !labels || !arrol_aligned16(hidden) || !arrol_aligned16(w1)) return ARROL_EINVAL;
    const GradPlan p = make_grad_plan(n_rows, d, m, delta_terms);
    const int mt = delta_terms * m;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < p.total) return ARROL_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    float* score = reinterpret_cast<float*>(ws + p.off_score);
    float* prob = reinterpret_cast<float*>(ws + p.off_prob);
    float* resid = reinterpret_cast<float*>(ws + p.off_resid);
    float* bsum = reinterpret_cast<float*>(ws + p.off_bsum);
    const int n_rblocks = (n_rows + 1023) / 1024;
    uint16_t* ht = reinterpret_cast<uint16_t*>(ws + p.off_ht);
    uint16_t* dt = reinterpret_cast<uint16_t*>(ws + p.off_dt);                       // [hi; lo]: delta_terms * m rows
    uint16_t* dt_lo = delta_terms == 2 ? dt + static_cast<int64_t>(m) * p.n_pad : nullptr;
    float* unit = reinterpret_cast<float*>(ws + p.off_unit);
    float* slab = reinterpret_cast<float*>(ws + p.off_slab);

    // forward pass: relu(pre) is kept for the backward pass; only with d not a multiple of 64 the one-launch tile
    // kernel runs, whose pre-activations are recomputed below
    MlpArgs a = {};
    a.hidden = static_cast<const uint16_t*>(hidden); a.row_stride = row_stride_elems; a.row_index = row_index;
    a.w1 = static_cast<const uint16_t*>(w1); a.a_stride = d; a.b1 = b1; a.w2 = w2; a.b2 = b2;
    a.n_rows = n_rows; a.d = d; a.m = m; a.score_out = score; a.prob_out = prob;
    float* act = reinterpret_cast<float*>(ws + p.off_act);
    float* partial = reinterpret_cast<float*>(ws + p.off_small);
    const ForwardPath path = pick_forward(n_rows, d, m, row_stride_elems, row_index != nullptr);
    const bool kept = path != kPathTile;
    int rc;
    if (kept)
        rc = enqueue_forward(path, hidden, row_stride_elems, row_index, w1, b1, w2, n_rows, d, m, partial, act, p.n_pad, st);
    else
        rc = launch_mlp<kForward>(a, dim3(p.n_rb), st);
    if (rc != ARROL_OK) return rc;
    const int n_ub = (m + unit_block(path) - 1) / unit_block(path);
    if (arrol_launch_failed()) return arrol_launch_status();
    const bool in_place = wgrad_in_place(d, row_stride_elems, row_index != nullptr);
    const int n_pblocks = (n_rows + kPartRows - 1) / kPartRows;
    const bool sums_ride = in_place && p.w_rows != 256;
    const bool fused = kept && n_rows <= (sums_ride ? kFusedRows : kFusedRowsAlone) && static_cast<int64_t>(n_rows) * m <= kFusedSize;
    const MlpSums sums = {fused ? unit : nullptr, bsum, n_pblocks, n_rows, m, grad_w2, grad_b1, loss_out, grad_b2};
    const int n_groups = (m + kPartRows / ARROL_WAVE - 1) / (kPartRows / ARROL_WAVE);
    if (fused) {
        arrol_launch(mlp_score_delta_kernel, dim3(static_cast<unsigned>(n_pblocks) * n_groups), dim3(kPartRows), 0, st, partial, n_ub, b2, labels, act,
                     static_cast<int64_t>(p.n_pad), w2, n_rows, p.n_pad, m, n_groups, dt, dt_lo, unit, bsum);
        if (!sums_ride) arrol_launch(mlp_sums_kernel, dim3((m + 255) / 256, 2), dim3(256), 0, st, sums);
    } else if (kept) {
        // scores from the partials, residuals and loss terms in one launch; delta^T, the per-unit sums, the loss
        // and dL/db2 in the next
        arrol_launch(mlp_finish_residual_kernel, dim3(n_rblocks), dim3(1024), 0, st, partial, n_ub, b2, labels, n_rows,
                     resid, bsum);
        arrol_launch(mlp_delta_kernel, dim3(m), dim3(kDeltaThreads), 0, st, act, static_cast<int64_t>(p.n_pad), resid, w2,
                     n_rows, p.n_pad, dt, dt_lo, grad_w2, grad_b1, bsum, n_rblocks, loss_out, grad_b2);
    } else {
        arrol_launch(mlp_residual_kernel, dim3(n_rblocks), dim3(1024), 0, st, score, prob, labels, n_rows, resid, bsum);
        arrol_launch(mlp_residual_finish_kernel, dim3(1), dim3(1), 0, st, bsum, n_rblocks, n_rows, loss_out, grad_b2);
        a.resid = resid; a.delta_t = dt; a.delta_lo = dt_lo; a.delta_stride = p.n_pad; a.unit_partial = unit;
        rc = launch_mlp<kDelta>(a, dim3(p.n_rb), st);
        if (rc != ARROL_OK) return rc;
        arrol_launch(reduce_rows_f32_kernel<8>, dim3((m + 31) / 32), dim3(256), 0, st, unit, p.n_rb,
                     static_cast<int64_t>(2) * m, static_cast<int64_t>(m), 1.f, grad_w2);
        arrol_launch(reduce_rows_f32_kernel<8>, dim3((m + 31) / 32), dim3(256), 0, st, unit + m, p.n_rb,
                     static_cast<int64_t>(2) * m, static_cast<int64_t>(m), 1.f, grad_b1);
    }
    if (arrol_launch_failed()) return arrol_launch_status();
    const int64_t width = static_cast<int64_t>(m) * d;
    if (in_place) {
        // dL/dW1 = delta^T . H over the rollouts, the hidden states read in place
        float* rslab = reinterpret_cast<float*>(ws + p.off_rslab);
        MlpRingArgs g = {};
        // partials [K split][term][m][d] of terms as rows of their own are delta_terms * r_splits slabs of m * d values
        const bool stacked = p.w_rows == 256 || p.w_stacked;
        const int n_slabs = stacked ? p.r_splits * delta_terms : p.r_splits;
        g.a = dt; g.a_stride = static_cast<unsigned>(p.n_pad) * 2; g.a_rows = mt;
        g.b = a.hidden; g.b_stride = static_cast<unsigned>(row_stride_elems * 2);
        g.b_rows = d; g.b_k_rows = n_rows;
        g.n_k64 = (n_rows + 63) / 64; g.k64_per_split = p.r_k64_per_split;
        g.c_out = n_slabs > 1 ? rslab : grad_w1; g.c_stride = d;
        if (p.w_rows != 256) {
            g.a_rows = stacked ? mt : m;
            const int terms = stacked ? 1 : delta_terms;
            rc = p.w_rows == 64    ? launch_wgrad_mid<Wgrad64>(g, terms, p.r_splits, sums, st)
                 : p.w_groups == 2 ? launch_wgrad_mid<Wgrad128>(g, terms, p.r_splits, sums, st)
                                   : launch_wgrad_mid<Wgrad128Two>(g, terms, p.r_splits, sums, st);
            if (rc != ARROL_OK) return rc;
        } else {
            rc = launch_mlp_ring<kWgrad>(g, dim3(p.r_cb, p.r_gt, p.r_splits), st);
            if (rc != ARROL_OK) return rc;
        }
        if (n_slabs > 1)
            launch_reduce_slabs(rslab, n_slabs, width, grad_w1, st);
        return arrol_launch_status();
    }
    // gathered rows or d not a multiple of 64: H^T, then the tile kernel
    arrol_launch(mlp_transpose_kernel, dim3(p.n_pad / 64, (d + 63) / 64), dim3(256), 0, st,
                 a.hidden, row_stride_elems, row_index, n_rows, d, p.n_pad, ht);
    MlpArgs g = {};
    g.hidden = ht; g.row_stride = p.n_pad; g.row_index = nullptr;
    g.w1 = dt; g.a_stride = p.n_pad;
    const int n_slabs = p.splits * delta_terms;
    g.n_rows = d; g.d = p.n_pad; g.m = mt;
    g.c_out = n_slabs > 1 ? slab : grad_w1; g.c_stride = d; g.kc_per_split = p.kc_per_split;
    rc = launch_mlp<kWgrad>(g, dim3(p.n_cb, p.splits, p.n_groups), st);
    if (rc != ARROL_OK) return rc;
    if (n_slabs > 1)
        launch_reduce_slabs(slab, n_slabs, width, grad_w1, st);
    return arrol_launch_status();
}

extern "C" int arrol_score_mlp_kernels(int32_t n_rows, int32_t d, int32_t m, int64_t row_stride_elems, int32_t gathered,
                                       int32_t delta_terms, int32_t* forward, int32_t* weight_gradient, int32_t* splits) {
    if (n_rows < 1 || d < 8 || (d & 7) || m < 1 || row_stride_elems < d || delta_terms < 0 || delta_terms > 2 || !forward ||
        !weight_gradient || !splits)
        return ARROL_EINVAL;
    const auto pick = delta_terms ? pick_forward : pick_score;
    *forward = pick(n_rows, d, m, row_stride_elems, gathered != 0);
    *weight_gradient = -1;
    *splits = 0;
    if (delta_terms) {
        const GradPlan p = make_grad_plan(n_rows, d, m, delta_terms);
        const bool in_place = wgrad_in_place(d, row_stride_elems, gathered != 0);
        *weight_gradient = !in_place ? 0 : p.w_rows != 256 ? 1 : 2;
        *splits = in_place ? p.r_splits : p.splits;
    }
    return ARROL_OK;
}

extern "C" int arrol_score_mlp_tiles(int32_t n_rows, int32_t d, int32_t m, int64_t row_stride_elems, int32_t gathered,
                                     int32_t delta_terms, int32_t* forward_groups_out, int32_t* gradient_rows, int32_t* gradient_groups) {
    int32_t forward, gradient, splits;
    if (!forward_groups_out || !gradient_rows || !gradient_groups) return ARROL_EINVAL;
    const int rc = arrol_score_mlp_kernels(n_rows, d, m, row_stride_elems, gathered, delta_terms, &forward, &gradient, &splits);
    if (rc != ARROL_OK) return rc;
    *forward_groups_out = forward_groups(static_cast<ForwardPath>(forward), n_rows, d, m);
    *gradient_rows = 0;
    *gradient_groups = 0;
    if (gradient > 0) {
        const GradPlan p = make_grad_plan(n_rows, d, m, delta_terms);
        *gradient_rows = p.w_rows;
        *gradient_groups = p.w_rows == 256 ? 1 : p.w_groups;
    }
    return ARROL_OK;
}
