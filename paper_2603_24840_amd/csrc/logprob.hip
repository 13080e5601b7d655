// arrol_logprob: per-token log pi(o_t | o_<t) on the re-batched survivors
// (policy term of GRPO's importance ratio, Sec. 3; computed by the frontend on the
// survivors, Sec. 4.3 (ii), Alg. 1).
//
//   logprob_t = z_t[y_t] - logsumexp_v z_t[v],   z_t = W h_t
//
// One fused kernel: bf16 MFMA (v_mfma_f32_32x32x16_bf16) LM-head contraction with the
// vocabulary tiled, an online (running max / running sum) logsumexp and the target-logit
// capture applied to each accumulator tile while it is still in registers.  The [T, V]
// logits never reach memory.  The product is computed transposed, Z^T = W H^T, so that in
// the MFMA result layout a lane's 16 accumulator values of a 32x32 block belong to ONE token
// (column = lane % 32) and 16 different vocabulary rows: the softmax reduction over the
// vocabulary is then lane-local, and the only cross-lane work is one merge at the very end.
//
// Work decomposition: grid = token blocks (BN tokens) x vocabulary splits; a workgroup walks
// the vocabulary tiles (BM rows) of its split and, inside each, the K chunks (BK) of d.
// Every (split, token) writes a partial (max, sumexp, target logit); a small second kernel
// merges the splits.  Workgroup ids are mapped so that the workgroups resident on one XCD
// (ids congruent mod 8) form a (few token blocks) x (all splits) patch and share their
// H and W tiles through that XCD's L2.
#include <type_traits>

#include "common.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;  // finite stand-in for "no logit seen yet"
constexpr int kXcds = 8;
constexpr int kCuPerXcd = 32;
constexpr int kSplitsFirst = 8;      // see map_workgroup

template <int BM_, int BN_, int BK_, int WM_, int WN_>
struct Tile {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_;
    static constexpr int NT = WM * WN * ARROL_WAVE;       // threads per workgroup
    static constexpr int TM = BM / WM / 32;               // 32-row vocab blocks per wave
    static constexpr int TN = BN / WN / 32;               // 32-token blocks per wave
    static constexpr int CPR = BK / 8;                    // 16-byte chunks per tile row
    static constexpr int ROWS_PER_PASS = NT / CPR;
    static constexpr int PA = BM / ROWS_PER_PASS;         // load passes for the W tile
    static constexpr int PB = BN / ROWS_PER_PASS;         // load passes for the H tile
    static constexpr int STAGE_BYTES = (BM + BN) * BK * 2;
    static constexpr int LDS_BYTES = 2 * STAGE_BYTES;
    static_assert(BK == 64, "the LDS swizzle below assumes 128-byte tile rows");
    static_assert(BM % (WM * 32) == 0 && BN % (WN * 32) == 0, "wave tiles are made of 32x32 blocks");
    static_assert(BM % ROWS_PER_PASS == 0 && BN % ROWS_PER_PASS == 0 && ROWS_PER_PASS % 16 == 0, "load passes");
};

// Position of 16-byte chunk c of tile row r inside a [rows][64] bf16 LDS tile.  The XOR
// spreads the 16 rows that one quarter-wave reads at the same k over all 64 banks.
__device__ __forceinline__ int lds_chunk_offset(int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); }

struct LogprobArgs {
    const uint16_t* H;      // [T, d]
    const uint16_t* W;      // [V, d]
    const int32_t* targets; // [T]
    float* part;            // [n_sp][3][T]  (max, sumexp, target logit)
    int64_t T;
    int V, d;
    int n_tb, n_sp, n_vt;
    int band, n_long;       // work order: n_long bands of `band` token blocks, the rest one shorter (map_workgroup)
};

// Per-lane online-softmax state: the lane owns token (wave token base + j*32 + lane%32), j < TN.
template <int TN>
struct LaneState {
    float run_m[TN], run_s[TN], tgt_z[TN];
    int tgt[TN];
};

// Folds one finished accumulator tile into the running (max, sumexp, target logit) and clears it.
// acc[i][j][v] is the logit of vocab row vrow0 + i*32 + (v/4)*8 + lh*4 + v%4 for the lane's token of
// block j (MFMA 32x32 result layout); WROWS = vocab rows per wave tile.
template <int TM, int TN, int WROWS>
__device__ __forceinline__ void tile_epilogue(f32x16 (&acc)[TM][TN], LaneState<TN>& st, int vrow0, int V, int lh) {
    if (vrow0 + WROWS > V) {  // tile hangs over the end of the vocabulary
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const bool dead = vrow0 + i * 32 + (v >> 2) * 8 + lh * 4 + (v & 3) >= V;
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j][v] = dead ? -INFINITY : acc[i][j][v];
            }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int rel = st.tgt[j] - vrow0;
        const bool mine = rel >= 0 && rel < WROWS && ((rel >> 2) & 1) == lh;
        if (__any(mine)) {
            const int code = mine ? ((rel >> 5) * 16 + ((rel & 31) >> 3) * 4 + (rel & 3)) : -1;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (code == i * 16 + v) st.tgt_z[j] = acc[i][j][v];
        }
        float mx = acc[0][j][0];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc[i][j][v]);
        const float m_new = fmaxf(st.run_m[j], mx);
        const float neg = -m_new * kLog2e;
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                sum += __builtin_amdgcn_exp2f(fmaf(acc[i][j][v], kLog2e, neg));
                acc[i][j][v] = 0.f;
            }
        // difference first: exactly 0 when the maximum did not move (also for the -1e30 sentinel)
        st.run_s[j] = st.run_s[j] * __builtin_amdgcn_exp2f((st.run_m[j] - m_new) * kLog2e) + sum;
        st.run_m[j] = m_new;
    }
}

// End of a workgroup's vocabulary range: merge the two lane halves (same token, different vocab
// rows), then the WM waves that share a token range (through LDS, `red` = [WM][3][BN] floats, the
// staging memory being idle by now), and write the (max, sumexp, target logit) partial of split sp.
template <int TN, int WM, int WN, int BN, int NT>
__device__ __forceinline__ void write_partials(LaneState<TN>& st, float* red, int wm, int wn, int l31, int lh,
                                               int tid, int64_t tok0, int64_t T, int sp, float* part) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const float om = __shfl_xor(st.run_m[j], 32, ARROL_WAVE);
        const float os = __shfl_xor(st.run_s[j], 32, ARROL_WAVE);
        const float oz = __shfl_xor(st.tgt_z[j], 32, ARROL_WAVE);
        const float m = fmaxf(st.run_m[j], om);
        st.run_s[j] = st.run_s[j] * __builtin_amdgcn_exp2f((st.run_m[j] - m) * kLog2e) +
                      os * __builtin_amdgcn_exp2f((om - m) * kLog2e);
        st.run_m[j] = m;
        st.tgt_z[j] += oz;
    }
    if (lh == 0) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = wn * (BN / WN) + j * 32 + l31;
            red[(wm * 3 + 0) * BN + col] = st.run_m[j];
            red[(wm * 3 + 1) * BN + col] = st.run_s[j];
            red[(wm * 3 + 2) * BN + col] = st.tgt_z[j];
        }
    }
    __syncthreads();
    for (int col = tid; col < BN; col += NT) {
        const int64_t t = tok0 + col;
        if (t >= T) continue;
        float m = red[col], s = red[BN + col], z = red[2 * BN + col];
#pragma unroll
        for (int w = 1; w < WM; ++w) {
            const float om = red[(w * 3 + 0) * BN + col], os = red[(w * 3 + 1) * BN + col];
            const float mm = fmaxf(m, om);
            s = s * __builtin_amdgcn_exp2f((m - mm) * kLog2e) + os * __builtin_amdgcn_exp2f((om - mm) * kLog2e);
            m = mm;
            z += red[(w * 3 + 2) * BN + col];
        }
        float* p = part + static_cast<int64_t>(sp) * 3 * T + t;
        p[0] = m;
        p[T] = s;
        p[2 * T] = z;
    }
}

// The same for the 16x16x32 MFMA result layout: acc[i][j][v] is the logit of vocab row vrow0 + i*16 + lq*4 + v
// (lq = lane / 16) for the lane's token of block j (token j*16 + lane%16 of the wave's range).  The accumulators
// are left as they are (the next tile's first MFMAs take 0 as their addend).
template <int TI, int TJ, int WROWS>
__device__ __forceinline__ void tile_epilogue16(f32x4 (&acc)[TI][TJ], LaneState<TJ>& st, int vrow0, int V, int lq,
                                                const int (&tgt)[TJ]) {
    if (vrow0 + WROWS > V) {  // tile hangs over the end of the vocabulary
        const int lim = V - vrow0 - lq * 4;   // rows of this lane from here on are past the end: one value per tile,
#pragma unroll                                // compared with constants (nothing per (i, v) to keep in registers)
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const bool dead = i * 16 + v >= lim;
#pragma unroll
                for (int j = 0; j < TJ; ++j) acc[i][j][v] = dead ? -INFINITY : acc[i][j][v];
            }
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        const int rel = tgt[j] - vrow0;
        const bool mine = rel >= 0 && rel < WROWS && ((rel >> 2) & 3) == lq;
        if (__any(mine)) {
            const int code = mine ? ((rel >> 4) * 4 + (rel & 3)) : -1;
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (code == i * 4 + v) st.tgt_z[j] = acc[i][j][v];
        }
        float mx = acc[0][j][0];
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) mx = fmaxf(mx, acc[i][j][v]);
        const float m_new = fmaxf(st.run_m[j], mx);
        const float neg = -m_new * kLog2e;
        // of more than 8 rows in two sums: one of all 52 terms rounds more than 32 terms do, and waits on itself longer
        constexpr int kSums = TI > 8 ? 2 : 1;
        float part[kSums] = {};
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[v % kSums] += __builtin_amdgcn_exp2f(fmaf(acc[i][j][v], kLog2e, neg));
        const float sum = kSums == 2 ? part[0] + part[kSums - 1] : part[0];
        // difference first: exactly 0 when the maximum did not move (also for the -1e30 sentinel)
        st.run_s[j] = st.run_s[j] * __builtin_amdgcn_exp2f((st.run_m[j] - m_new) * kLog2e) + sum;
        st.run_m[j] = m_new;
        __builtin_amdgcn_sched_barrier(0);   // one token column at a time: keeps the temporaries of the exp chains few
    }
}

// End of a workgroup's vocabulary range, 16x16 layout: merge the four lane quarters (same token, different
// vocab rows), then the WM waves that share a token range through LDS, and write the partial of split sp.
template <int TJ, int WM, int WN, int BN, int NT>
__device__ __forceinline__ void write_partials16(LaneState<TJ>& st, float* red, int wm, int wn, int l15, int lq,
                                                 int tid, int64_t tok0, int64_t T, int sp, float* part) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
#pragma unroll
        for (int msk = 16; msk <= 32; msk <<= 1) {
            const float om = __shfl_xor(st.run_m[j], msk, ARROL_WAVE);
            const float os = __shfl_xor(st.run_s[j], msk, ARROL_WAVE);
            const float oz = __shfl_xor(st.tgt_z[j], msk, ARROL_WAVE);
            const float m = fmaxf(st.run_m[j], om);
            st.run_s[j] = st.run_s[j] * __builtin_amdgcn_exp2f((st.run_m[j] - m) * kLog2e) +
                          os * __builtin_amdgcn_exp2f((om - m) * kLog2e);
            st.run_m[j] = m;
            st.tgt_z[j] += oz;
        }
    }
    if (lq == 0) {
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            const int col = wn * (BN / WN) + j * 16 + l15;
            red[(wm * 3 + 0) * BN + col] = st.run_m[j];
            red[(wm * 3 + 1) * BN + col] = st.run_s[j];
            red[(wm * 3 + 2) * BN + col] = st.tgt_z[j];
        }
    }
    __syncthreads();
    for (int col = tid; col < BN; col += NT) {
        const int64_t t = tok0 + col;
        if (t >= T) continue;
        float m = red[col], s = red[BN + col], z = red[2 * BN + col];
#pragma unroll
        for (int w = 1; w < WM; ++w) {
            const float om = red[(w * 3 + 0) * BN + col], os = red[(w * 3 + 1) * BN + col];
            const float mm = fmaxf(m, om);
            s = s * __builtin_amdgcn_exp2f((m - mm) * kLog2e) + os * __builtin_amdgcn_exp2f((om - mm) * kLog2e);
            m = mm;
            z += red[(w * 3 + 2) * BN + col];
        }
        float* p = part + static_cast<int64_t>(sp) * 3 * T + t;
        p[0] = m;
        p[T] = s;
        p[2 * T] = z;
    }
}

// workgroup id -> (token block, vocab split).  Ids congruent mod 8 land on the same XCD, and a round of 256 workgroups
// (one per compute unit: the tile kernels take most of a unit's LDS) gives each XCD 32 consecutive positions of the work order
// (the last round spreads what is left evenly).  The order runs through bands of 5 to 8 token blocks, in
// each band with the split fastest where there are up to 8 (1.5-2 % faster than the other way round at 8,000 to 33,000
// tokens), the token block fastest otherwise (0.6 % at 4,096 tokens x 16 splits), so the 32 resident workgroups of an
// XCD are a patch of about 6 token blocks x 5 splits that shares its H and W tiles through the XCD's L2, for any
// number of token blocks.  Dealing token blocks to the XCDs instead leaves 6 of the 8 idle at 311 tokens (with
// 151,936 x 2048 in the ring kernel 1.00 ms, 0.26 this way) and makes every XCD read all of W up to some 10,000 tokens (1,000
// tokens: 1.00 ms and 0.50).
__device__ __forceinline__ bool map_workgroup(const LogprobArgs& a, int& tb, int& sp, int& vt_lo, int& vt_hi) {
    constexpr int kRound = kXcds * kCuPerXcd;
    const int round0 = static_cast<int>(blockIdx.x) / kRound * kRound, id = static_cast<int>(blockIdx.x) - round0;
    const int64_t left = static_cast<int64_t>(a.n_tb) * a.n_sp - round0;
    const int in_round = left < kRound ? static_cast<int>(left) : kRound;
    const int per_xcd = (in_round + kXcds - 1) / kXcds;
    const int pos = id % kXcds * per_xcd + id / kXcds;
    if (id / kXcds >= per_xcd || pos >= in_round) return false;
    int64_t w = static_cast<int64_t>(round0) + pos;
    // n_long bands of `band` token blocks, then bands of band - 1
    const int64_t in_long = static_cast<int64_t>(a.n_long) * a.band * a.n_sp;
    int tb0 = 0, size = a.band;
    if (w >= in_long) { w -= in_long; tb0 = a.n_long * a.band; --size; }
    const int64_t per_band = static_cast<int64_t>(size) * a.n_sp;
    const int b = static_cast<int>(w / per_band), r = static_cast<int>(w - b * per_band);
    const int tbi = a.n_sp <= kSplitsFirst ? r / a.n_sp : r % size;
    sp = a.n_sp <= kSplitsFirst ? r - tbi * a.n_sp : r / size;
    tb = tb0 + b * size + tbi;
    vt_lo = static_cast<int>(static_cast<int64_t>(a.n_vt) * sp / a.n_sp);
    vt_hi = static_cast<int>(static_cast<int64_t>(a.n_vt) * (sp + 1) / a.n_sp);
    return true;
}

// ---------------------------------------------------------------------------------------------
// General kernel (any d that is a multiple of 8): global -> registers -> LDS, two LDS stages.
// ---------------------------------------------------------------------------------------------
template <class C>
__global__ __launch_bounds__(C::NT) void logprob_kernel(LogprobArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int BM = C::BM, BN = C::BN, BK = C::BK, TM = C::TM, TN = C::TN;

    int tb, sp, vt_lo, vt_hi;
    if (!map_workgroup(a, tb, sp, vt_lo, vt_hi)) return;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int l31 = lane & 31, lh = lane >> 5;

    // ---- global -> register -> LDS staging geometry ---------------------------------------
    const int ld_c = tid % C::CPR;             // 16-byte chunk inside the 128-byte row segment
    const int ld_r = tid / C::CPR;             // tile row of pass 0
    const int ld_lds = lds_chunk_offset(ld_r, ld_c);  // rows of later passes differ by multiples of 16
    const int64_t tok0 = static_cast<int64_t>(tb) * BN;
    const int n_kc = (a.d + BK - 1) / BK;
    const int total_it = (vt_hi - vt_lo) * n_kc;

    uint4 stage[C::PA + C::PB];
    int ld_vt = vt_lo, ld_kc = 0;              // chunk the next issue_loads() fetches
    auto issue_loads = [&]() {
        const int k = ld_kc * BK + ld_c * 8;
        const bool k_ok = k < a.d;
        const int64_t v0 = static_cast<int64_t>(ld_vt) * BM;
#pragma unroll
        for (int p = 0; p < C::PA; ++p) {
            int64_t row = v0 + ld_r + p * C::ROWS_PER_PASS;
            row = row < a.V ? row : a.V - 1;
            stage[p] = k_ok ? *reinterpret_cast<const uint4*>(a.W + row * a.d + k) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < C::PB; ++p) {
            int64_t row = tok0 + ld_r + p * C::ROWS_PER_PASS;
            row = row < a.T ? row : a.T - 1;
            stage[C::PA + p] = k_ok ? *reinterpret_cast<const uint4*>(a.H + row * a.d + k) : make_uint4(0, 0, 0, 0);
        }
        if (++ld_kc == n_kc) { ld_kc = 0; ++ld_vt; }
    };
    auto store_stage = [&](int buf) {
        unsigned char* sa = lds + buf * C::STAGE_BYTES + ld_lds;
        unsigned char* sb = sa + BM * BK * 2;
#pragma unroll
        for (int p = 0; p < C::PA; ++p) *reinterpret_cast<uint4*>(sa + p * C::ROWS_PER_PASS * 128) = stage[p];
#pragma unroll
        for (int p = 0; p < C::PB; ++p) *reinterpret_cast<uint4*>(sb + p * C::ROWS_PER_PASS * 128) = stage[C::PA + p];
    };

    LaneState<TN> st;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        st.run_m[j] = kNegBig; st.run_s[j] = 0.f; st.tgt_z[j] = 0.f;
        const int64_t t = tok0 + wn * (BN / C::WN) + j * 32 + l31;
        st.tgt[j] = t < a.T ? a.targets[t] : -1;
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // fragment read offsets: row (wave base + i*32 + l31), chunk kk*2 + lh
    const int a_row0 = wm * (BM / C::WM) + l31;
    const int b_row0 = wn * (BN / C::WN) + l31;
    const int swz = (l31 >> 1) & 7;            // same for every 32-row block of the wave

    if (total_it > 0) {
        issue_loads();
        store_stage(0);
        __syncthreads();
    }
    int vt = vt_lo, kc = 0;
    for (int it = 0; it < total_it; ++it) {
        const bool more = it + 1 < total_it;
        if (more) issue_loads();
        const unsigned char* sa = lds + (it & 1) * C::STAGE_BYTES;
        const unsigned char* sb = sa + BM * BK * 2;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            const int coff = ((kk * 2 + lh) ^ swz) << 4;
            bf16x8 fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                fa[i] = *reinterpret_cast<const bf16x8*>(sa + (a_row0 + i * 32) * 128 + coff);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[j] = *reinterpret_cast<const bf16x8*>(sb + (b_row0 + j * 32) * 128 + coff);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        if (more) store_stage((it + 1) & 1);
        __syncthreads();

        if (++kc == n_kc) {
            tile_epilogue<TM, TN, BM / C::WM>(acc, st, vt * BM + wm * (BM / C::WM), a.V, lh);
            kc = 0;
            ++vt;
        }
    }
    write_partials<TN, C::WM, C::WN, BN, C::NT>(st, reinterpret_cast<float*>(lds), wm, wn, l31, lh, tid, tok0,
                                                 a.T, sp, a.part);
}

// ---------------------------------------------------------------------------------------------
// Fast kernel (d a multiple of 64): global -> LDS directly (no staging registers) into a ring of
// RING K32 slots (32 k-values = 64 bytes of each of the BM + BN tile rows); the contraction runs on
// v_mfma_f32_16x16x32_bf16, one whole K32 slot per instruction: 8 x 4 blocks of 16 vocabulary rows x 16 tokens
// per wave.  (In a register-only loop on random operands this shape sustains 2.0 PFLOP/s under the part's
// power limit, the 32x32x16 shape 1.8; the kernel as a whole gains 2-3 % on the workloads' data.)
//
// Loads always fetch whole 128-byte lines of a row, i.e. the two K32 halves that go to two
// consecutive slots (a "pair").  The L1 path moves 64 bytes per clock, so a pair costs as many L1
// cycles as half of its MFMA time; to keep that evenly spread, the W lines ("A") of a pair are
// requested during one K32 iteration and its H lines ("B") during the next, two load instructions before the
// iteration's barrier and two right behind it.  The pipeline per iteration i (chunk i lives in slot i % RING, its
// fragments are in registers when the iteration starts):
//   rows 0-2 of MFMAs (a row = one vocabulary block x the 4 token blocks); W fragment r of slot i+1 is read
//               into the registers of W fragment r as soon as row r has been issued (the W part of slot i+1
//               was certified one barrier earlier);
//   the wait for this wave's older loads, the workgroup barrier;
//   the H fragments of slot i+1 (certified just now) into the second H fragment set, then rows 3-7 with the
//               remaining W fragment reads between them: five rows of MFMAs cover the eight waves' reads
//               queueing on the LDS, so the matrix pipe never waits for an LDS round trip behind a barrier.
// The barrier inside iteration i certifies the W part of slot i+2 and the H part of slot i+1; every read of
// slot i has completed by then (they were issued during iteration i-1 and at the start of iteration i), so
// slot i is free for refilling from there on.
// The first chunk of every vocabulary tile takes the constant 0 as its MFMA addend, so the epilogue never
// clears the accumulators.
// (ring_nt.h holds the 32x32x16 form of this pipeline in a general form - row strides, K ranges, an epilogue
// after the walk - for the MLP head's kernels, which walk one tile per workgroup.)
// ---------------------------------------------------------------------------------------------
template <int BM_, int BN_, int WM_, int WN_>
struct RingTile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
    static constexpr int NT = WM * WN * ARROL_WAVE;
    static constexpr int NW = WM * WN;
    static constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    static constexpr int RING = 5;
    static constexpr int SLOT_BYTES = (BM + BN) * 64;
    static constexpr int LDS_BYTES = RING * SLOT_BYTES;
    static constexpr int G = BM / 16 / NW;                  // 16-row load groups per wave and operand
    static constexpr int LOADS = 2 * G;                     // load instructions per wave and iteration
    static_assert(BM == BN, "W and H tiles are loaded by the same code in alternate iterations");
    static_assert(BM % (16 * NW) == 0, "whole 16-row load groups per wave");
    static_assert(LOADS == 4, "the hand-placed schedule below");
};

template <int N>
__device__ __forceinline__ void wait_vmcnt() {  // s_waitcnt vmcnt(N) only (gfx9 encoding: bits 3:0 and 15:14), N <= 63
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

template <class C>
__global__ __launch_bounds__(C::NT) void logprob_ring_kernel(LogprobArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int BM = C::BM, BN = C::BN, RING = C::RING;
    constexpr int TI = BM / C::WM / 16, TJ = BN / C::WN / 16;   // 16 x 16 blocks per wave: vocabulary x tokens
    typedef __attribute__((address_space(3))) void* lds_ptr_t;

    int tb, sp, vt_lo, vt_hi;
    if (!map_workgroup(a, tb, sp, vt_lo, vt_hi)) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int l15 = lane & 15, lq = lane >> 4;
    const int64_t tok0 = static_cast<int64_t>(tb) * BN;
    const int n_k64 = a.d / 64;

    // ---- loader geometry: one instruction moves 16 rows x 64 bytes; lane -> (row lane/4, physical
    //      16-byte position lane%4), which holds logical chunk (lane%4) ^ g(row), g(row) = 2 * ((row/4)%2)
    //      (see the fragment reads) -----------
    const int ld_row = lane >> 2;
    const int ld_kb = ((lane & 3) ^ (((lane >> 4) & 1) << 1)) * 16;   // byte offset inside the K32 half
    // Addresses are (wave-uniform 64-bit base in SGPRs) + (per-lane 32-bit byte offset): the base
    // carries tile and K position, the lane offset the row inside the tile (clamped at the end of the
    // vocabulary / token range, so every load stays inside W and H) and the swizzled chunk.
    const int64_t row_bytes = static_cast<int64_t>(a.d) * 2;
    const int64_t tile_bytes = BM * row_bytes;
    unsigned a_voff[C::G], b_voff[C::G];
    {
        const int rows_valid = static_cast<int>(a.T - tok0 < BN ? a.T - tok0 : BN);
#pragma unroll
        for (int g = 0; g < C::G; ++g) {
            int r = (wave * C::G + g) * 16 + ld_row;
            r = r < rows_valid ? r : rows_valid - 1;
            b_voff[g] = static_cast<unsigned>(r) * static_cast<unsigned>(row_bytes) + ld_kb;   // < 256 rows x 16 KiB
        }
    }
    auto point_at_tile = [&](int vt) {
        const int left = a.V - vt * BM;                                      // vt * BM < V + BM: no overflow
        const int rows_valid = left < BM ? (left > 0 ? left : 1) : BM;       // left <= 0 only past the last pair
#pragma unroll
        for (int g = 0; g < C::G; ++g) {
            int r = (wave * C::G + g) * 16 + ld_row;
            r = r < rows_valid ? r : rows_valid - 1;
            a_voff[g] = static_cast<unsigned>(r) * static_cast<unsigned>(row_bytes) + ld_kb;
        }
    };
    // two load streams, each walking the pairs (pair = two K32 slots = one 128-byte line per row) of the
    // workgroup's vocabulary range: W lines (A) and H lines (B).  Past the last pair both keep requesting lines
    // that exist (W: the last line again; H: its tile from the start) into ring slots nobody reads any more,
    // so the loop below needs no variant without loads.
    int a_vt = vt_lo, a_k64 = 0, a_slot = 0;
    int b_k64 = 0, b_slot = 0;
    const char* a_base = reinterpret_cast<const char*>(a.W) + a_vt * tile_bytes;
    const char* b_base = reinterpret_cast<const char*>(a.H) + tok0 * row_bytes;
    point_at_tile(a_vt);
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((lds_ptr_t)lds));
    // The q-th (q = 2*g + h) of the LOADS load instructions of a group: 16-row group g of this wave, K32
    // half h (-> first / second slot of the pair).  `stream` picks W lines or H lines at compile time.  Written as asm
    // so that the compiler keeps its own LDS wait counters exact; completion is tracked by hand with
    // s_waitcnt vmcnt + the workgroup barrier.
    auto issue_one = [&](auto stream, int q) {
        constexpr bool is_b = decltype(stream)::value;
        const int g = q >> 1, h = q & 1;
        const int slot0 = is_b ? b_slot : a_slot;
        const int s_h = h == 0 ? slot0 : (slot0 + 1 == RING ? 0 : slot0 + 1);
        const int r0 = (wave * C::G + g) * 16;
        const unsigned dst = lds0 + s_h * C::SLOT_BYTES + (is_b ? BM * 64 : 0) + r0 * 64;
        const char* base = (is_b ? b_base : a_base) + h * 64;
        const unsigned voff = is_b ? b_voff[g] : a_voff[g];
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(dst) : "memory");
    };
    auto advance = [&](auto stream) {
        constexpr bool is_b = decltype(stream)::value;
        if (is_b) {
            b_base += 128;
            if (++b_k64 == n_k64) { b_k64 = 0; b_base -= row_bytes; }   // next vocabulary tile: H rewinds
            b_slot = b_slot + 2 >= RING ? b_slot + 2 - RING : b_slot + 2;
        } else {
            if (a_vt < vt_hi) {
                a_base += 128;
                if (++a_k64 == n_k64) {   // next vocabulary tile: W moves on by a tile minus the row just walked
                    a_k64 = 0;
                    ++a_vt;
                    if (a_vt < vt_hi) {
                        a_base += tile_bytes - row_bytes;
                        point_at_tile(a_vt);
                    } else {
                        a_base -= 128;   // past the last pair: keep requesting the last line (nobody reads that slot any more)
                    }
                }
            }
            a_slot = a_slot + 2 >= RING ? a_slot + 2 - RING : a_slot + 2;
        }
    };
    auto issue_group = [&](auto stream) {
#pragma unroll
        for (int q = 0; q < C::LOADS; ++q) issue_one(stream, q);
        advance(stream);
    };
    constexpr std::false_type kA{};   // W lines
    constexpr std::true_type kB{};    // H lines

    LaneState<TJ> st;
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        st.run_m[j] = kNegBig; st.run_s[j] = 0.f; st.tgt_z[j] = 0.f;
    }
    // tokens of this wave: tok_wave + 0 .. 63; the first tgt_valid of them exist (both wave-uniform)
    const int64_t tok_wave = tok0 + wn * (BN / C::WN);
    const int32_t* tgt_wave = a.targets + (tok_wave < a.T ? tok_wave : 0);
    const int tgt_valid = tok_wave < a.T ? static_cast<int>(a.T - tok_wave < BN / C::WN ? a.T - tok_wave : BN / C::WN) : 0;
    f32x4 acc[TI][TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

    // fragment reads: one MFMA takes the whole K32 of a slot: row (wave base + i*16 + lane%16), 16-byte chunk
    // lane/16 at position chunk ^ g(row).  Measured on the device: a 128-bit LDS read serves per cycle the 16
    // lanes that share lane bit 5 and the parity of lane bits 2, 3, 4, so two lanes of a half-wave that fall on
    // the same 16-byte bank group must differ in an odd number of those bits.  Here the bank group is
    // (row%4, position) = (l1 l0, l5 ^ l2, l4): the two lanes of a half-wave that share one differ in l3 alone.
    // (The 32x32 kernel's swizzle (row/4)%4 makes them differ in l2 and l4: two-way conflicts on every read.)
    const int swz = ((l15 >> 2) & 1) << 1;
    const int a_off = (wm * (BM / C::WM) + l15) * 64 + ((lq ^ swz) << 4);
    const int b_off = BM * 64 + (wn * (BN / C::WN) + l15) * 64 + ((lq ^ swz) << 4);
    bf16x8 fa[TI], fbe[TJ], fbo[TJ];   // W fragments (reloaded row by row), H fragments of even / odd iterations
    auto read_a = [&](const unsigned char* base, int i) {
        fa[i] = *reinterpret_cast<const bf16x8*>(base + a_off + i * 16 * 64);
    };
    auto read_b = [&](bf16x8 (&fb)[TJ], const unsigned char* base, int j) {
        fb[j] = *reinterpret_cast<const bf16x8*>(base + b_off + j * 16 * 64);
    };

    // Load schedule (pair p = chunks 2p, 2p+1 -> slots 2p % RING, (2p+1) % RING):
    //   up front           A(0), B(0), A(1)
    //   iteration 2p-2     B(p)   (even iterations, p >= 1)
    //   iteration 2p-3     A(p)   (odd iterations,  p >= 2)
    // The barrier inside iteration i needs every group requested before iteration i to have landed
    // (W part of slot i+2, H part of slot i+1), i.e. only this iteration's own loads may be in flight.
    issue_group(kA); issue_group(kB); issue_group(kA);
    wait_vmcnt<C::LOADS>();
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TJ; ++j) read_b(fbe, lds, j);
#pragma unroll
    for (int i = 0; i < TI - 2; ++i) read_a(lds, i);
    int slot = 0;
    // One K32 chunk: 32 MFMAs, vocabulary block by vocabulary block.  W fragment i of the next slot (its W part
    // was certified one barrier earlier) is read into fa[i] once row i of MFMAs has been issued - the last two
    // only at the start of the next iteration, long before their rows.  The workgroup barrier sits after the third
    // row; the H fragments of the next slot are read right after it into the other fragment set, with five rows of
    // MFMAs to cover the 8 waves' reads queueing on the LDS.  Two of the four loads go out before the barrier and
    // two right behind it: of the placements tried at the benchmark sizes (all four before it, barrier after row
    // 1 ... 5, loads spread over the rows) this one was the fastest on the workloads' data (+4-6 % over all four
    // before a barrier after row 3) and fetched the fewest bytes from beyond the L2; on all-zero operands it is 8 %
    // slower than that one.  Even iterations (stream = H lines) compute on fbe, odd ones on fbo.
    // `first`: first chunk of a vocabulary tile - the addend is the constant 0, so the accumulators are never cleared.
    auto iteration = [&](auto stream, auto first) {
        constexpr bool is_b = decltype(stream)::value;
        constexpr bool is_first = decltype(first)::value;
        const unsigned char* cur = lds + slot * C::SLOT_BYTES;
        slot = slot + 1 == RING ? 0 : slot + 1;
        const unsigned char* nxt = lds + slot * C::SLOT_BYTES;
        bf16x8 (&fb)[TJ] = is_b ? fbe : fbo;
        bf16x8 (&fbn)[TJ] = is_b ? fbo : fbe;
        // consecutive MFMAs always share an operand: token blocks ascend on even rows and descend on odd ones
        // (in a register-only loop under the power limit this order sustained 4 % more than plain row-major)
        auto row = [&](int i) {
#pragma unroll
            for (int jj = 0; jj < TJ; ++jj) {
                const int j = (i & 1) ? TJ - 1 - jj : jj;
                if constexpr (is_first) {
                    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], zero, 0, 0, 0);
                } else {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
                }
            }
        };
        read_a(cur, 6); read_a(cur, 7);
        __builtin_amdgcn_sched_barrier(0);
        row(0);
        __builtin_amdgcn_sched_barrier(0);
        read_a(nxt, 0);
        issue_one(stream, 0);
        issue_one(stream, 1);
        __builtin_amdgcn_sched_barrier(0);
        row(1);
        __builtin_amdgcn_sched_barrier(0);
        read_a(nxt, 1);
        __builtin_amdgcn_sched_barrier(0);
        row(2);
        __builtin_amdgcn_sched_barrier(0);
        // everything this wave requested before this iteration has landed (vmcnt counts in order: its two loads of
        // this iteration may fly, the two it issued behind the previous barrier may not); its own LDS reads are
        // complete (the last one was issued a row of MFMAs ago); then all waves agree
        wait_vmcnt<2>();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0) only
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TJ; ++j) read_b(fbn, nxt, j);                    // H part of slot i+1: certified just now
        __builtin_amdgcn_sched_barrier(0);
        row(3);
        __builtin_amdgcn_sched_barrier(0);
        read_a(nxt, 2);                                                      // behind every wave's H reads in the LDS queue
        issue_one(stream, 2);
        issue_one(stream, 3); advance(stream);
        __builtin_amdgcn_sched_barrier(0);
        row(4);
        __builtin_amdgcn_sched_barrier(0);
        read_a(nxt, 3);
        __builtin_amdgcn_sched_barrier(0);
        row(5);
        __builtin_amdgcn_sched_barrier(0);
        read_a(nxt, 4); read_a(nxt, 5);
        __builtin_amdgcn_sched_barrier(0);
        row(6);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_sched_barrier(0);
        row(7);
        __builtin_amdgcn_sched_barrier(0);
        // (the scheduling fence after the last row matters: without it the compiler lets the next iteration's first
        // reads drift up into this one and the kernel loses 10 %)
    };
    static_assert(TI == 8 && TJ == 4, "the hand-placed schedule above");
    for (int vt = vt_lo; vt < vt_hi; ++vt) {
        iteration(kB, std::true_type{});
        iteration(kA, std::false_type{});
        for (int k = 1; k < n_k64; ++k) {
            iteration(kB, std::false_type{});
            iteration(kA, std::false_type{});
        }
        {
            // the lane's targets are fetched again for every tile (from cache) instead of living in registers through
            // the K loop: tgt_wave (wave-uniform) points at the wave's first token, of which tgt_valid exist
            int tgt[TJ];
#pragma unroll
            for (int j = 0; j < TJ; ++j) tgt[j] = j * 16 + l15 < tgt_valid ? tgt_wave[j * 16 + l15] : -1;
            tile_epilogue16<TI, TJ, BM / C::WM>(acc, st, vt * BM + wm * (BM / C::WM), a.V, lq, tgt);
        }
        // The fragments of the next chunk are read again here rather than kept across the epilogue: held, their
        // 64 registers pushed the epilogue into scratch memory, whose latency nothing hides (every wave of the
        // workgroup is in its epilogue at the same time).  The slot is certified and not yet released.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        {
            const unsigned char* nxt = lds + slot * C::SLOT_BYTES;
#pragma unroll
            for (int j = 0; j < TJ; ++j) read_b(fbe, nxt, j);
#pragma unroll
            for (int i = 0; i < TI - 2; ++i) read_a(nxt, i);   // the last two: at the start of the iteration
        }
    }
    wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __syncthreads();   // every fragment read and every load into LDS has finished
    write_partials16<TJ, C::WM, C::WN, BN, C::NT>(st, reinterpret_cast<float*>(lds), wm, wn, l15, lq, tid, tok0,
                                                   a.T, sp, a.part);
}

// ---------------------------------------------------------------------------------------------
// Block kernel (d a multiple of 64, up to some 600 tokens): 16 TI WM vocabulary rows x 64 TJ tokens per workgroup of WM x 4
// wavefronts (WM is 2, of the 208 x 256 form 1): other forms of the tile above for batches that would leave much of a 256-token block empty
// or of the chip idle.
//
// What bounds it is the bytes in flight: W comes from HBM, every line once, some 1.2 us away under load; the loads of a
// wavefront complete in order, so H's, from the L2, wait behind them; and the LDS holds under three K64 steps.  So a step
// ("pair" of K32 chunks, slots of whole 128-byte lines per operand, NA of W and NB of H) has one barrier, and everything
// that hides latency hangs on it: all fragments of the next chunk are read ahead into a second register set, so that at the
// barrier of pair p (in its second chunk, behind row BAR of MFMAs) both of pair p's slots are free, and the loads of H(p + NB)
// and W(p + NA) all go out right behind it.  The barrier certifies pair p + 1.
// Every split starts at another place of the K extent and wraps around: all of them at the same offset of rows a power of
// two apart meet in the same memory channels (128 tokens: 151 us against 119).
//
// Measured at 151,936 x 2048, all on one card and as HIP graphs (before: for up to 128 tokens W straight to registers, else the
// ring kernel; other cards and a profiler's run differ by up to 5 %): 64 tokens 134 -> 111 us (5.6 TB/s of W), 128: 153 -> 119,
// 192: 177 -> 136, 311: 262 -> 193, 384: 264 -> 222.  At 311 tokens with W always
// from the L2 it would be 160, without any loads 130.  Tried and slower: W and H fetched by different wavefronts, each with
// its own order (311 tokens: 242); W straight to registers, several steps ahead (128 tokens: 148; half lines at a time).
//
// 208 x 256 (WM = 1, four wavefronts with the registers of a SIMD each) is for 193 to 256 tokens (and two blocks of them) where it needs no
// more rounds of workgroups than the ring kernel: with an lm_head beyond 256 MiB, vocabularies of 40,961 to 53,248, 81,921 to 106,496 and
// 131,073 to 159,744 rows, so 151,936 but not 128,256.  There 256 x 256 tiles leave room for two K64 steps and the ring kernel, in
// 32-column slots of them, waits for W.  13 x 4 MFMAs a chunk fill the registers with one set of W's
// fragments, so a fragment's successor is read over it; three steps of W fit the LDS.  At 151,936 x 2048 and 200 / 256 tokens 171 / 171 ->
// 158 / 158 us (ring kernel before), 100,352 x 2048 119 / 125 -> 106 / 107, 49,152 x 4096 124 / 121 -> 98 / 102, 50,000 x 3072 with 512 152 -> 139.
// Of the 158, 119 are left without loads and 138 with W from the L2.  (The compiler keeps 139 scalars of it in vector registers; a step reads two
// back.)  In the same manner 208 x 320 spills, 160 x 320 gains 2 % at 311
// tokens and loses 3 at others, and tiles of even shares of 16-row units instead of 208 rows and a short last round gain nothing.
//
// Slot layout: 16-byte chunk c of row r sits at position c ^ (r & 6) of its 128-byte row: by the serving rule given at the
// ring kernel's fragment reads, lanes that share a bank group differ in lane bit 3 alone: no conflicts.
// ---------------------------------------------------------------------------------------------
template <int TI_, int TJ_, int NA_, int NB_, int WM_ = 2>
struct BlockTile {
    static constexpr int TI = TI_, TJ = TJ_, NA = NA_, NB = NB_;
    static constexpr int WM = WM_, WN = 4, NW = WM * WN, NT = NW * ARROL_WAVE;
    static constexpr int BM = 16 * TI * WM, BN = 16 * TJ * WN;
    static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128;   // one slot: K64 of an operand
    static constexpr int LDS_BYTES = NA * A_BYTES + NB * B_BYTES;
    static constexpr int GA = BM / 8;                              // load instructions (8 rows x 128 bytes) per slot of W
    static constexpr int LA = (GA + NW - 1) / NW, LB = BN / 8 / NW, L = LA + LB;   // per wavefront; surplus ones repeat the last
    static constexpr bool ONE_SET = WM == 1;                       // of W's fragments: of two, 13 rows x 4 would not fit the registers
    static constexpr int BAR = TI >= 8 ? 1 : 0;
    static constexpr int PER_ROW = 3;                              // loads behind each row of MFMAs from BAR on
    // in flight at the barrier of pair p + 1: what was requested after H(p + 2)
    static constexpr int FLY = (NA > NB ? LA : 0) + (NB - 2) * L;
    static_assert(LDS_BYTES <= 163840 && WM * 3 * BN * 4 <= LDS_BYTES, "LDS (write_partials16 needs the latter)");
    static_assert(NB >= 2 && (NA == NB || NA == NB + 1), "order of the loads");
    static_assert((TI - BAR) * PER_ROW >= L, "all loads in the second chunk");
};

template <class C, bool STREAM = false>   // STREAM: W's lines come from memory, and are read once but for a workgroup's last NA slots (kStreamElements)
__global__ __launch_bounds__(C::NT) void logprob_block_kernel(LogprobArgs a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int BM = C::BM, BN = C::BN, TI = C::TI, TJ = C::TJ, NA = C::NA, NB = C::NB, L = C::L;
    typedef __attribute__((address_space(3))) void* lds_ptr_t;

    int tb, sp, vt_lo, vt_hi;
    if (!map_workgroup(a, tb, sp, vt_lo, vt_hi)) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int l15 = lane & 15, lq = lane >> 4;
    const int64_t tok0 = static_cast<int64_t>(tb) * BN;
    const int n_k64 = a.d / 64;

    // ---- loader: lane -> (row lane/8 of an 8-row group, position lane%8); rows past the end repeat the last one
    const unsigned ld_kb = ((lane & 7) ^ ((lane >> 3) & 6)) * 16;
    const int64_t row_bytes = static_cast<int64_t>(a.d) * 2;
    const int64_t tile_bytes = BM * row_bytes;
    unsigned a_voff[C::LA], b_voff[C::LB];
    auto a_group = [&](int q) { const int g = wave * C::LA + q; return g < C::GA ? g : C::GA - 1; };
    auto point_at_tile = [&](int vt) {
        const int left = a.V - vt * BM, last = (left < BM ? left : BM) - 1;
#pragma unroll
        for (int q = 0; q < C::LA; ++q) {
            const int r = a_group(q) * 8 + (lane >> 3);
            a_voff[q] = static_cast<unsigned>(r < last ? r : last) * static_cast<unsigned>(row_bytes) + ld_kb;
        }
    };
    {
        const int last = static_cast<int>(a.T - tok0 < BN ? a.T - tok0 : BN) - 1;
#pragma unroll
        for (int q = 0; q < C::LB; ++q) {
            const int r = (wave * C::LB + q) * 8 + (lane >> 3);
            b_voff[q] = static_cast<unsigned>(r < last ? r : last) * static_cast<unsigned>(row_bytes) + ld_kb;
        }
    }
    const int k_start = sp % n_k64;
    int a_vt = vt_lo, a_k = k_start, a_slot = 0, b_k = k_start, b_slot = 0;
    const char* a_base = reinterpret_cast<const char*>(a.W) + vt_lo * tile_bytes + k_start * 128;
    const char* b_base = reinterpret_cast<const char*>(a.H) + tok0 * row_bytes + k_start * 128;
    point_at_tile(vt_lo);
    const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<size_t>((lds_ptr_t)lds));
    // the n-th load instruction of a pair: its H lines, then its W lines
    auto issue_one = [&](int n) {
        const bool b = n < C::LB;
        const unsigned dst = b ? lds0 + NA * C::A_BYTES + b_slot * C::B_BYTES + (wave * C::LB + n) * 1024
                               : lds0 + a_slot * C::A_BYTES + a_group(n - C::LB) * 1024;
        const unsigned voff = b ? b_voff[b ? n : 0] : a_voff[b ? 0 : n - C::LB];
        if (!b && STREAM) asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(a_base), "s"(dst) : "memory");
        else asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(b ? b_base : a_base), "s"(dst) : "memory");
    };
    auto advance_a = [&]() {
        a_slot = a_slot + 1 == NA ? 0 : a_slot + 1;
        a_base += 128;
        if (++a_k == n_k64) { a_k = 0; a_base -= row_bytes; }
        if (a_k == k_start && a_vt + 1 < vt_hi) {      // past the last tile: its lines again, into slots nobody reads
            if (C::ONE_SET) asm volatile("");          // a branch: here the compiler would form the next tile's offsets every time
            a_base += tile_bytes;
            point_at_tile(++a_vt);
        }
    };
    auto advance_b = [&]() {
        b_slot = b_slot + 1 == NB ? 0 : b_slot + 1;
        b_base += 128;
        if (++b_k == n_k64) { b_k = 0; b_base -= row_bytes; }
    };

    LaneState<TJ> st;
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        st.run_m[j] = kNegBig; st.run_s[j] = 0.f; st.tgt_z[j] = 0.f;
    }
    // tokens of this wave: tok_wave + 0 .. 16 TJ - 1; the first tgt_valid of them exist (both wave-uniform)
    const int64_t tok_wave = tok0 + wn * (BN / C::WN);
    const int32_t* tgt_wave = a.targets + (tok_wave < a.T ? tok_wave : 0);
    const int tgt_valid = tok_wave < a.T ? static_cast<int>(a.T - tok_wave < BN / C::WN ? a.T - tok_wave : BN / C::WN) : 0;
    f32x4 acc[TI][TJ];
    const unsigned f_off[2] = {static_cast<unsigned>(l15 * 128 + ((lq ^ (l15 & 6)) << 4)),
                               static_cast<unsigned>(l15 * 128 + (((lq + 4) ^ (l15 & 6)) << 4))};
    bf16x8 fa[C::ONE_SET ? 1 : 2][TI], fb[2][TJ];   // fragments of a pair's first / second chunk
    auto read_a = [&](int slot, int h, int i) {
        fa[C::ONE_SET ? 0 : h][i] = *reinterpret_cast<const bf16x8*>(lds + (f_off[h] + slot * C::A_BYTES + wm * (BM / C::WM) * 128) + i * 2048);
    };
    auto read_b = [&](int slot, int h, int j) {
        fb[h][j] = *reinterpret_cast<const bf16x8*>(lds + (f_off[h] + NA * C::A_BYTES + slot * C::B_BYTES + wn * (BN / C::WN) * 128) + j * 2048);
    };
    // up front: W(0) where W has a slot more, then H(p), W(p + NA - NB) for every slot of H
    if (NA > NB) {
#pragma unroll
        for (int n = C::LB; n < L; ++n) issue_one(n);
        advance_a();
    }
#pragma unroll
    for (int p = 0; p < NB; ++p) {
#pragma unroll
        for (int n = 0; n < L; ++n) issue_one(n);
        advance_b();
        advance_a();
    }
    wait_vmcnt<C::FLY + L>();
    __syncthreads();
    int sa = 0, sb = 0;   // slots of the pair in work; from the start of its second chunk on, of the next
    auto read_first = [&]() {
#pragma unroll
        for (int j = 0; j < TJ; ++j) read_b(sb, 0, j);
#pragma unroll
        for (int i = 0; i < TI; ++i) read_a(sa, 0, i);
    };
    read_first();
    // One K32 chunk: TI rows of TJ MFMAs (token blocks in snake order, so that consecutive ones share an operand).
    // `first`: first chunk of a vocabulary tile - the addend is the constant 0, so the accumulators are never cleared.
    auto chunk = [&](auto second, auto first) {
        constexpr int h = decltype(second)::value ? 1 : 0, hn = 1 - h;
        if (h) { sa = sa + 1 == NA ? 0 : sa + 1; sb = sb + 1 == NB ? 0 : sb + 1; }
        auto mfma = [&](int i, int jj) {
            const int j = (i & 1) ? TJ - 1 - jj : jj;
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[C::ONE_SET ? 0 : h][i], fb[h][j], decltype(first)::value ? zero : acc[i][j], 0, 0, 0);
        };
        auto next_pair = [&]() {
            // the next pair has landed, for every wavefront, and everybody's fragments of this one are in registers
            wait_vmcnt<C::FLY>();
            __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0) only
            __syncthreads();
        };
        if constexpr (C::ONE_SET) {
            // One wavefront to a SIMD: nobody fills the matrix pipe while it issues anything else, so at most a read and a load follow each
            // MFMA.  A fragment of W is read over its predecessor once that one's row has been issued.
            constexpr int FROM = h ? C::BAR + 1 : 0;   // rows before the barrier
            static_assert((TI - C::BAR - 1) * TJ >= L && (TI - FROM) * TJ >= TJ + FROM, "all loads in the second chunk, all reads");
#pragma unroll
            for (int i = 0; i < TI; ++i) {
#pragma unroll
                for (int jj = 0; jj < TJ; ++jj) {
                    mfma(i, jj);
                    const int n = (i - FROM) * TJ + jj;     // MFMAs behind the barrier
                    if (n >= 0) {
                        if (h && n < L) issue_one(n);
                        if (n < TJ) read_b(sb, hn, n);
                        else if (n < TJ + FROM) read_a(sa, hn, n - TJ);
                        else if (i > FROM && jj == TJ - 1) read_a(sa, hn, i - 1);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (h && i == C::BAR) next_pair();
            }
            read_a(sa, hn, TI - 1);
            __builtin_amdgcn_sched_barrier(0);
            if (h) { advance_b(); advance_a(); }
            return;
        }
#pragma unroll
        for (int i = 0; i < TI; ++i) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int jj = 0; jj < TJ; ++jj) mfma(i, jj);
            __builtin_amdgcn_sched_barrier(0);
            if (i == C::BAR) {
                if (h) next_pair();
#pragma unroll
                for (int j = 0; j < TJ; ++j) read_b(sb, hn, j);
#pragma unroll
                for (int q = 0; q < (TI > 4 ? 2 : TI); ++q) read_a(sa, hn, q);
            }
            if (TI > 4 && i > C::BAR) {
                if (2 * (i - C::BAR) < TI) read_a(sa, hn, 2 * (i - C::BAR));
                if (2 * (i - C::BAR) + 1 < TI) read_a(sa, hn, 2 * (i - C::BAR) + 1);
            }
            if (h && i >= C::BAR) {
#pragma unroll
                for (int q = 0; q < C::PER_ROW; ++q)
                    if ((i - C::BAR) * C::PER_ROW + q < L) issue_one((i - C::BAR) * C::PER_ROW + q);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (h) { advance_b(); advance_a(); }
    };
    for (int vt = vt_lo; vt < vt_hi; ++vt) {
        chunk(std::false_type{}, std::true_type{});
        chunk(std::true_type{}, std::false_type{});
        for (int k = 1; k < n_k64; ++k) {
            chunk(std::false_type{}, std::false_type{});
            chunk(std::true_type{}, std::false_type{});
        }
        int tgt[TJ];
#pragma unroll
        for (int j = 0; j < TJ; ++j) tgt[j] = j * 16 + l15 < tgt_valid ? tgt_wave[j * 16 + l15] : -1;
        tile_epilogue16<TI, TJ, BM / C::WM>(acc, st, vt * BM + wm * (BM / C::WM), a.V, lq, tgt);
        // read again rather than kept across the epilogue; the slots are certified and not yet released
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        read_first();
    }
    wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __syncthreads();   // every fragment read and every load into LDS has finished
    write_partials16<TJ, C::WM, C::WN, BN, C::NT>(st, reinterpret_cast<float*>(lds), wm, wn, l15, lq, tid, tok0,
                                                   a.T, sp, a.part);
}

// Merges the splits.  256 / GROUPS tokens per workgroup, GROUPS lanes per token that take every GROUPS-th split and
// are merged through LDS in index order.  One lane per token walks the many splits of a short batch one dependent load
// after the other: at 64 tokens x 256 splits the whole call took 217 us, with 16 lanes 150 (up to 8 splits one lane is
// as fast and needs no merge).
template <int GROUPS>
__global__ __launch_bounds__(256) void logprob_finalize_kernel(
    const float* __restrict__ part, const int32_t* __restrict__ targets, int64_t T, int V, int n_sp,
    float* __restrict__ logprob_out, float* __restrict__ lse_out) {
    constexpr int TOK = 256 / GROUPS, UNROLL = 4;
    const int tok = threadIdx.x % TOK, grp = threadIdx.x / TOK;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * TOK + tok;
    float m = kNegBig, s = 0.f, z = 0.f;
    auto merge = [&](float om, float os, float oz) {
        const float mm = fmaxf(m, om);
        s = s * exp2f((m - mm) * kLog2e) + os * exp2f((om - mm) * kLog2e);
        m = mm;
        z += oz;
    };
    if (t < T) {
        for (int sp0 = grp; sp0 < n_sp; sp0 += GROUPS * UNROLL) {
            float om[UNROLL], os[UNROLL], oz[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int sp = sp0 + u * GROUPS;
                const float* p = part + static_cast<int64_t>(sp < n_sp ? sp : sp0) * 3 * T + t;
                om[u] = p[0]; os[u] = p[T]; oz[u] = p[2 * T];
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                if (sp0 + u * GROUPS < n_sp) merge(om[u], os[u], oz[u]);
        }
    }
    if (GROUPS > 1) {
        __shared__ float red[3][GROUPS][TOK];
        red[0][grp][tok] = m; red[1][grp][tok] = s; red[2][grp][tok] = z;
        __syncthreads();
        if (grp) return;
        for (int g = 1; g < GROUPS; ++g) merge(red[0][g][tok], red[1][g][tok], red[2][g][tok]);
    }
    if (t >= T) return;
    const float lse = m + logf(s);
    const int y = targets[t];
    logprob_out[t] = (y >= 0 && y < V) ? z - lse : __builtin_nanf("");
    if (lse_out) lse_out[t] = lse;
}

using MainTile = Tile<256, 256, 64, 2, 4>;
using FastTile = RingTile<256, 256, 2, 4>;
static_assert(MainTile::BM == FastTile::BM && MainTile::BN == FastTile::BN, "one plan serves both kernels");

using Block64 = BlockTile<8, 1, 4, 3>;     // 256 vocabulary rows x 64 tokens
using Block128 = BlockTile<8, 2, 3, 3>;    // 256 x 128
using Block192 = BlockTile<8, 3, 3, 2>;    // 256 x 192
using Block256 = BlockTile<13, 4, 3, 2, 1>; // 208 x 256
using Block320 = BlockTile<5, 5, 3, 2>;    // 160 x 320

enum LogprobForm { kFormRing, kForm64, kForm128, kForm192, kForm256, kForm320, kForms };
struct FormSize { int bm, bn; double step; };
// Vocabulary rows and tokens of a workgroup's tile; microseconds per K64 step of a tile when the chip is full, measured over
// 50,000 to 151,936 x 1024 to 4096 with up to 640 tokens (from there on the ring kernel's step falls to 1.45).
// They choose within 2 % of the best form at most of 15 vocabularies and widths x 14 token counts; the worst: 65,536 x 4096 with 250
// tokens (ring 170 us, 256 x 128 tiles 140), 65,536 x 2048 with 577 to 640 (256 x 192 and 160 x 320 170 us, the ring 159).
constexpr FormSize kFormSize[kForms] = {{FastTile::BM, FastTile::BN, 1.66}, {Block64::BM, Block64::BN, 1.15}, {Block128::BM, Block128::BN, 1.25},
                                        {Block192::BM, Block192::BN, 1.42}, {Block256::BM, Block256::BN, 1.45}, {Block320::BM, Block320::BN, 1.42}};
// The 208 x 256 form beats the ring kernel, where both take as many rounds, by 5 to 24 % while W comes from memory, and loses 3 to 10 % where
// the 256 MiB cache in front of it holds W from the call before (28 vocabularies and widths x 200, 256 and 512 tokens: 50,257 x 2048
// 51 -> 54 us, 100,003 x 1280 64 -> 67, 100,003 x 1536 90 -> 82, 151,936 x 1024 87 -> 83): it is taken from that size on.  Where other data
// passes between the calls a smaller W comes from memory too, and the line costs what it saves elsewhere: 256 tokens x 50,257 x 2048 after
// 1 GB read 80 -> 67 us, after 600 MB written 112 -> 86.
constexpr int64_t kCachedElements = 128 << 20;
// A W beyond 9/8 of that cache, read by one token block, is loaded past the caches (nt): they keep nothing of it for the next call, and H stays in the
// L2.  The same W again and again, us: 16 tokens x 151,936 x 4096 212 -> 188, 64 x 151,936 x 2048 112 -> 105 (5.9 TB/s), 128 x 122 -> 118,
// 192 x 139 -> 135, 311 x 214 -> 212, 300 x 128,256 x 4096 358 -> 352; just above the line (1,344 to 4,096 wide) 1 to 64 tokens 2 to 6 %, 128 2 to
// 4, 192 and 311 even; below it, where the cache has W, plain loads: 128 x 64,000 x 2048 would go 48 -> 51, 64 x 32,000 x 4096 45 -> 59.  After
// 600 MB written in between, which the plain loads have to push out of the cache: 64 x 73,984 x 2048 110 -> 70, and below the line
// 64 x 64,000 x 2048 would go 98 -> 56.  The 208 x 256 form and two token blocks (384 tokens) are even with it.
constexpr int64_t kStreamElements = kCachedElements / 8 * 9;
constexpr int kSmallestBM = Block320::BM, kLargestBN = Block320::BN, kBlockTokens = 640;

// The ring and block kernels give a lane its row of a tile as a 32-bit byte offset; of longer rows the general kernel's are 64-bit.
constexpr bool offsets_fit(int form, int d) {
    const FormSize f = kFormSize[form];
    return 2ll * d * ((f.bm > f.bn ? f.bm : f.bn) - 1) + 128 <= UINT32_MAX;
}

struct Plan { int form, n_tb, n_vt, n_sp, band, n_long; bool general, stream; };

// Vocabulary splits of n_tb token blocks x n_vt tiles, and what they cost, in tiles one after the other.
double pick_splits(int n_tb, int n_vt, int& n_sp) {
    constexpr int kRound = kXcds * kCuPerXcd;
    // A launch takes rounds of 256 workgroups x the vocabulary tiles of the longest split (plus about a quarter of a
    // tile's time per workgroup to start and finish).  Candidates: the split counts that just fill 1 ... 8 rounds, and
    // 4 ... 12.  Fewer than 6 splits widen an XCD's patch to more token blocks and fetch more operand slices per K
    // step (an eighth of a per cent each); where costs tie the smallest wins.  At 32,768 tokens this gives 6 (27.5 ms;
    // 12 splits: 28.5).  From 16 rounds on the last one no longer matters: 6, which at the benchmark shapes (T of
    // 290,000 to 2.4 million) measured 0.4-2.1 % faster than 4, 5, 7 or 8.
    if (static_cast<int64_t>(n_tb) * 6 >= 16 * kRound) {
        n_sp = n_vt < 6 ? n_vt : 6;
        return static_cast<double>(n_tb) * n_sp / kRound * ((n_vt + n_sp - 1) / n_sp);
    }
    double best = -1.0;
    n_sp = 1;
    for (int c = 0; c < 17; ++c) {
        int64_t sp = c < 9 ? c + 4 : static_cast<int64_t>(kRound) * (c - 8) / n_tb;
        if (sp > n_vt) sp = n_vt;
        if (sp < 1) continue;
        const int64_t tiles = (n_vt + sp - 1) / sp;
        if (sp > 12) sp = (n_vt + tiles - 1) / tiles;         // no more splits than the longest one needs
        const int64_t rounds = (n_tb * sp + kRound - 1) / kRound;
        const double slices = sp >= 6 ? 11.3 : sp + 32.0 / static_cast<double>(sp);
        const double cost = static_cast<double>(rounds) * (static_cast<double>(tiles) + 0.25) * (1.0 + 0.00125 * slices);
        if (best < 0.0 || cost < best || (cost == best && sp < n_sp)) { best = cost; n_sp = static_cast<int>(sp); }
    }
    return best;
}

Plan make_plan(int64_t T, int V, int d, int n_splits) {
    Plan p = {};
    // The form whose tiles come out cheapest.  At 151,936 x 2048: 64-, 128- and 192-token blocks for up to as many tokens,
    // 208 x 256 up to 256, 160 x 320 up to 320, 2 x 192 up to 384, the ring to 512 (262 us; 3 x 192: 308), 3 x 192 to 576.
    double best = -1.0;
    for (int f = 0; f < kForms; ++f) {
        if (f != kFormRing && (d % 64 || T > kBlockTokens || !offsets_fit(f, d))) continue;
        if (f == kForm256 && static_cast<int64_t>(V) * d <= kCachedElements) continue;
        const int n_tb = static_cast<int>((T + kFormSize[f].bn - 1) / kFormSize[f].bn), n_vt = (V + kFormSize[f].bm - 1) / kFormSize[f].bm;
        const int cap = (V + MainTile::BM - 1) / MainTile::BM;        // of splits given: <= n_vt for every form
        int sp = n_splits < cap ? n_splits : cap;
        double tiles;
        if (n_splits > 0)
            tiles = static_cast<double>((static_cast<int64_t>(n_tb) * sp + 255) / 256 * ((n_vt + sp - 1) / sp));
        else
            tiles = pick_splits(n_tb, n_vt, sp);
        const double cost = tiles * kFormSize[f].step;
        if (best < 0.0 || cost < best) { best = cost; p.form = f; p.n_tb = n_tb; p.n_vt = n_vt; p.n_sp = sp; }
    }
    p.general = d % 64 || !offsets_fit(p.form, d);
    p.stream = !p.general && p.form != kFormRing && p.form != kForm256 && p.n_tb == 1 && static_cast<int64_t>(V) * d > kStreamElements;
    const int bands = (p.n_tb + 3) / 6 > 1 ? (p.n_tb + 3) / 6 : 1;
    p.band = (p.n_tb + bands - 1) / bands;
    p.n_long = p.n_tb - (p.band - 1) * bands;
    return p;
}

template <void (*KERNEL)(LogprobArgs), class C>
int launch_logprob(dim3 grid, hipStream_t st, const LogprobArgs& a) {
    static arrol_device_flags lds_ok;
    if (!arrol_allow_lds(KERNEL, C::LDS_BYTES, lds_ok)) return ARROL_EHIP;
    arrol_launch(KERNEL, grid, dim3(C::NT), C::LDS_BYTES, st, a);
    return ARROL_OK;
}

template <class C>
int launch_block(bool stream, dim3 grid, hipStream_t st, const LogprobArgs& a) {
    return stream ? launch_logprob<logprob_block_kernel<C, true>, C>(grid, st, a) : launch_logprob<logprob_block_kernel<C>, C>(grid, st, a);
}

}  // namespace

extern "C" size_t arrol_logprob_workspace_bytes(int64_t T, int32_t V, int32_t d, int32_t n_splits) {
    if (T <= 0 || V < 1 || n_splits < 0) return 0;
    const Plan p = make_plan(T, V, d, n_splits);
    // Partials per token x tokens.  The plan's own split count falls from one batch to the next larger one, so the
    // answer for n_splits = 0 is what no smaller batch exceeds: a workspace sized for the largest batch serves all of
    // them.  make_plan takes up to 12 splits or, of few token blocks, 8 rounds of workgroups, and 6 from 16 rounds on.
    int64_t rows = static_cast<int64_t>(p.n_sp) * T;
    if (n_splits == 0) {
        constexpr int64_t kRound = kXcds * kCuPerXcd, kTwelve = 16 * kRound / 6 * MainTile::BN;   // tokens of 16 rounds
        int64_t most = 8 * kRound * kLargestBN;
        most = most > 6 * T ? most : 6 * T;
        const int64_t twelve = 12 * (T < kTwelve ? T : kTwelve);
        most = most > twelve ? most : twelve;
        const int64_t most_splits = (V + kSmallestBM - 1) / kSmallestBM;
        most = most < most_splits * T ? most : most_splits * T;
        rows = rows > most ? rows : most;
    }
    return (static_cast<size_t>(rows) * 3 * sizeof(float) + 255) & ~static_cast<size_t>(255);
}

extern "C" int arrol_logprob(const void* hidden, const void* lm_head, const int32_t* targets,
                             int64_t T, int32_t V, int32_t d, float* logprob_out, float* lse_out,
                             int32_t n_splits, void* workspace, size_t workspace_bytes, void* stream) {
    if (T < 0 || V < 1 || d < 8 || (d & 7) || n_splits < 0) return ARROL_EINVAL;
    if (T == 0) return ARROL_OK;
    if (!hidden || !lm_head || !targets || !logprob_out || !arrol_aligned16(hidden) || !arrol_aligned16(lm_head))
        return ARROL_EINVAL;
    const Plan p = make_plan(T, V, d, n_splits);
    // whole rounds of 256, then the rest spread over the 8 XCDs
    const int64_t grid = (static_cast<int64_t>(p.n_tb) * p.n_sp + kXcds - 1) / kXcds * kXcds;
    if (grid > INT32_MAX - 256 || static_cast<int64_t>(p.n_vt) * (d / 64) > INT32_MAX - 64) return ARROL_EINVAL;
    if (!workspace || !arrol_aligned16(workspace) || workspace_bytes < arrol_logprob_workspace_bytes(T, V, d, n_splits))
        return ARROL_EWORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    LogprobArgs a;
    a.H = static_cast<const uint16_t*>(hidden);
    a.W = static_cast<const uint16_t*>(lm_head);
    a.targets = targets;
    a.part = static_cast<float*>(workspace);
    a.T = T; a.V = V; a.d = d;
    a.n_tb = p.n_tb; a.n_sp = p.n_sp; a.n_vt = p.n_vt; a.band = p.band; a.n_long = p.n_long;
    const dim3 g(static_cast<unsigned>(grid));
    int rc;
    if (p.general) rc = launch_logprob<logprob_kernel<MainTile>, MainTile>(g, st, a);
    else if (p.form == kForm64) rc = launch_block<Block64>(p.stream, g, st, a);
    else if (p.form == kForm128) rc = launch_block<Block128>(p.stream, g, st, a);
    else if (p.form == kForm192) rc = launch_block<Block192>(p.stream, g, st, a);
    else if (p.form == kForm256) rc = launch_logprob<logprob_block_kernel<Block256>, Block256>(g, st, a);
    else if (p.form == kForm320) rc = launch_block<Block320>(p.stream, g, st, a);
    else rc = launch_logprob<logprob_ring_kernel<FastTile>, FastTile>(g, st, a);
    if (rc != ARROL_OK) return rc;
    if (arrol_launch_failed()) return arrol_launch_status();
    if (p.n_sp > 8)
        arrol_launch(logprob_finalize_kernel<16>, dim3(static_cast<unsigned>((T + 15) / 16)), dim3(256), 0, st,
                     static_cast<const float*>(workspace), targets, T, V, p.n_sp, logprob_out, lse_out);
    else
        arrol_launch(logprob_finalize_kernel<1>, dim3(static_cast<unsigned>((T + 255) / 256)), dim3(256), 0, st,
                     static_cast<const float*>(workspace), targets, T, V, p.n_sp, logprob_out, lse_out);
    return arrol_launch_status();
}

extern "C" int arrol_logprob_kernel(int64_t T, int32_t V, int32_t d, int32_t n_splits, int32_t* kernel, int32_t* tile_rows,
                                    int32_t* tile_tokens, int32_t* splits) {
    if (T < 1 || V < 1 || d < 8 || (d & 7) || n_splits < 0 || !kernel || !tile_rows || !tile_tokens || !splits) return ARROL_EINVAL;
    const Plan p = make_plan(T, V, d, n_splits);
    *kernel = p.general ? 0 : p.form == kFormRing ? 1 : 2;
    *tile_rows = kFormSize[p.form].bm;
    *tile_tokens = kFormSize[p.form].bn;
    *splits = p.n_sp;
    return ARROL_OK;
}

extern "C" int arrol_logprob_streamed(int64_t T, int32_t V, int32_t d, int32_t n_splits, int32_t* streamed) {
    if (T < 1 || V < 1 || d < 8 || (d & 7) || n_splits < 0 || !streamed) return ARROL_EINVAL;
    *streamed = make_plan(T, V, d, n_splits).stream ? 1 : 0;
    return ARROL_OK;
}
