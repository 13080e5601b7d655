// The paper's practical pruning policy (App. A.4 "Calibration Mapping and Survival Probability Design";
// Alg. 1, backend): binned posterior calibration of the sigmoid-normalised head score, survival
// probability with the keep-rate bias found by binary search, Bernoulli pruning with caller-supplied
// uniforms and an order-preserving stream compaction of the survivors.
#include "common.h"

namespace {

constexpr int kHistThreads = 256;
constexpr int kHistOneThreads = 1024;
constexpr int kHistOneMax = 16384;    // entries one workgroup takes alone: 16 per thread, 4.3 us with 128 bins and 5.2 with 2,048
                                      // where two launches take 5.8 and 7.2
constexpr int kMaxBins = 2048;        // two fp64 tables of kMaxBins entries fit in LDS
constexpr int kPruneThreads = 1024;
constexpr int kBisectIters = 64;
static_assert(64 * 32 == kMaxBins, "the last form of the calibration takes every bin count");

// b(s') = min(B-1, floor(B s')), product in fp32 (App. A.4)
__device__ __forceinline__ int bin_of(float s_norm, int B) {
    int b = static_cast<int>(floorf(s_norm * static_cast<float>(B)));
    b = b < 0 ? 0 : b;
    return b < B - 1 ? b : B - 1;
}

__global__ void zero_counts_kernel(int64_t* c_pos, int64_t* c_neg, int B) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < B) { c_pos[i] = 0; c_neg[i] = 0; }
}

// Eq. 1: per-workgroup histograms in LDS, merged with 64-bit atomics (integer: order-free)
__global__ __launch_bounds__(kHistThreads) void histogram_kernel(
    const float* __restrict__ s_norm, const uint8_t* __restrict__ label, int64_t M, int B,
    unsigned long long* __restrict__ c_pos, unsigned long long* __restrict__ c_neg) {
    extern __shared__ unsigned int hist[];   // [2][B]
    for (int i = threadIdx.x; i < 2 * B; i += kHistThreads) hist[i] = 0;
    __syncthreads();
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kHistThreads;
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * kHistThreads + threadIdx.x; k < M; k += stride)
        atomicAdd(&hist[(label[k] ? 0 : B) + bin_of(s_norm[k], B)], 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < B; i += kHistThreads) {
        if (hist[i]) atomicAdd(&c_pos[i], static_cast<unsigned long long>(hist[i]));
        if (hist[B + i]) atomicAdd(&c_neg[i], static_cast<unsigned long long>(hist[B + i]));
    }
}

// The same for a short buffer: one workgroup whose LDS histogram is the result, so nothing has to be zeroed first (one
// launch instead of two; 4,096 entries, 128 bins: 5.6 us of kernels before, 2.6 now).  Lanes that count in the same word
// wait for each other, and a head at cold start puts nearly all scores into one bin, so a bin has COPIES words side by
// side, of which a lane takes the one of its number (16,384 entries in one bin of 128: 12.5 us with one word a bin, 4.3
// with eight; in two launches 6.2).
template <int COPIES>
__global__ __launch_bounds__(kHistOneThreads) void histogram_one_kernel(
    const float* __restrict__ s_norm, const uint8_t* __restrict__ label, int M, int B, int64_t* __restrict__ c_pos,
    int64_t* __restrict__ c_neg) {
    constexpr int VEC = COPIES >= 4 ? 4 : 1;
    typedef unsigned int words __attribute__((ext_vector_type(VEC)));
    extern __shared__ __attribute__((aligned(16))) unsigned int hist[];   // [2][B][COPIES]
    for (int i = threadIdx.x; i < 2 * B * COPIES / VEC; i += kHistOneThreads) reinterpret_cast<words*>(hist)[i] = words(0u);
    __syncthreads();
    const int copy = threadIdx.x % COPIES;
    for (int k0 = threadIdx.x; k0 < M; k0 += kHistOneThreads * 4) {
        float s[4];
        uint8_t l[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + u * kHistOneThreads;
            s[u] = k < M ? s_norm[k] : 0.f;
            l[u] = k < M ? label[k] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (k0 + u * kHistOneThreads < M) atomicAdd(&hist[((l[u] ? 0 : B) + bin_of(s[u], B)) * COPIES + copy], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * B; i += kHistOneThreads) {
        unsigned int sum = 0;
#pragma unroll
        for (int c = 0; c < COPIES / VEC; ++c) {
            const words x = reinterpret_cast<const words*>(hist)[i * (COPIES / VEC) + c];
#pragma unroll
            for (int v = 0; v < VEC; ++v) sum += x[v];
        }
        (i < B ? c_pos[i] : c_neg[i - B]) = sum;
    }
}

// Likelihoods, Bayes posterior, survival probability and the bisection for delta; one workgroup, fp64.
// What bounds it is the serial chain of 64 halvings, each a sum over the bins.  LEVELS halvings are taken at once: the
// 2^LEVELS - 1 midpoints that they can ask for form a binary tree, LPM lanes with PER_LANE bins each in their registers
// sum at each node (numbered as a heap), and every thread walks the decisions down the tree behind one barrier.
// Midpoints are those of one halving after the other.  128 bins: 31.3 us with a sum over the whole workgroup and two
// barriers per halving, now 7.7 (other sizes at the launch).
template <int LEVELS, int LPM, int PER_LANE>
__global__ __launch_bounds__((1 << LEVELS) * LPM) void calibrate_kernel(
    const int64_t* __restrict__ c_pos, const int64_t* __restrict__ c_neg, int B, arrol_policy pol,
    float* __restrict__ q_lut, float* __restrict__ p_lut, double* __restrict__ delta_out) {
    constexpr int NODES = 1 << LEVELS, NT = NODES * LPM, WAVES = NT / ARROL_WAVE;
    static_assert(kBisectIters % LEVELS == 0 && (LPM == 16 || LPM == 64), "a node's lanes lie in one wavefront");
    // off_s: lambda (rho - q), what a bin adds to kappa + delta
    constexpr int MAX_B = PER_LANE * LPM;                               // the bins of a node's lanes sit in registers
    __shared__ double q_s[MAX_B], off_s[MAX_B], w_s[MAX_B];
    __shared__ double node_sum[2][NODES];
    __shared__ int64_t cnt[2][WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t tp = 0, tn = 0;
    for (int b = tid; b < B; b += NT) { tp += c_pos[b]; tn += c_neg[b]; }
    tp = wave_sum_i64(tp);
    tn = wave_sum_i64(tn);
    if (lane == 0) { cnt[0][wave] = tp; cnt[1][wave] = tn; }
    __syncthreads();
    tp = tn = 0;
    for (int w = 0; w < WAVES; ++w) { tp += cnt[0][w]; tn += cnt[1][w]; }
    const double np = static_cast<double>(tp), nn = static_cast<double>(tn);
    const double alpha = pol.alpha, kappa = pol.kappa, rho = pol.rho, lam = pol.lambda;
    const double p_min = pol.p_min, p_max = pol.p_max;
    const double pi = (np + nn) > 0.0 ? np / (np + nn) : 0.5;
    for (int b = tid; b < B; b += NT) {
        const double cp = static_cast<double>(c_pos[b]), cn = static_cast<double>(c_neg[b]);
        const double like_pos = (cp + alpha) / (np + alpha * B);
        const double like_neg = (cn + alpha) / (nn + alpha * B);
        const double num = pi * like_pos, den = num + (1.0 - pi) * like_neg;
        const double q = den > 0.0 ? num / den : pi;
        q_s[b] = q;
        off_s[b] = lam * (rho - q);
        w_s[b] = (np + nn) > 0.0 ? (cp + cn) / (np + nn) : 1.0 / B;
    }
    __syncthreads();
    const int my_node = tid / LPM, my_lane = tid % LPM;
    double off[PER_LANE], wgt[PER_LANE];
#pragma unroll
    for (int k = 0; k < PER_LANE; ++k) {
        const int b = k * LPM + my_lane;
        off[k] = b < B ? off_s[b] : 0.0;
        wgt[k] = b < B ? w_s[b] : 0.0;          // adds nothing
    }
    double lo = p_min - kappa - lam, hi = p_max - kappa + lam;
    for (int it = 0; it < kBisectIters / LEVELS; ++it) {
        // my node's midpoint: down from the root by the bits below its top one (node 0 repeats the root)
        double l = lo, h = hi;
#pragma unroll
        for (int bit = LEVELS - 2; bit >= 0; --bit) {
            if (my_node >= (2 << bit)) {
                const double mid = 0.5 * (l + h);
                if ((my_node >> bit) & 1) l = mid; else h = mid;
            }
        }
        const double base = kappa + 0.5 * (l + h);
        double e = 0.0;
#pragma unroll
        for (int k = 0; k < PER_LANE; ++k) e = fma(wgt[k], fmin(fmax(base + off[k], p_min), p_max), e);
        const auto add = [](double x, double y) { return x + y; };
        if constexpr (LPM == 64) { e = wave_step<32>(e, add); e = wave_step<16>(e, add); }
        e = wave_step<8>(e, add);
        e = wave_step<4>(e, add);
        e = wave_step<2>(e, add);
        e = wave_step<1>(e, add);
        if (my_lane == 0) node_sum[it & 1][my_node] = e;
        __syncthreads();
        // bit n: the sum at node n is too small (the midpoint becomes the lower end)
        const uint64_t small = __ballot(node_sum[it & 1][lane % NODES] < kappa);
        int node = 1;                            // 1 the root, 2n the lower half of node n, 2n + 1 the upper
#pragma unroll
        for (int level = 0; level < LEVELS; ++level) {
            const double m = 0.5 * (lo + hi);
            const int up = static_cast<int>((small >> node) & 1u);
            if (up) lo = m; else hi = m;
            node = 2 * node + up;
        }
    }
    const double delta = 0.5 * (lo + hi);
    for (int b = tid; b < B; b += NT) {
        const double q = q_s[b], p = kappa + delta + lam * (rho - q);
        q_lut[b] = static_cast<float>(q);
        p_lut[b] = static_cast<float>(p < p_min ? p_min : (p > p_max ? p_max : p));
    }
    if (tid == 0 && delta_out) *delta_out = delta;
}

// Alg. 1: survival probability lookup, Bernoulli decision u < p, survivors compacted in rollout order
// (ballot + popcount inside a wave, LDS carry across waves and chunks).  One workgroup.
__global__ __launch_bounds__(kPruneThreads) void prune_bernoulli_kernel(
    const float* __restrict__ s_norm, const float* __restrict__ uniforms, int N, const float* __restrict__ p_lut,
    int B, float* __restrict__ p_out, uint8_t* __restrict__ keep_mask, int32_t* __restrict__ survivor_idx,
    int32_t* __restrict__ n_survivors) {
    __shared__ int wave_tot[kPruneThreads / ARROL_WAVE];
    __shared__ int carry_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) carry_s = 0;
    __syncthreads();
    for (int i0 = 0; i0 < N; i0 += kPruneThreads) {
        const int i = i0 + tid;
        bool keep = false;
        if (i < N) {
            const float p = p_lut[bin_of(s_norm[i], B)];
            keep = uniforms[i] < p;
            if (p_out) p_out[i] = p;
            keep_mask[i] = keep ? 1 : 0;
        }
        const uint64_t ballot = __ballot(keep);
        if (lane == 0) wave_tot[wave] = __popcll(ballot);
        __syncthreads();
        int before = carry_s;
        for (int w = 0; w < wave; ++w) before += wave_tot[w];
        if (keep) survivor_idx[before + __popcll(ballot & ((1ull << lane) - 1ull))] = i;
        __syncthreads();
        if (tid == kPruneThreads - 1) carry_s = before + __popcll(ballot);
        __syncthreads();
    }
    const int n = carry_s;
    for (int i = n + tid; i < N; i += kPruneThreads) survivor_idx[i] = -1;   // unused tail: "no rollout"
    if (tid == 0) *n_survivors = n;
}

bool policy_ok(const arrol_policy& p) {
    return p.kappa >= 0.f && p.kappa <= 1.f && p.rho >= 0.f && p.rho <= 1.f && p.lambda >= 0.f &&
           p.p_min >= 0.f && p.p_max <= 1.f && p.p_min <= p.p_max && p.alpha >= 0.f;
}

}  // namespace

extern "C" int arrol_histogram(const float* s_norm, const uint8_t* label, int64_t M, int32_t B,
                               int64_t* c_pos, int64_t* c_neg, void* stream) {
    if (M < 0 || B < 1 || B > kMaxBins || !c_pos || !c_neg) return ARROL_EINVAL;
    if (M > 0 && (!s_norm || !label)) return ARROL_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (M <= kHistOneMax) {
        // Up to 4,096 entries one word a bin is no slower than two launches even with all scores in one bin (4.8 us against
        // 6.0); beyond, eight words as far as 64 KiB of LDS reach, else four.
        const auto launch = [&](auto kernel, int copies) {
            arrol_launch(kernel, dim3(1), dim3(kHistOneThreads), 2 * B * copies * sizeof(unsigned int), st, s_norm, label,
                         static_cast<int>(M), B, c_pos, c_neg);
        };
        if (M <= 4096) launch(histogram_one_kernel<1>, 1);
        else if (B <= 1024) launch(histogram_one_kernel<8>, 8);
        else launch(histogram_one_kernel<4>, 4);
        return arrol_launch_status();
    }
    arrol_launch(zero_counts_kernel, dim3((B + 255) / 256), dim3(256), 0, st, c_pos, c_neg, B);
    if (arrol_launch_failed()) return arrol_launch_status();
    int64_t blocks = (M + kHistThreads * 16 - 1) / (kHistThreads * 16);
    blocks = blocks < 1 ? 1 : (blocks > 1024 ? 1024 : blocks);
    arrol_launch(histogram_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kHistThreads),
                       2 * B * sizeof(unsigned int), st, s_norm, label, M, B,
                       reinterpret_cast<unsigned long long*>(c_pos), reinterpret_cast<unsigned long long*>(c_neg));
    return arrol_launch_status();
}

extern "C" int arrol_calibrate(const int64_t* c_pos, const int64_t* c_neg, int32_t B, arrol_policy pol,
                               float* q_lut, float* p_lut, double* delta, void* stream) {
    if (B < 1 || B > kMaxBins || !c_pos || !c_neg || !q_lut || !p_lut || !policy_ok(pol)) return ARROL_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Measured (before: 31 us up to 256 bins, 37, 45, 63 at 512, 1024, 2048): 15 midpoints at once 7.7 and 8.8 us up to
    // 128 and 256 bins; beyond that the sums of 15 midpoints cost more than the rounds they save (21 us at 1024 against
    // 15 with 3 midpoints, one wavefront each): 12, 15 and 20 us.
    const auto launch = [&](auto kernel) {
        arrol_launch(kernel, dim3(1), dim3(256), 0, st, c_pos, c_neg, B, pol, q_lut, p_lut, delta);
    };
    if (B <= 128) launch(calibrate_kernel<4, 16, 8>);
    else if (B <= 256) launch(calibrate_kernel<4, 16, 16>);
    else if (B <= 512) launch(calibrate_kernel<2, 64, 8>);
    else if (B <= 1024) launch(calibrate_kernel<2, 64, 16>);
    else launch(calibrate_kernel<2, 64, 32>);
    return arrol_launch_status();
}

extern "C" int arrol_prune_bernoulli(const float* s_norm, const float* uniforms, int32_t N, const float* p_lut,
                                     int32_t B, float* p_out, uint8_t* keep_mask, int32_t* survivor_idx,
                                     int32_t* n_survivors, void* stream) {
    if (N < 0 || B < 1 || B > kMaxBins || !p_lut || !n_survivors) return ARROL_EINVAL;
    if (N > 0 && (!s_norm || !uniforms || !keep_mask || !survivor_idx)) return ARROL_EINVAL;
    arrol_launch(prune_bernoulli_kernel, dim3(1), dim3(kPruneThreads), 0, static_cast<hipStream_t>(stream),
                       s_norm, uniforms, N, p_lut, B, p_out, keep_mask, survivor_idx, n_survivors);
    return arrol_launch_status();
}
