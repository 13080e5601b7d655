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
constexpr int kMaxBins4 = 512;        // of the calibration's rounds of 15 points; 7 beyond
constexpr int kPruneThreads = 1024;
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

// Bins of the calibration: posterior, what a bin adds to kappa + delta, and its weight in the mean.
struct CalibrationBin { double q, off, w; };
__host__ __device__ inline double calibration_prior(double np, double nn) { return (np + nn) > 0.0 ? np / (np + nn) : 0.5; }
__host__ __device__ inline CalibrationBin calibration_bin(double cp, double cn, double np, double nn, double pi, int B, const arrol_policy& pol) {
    const double alpha = pol.alpha;
    const double like_pos = (cp + alpha) / (np + alpha * B);
    const double like_neg = (cn + alpha) / (nn + alpha * B);
    const double num = pi * like_pos, den = num + (1.0 - pi) * like_neg;
    const double q = den > 0.0 ? num / den : pi;
    return {q, static_cast<double>(pol.lambda) * (static_cast<double>(pol.rho) - q), (np + nn) > 0.0 ? (cp + cn) / (np + nn) : 1.0 / B};
}

// The search for delta: where sum_b w_b clip(kappa + delta + off_b, p_min, p_max), which rises with delta in straight pieces, reaches kappa.
// A round asks for the sums at 2^LOG - 1 points of the bracket; the bracket then is between the last point whose sum is too small and
// the next.  Rounds of equal steps gain LOG bits each.  Once both ends' sums are known and the bracket is some 2 / B of its start (every bin
// has two kinks), every other round's points lie around the secant's root, at distances that fall by powers of two: between two kinks one
// such round leaves a few ulps, which the last rounds of equal steps share.  Later than round 7 kinks crowd around the root and equal
// steps alone are quicker.  It ends as 64 halvings would: no double between the ends, or 2^-63 of the start.  At most four rounds of the
// second kind and 63 / LOG of the first: 20 of four bits, 25 of three.  Score buffers of 512 to 262,144 entries, kappa 0.25 to 0.625: 4 to 11
// rounds up to 512 bins (LOG 4), 5 to 14 beyond (LOG 3).
template <int LOG>
struct DeltaSearch {
    static constexpr int NODES = 1 << LOG, ROUNDS = 2 * ((64 + LOG - 1) / LOG);      // (more than there can be)
    static_assert(LOG == 3 || LOG == 4);
    double kappa, lo, hi, enough, root = 0.0, sum_lo = 0.0, sum_hi = 0.0;
    bool known_lo = false, known_hi = false, secant = false;     // the ends' sums; the kind of this round
    __host__ __device__ explicit DeltaSearch(const arrol_policy& pol)
        : kappa(pol.kappa), lo(static_cast<double>(pol.p_min) - kappa - static_cast<double>(pol.lambda)),
          hi(static_cast<double>(pol.p_max) - kappa + static_cast<double>(pol.lambda)), enough((hi - lo) * 0x1p-63) {}
    __host__ __device__ bool begin_round() {
        const double width = hi - lo, middle = lo + 0.5 * width;
        if (width <= enough || middle <= lo || middle >= hi) return false;
        root = secant ? lo + (kappa - sum_lo) / (sum_hi - sum_lo) * width : 0.0;
        return true;
    }
    __host__ __device__ double point(int j, int it) const {      // ascending; 0: the start's lower end, then the upper
        if (j == 0) return it == 0 ? lo : hi;
        const double width = hi - lo;
        if (!secant) return fma(width, j * (1.0 / NODES), lo);
        const int m = j - NODES / 2, rank = m < 0 ? -m : m;      // steps of 2^-46 ... 2^-4 (2^-6) of the bracket
        const int e = LOG == 4 ? 53 - 7 * rank : 66 - 20 * rank;
        const double step = m == 0 ? 0.0 : width * __builtin_bit_cast(double, static_cast<long long>(1023 - e) << 52);
        return fmin(fmax(m < 0 ? root - step : root + step, lo), hi);
    }
    // false: kappa is below what any delta gives, or above
    __host__ __device__ bool in_reach(int it, double end_sum) {
        if (it == 0 && end_sum >= kappa) { hi = lo; return false; }
        if (it == 1 && !known_hi && end_sum < kappa) { lo = hi; return false; }
        return true;
    }
    // `first` of the points 1 ... NODES - 1 is the first whose sum is large enough (NODES: none)
    template <class Sum>
    __host__ __device__ void end_round(int it, int B, int first, Sum sum_at) {
        const double new_lo = first > 1 ? point(first - 1, it) : lo, new_hi = first < NODES ? point(first, it) : hi;
        if (first > 1) { sum_lo = sum_at(first - 1); known_lo = true; }
        if (first < NODES) { sum_hi = sum_at(first); known_hi = true; }
        lo = new_lo;
        hi = new_hi;
        secant = known_lo && known_hi && it < 7 && (4ll << (it + 1) * LOG) >= 2 * B && !secant;
    }
};

// Likelihoods, Bayes posterior, survival probability and the search for delta; one workgroup, fp64.
// What bounds it is the serial chain of sums over the bins: 2^LOG - 1 points at once, LPM lanes with PER_LANE bins each in their registers a
// point, behind one barrier (some 0.4 us a round at 128 bins, 1.1 at 2,048).
template <int LOG, int LPM, int PER_LANE>
__global__ __launch_bounds__((1 << LOG) * LPM) void calibrate_kernel(
    const int64_t* __restrict__ c_pos, const int64_t* __restrict__ c_neg, int B, arrol_policy pol,
    float* __restrict__ q_lut, float* __restrict__ p_lut, double* __restrict__ delta_out) {
    constexpr int NODES = 1 << LOG, NT = NODES * LPM, WAVES = NT / ARROL_WAVE;
    static_assert(LPM == 16 || LPM == 64, "a point's lanes lie in one wavefront");
    constexpr int MAX_B = PER_LANE * LPM;                               // the bins of a point's lanes sit in registers
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
    const double kappa = pol.kappa, rho = pol.rho, lam = pol.lambda, p_min = pol.p_min, p_max = pol.p_max;
    const double pi = calibration_prior(np, nn);
    for (int b = tid; b < B; b += NT) {
        const CalibrationBin x = calibration_bin(static_cast<double>(c_pos[b]), static_cast<double>(c_neg[b]), np, nn, pi, B, pol);
        q_s[b] = x.q;
        off_s[b] = x.off;
        w_s[b] = x.w;
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
    DeltaSearch<LOG> search(pol);
    for (int it = 0; it < search.ROUNDS; ++it) {     // the same in every thread
        if (!search.begin_round()) break;
        const double base = kappa + search.point(my_node, it);
        double e = 0.0;
#pragma unroll
        for (int k = 0; k < PER_LANE; ++k) e = fma(wgt[k], fmin(fmax(base + off[k], p_min), p_max), e);
        const auto add = [](double x, double y) { return x + y; };
        if constexpr (LPM == 64) { e = wave_step<32>(e, add); e = wave_step<16>(e, add); }
        e = wave_step<8>(e, add);
        e = wave_step<4>(e, add);
        e = wave_step<2>(e, add);
        e = wave_step<1>(e, add);
        const double* sums = node_sum[it & 1];
        if (my_lane == 0) node_sum[it & 1][my_node] = e;
        __syncthreads();
        if (!search.in_reach(it, sums[0])) break;
        const uint64_t large = __ballot(sums[lane % NODES] >= kappa) & ((1ull << NODES) - 2);
        search.end_round(it, B, large ? __builtin_ctzll(large) : NODES, [&](int j) { return sums[j]; });
    }
    const double delta = 0.5 * (search.lo + search.hi);
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
    // us a call, halvings (15 midpoints at once up to 256 bins, 3 beyond) and this, mean and most of 36 score buffers of 1,024 to 262,144 entries at
    // kappa 0.25 to 0.625: 128 bins 8.1 and 5.4 / 7.0, 256 9.3 and 6.1 / 7.9, 512 12.6 and 8.6 / 11.1, 1,024 15.5 and 9.9 / 11.7, 2,048
    // 20.8 and 15.2 / 16.2.  From 257 bins on a wavefront sums a point, and beyond 512 seven points a round: 15 of 32 bins a lane would need
    // more registers than 1,024 threads have.
    const auto launch = [&](auto kernel, int threads) {
        arrol_launch(kernel, dim3(1), dim3(threads), 0, st, c_pos, c_neg, B, pol, q_lut, p_lut, delta);
    };
    if (B <= 128) launch(calibrate_kernel<4, 16, 8>, 256);
    else if (B <= 256) launch(calibrate_kernel<4, 16, 16>, 256);
    else if (B <= kMaxBins4) launch(calibrate_kernel<4, 64, 8>, 1024);
    else if (B <= 1024) launch(calibrate_kernel<3, 64, 16>, 512);
    else launch(calibrate_kernel<3, 64, 32>, 512);
    return arrol_launch_status();
}

namespace {
template <int LOG>
void search_on_host(const CalibrationBin* bins, int B, const arrol_policy& pol, int32_t* rounds, double* delta) {
    DeltaSearch<LOG> search(pol);
    double sums[DeltaSearch<LOG>::NODES];
    for (*rounds = 0; *rounds < search.ROUNDS && search.begin_round(); ++*rounds) {
        int first = search.NODES;
        for (int j = search.NODES - 1; j >= 0; --j) {
            const double base = search.kappa + search.point(j, *rounds);
            sums[j] = 0.0;
            for (int b = 0; b < B; ++b)
                sums[j] = fma(bins[b].w, fmin(fmax(base + bins[b].off, static_cast<double>(pol.p_min)), static_cast<double>(pol.p_max)), sums[j]);
            if (j > 0 && sums[j] >= search.kappa) first = j;
        }
        if (!search.in_reach(*rounds, sums[0])) { ++*rounds; break; }
        search.end_round(*rounds, B, first, [&](int j) { return sums[j]; });
    }
    *delta = 0.5 * (search.lo + search.hi);
}
}  // namespace

extern "C" int arrol_calibrate_search(const int64_t* c_pos, const int64_t* c_neg, int32_t B, arrol_policy pol, int32_t* rounds, double* delta) {
    if (B < 1 || B > kMaxBins || !c_pos || !c_neg || !rounds || !delta || !policy_ok(pol)) return ARROL_EINVAL;
    int64_t tp = 0, tn = 0;
    for (int b = 0; b < B; ++b) { tp += c_pos[b]; tn += c_neg[b]; }
    const double np = static_cast<double>(tp), nn = static_cast<double>(tn);
    CalibrationBin bins[kMaxBins];
    for (int b = 0; b < B; ++b)
        bins[b] = calibration_bin(static_cast<double>(c_pos[b]), static_cast<double>(c_neg[b]), np, nn, calibration_prior(np, nn), B, pol);
    if (B <= kMaxBins4) search_on_host<4>(bins, B, pol, rounds, delta);
    else search_on_host<3>(bins, B, pol, rounds, delta);
    return ARROL_OK;
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
