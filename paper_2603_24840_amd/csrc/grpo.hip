// GRPO on the surviving rollouts (Sec. 3 "Group-Relative Policy Optimization"; the frontend step of Alg. 1
// that follows the log-probs): the group-relative advantage and the clipped-ratio objective with its derivative
// with respect to the per-token log-probabilities that arrol_logprob produces.  A few bytes per token and a
// handful of groups: latency-bound kernels, written for fixed summation order and fp64 decisions rather than
// for bandwidth.
#include "common.h"

namespace {

__device__ __forceinline__ void group_range(const int64_t* group_offsets, int g, int64_t N, int64_t& lo, int64_t& hi) {
    lo = group_offsets[g];
    hi = group_offsets[g + 1];
    lo = lo < 0 ? 0 : (lo > N ? N : lo);
    hi = hi < lo ? lo : (hi > N ? N : hi);
}

// Zeros for those of the 64 rollouts from c0 on that no group holds, by one wavefront, while others work on the groups: each
// lane marks what every 64th group holds of them, whatever the order of the offsets.  Nothing that a group writes is touched.
__device__ void zero_outside(const int64_t* __restrict__ group_offsets, int64_t N, int n_groups, int64_t c0, float* __restrict__ advantage,
                             float* __restrict__ seq_weight) {
    constexpr int kInFlight = 8;
    uint64_t held = 0;
    for (int g0 = threadIdx.x; g0 < n_groups; g0 += kInFlight * ARROL_WAVE) {
        int64_t lo[kInFlight], hi[kInFlight];
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {    // past the end the lane's first one again, so that no load waits on a branch
            const int g = g0 + k * ARROL_WAVE < n_groups ? g0 + k * ARROL_WAVE : g0;
            lo[k] = group_offsets[g];
            hi[k] = group_offsets[g + 1];
        }
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            const int first = static_cast<int>(min(max(lo[k], c0), c0 + ARROL_WAVE) - c0), end = static_cast<int>(min(max(hi[k], c0), c0 + ARROL_WAVE) - c0);
            if (first < end) held |= ~0ull >> (ARROL_WAVE - (end - first)) << first;
        }
    }
    held = wave_reduce(held, [](uint64_t a, uint64_t b) { return a | b; });
    const int64_t i = c0 + threadIdx.x;
    if (i < N && !(held >> threadIdx.x & 1)) {
        advantage[i] = 0.f;
        if (seq_weight) seq_weight[i] = 0.f;
    }
}

__global__ __launch_bounds__(256) void grpo_zero_kernel(int64_t N, float* __restrict__ advantage, float* __restrict__ seq_weight) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= N) return;
    advantage[i] = 0.f;
    if (seq_weight) seq_weight[i] = 0.f;
}

// one wavefront per group; with one more for every 64 rollouts these write the zeros
__global__ __launch_bounds__(ARROL_WAVE) void grpo_advantage_kernel(
    const float* __restrict__ reward, const int64_t* __restrict__ group_offsets, int64_t N, int n_groups, int ddof,
    double eps, float* __restrict__ advantage, float* __restrict__ seq_weight) {
    const int g = blockIdx.x;
    if (g >= n_groups) return zero_outside(group_offsets, N, n_groups, static_cast<int64_t>(g - n_groups) * ARROL_WAVE, advantage, seq_weight);
    int64_t lo, hi;
    group_range(group_offsets, g, N, lo, hi);
    const int64_t n = hi - lo;
    if (n == 0) return;
    double s = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += ARROL_WAVE) s += static_cast<double>(reward[i]);
    const double mean = wave_sum_f64(s) / static_cast<double>(n);
    double q = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += ARROL_WAVE) {
        const double dv = static_cast<double>(reward[i]) - mean;
        q += dv * dv;
    }
    q = wave_sum_f64(q);
    const double stdv = n - ddof > 0 ? sqrt(q / static_cast<double>(n - ddof)) : 0.0;
    const double den = stdv + eps;
    const float wgt = static_cast<float>(1.0 / (static_cast<double>(n) * static_cast<double>(n_groups)));
    for (int64_t i = lo + threadIdx.x; i < hi; i += ARROL_WAVE) {
        const double dv = static_cast<double>(reward[i]) - mean;
        advantage[i] = den > 0.0 ? static_cast<float>(dv / den) : 0.f;
        if (seq_weight) seq_weight[i] = wgt;
    }
}

constexpr int kSegments = 8;           // most workgroups per rollout

// the workgroup's sums of s and c, in thread 0
template <int WAVES>
__device__ __forceinline__ void workgroup_sums(double& s, long long& c, double (&sh_s)[WAVES], long long (&sh_c)[WAVES]) {
    s = wave_sum_f64(s);
    c = wave_sum_i64(c);
    const int lane = threadIdx.x & (ARROL_WAVE - 1), wave = threadIdx.x / ARROL_WAVE;
    if (lane == 0) { sh_s[wave] = s; sh_c[wave] = c; }
    __syncthreads();
    if (threadIdx.x == 0) {
        s = 0.0;
        c = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) { s += sh_s[w]; c += sh_c[w]; }
    }
}

// exp(-u) and exp(u), |u| < 700, from one reduction u = k ln 2 + r: exp(+-r) = 1 + ((cosh r - 1) +- sinh r), both by their Taylor series in r^2
// (|r| <= 0.347: what is left out is below 1e-17 of them).  25 instructions where an exponential and a reciprocal took some 50.  Each is
// within 1.24 ulp of the true value, 0.33 in the root mean square (1 million of them each in +-690, +-20 and normal ones of 0.2), and
// exactly 1 at 0; the library's exponential and its reciprocal had 0.85 and 1.49, 0.30 and 0.45.
__device__ __forceinline__ void exp_both(double u, double& down, double& up) {
    const double k = rint(u * 1.4426950408889634);
    // ln 2 in 42 bits and what they leave of it: k times the first is exact, and so is the difference
    const double r = fma(-k, 5.497923018708371e-14, fma(-k, 0.6931471805598903, u)), t = r * r;
    double c = 1.0 / 479001600.0, s = 1.0 / 6227020800.0;            // 1 / 12!, 1 / 13!
    c = fma(c, t, 1.0 / 3628800.0);
    s = fma(s, t, 1.0 / 39916800.0);
    c = fma(c, t, 1.0 / 40320.0);
    s = fma(s, t, 1.0 / 362880.0);
    c = fma(c, t, 1.0 / 720.0);
    s = fma(s, t, 1.0 / 5040.0);
    c = fma(c, t, 1.0 / 24.0);
    s = fma(s, t, 1.0 / 120.0);
    c = fma(c, t, 0.5);
    s = fma(s, t, 1.0 / 6.0);
    c *= t;
    s = fma(s * t, r, r);
    const int e = static_cast<int>(k);
    down = ldexp(1.0 + (c - s), -e);
    up = ldexp(1.0 + (c + s), e);
}

// n_seg workgroups per rollout, each with an equal part of its tokens: partial[i n_seg + q] = weight_i * (1/L_i) * sum_t term_t,
// clipped[..] = tokens on the clipped branch.  Bound by latency (64-bit exponentials behind two loads, 12 bytes a token): the
// loads of up to four tokens go out together, their arithmetic is interleaved, and long rollouts get enough wavefronts to hide the rest.
template <int kObjThreads>
__global__ __launch_bounds__(kObjThreads) void grpo_objective_kernel(
    const float* __restrict__ logp, const float* __restrict__ logp_ref, const int64_t* __restrict__ cu, int64_t T,
    const float* __restrict__ advantage, const float* __restrict__ seq_weight, double eps_low, double eps_high,
    double beta, float* __restrict__ grad_logp, double* __restrict__ partial, int64_t* __restrict__ clipped) {
    __shared__ double sh_s[kObjThreads / ARROL_WAVE];
    __shared__ long long sh_c[kObjThreads / ARROL_WAVE];
    const int i = blockIdx.x, n_seg = gridDim.y, out = i * n_seg + blockIdx.y;
    int64_t lo = cu[i], hi = cu[i + 1];
    lo = lo < 0 ? 0 : (lo > T ? T : lo);
    hi = hi < lo ? lo : (hi > T ? T : hi);
    const int64_t L = hi - lo;
    if (n_seg > 1) {
        const int64_t part = (L + n_seg - 1) / n_seg;
        lo = lo + blockIdx.y * part < hi ? lo + blockIdx.y * part : hi;
        hi = lo + part < hi ? lo + part : hi;
    }
    if (lo == hi) {
        if (threadIdx.x == 0) { partial[out] = 0.0; clipped[out] = 0; }
        return;
    }
    const double A = static_cast<double>(advantage[i]);
    const double scale = static_cast<double>(seq_weight[i]) / static_cast<double>(L);
    const double r_lo = 1.0 - eps_low, r_hi = 1.0 + eps_high;
    double s = 0.0;
    long long c = 0;
    // the tokens t0, t0 + kObjThreads, ...: as many as `step` says, as far as they are there
    const auto tokens = [&](auto step, int64_t t0) {
        constexpr int N = decltype(step)::value;
        if (t0 >= hi) return;
        float ref[N], lp[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int64_t t = t0 + k * kObjThreads < hi ? t0 + k * kObjThreads : t0;   // a load that may be skipped would be waited for
            ref[k] = logp_ref[t];
            lp[k] = logp[t];
        }
        double u[N], ratio[N], eu[N];
        bool far = false;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            u[k] = static_cast<double>(ref[k]) - static_cast<double>(lp[k]);
            exp_both(u[k], ratio[k], eu[k]);
            far = far || !(fabs(u[k]) < 700.0);
        }
        if (__builtin_expect(__ballot(far) != 0, 0)) {                 // a lane past the ends of the exponentials' range, infinite or undefined
            asm volatile("");                // (a branch: the compiler would take both sides)
#pragma unroll 1
            for (int k = 0; k < N; ++k)
                if (!(fabs(u[k]) < 700.0)) {
                    ratio[k] = exp(-u[k]);
                    eu[k] = exp(u[k]);
                }
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {       // beside each other: dead ones repeat the first and are not counted
            const int64_t t = t0 + k * kObjThreads;
            const bool live = t < hi;
            const double plain = ratio[k] * A;
            const double clamped = fmin(fmax(ratio[k], r_lo), r_hi) * A;
            const double term = fmin(plain, clamped) - beta * (eu[k] - u[k] - 1.0);
            s += live ? term : 0.0;
            c += live && clamped < plain ? 1 : 0;
            if (grad_logp && live) {
                const double d = (plain <= clamped ? plain : 0.0) - beta * (1.0 - eu[k]);
                grad_logp[t] = static_cast<float>(d * scale);
            }
        }
    };
    // Four tokens a thread at a time while there are more than three, then two, then one: a step's arithmetic is done whether its tokens are
    // there or not.  By each rollout's own length: with one number for all, of their mean, 255 rollouts of 64 tokens and one of
    // 8,192 took 12.7 us (now 8.9), 512 of 1,200 6.6 (5.9), of 2,500 8.6 (7.4), of 250 5.3 (4.9); with four always, and the missing ones
    // skipped one by one, 11.9, 6.2, 8.2 and 5.1.
    int64_t t0 = lo + threadIdx.x;
    const auto left = [&] { return hi - t0 + threadIdx.x; };
    for (; left() > 3 * kObjThreads; t0 += 4 * kObjThreads) tokens(std::integral_constant<int, 4>{}, t0);
    if (left() > kObjThreads) {
        tokens(std::integral_constant<int, 2>{}, t0);
        t0 += 2 * kObjThreads;
    }
    tokens(std::integral_constant<int, 1>{}, t0);
    workgroup_sums(s, c, sh_s, sh_c);
    if (threadIdx.x == 0) {
        partial[out] = s * scale;
        clipped[out] = c;
    }
}

// one workgroup: J = the partials' sum in a fixed order
template <int kFinishThreads>
__global__ __launch_bounds__(kFinishThreads) void grpo_finish_kernel(const double* __restrict__ partial,
                                                                     const int64_t* __restrict__ clipped, int64_t n,
                                                                     double* __restrict__ objective_out,
                                                                     int64_t* __restrict__ n_clipped) {
    __shared__ double sh_s[kFinishThreads / ARROL_WAVE];
    __shared__ long long sh_c[kFinishThreads / ARROL_WAVE];
    double s = 0.0;
    long long c = 0;
    constexpr int kInFlight = kFinishThreads > 256 ? 4 : 1;
    for (int64_t i0 = threadIdx.x; i0 < n; i0 += kFinishThreads * kInFlight) {
        double x[kInFlight];
        int64_t y[kInFlight];
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            const int64_t i = i0 + k * kFinishThreads < n ? i0 + k * kFinishThreads : i0;
            x[k] = partial[i];
            y[k] = clipped[i];
        }
#pragma unroll
        for (int k = 0; k < kInFlight; ++k)
            if (i0 + k * kFinishThreads < n) { s += x[k]; c += y[k]; }
    }
    workgroup_sums(s, c, sh_s, sh_c);
    if (threadIdx.x == 0) {
        if (objective_out) *objective_out = s;
        if (n_clipped) *n_clipped = c;
    }
}

}  // namespace

extern "C" int arrol_grpo_advantage(const float* reward, const int64_t* group_offsets, int64_t N, int32_t n_groups,
                                    int32_t ddof, float eps, float* advantage, float* seq_weight, void* stream) {
    if (N < 0 || n_groups < 0 || (ddof != 0 && ddof != 1) || !(eps >= 0.f)) return ARROL_EINVAL;
    if (n_groups == 0 || N == 0) return ARROL_OK;
    if (!reward || !group_offsets || !advantage) return ARROL_EINVAL;
    arrol_launch(grpo_advantage_kernel, dim3(n_groups), dim3(ARROL_WAVE), 0, static_cast<hipStream_t>(stream),
                       reward, group_offsets, N, n_groups, ddof, static_cast<double>(eps), advantage, seq_weight);
    return arrol_launch_status();
}

extern "C" int arrol_grpo_advantage_all(const float* reward, const int64_t* group_offsets, int64_t N, int32_t n_groups,
                                        int32_t ddof, float eps, float* advantage, float* seq_weight, void* stream) {
    if (N < 0 || n_groups < 0 || (ddof != 0 && ddof != 1) || !(eps >= 0.f)) return ARROL_EINVAL;
    if (N == 0) return ARROL_OK;
    if (!advantage || (n_groups > 0 && (!reward || !group_offsets))) return ARROL_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // Every wavefront of the zeros looks at every offset, 512 at a time: one launch up to 2,048 groups (2,048 groups of 16,384
    // rollouts 5.2 us; of 32,768 rollouts 4,096 groups 8.7 in one launch and 4,097 5.5 in two)
    if (n_groups > 0 && n_groups <= 2048 && N <= 65536) {
        const unsigned zeros = static_cast<unsigned>((N + ARROL_WAVE - 1) / ARROL_WAVE);
        arrol_launch(grpo_advantage_kernel, dim3(n_groups + zeros), dim3(ARROL_WAVE), 0, st, reward, group_offsets, N, n_groups, ddof,
                     static_cast<double>(eps), advantage, seq_weight);
        return arrol_launch_status();
    }
    const int64_t blocks = (N + 255) / 256;
    if (blocks > INT32_MAX) return ARROL_EINVAL;
    arrol_launch(grpo_zero_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, N, advantage, seq_weight);
    if (arrol_launch_failed()) return arrol_launch_status();
    return arrol_grpo_advantage(reward, group_offsets, N, n_groups, ddof, eps, advantage, seq_weight, stream);
}

extern "C" size_t arrol_grpo_objective_workspace_bytes(int32_t n_seq) {
    return n_seq < 0 ? 0 : static_cast<size_t>(n_seq) * 16;
}

extern "C" int arrol_grpo_objective(const float* logp, const float* logp_ref, const int64_t* cu_seqlens, int64_t T,
                                    int32_t n_seq, const float* advantage, const float* seq_weight, float eps_low,
                                    float eps_high, float beta, double* objective_out, float* grad_logp,
                                    int64_t* n_clipped, void* workspace, size_t workspace_bytes, void* stream) {
    if (T < 0 || n_seq < 0 || !(eps_low >= 0.f && eps_low <= 1.f) || !(eps_high >= 0.f) || !(beta >= 0.f))
        return ARROL_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n_seq == 0) {
        arrol_launch(grpo_finish_kernel<256>, dim3(1), dim3(256), 0, st, nullptr, nullptr, 0, objective_out, n_clipped);
        return arrol_launch_status();
    }
    if (!cu_seqlens || !advantage || !seq_weight || (T > 0 && (!logp || !logp_ref))) return ARROL_EINVAL;
    const int64_t room = static_cast<int64_t>(workspace_bytes / 16 / static_cast<size_t>(n_seq));   // partials per rollout
    if (!workspace || !arrol_aligned16(workspace) || room < 1) return ARROL_EWORKSPACE;
    // Rollouts are cut into parts of some 1,024 tokens where there are too few to fill the chip, up to 256 parts in all (one of
    // 20,000 tokens: 17.3 us whole, 7.2 in 8; 32 of 1,024 to 8,192: 9.7 and 5.9; but 256 of 2,000 6.0 and 7.5 in 4), and, of 3 million
    // tokens and more, where whole ones leave the units uneven (1,024 of 1,024 to 8,192: 25.3 and 22.6 in 4).
    int64_t n_seg = T < 800 ? 1 : (2 * (T / n_seq) + 1023) / 1024;      // (one of 700: 4.1 us whole, 4.4 in parts)
    const int64_t most = (T >= 3000000 ? 4096 : 256) / n_seq;
    n_seg = n_seg < kSegments ? n_seg : kSegments;
    n_seg = n_seg < most ? n_seg : most;
    n_seg = n_seg < room ? n_seg : room;
    n_seg = n_seg > 1 ? n_seg : 1;
    const int64_t n_parts = n_seq * n_seg;
    double* partial = static_cast<double*>(workspace);
    int64_t* clipped = reinterpret_cast<int64_t*>(partial + n_parts);
#define ARROL_OBJECTIVE(N)                                                                                                     \
    arrol_launch(grpo_objective_kernel<N>, dim3(n_seq, static_cast<unsigned>(n_seg)), dim3(N), 0, st, logp, logp_ref, cu_seqlens, T, \
                 advantage, seq_weight, static_cast<double>(eps_low), static_cast<double>(eps_high), static_cast<double>(beta),     \
                 grad_logp, partial, clipped)
    // wider workgroups shorten a long rollout's chain while the chip has room for them (one token at a time: 512 rollouts of 512 to 4,096
    // tokens 10.5 us with 512 threads, 11.3 with 256; 4,096 of 256 to 2,048 30.0 and 26.1)
    if (n_seg == 1 && T / n_seq > 1024 && n_seq <= 1024) ARROL_OBJECTIVE(512);
    else ARROL_OBJECTIVE(256);
#undef ARROL_OBJECTIVE
    // many: four partials a thread at a time; 256 threads are quicker to add up (one rollout: 4.2 us the call, 4.7 with 1,024)
    if (n_parts <= 1024)
        arrol_launch(grpo_finish_kernel<256>, dim3(1), dim3(256), 0, st, partial, clipped, n_parts, objective_out, n_clipped);
    else
        arrol_launch(grpo_finish_kernel<1024>, dim3(1), dim3(1024), 0, st, partial, clipped, n_parts, objective_out, n_clipped);
    return arrol_launch_status();
}
