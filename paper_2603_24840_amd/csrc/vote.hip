// arrol_weighted_vote: rank-weighted answer vote (Sec. 4.4).  One wavefront per question,
// lane i owns candidate i.  Ranks are doubled average ranks, so everything after the fp32
// comparisons is integer and the result does not depend on candidate order.
#include "common.h"

namespace {

constexpr int kVoteThreads = 256;
constexpr int kQuestionsPerBlock = kVoteThreads / ARROL_WAVE;

// What bounds it is the chain of instructions of one wavefront.  The scores lie in LDS and are compared four at a time
// (a broadcast read each); slots beyond C hold NaN, which is neither below nor equal to anything.  Tallies: with
// TALLY_IN_LDS (up to kVoteLdsAnswers answer ids) every candidate adds its rank, and a one above 16 bits of it, to its
// answer's word, else the lanes sweep the ids 64 at a time over all candidates.  512 questions of 64 candidates and 16
// ids took 10.2 us with both loops shuffling candidate by candidate.
constexpr int kVoteLdsAnswers = 1024;

template <bool TALLY_IN_LDS>
__global__ __launch_bounds__(kVoteThreads) void vote_kernel(
    const float* __restrict__ prob, const int32_t* __restrict__ answer_id, int n_questions, int C,
    int n_answers, int32_t* __restrict__ winner, int64_t* __restrict__ tally) {
    extern __shared__ unsigned int words[];                     // TALLY_IN_LDS: [kQuestionsPerBlock][n_answers]
    __shared__ __attribute__((aligned(16))) float score[kQuestionsPerBlock][ARROL_WAVE];
    const int lane = threadIdx.x & (ARROL_WAVE - 1);
    const int wave = threadIdx.x / ARROL_WAVE;
    const int question = blockIdx.x * kQuestionsPerBlock + wave;
    if (question >= n_questions) return;                        // whole wave; nothing below waits for other waves
    const int64_t base = static_cast<int64_t>(question) * C;
    const bool has = lane < C;
    const float q = has ? prob[base + lane] : __builtin_nanf("");
    int ans = has ? answer_id[base + lane] : -1;
    if (ans < 0 || ans >= n_answers) ans = -1;  // takes no part
    score[wave][lane] = q;
    unsigned int* mine = words + static_cast<size_t>(wave) * n_answers;
    if (TALLY_IN_LDS)
        for (int a = lane; a < n_answers; a += ARROL_WAVE) mine[a] = 0u;
    wave_lds_exchange();
    const float4* others = reinterpret_cast<const float4*>(score[wave]);
    int below = 0, equal = 0;
    const auto compare = [&](auto reads) {
#pragma unroll
        for (int j = 0; j < decltype(reads)::value; ++j) {
            const float4 o = others[j];
            below += (o.x < q ? 1 : 0) + (o.y < q ? 1 : 0) + (o.z < q ? 1 : 0) + (o.w < q ? 1 : 0);
            equal += (o.x == q ? 1 : 0) + (o.y == q ? 1 : 0) + (o.z == q ? 1 : 0) + (o.w == q ? 1 : 0);
        }
    };
    if (C <= 16) compare(std::integral_constant<int, 4>{});
    else if (C <= 32) compare(std::integral_constant<int, 8>{});
    else compare(std::integral_constant<int, ARROL_WAVE / 4>{});
    const int rank2 = 2 * below + equal - (q == q ? 1 : 0);     // the candidate itself is not one of the equal ones
    if (TALLY_IN_LDS) {
        if (ans >= 0) atomicAdd(&mine[ans], static_cast<unsigned int>(rank2) | 0x10000u);   // at most 64 * 126 below
        wave_lds_exchange();
    }
    // lanes sweep the answer ids 64 at a time; each keeps its best (tally, lowest id) key
    int64_t best = -1;
    for (int a0 = 0; a0 < n_answers; a0 += ARROL_WAVE) {
        const int a = a0 + lane;
        int t = 0;
        bool occurs = false;
        if (TALLY_IN_LDS) {
            const unsigned int w = a < n_answers ? mine[a] : 0u;
            t = static_cast<int>(w & 0xffffu);
            occurs = w >= 0x10000u;
        } else {
            for (int j = 0; j < C; ++j)
                if (wave_bcast(ans, j) == a) { t += wave_bcast(rank2, j); occurs = true; }
        }
        if (a < n_answers) {
            if (tally) tally[static_cast<int64_t>(question) * n_answers + a] = t;
            if (occurs) {
                const int64_t key = (static_cast<int64_t>(t) << 32) | static_cast<int64_t>(0x7fffffff - a);
                best = key > best ? key : best;
            }
        }
    }
    best = wave_max_i64(best);
    if (lane == 0) winner[question] = best < 0 ? -1 : static_cast<int32_t>(0x7fffffff - (best & 0x7fffffffll));
}

}  // namespace

extern "C" int arrol_weighted_vote(const float* prob, const int32_t* answer_id, int32_t n_questions,
                                   int32_t C, int32_t n_answers, int32_t* winner, int64_t* tally,
                                   void* stream) {
    if (n_questions < 0 || C < 1 || C > ARROL_MAX_GROUP || n_answers < 1) return ARROL_EINVAL;
    if (n_questions == 0) return ARROL_OK;
    if (!prob || !answer_id || !winner) return ARROL_EINVAL;
    const int grid = (n_questions + kQuestionsPerBlock - 1) / kQuestionsPerBlock;
    const bool in_lds = n_answers <= kVoteLdsAnswers;
    const size_t lds = in_lds ? sizeof(unsigned int) * kQuestionsPerBlock * n_answers : 0;
    arrol_launch(in_lds ? vote_kernel<true> : vote_kernel<false>, dim3(grid), dim3(kVoteThreads), lds,
                 static_cast<hipStream_t>(stream), prob, answer_id, n_questions, C, n_answers, winner, tally);
    return arrol_launch_status();
}
