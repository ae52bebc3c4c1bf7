// Evaluation from the order index for tolerances of more than
// kIndexMaxViolations violating pairs: the index evaluator's tiles with
// binary violation counters (gfx950).  One 8-byte order word replaces the 64
// FP32 values the direct kernel reads per column, and the kernel is bound, as
// at small tolerances, by its chain of order-word reads and by the counters'
// registers: 2048 series of 6-20 columns on 20000 x 500, both directions,
// k = 5, take 226 us with the direct kernel and 22.7 us here.  That is with
// 2 pairs per batch of loads; 4 (100 VGPRs, 4 waves per SIMD) take 27.4 us,
// and 1 word per lane with 4 pairs 23.8 us.
#include "ebic_index_eval.h"

namespace ebic {
namespace {

// Tolerances above kIndexMaxViolations (binary counters, KM = 2^bits - 1 >=
// k): whole candidates with 1 word per lane up to 128 words and 2 up to
// kAlignedThreads lanes, flattened tiles of 2 words per lane beyond.
template <int KM, int U>
void launch_index_binary(const IndexRun &R, const EvalArgs &e, bool ties,
                                hipStream_t stream) {
    if (R.W <= kBlock / 2)
        launch_aligned<KM, U, 1>(R, e, ties, stream);
    else if (R.W <= 2 * kAlignedThreads)
        launch_aligned<KM, U, 2>(R, e, ties, stream);
    else {
        constexpr int V = kWordsPerLane;
        const int64_t total = (int64_t)R.P * ((R.W + V - 1) / V);
        const dim3 grid((unsigned)((total + kBlock - 1) / kBlock));
        launch_index_t<KM, U, V, false>(R, 0, grid, dim3(kBlock), e, ties, stream);
    }
}

}  // namespace

void launch_eval_index_binary(const IndexRun &R, const EvalArgs &e, bool ties,
                              hipStream_t stream) {
    if (e.k <= 7)
        launch_index_binary<7, 2>(R, e, ties, stream);
    else
        launch_index_binary<kIndexBinaryViolations, 2>(R, e, ties, stream);
}

}  // namespace ebic
