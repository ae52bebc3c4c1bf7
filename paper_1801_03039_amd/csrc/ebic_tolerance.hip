// Evaluation from the order index for tolerances of more than
// kIndexMaxViolations violating pairs: the index evaluator's tiles with
// wider violation counters (gfx950).  One 8-byte order word replaces the 64
// FP32 values the direct kernel reads per column: 2048 series of 6-20 columns
// on 20000 x 500, both directions, k = 5, take 226 us with the direct kernel
// and 16.5 us here (22.7 with the violations added pair by pair and 2 pairs
// per batch of loads).  The counters' registers limit the waves (90 VGPRs, 5
// per SIMD), so tolerances of 4 to 7 have a class of their own.
#include "ebic_index_eval.h"

namespace ebic {
namespace {

// KM = 2^bits - 1 >= k: whole candidates with 1 word per lane up to 128 words
// and 2 up to kAlignedThreads lanes (20000 rows: 16.5 us; 23.8 with 1 word),
// flattened tiles of 2 words per lane beyond.
template <int KM, int U>
void launch_index_wide(const IndexRun &R, const EvalArgs &e, hipStream_t stream) {
    if (R.W <= kBlock / 2)
        launch_aligned<KM, U, 1>(R, e, stream);
    else if (R.W <= 2 * kAlignedThreads)
        launch_aligned<KM, U, 2>(R, e, stream);
    else {
        constexpr int V = kWordsPerLane;
        const int64_t total = (int64_t)R.P * ((R.W + V - 1) / V);
        const dim3 grid((unsigned)((total + kBlock - 1) / kBlock));
        launch_index_t<KM, U, V, false>(R, 0, grid, dim3(kBlock), e, stream);
    }
}

}  // namespace

void launch_eval_index_wide(const IndexRun &R, const EvalArgs &e, hipStream_t stream) {
    if (e.k <= 7)
        launch_index_wide<7, kUnroll>(R, e, stream);
    else
        launch_index_wide<kIndexWideViolations, kUnroll>(R, e, stream);
}

}  // namespace ebic
