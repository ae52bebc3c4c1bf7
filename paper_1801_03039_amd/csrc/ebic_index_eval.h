// The single-run index evaluator: its kernel and the launch of one of its
// tilings (gfx950).  Included by the .hip files that instantiate it.
//
// What bounds it: at the sizes of a search all workgroups are resident at
// once, and a launch lasts as long as the slowest workgroup's chain of
// dependent reads (offsets, columns, one batch of order words after the
// other), each about a microsecond; larger launches are bound by the order
// words they read.  Both leave room only where the instructions between the
// reads are few: with the offsets of the order rows formed while staging, the
// four-pair adders and the tied rows kept out of the loop, a pair takes about
// 17 VALU operations per lane for 2 words in both directions at k = 1 (60
// before), and 2048 series on 20000 x 200 take 10.2 us (11.6), 12288 series
// on 20000 x 500 50 us (61), 1024 series on 100003 x 101 at k = 2 18.2 us
// (20.5, rising only) and 20.6 (27.7, both directions).
#pragma once

#include <algorithm>

#include "ebic_device.h"

namespace ebic {
namespace {

// Waves per SIMD that the registers of the 2-word falling-trend kernels leave
// room for: as many as with the fast loop alone, which the other loop would
// exceed by a few registers (12288 series on 20000 rows, k = 1: 43.1 us with
// 8 waves, 47.4 with 7; 2048 series, k = 5: 16.4 with 5, 19.0 with 4).
constexpr int min_waves(int K, bool NEG, int V, bool ALIGNED, bool OFF32) {
    if (!NEG || V != 2) return 1;
    if (K == 7) return 5;
    if (K <= 1) return OFF32 || !ALIGNED ? 8 : 1;
    return K == 3 && OFF32 ? 6 : 1;
}

template <int K, bool NEG, int U, int V, bool ALIGNED, bool OFF32, bool TAIL>
__global__ __launch_bounds__(kAlignedThreads, min_waves(K, NEG, V, ALIGNED, OFF32)) void eval_index_kernel(
    IndexRun R, uint32_t cpw, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ cols, int64_t n_entries, int32_t sigma,
    uint64_t *__restrict__ masks, unsigned long long *__restrict__ acc,
    int32_t *__restrict__ counts, double *__restrict__ fitness, int32_t stage) {
    __shared__ TileLds lds;
    extern __shared__ uint64_t s_stage[];
    index_tile<K, NEG, U, V, ALIGNED, OFF32, TAIL>(R, blockIdx.x, cpw, offsets, cols, n_entries,
                                                   sigma, masks, acc, counts, fitness, lds,
                                                   StageLds(s_stage, stage));
}

template <int K, int U, int V, bool ALIGNED, bool OFF32, bool TAIL>
void launch_index_o(const IndexRun &R, uint32_t cpw, dim3 grid, dim3 block, const EvalArgs &e,
                    hipStream_t stream) {
    // Room for the series of a workgroup at their mean length and a quarter
    // more (n_entries may count room past the last series, which only makes
    // the area larger).
    const int64_t series = ALIGNED ? cpw : 2 + kBlock / ((R.W + V - 1) / V);
    const int32_t stage = stage_entries(series * (e.n_entries / e.P + 1) * 5 / 4);
    const unsigned lds = stage_bytes(stage);
    if (e.negative)
        hipLaunchKernelGGL((eval_index_kernel<K, true, U, V, ALIGNED, OFF32, TAIL>), grid, block,
                           lds, stream, R, cpw, e.offsets, e.cols, e.n_entries, e.sigma, e.masks,
                           e.acc, e.counts, e.fitness, stage);
    else
        hipLaunchKernelGGL((eval_index_kernel<K, false, U, V, ALIGNED, OFF32, TAIL>), grid, block,
                           lds, stream, R, cpw, e.offsets, e.cols, e.n_entries, e.sigma, e.masks,
                           e.acc, e.counts, e.fitness, stage);
}

// 32-bit index offsets when the whole index is below 4 GiB.
template <int K, int U, int V, bool ALIGNED, bool TAIL = false>
void launch_index_t(const IndexRun &R, uint32_t cpw, dim3 grid, dim3 block,
                           const EvalArgs &e, hipStream_t stream) {
    const uint64_t bytes = (uint64_t)R.m * (uint64_t)R.m * (uint64_t)R.wpad * 8ull;
    if (bytes <= 0xFFFFFFFFull)
        launch_index_o<K, U, V, ALIGNED, true, TAIL>(R, cpw, grid, block, e, stream);
    else
        launch_index_o<K, U, V, ALIGNED, false, TAIL>(R, cpw, grid, block, e, stream);
}

// Whole-candidate workgroups.  With 4 words per lane, as many candidates as
// fit in 256 lanes.  With 1 or 2, the candidate count (up to 320 lanes) that
// leaves the fewest idle lanes in the workgroup's whole waves: e.g. 2
// candidates of 157 lanes in 5 waves instead of 1 in 3 waves with 35 idle
// lanes (measured 6% faster at 20000 rows, 7% at 5000; with 4 words per
// lane the same rule was slower).
template <int K, int U, int V, bool TAIL = false>
void launch_aligned(const IndexRun &R, const EvalArgs &e, hipStream_t stream) {
    const int64_t Wg = (R.W + V - 1) / V;
    int64_t cpw = kBlock / Wg;
    if (V <= 2) {
        int64_t best = INT64_MAX;
        for (int64_t c = 1; c <= kBlock && c * Wg <= kAlignedThreads; ++c) {
            const int64_t th = (c * Wg + kWave - 1) / kWave * kWave;
            const int64_t idle = (th - c * Wg) * 4096 / th;   // idle share, 1/4096 units
            if (idle < best) {
                best = idle;
                cpw = c;
            }
        }
    }
    // Few lanes and many series: further waves, which only stage, until a lane
    // has about 4 entries (4096 series of 20-28 columns on 60 rows, both
    // directions, k = 1: 9.0 us with the 64 lanes of the series, 5.1 with 256).
    const dim3 grid((unsigned)((R.P + cpw - 1) / cpw));
    int64_t stagers = std::min<int64_t>(cpw * (e.n_entries / R.P + 1) / 4, kBlock);
    if ((int64_t)grid.x * kBlock > INT32_MAX) stagers = 0;   // (a launch's lanes are limited)
    const int64_t threads = (std::max(cpw * Wg, stagers) + kWave - 1) / kWave * kWave;
    launch_index_t<K, U, V, true, TAIL>(R, (uint32_t)cpw, grid, dim3((unsigned)threads), e,
                                        stream);
}

}  // namespace
}  // namespace ebic
