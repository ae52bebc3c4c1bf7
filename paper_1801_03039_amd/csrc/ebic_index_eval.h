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

#include "ebic_device.h"

namespace ebic {
namespace {

template <int K, bool NEG, int U, int V, bool ALIGNED, bool OFF32, bool TAIL>
__global__ __launch_bounds__(kAlignedThreads) void eval_index_kernel(
    IndexRun R, uint32_t cpw, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ cols, int64_t n_entries, int32_t sigma,
    uint64_t *__restrict__ masks, unsigned long long *__restrict__ acc,
    int32_t *__restrict__ counts, double *__restrict__ fitness) {
    __shared__ TileLds lds;
    index_tile<K, NEG, U, V, ALIGNED, OFF32, TAIL>(R, blockIdx.x, cpw, offsets, cols, n_entries,
                                                   sigma, masks, acc, counts, fitness, lds);
}

template <int K, int U, int V, bool ALIGNED, bool OFF32, bool TAIL>
void launch_index_o(const IndexRun &R, uint32_t cpw, dim3 grid, dim3 block, const EvalArgs &e,
                    hipStream_t stream) {
    if (e.negative)
        hipLaunchKernelGGL((eval_index_kernel<K, true, U, V, ALIGNED, OFF32, TAIL>), grid, block,
                           0, stream, R, cpw, e.offsets, e.cols, e.n_entries, e.sigma, e.masks,
                           e.acc, e.counts, e.fitness);
    else
        hipLaunchKernelGGL((eval_index_kernel<K, false, U, V, ALIGNED, OFF32, TAIL>), grid, block,
                           0, stream, R, cpw, e.offsets, e.cols, e.n_entries, e.sigma, e.masks,
                           e.acc, e.counts, e.fitness);
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
    const int64_t threads = (cpw * Wg + kWave - 1) / kWave * kWave;
    const dim3 grid((unsigned)((R.P + cpw - 1) / cpw));
    launch_index_t<K, U, V, true, TAIL>(R, (uint32_t)cpw, grid, dim3((unsigned)threads), e,
                                        stream);
}

}  // namespace
}  // namespace ebic
