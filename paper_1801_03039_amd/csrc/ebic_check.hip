// Duplicate columns of host populations, found on the device (gfx950).
//
// The host-array entry points refuse series that repeat a column.  Checking
// every column on the host costs about a nanosecond a column, more than the
// evaluation of a large pool; here a wave takes a series, lane t its t-th
// column, and every column is compared with all of them (a broadcast read
// and a compare per column).  Bound by the launch at a pool's size: 12288
// series of 3-20 columns take 5.7 us, against about 110 us on the host (a
// whole call from host arrays 231 -> 112 us).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ebic_internal.h"

namespace ebic {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

// counts[c] = -1 for every series c that repeats a column; others are left
// alone.  The offsets have been checked: they increase from 0.
__global__ __launch_bounds__(kBlock) void repeats_kernel(const int32_t *__restrict__ offsets,
                                                         const int32_t *__restrict__ cols,
                                                         int32_t P,
                                                         int32_t *__restrict__ counts) {
    const int64_t c = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (c >= P) return;   // whole waves leave
    const int lane = threadIdx.x & 63;
    const int32_t start = offsets[c], L = offsets[c + 1] - start;
    bool repeated = false;
    for (int32_t i0 = 0; i0 < L; i0 += 64) {
        const int32_t i = i0 + lane;
        const int32_t x = i < L ? cols[start + i] : 0;
        for (int32_t j0 = 0; j0 <= i0; j0 += 64) {
            const int32_t y = j0 == i0 ? x : cols[start + j0 + lane];   // a full block if j0 < i0
            const int32_t n = L - j0 < 64 ? L - j0 : 64;
            for (int32_t j = 0; j < n; ++j) {
                const int32_t z = __builtin_amdgcn_readlane(y, j);
                repeated |= i < L && j0 + j < i && z == x;
            }
        }
    }
    if (__ballot(repeated) != 0ull && lane == 0) counts[c] = -1;
}

}  // namespace

hipError_t launch_mark_repeats(const int32_t *offsets, const int32_t *cols, int32_t P,
                               int32_t *counts, hipStream_t stream) {
    if (P < 1) return hipSuccess;
    hipLaunchKernelGGL(repeats_kernel, dim3((unsigned)((P + kWaves - 1) / kWaves)), dim3(kBlock),
                       0, stream, offsets, cols, P, counts);
    return hipGetLastError();
}

}  // namespace ebic
