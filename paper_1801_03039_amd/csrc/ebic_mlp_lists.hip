// The lists behind the surrogate's embedding gradients (gfx950): the entries
// of a batch by column (position and candidate of every occurrence, in
// candidate-then-series order) and its candidates by series length.
//
// Both are stable counting sorts of small keys, in three launches: a wave
// counts the keys of its tile of items in LDS; the tiles' counts are summed
// per key; a wave places its tile's items, 64 at a time, behind what came
// before.  Within a wave, items of one key are ranked by the ballots of the
// key's bits, so the order is that of the items.  Bound by the launches and
// by a tile's chain of LDS updates: 94000 entries over 500 columns take 21 us
// (count 6.1, scan 6.5, place 8.0; on the host, with five blocking copies,
// about 190 us).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "ebic_mlp.h"

namespace ebic {
namespace mlp {
namespace {

constexpr int kWave = 64;
constexpr int64_t kTileItems = 256;    // items per tile, more if that makes over kMaxTiles
constexpr int64_t kMaxTiles = 1024;
constexpr int kGroup = 4;              // batches of 64 items whose keys are in flight
constexpr int kScanSegs = 16;          // the scan's lanes per key
constexpr int32_t kMaxKeys = 8192;     // LDS counters of a wave (32 KiB)

// One sort: items 0 .. n - 1 with keys in [0, keys); by column the key is
// cols[i], by length it is off[i + 1] - off[i].
struct Sort {
    int64_t n;
    int32_t keys, tiles;
    int64_t per;       // items per tile
    int32_t *hist;     // [tiles][keys]: counts, then items of earlier tiles
    int32_t *total;    // [keys]
    int32_t *start;    // [keys + 1]
};
struct Lists {
    Sort col, len;
    const int32_t *off, *cols;
    int32_t *owner;    // candidate of each entry
    int32_t *occ_pos, *occ_b, *len_b;
};

__device__ __forceinline__ int32_t key_of(const Lists &a, bool by_col, int64_t i) {
    return by_col ? a.cols[i] : a.off[i + 1] - a.off[i];
}

// Counts of a tile's keys.  Workgroup = one wave = one tile; the workgroups
// after the tiles write the owners of 64 candidates' entries each.
__global__ __launch_bounds__(kWave) void lists_count_kernel(Lists a) {
    extern __shared__ int32_t cnt[];
    const int lane = threadIdx.x;
    const int32_t tiles = a.col.tiles + a.len.tiles;
    if ((int)blockIdx.x >= tiles) {
        const int64_t b = (int64_t)((int)blockIdx.x - tiles) * kWave + lane;
        if (b < a.len.n)
            for (int32_t e = a.off[b], e1 = a.off[b + 1]; e < e1; ++e) a.owner[e] = (int32_t)b;
        return;
    }
    const bool by_col = (int)blockIdx.x < a.col.tiles;
    const Sort &s = by_col ? a.col : a.len;
    const int32_t tile = by_col ? (int32_t)blockIdx.x : (int32_t)blockIdx.x - a.col.tiles;
    for (int32_t k = lane; k < s.keys; k += kWave) cnt[k] = 0;
    __syncthreads();
    const int64_t lo = tile * s.per, hi = lo + s.per < s.n ? lo + s.per : s.n;
    for (int64_t i0 = lo + lane; i0 < hi; i0 += kWave * kGroup) {
        int32_t key[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u)
            key[u] = i0 + kWave * u < hi ? key_of(a, by_col, i0 + kWave * u) : -1;
#pragma unroll
        for (int u = 0; u < kGroup; ++u)
            if (key[u] >= 0) atomicAdd(&cnt[key[u]], 1);
    }
    __syncthreads();
    for (int32_t k = lane; k < s.keys; k += kWave) s.hist[(int64_t)tile * s.keys + k] = cnt[k];
}

// hist[t][k] <- items of key k in tiles before t; total[k] <- items of key k.
// Workgroup = 64 keys, kScanSegs ranges of tiles each.
__global__ __launch_bounds__(kWave *kScanSegs) void lists_scan_kernel(Lists a) {
    __shared__ int32_t part[kScanSegs][kWave];
    const int32_t col_blocks = (a.col.keys + kWave - 1) / kWave;
    const bool by_col = (int)blockIdx.x < col_blocks;
    const Sort &s = by_col ? a.col : a.len;
    const int32_t k = (by_col ? (int32_t)blockIdx.x : (int32_t)blockIdx.x - col_blocks) * kWave +
                      (int32_t)(threadIdx.x % kWave);
    const int seg = threadIdx.x / kWave;
    const int32_t each = (s.tiles + kScanSegs - 1) / kScanSegs;
    const int32_t t0 = min(seg * each, s.tiles), t1 = min(t0 + each, s.tiles);
    int32_t sum = 0;
    if (k < s.keys) {
#pragma unroll 8
        for (int32_t t = t0; t < t1; ++t) sum += s.hist[(int64_t)t * s.keys + k];
    }
    part[seg][threadIdx.x % kWave] = sum;
    __syncthreads();
    if (k >= s.keys) return;
    int32_t before = 0, all = 0;
    for (int i = 0; i < kScanSegs; ++i) {
        const int32_t x = part[i][threadIdx.x % kWave];
        before += i < seg ? x : 0;
        all += x;
    }
    if (seg == 0) s.total[k] = all;
    for (int32_t t = t0; t < t1; t += 8) {
        int32_t x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = t + u < t1 ? s.hist[(int64_t)(t + u) * s.keys + k] : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (t + u < t1) s.hist[(int64_t)(t + u) * s.keys + k] = before;
            before += x[u];
        }
    }
}

// Places a tile's items.  Workgroup = one wave = one tile, which first sums
// the keys' totals (the first tile also writes them as the lists' starts).
__global__ __launch_bounds__(kWave) void lists_place_kernel(Lists a) {
    extern __shared__ int32_t next[];   // per key: the place of its next item
    const bool by_col = (int)blockIdx.x < a.col.tiles;
    const Sort &s = by_col ? a.col : a.len;
    const int32_t tile = by_col ? (int32_t)blockIdx.x : (int32_t)blockIdx.x - a.col.tiles;
    const int lane = threadIdx.x;
    int32_t carry = 0;
    constexpr int kScan = 8;   // batches of 64 keys whose counts are in flight
    for (int32_t k0 = 0; k0 < s.keys; k0 += kWave * kScan) {
        int32_t c[kScan], before[kScan];
#pragma unroll
        for (int u = 0; u < kScan; ++u) {
            const int32_t k = k0 + kWave * u + lane;
            c[u] = k < s.keys ? s.total[k] : 0;
            before[u] = k < s.keys ? s.hist[(int64_t)tile * s.keys + k] : 0;
        }
#pragma unroll
        for (int u = 0; u < kScan; ++u) {
            const int32_t k = k0 + kWave * u + lane;
            int32_t x = c[u];
            for (int d = 1; d < kWave; d <<= 1) {
                const int32_t y = __shfl_up(x, d);
                if (lane >= d) x += y;
            }
            const int32_t first = carry + x - c[u];
            if (k < s.keys) {
                next[k] = first + before[u];
                if (tile == 0) s.start[k] = first;
            }
            carry += __shfl(x, kWave - 1);
        }
    }
    if (tile == 0 && lane == 0) s.start[s.keys] = carry;
    __syncthreads();
    const int bits = s.keys > 1 ? 32 - __clz(s.keys - 1) : 0;
    const int64_t lo = tile * s.per, hi = lo + s.per < s.n ? lo + s.per : s.n;
    for (int64_t g0 = lo; g0 < hi; g0 += kWave * kGroup) {
        int32_t keys[kGroup], owner[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const int64_t i = g0 + kWave * u + lane;
            keys[u] = i < hi ? key_of(a, by_col, i) : 0;
            owner[u] = by_col && i < hi ? a.owner[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const int64_t i = g0 + kWave * u + lane;
            const bool have = i < hi;
            const int32_t key = keys[u];
            uint64_t same = __ballot(have);   // the lanes with this lane's key
            for (int b = 0; b < bits; ++b) {
                const bool set = (key >> b) & 1;
                const uint64_t m = __ballot(set);
                same &= set ? m : ~m;
            }
            const int32_t base = next[key];
            const int32_t rank = __popcll(same & ((1ull << lane) - 1ull));
            __syncthreads();
            if (have && rank == 0) next[key] = base + __popcll(same);
            __syncthreads();
            if (have && by_col) {
                a.occ_pos[base + rank] = (int32_t)i;
                a.occ_b[base + rank] = owner[u];
            } else if (have) {
                a.len_b[base + rank] = (int32_t)i;
            }
        }
    }
}

Sort make_sort(int64_t n, int32_t keys, int32_t *ws, int32_t *start) {
    Sort s{};
    s.n = n;
    s.keys = keys;
    s.per = std::max(kTileItems,
                     ((n + kMaxTiles - 1) / kMaxTiles + kWave - 1) / kWave * kWave);
    s.tiles = (int32_t)((n + s.per - 1) / s.per);
    s.hist = ws;
    s.total = ws ? ws + (int64_t)s.tiles * keys : nullptr;
    s.start = start;
    return s;
}

int64_t ws_ints(const Sort &s) { return ((int64_t)s.tiles + 1) * s.keys; }

}  // namespace

bool lists_on_device(int32_t M) { return M + 1 <= kMaxKeys; }

int64_t lists_workspace(int64_t B, int64_t L, int32_t M) {
    return ws_ints(make_sort(L, M, nullptr, nullptr)) +
           ws_ints(make_sort(B, M + 1, nullptr, nullptr)) + L;
}

hipError_t build_lists(const int32_t *off, const int32_t *cols, int32_t B, int64_t L, int32_t M,
                       int32_t *ws, int32_t *occ_start, int32_t *occ_pos, int32_t *occ_b,
                       int32_t *len_start, int32_t *len_b, hipStream_t s) {
    Lists a{};
    a.col = make_sort(L, M, ws, occ_start);
    ws += ws_ints(a.col);
    a.len = make_sort(B, M + 1, ws, len_start);
    ws += ws_ints(a.len);
    a.off = off;
    a.cols = cols;
    a.owner = ws;
    a.occ_pos = occ_pos;
    a.occ_b = occ_b;
    a.len_b = len_b;
    const dim3 tiles((unsigned)(a.col.tiles + a.len.tiles));
    const unsigned lds = (unsigned)sizeof(int32_t) * (unsigned)(M + 1);
    const dim3 count((unsigned)(a.col.tiles + a.len.tiles + (B + kWave - 1) / kWave));
    hipLaunchKernelGGL(lists_count_kernel, count, dim3(kWave), lds, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)((M + kWave - 1) / kWave + (M + 1 + kWave - 1) / kWave);
    hipLaunchKernelGGL(lists_scan_kernel, dim3(blocks), dim3(kWave * kScanSegs), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(lists_place_kernel, tiles, dim3(kWave), lds, s, a);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace ebic
