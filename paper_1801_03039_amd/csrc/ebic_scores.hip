// Step 6 output and the accuracy scores of Section 3 on the device:
//   * row-index lists from 64-row masks (prefix sums of popcounts, then a
//     scatter in increasing row order);
//   * the cell Jaccard index of every (found, expected) bicluster pair and
//     the recovery / relevance scores of Eqs. (2)-(3).
// Integer work throughout; the only floating point is one FP64 division per
// Jaccard index, the max over a row or column of the index matrix and two
// sums taken in index order, so results are bit-exact and deterministic.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <type_traits>

#include "ebic_internal.h"

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

__device__ inline uint64_t tail_word(uint64_t v, int64_t w, int64_t W, uint64_t tail) {
    return w == W - 1 ? v & tail : v;
}

// Union of a bicluster's mask planes for word w.  PL: the number of planes
// (1: one mask, 2: both trend directions) if the kernel is built for it, so
// that their loads are in flight together; 0: `planes` at run time.
template <int PL>
__device__ inline uint64_t plane_or(const uint64_t *m, int32_t planes, int64_t W, int64_t w) {
    uint64_t v = m[w];
    if constexpr (PL == 2) v |= m[W + w];
    if constexpr (PL == 0)
        for (int32_t p = 1; p < planes; ++p) v |= m[(int64_t)p * W + w];
    return v;
}

// f(integral_constant<int, PL>) for the plane count's kernel form.
template <class F>
void for_planes(int32_t planes, F &&f) {
    if (planes == 1) f(std::integral_constant<int, 1>{});
    else if (planes == 2) f(std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 0>{});
}

template <typename T>
__device__ inline T wave_sum(T v) {
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// Exclusive prefix sum of v over the 256 threads of the block; *total gets
// the block's sum.  s_wave holds kWaves partial sums.
template <typename T>
__device__ inline T block_exclusive_scan(T v, T *s_wave, T *total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    T x = v;
    for (int d = 1; d < 64; d <<= 1) {
        const T y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_wave[wid] = x;
    __syncthreads();
    T base = 0, tot = 0;
    for (int i = 0; i < kWaves; ++i) {
        const T t = s_wave[i];
        if (i < wid) base += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return base + x - v;
}

// offsets[k + 1] = number of rows in bicluster k.  One block per bicluster.
template <int PL>
__global__ __launch_bounds__(kBlock) void mask_count_kernel(const uint64_t *masks, int32_t planes,
                                                            int64_t W, uint64_t tail,
                                                            int64_t *offsets) {
    const int64_t k = blockIdx.x;
    const uint64_t *m = masks + k * planes * W;
    int64_t c = 0;
    for (int64_t w = threadIdx.x; w < W; w += kBlock)
        c += __popcll(tail_word(plane_or<PL>(m, planes, W, w), w, W, tail));
    c = wave_sum(c);
    __shared__ int64_t s[kWaves];
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int i = 0; i < kWaves; ++i) t += s[i];
        offsets[k + 1] = t;
    }
}

// In-place inclusive scan of offsets[1..K]; offsets[0] = 0.  One block.
__global__ __launch_bounds__(kBlock) void offsets_scan_kernel(int64_t *offsets, int32_t K) {
    __shared__ int64_t s_wave[kWaves];
    int64_t carry = 0;
    for (int32_t base = 0; base < K; base += kBlock) {
        const int32_t i = base + (int32_t)threadIdx.x;
        const int64_t v = i < K ? offsets[i + 1] : 0;
        int64_t total;
        const int64_t ex = block_exclusive_scan(v, s_wave, &total);
        if (i < K) offsets[i + 1] = carry + ex + v;
        carry += total;
    }
    if (threadIdx.x == 0) offsets[0] = 0;
}

// Row indices of bicluster k at rows[offsets[k] ...], increasing; entries at
// or beyond `capacity` are not written.  Block (k, s) writes the rows of the
// s-th chunk of `chunk` words; where they start follows from the popcounts
// of the words before, which the block reads again (16 chunks at most, so
// the masks are read 8 times on average, from L2).  A wave takes 16 words
// at a time: each word is made uniform, lane b holds its bit b, and the
// set lanes store neighbouring entries.  Bound by latency at a search's
// sizes: 100 lists from 20000 rows took 16.3 us with one block per
// bicluster and a thread per word, storing its bits one after the other,
// and take 5.2 us.
constexpr int64_t kScatterWords = 16 * kWaves;   // words per block and step
constexpr int64_t kScatterChunks = 16;           // blocks per bicluster at most
template <int PL>
__global__ __launch_bounds__(kBlock) void mask_scatter_kernel(const uint64_t *masks, int32_t planes,
                                                              int64_t W, uint64_t tail,
                                                              const int64_t *offsets, int32_t *rows,
                                                              int64_t capacity, int64_t chunk) {
    const int64_t k = blockIdx.x;
    const uint64_t *m = masks + k * planes * W;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t w_lo = (int64_t)blockIdx.y * chunk, w_hi = w_lo + chunk < W ? w_lo + chunk : W;
    __shared__ int64_t s_part[kWaves];
    __shared__ int32_t s_step[2][kWaves];
    int64_t before = 0;
    for (int64_t w = threadIdx.x; w < w_lo; w += kBlock)
        before += __popcll(plane_or<PL>(m, planes, W, w));
    before = wave_sum(before);
    if (lane == 0) s_part[wv] = before;
    __syncthreads();
    int64_t pos0 = offsets[k];
    for (int i = 0; i < kWaves; ++i) pos0 += s_part[i];
    int step = 0;
    for (int64_t w0 = w_lo; w0 < w_hi; w0 += kScatterWords, step ^= 1) {
        // lanes 0..15: the wave's 16 words and their exclusive prefix sums
        const int64_t w = w0 + 16 * wv + lane;
        const uint64_t v =
            lane < 16 && w < w_hi ? tail_word(plane_or<PL>(m, planes, W, w), w, W, tail) : 0ull;
        const int32_t c = __popcll(v);
        int32_t x = c;
        for (int d = 1; d < 16; d <<= 1) {
            const int32_t y = __shfl_up(x, d, 16);
            if ((lane & 15) >= d) x += y;
        }
        if (lane == 15) s_step[step][wv] = x;
        __syncthreads();   // (two sets: a wave may be one step ahead)
        int32_t base = 0, total = 0;
        for (int i = 0; i < kWaves; ++i) {
            const int32_t t = s_step[step][i];
            if (i < wv) base += t;
            total += t;
        }
        const int32_t first = base + x - c;
        for (int i = 0; i < 16; ++i) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, i);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), i);
            const int32_t at = __builtin_amdgcn_readlane(first, i);
            const uint64_t word = ((uint64_t)hi << 32) | lo;
            const int64_t pos =
                pos0 + at + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
            if (((word >> lane) & 1ull) && pos < capacity)
                rows[pos] = (int32_t)((w0 + 16 * wv + i) * 64 + lane);
        }
        pos0 += total;
    }
}

struct SetView {
    const uint64_t *masks;
    int32_t planes;
    const int32_t *off;
    const int32_t *cols;
};

// Whether the wave's lane value c occurs in list[0..n) before place `upto`.
// The entries are read once per wave, 64 at a time, and made uniform: every
// lane has to take part.
__device__ inline bool occurs(const int32_t *list, int32_t n, int32_t c, int32_t upto) {
    const int lane = threadIdx.x & 63;
    bool in = false;
    for (int32_t base = 0; base < n; base += 64) {
        const int32_t cnt = n - base < 64 ? n - base : 64;
        const int32_t x = base + lane < n ? list[base + lane] : 0;
        for (int32_t j = 0; j < cnt; ++j) {
            const int32_t entry = __builtin_amdgcn_readlane(x, j);
            in |= base + j < upto && entry == c;
        }
    }
    return in;
}

// Distinct columns of the list a[0..la) (each counted at its first place)
// and how many of them occur in b[0..lb), for lists of any length; the
// results are uniform over the wave.
__device__ inline void column_counts(const int32_t *a, int32_t la, const int32_t *b, int32_t lb,
                                     int32_t *distinct, int32_t *shared) {
    const int lane = threadIdx.x & 63;
    int32_t d = 0, s = 0;
    for (int32_t base = 0; base < la; base += 64) {
        const int32_t i = base + lane;
        const int32_t c = i < la ? a[i] : 0;
        const int32_t end = base + 64 < la ? base + 64 : la;
        const bool before = occurs(a, end, c, i);
        const bool in = occurs(b, lb, c, lb);
        const bool first = i < la && !before;
        d += __popcll(__ballot(first));
        s += __popcll(__ballot(first && in));
    }
    *distinct = d;
    *shared = s;
}

// J[f * E + e] for every pair; a wave takes one found bicluster and TE
// expected ones, whose words meet the found one's in registers (TE = 4 reads
// 6 words for 4 pairs of 2-plane and 1-plane masks, TE = 1 3 for one).
// The row counts are exact in T (32 bits up to INT32_MAX rows).  Bound by
// latency at a search's sizes: 100 x 20 biclusters of 20000 rows took 16.2
// us, most of it in column scans that waited for one entry after the other,
// and take 8.3 us.
template <typename T, int TE, int FP, int EP>
__global__ __launch_bounds__(kBlock) void jaccard_kernel(SetView fs, int32_t F, SetView es,
                                                         int32_t E, int64_t W, uint64_t tail,
                                                         double *J) {
    const int32_t groups = (E + TE - 1) / TE;
    const int64_t item = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (item >= (int64_t)F * groups) return;   // whole waves leave; no block barrier follows
    const int32_t f = (int32_t)(item / groups), e0 = (int32_t)(item % groups) * TE;
    const int lane = threadIdx.x & 63;
    const uint64_t *a = fs.masks + (int64_t)f * fs.planes * W;
    const uint64_t *b[TE];
    for (int i = 0; i < TE; ++i)   // past the last one: repeated, not stored
        b[i] = es.masks + (int64_t)(e0 + i < E ? e0 + i : E - 1) * es.planes * W;
    // The columns of lists of up to 64 entries, one per lane, are in flight
    // with the masks.
    const int32_t *ca = fs.cols + fs.off[f];
    const int32_t la = fs.off[f + 1] - fs.off[f];
    const int32_t xa = lane < la ? ca[lane] : 0;
    const int32_t *cb[TE];
    int32_t lb[TE], xb[TE];
    bool short_lists = la <= 64;
#pragma unroll
    for (int i = 0; i < TE; ++i) {
        const int32_t e = e0 + i < E ? e0 + i : E - 1;
        cb[i] = es.cols + es.off[e];
        lb[i] = es.off[e + 1] - es.off[e];
        xb[i] = lane < lb[i] ? cb[i][lane] : 0;
        short_lists = short_lists && lb[i] <= 64;
    }
    // four words per lane in flight; past the end the last word, ignored
    T na = 0, nb[TE] = {}, ni[TE] = {};
    constexpr int U = TE == 1 ? 4 : 2;
    for (int64_t w0 = lane; w0 < W; w0 += 64 * U) {
        uint64_t x[U], y[TE][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t w = w0 + 64 * u < W ? w0 + 64 * u : W - 1;
            x[u] = plane_or<FP>(a, fs.planes, W, w);
#pragma unroll
            for (int i = 0; i < TE; ++i) y[i][u] = plane_or<EP>(b[i], es.planes, W, w);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t w = w0 + 64 * u;
            const uint64_t keep = w < W - 1 ? ~0ull : (w == W - 1 ? tail : 0ull);
            na += (T)__popcll(x[u] & keep);
#pragma unroll
            for (int i = 0; i < TE; ++i) {
                nb[i] += (T)__popcll(y[i][u] & keep);
                ni[i] += (T)__popcll(x[u] & y[i][u] & keep);
            }
        }
    }
    na = wave_sum(na);
    bool first_a = lane < la;   // the lane's found column has not occurred before it
    if (short_lists)
        for (int32_t j = 0; j + 1 < la; ++j) {
            const int32_t c = __builtin_amdgcn_readlane(xa, j);
            first_a = first_a && !(j < lane && c == xa);
        }
#pragma unroll
    for (int i = 0; i < TE; ++i) {
        const int32_t e = e0 + i;
        if (e >= E) break;
        nb[i] = wave_sum(nb[i]);
        ni[i] = wave_sum(ni[i]);
        int32_t da, db, sh;   // distinct columns of each, shared ones
        if (short_lists) {
            bool in_b = false, first_b = lane < lb[i];
            for (int32_t j = 0; j < lb[i]; ++j) {
                const int32_t c = __builtin_amdgcn_readlane(xb[i], j);
                in_b |= c == xa;
                first_b = first_b && !(j < lane && c == xb[i]);
            }
            da = __popcll(__ballot(first_a));
            db = __popcll(__ballot(first_b));
            sh = __popcll(__ballot(first_a && in_b));
        } else {
            int32_t again;   // the shared columns counted from the other side: the same
            column_counts(ca, la, cb[i], lb[i], &da, &sh);
            column_counts(cb[i], lb[i], ca, la, &db, &again);
        }
        if (lane == 0) {
            const int64_t inter = (int64_t)ni[i] * sh;
            const int64_t uni = (int64_t)na * da + (int64_t)nb[i] * db - inter;
            J[(int64_t)f * E + e] = uni > 0 ? (double)inter / (double)uni : 0.0;
        }
    }
}

// acc + at(0) + at(1) + ... + at(n - 1) in that order, eight reads in flight.
template <class F>
__device__ inline double add_in_order(double acc, int32_t n, F &&at) {
    int32_t t = 0;
    for (; t + 8 <= n; t += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = at(t + u);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; t < n; ++t) acc += at(t);
    return acc;
}

// scores[0] = recovery, scores[1] = relevance.  One block: the maxima of a
// chunk of columns or rows of J are formed in parallel, then added in index
// order by one thread.  Recovery: kScoreCols columns at a time, each by the
// threads of its residue, whose maxima (bit patterns of values >= 0 order
// as integers) meet in LDS.  Relevance: kScoreRow lanes to a row.  Bound by
// latency (and by the ordered sum, one FP64 addition after the other, for
// long lists): 100 x 20 took 27.8 us with one thread per maximum, and takes
// 4.1 us.
constexpr int kScoreBlock = 1024;
constexpr int kScoreCols = 512;     // columns of a recovery chunk
constexpr int kScoreRow = 8;        // lanes per row of a relevance chunk
constexpr int kScoreRows = kScoreBlock / kScoreRow;
__global__ __launch_bounds__(kScoreBlock) void scores_kernel(const double *J, int32_t F, int32_t E,
                                                             double *scores) {
    __shared__ unsigned long long s_max[kScoreCols];
    __shared__ double s_row[kScoreRows];
    const int tid = threadIdx.x;
    double recovery = 0.0, relevance = 0.0;
    for (int32_t base = 0; base < E; base += kScoreCols) {
        const int32_t n = E - base < kScoreCols ? E - base : kScoreCols;
        if (tid < kScoreCols) s_max[tid] = 0ull;
        __syncthreads();
        const int32_t g = tid / n, c = tid - g * n, groups = kScoreBlock / n;
        if (g < groups) {
            double mx = 0.0;
            for (int32_t f = g; f < F; f += 8 * groups) {
                double v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int32_t r = f + u * groups;
                    v[u] = r < F ? J[(int64_t)r * E + base + c] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) mx = v[u] > mx ? v[u] : mx;
            }
            atomicMax(&s_max[c], (unsigned long long)__double_as_longlong(mx));
        }
        __syncthreads();
        if (tid == 0)
            recovery = add_in_order(recovery, n, [&](int32_t t) {
                return __longlong_as_double((long long)s_max[t]);
            });
        __syncthreads();
    }
    for (int32_t base = 0; base < F; base += kScoreRows) {
        const int32_t n = F - base < kScoreRows ? F - base : kScoreRows;
        const int32_t r = tid / kScoreRow, q = tid % kScoreRow;
        double mx = 0.0;
        if (r < n)
            for (int32_t e = q; e < E; e += 8 * kScoreRow) {
                double v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int32_t x = e + u * kScoreRow;
                    v[u] = x < E ? J[(int64_t)(base + r) * E + x] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) mx = v[u] > mx ? v[u] : mx;
            }
        for (int d = kScoreRow / 2; d >= 1; d >>= 1) {
            const double o = __shfl_xor(mx, d);
            mx = o > mx ? o : mx;
        }
        if (q == 0) s_row[r] = mx;
        __syncthreads();
        if (tid == 0)
            relevance = add_in_order(relevance, n, [&](int32_t t) { return s_row[t]; });
        __syncthreads();
    }
    if (tid == 0) {
        const bool none = F == 0 || E == 0;
        scores[0] = none ? 0.0 : recovery / (double)E;
        scores[1] = none ? 0.0 : relevance / (double)F;
    }
}

ebic_status arg_error(const std::string &msg) {
    ebic::set_thread_error(msg.c_str());
    return EBIC_E_ARG;
}

ebic_status hip_error(hipError_t e, const char *what) {
    ebic::set_thread_error((std::string(what) + ": " + hipGetErrorString(e)).c_str());
    return EBIC_E_DEVICE;
}

uint64_t tail_mask(int64_t n_rows) {
    const int r = (int)(n_rows % 64);
    return r == 0 ? ~0ull : ((1ull << r) - 1);
}

bool set_ok(const ebic_bicluster_set *s, const char *name, std::string *msg) {
    if (!s || s->struct_size < sizeof(ebic_bicluster_set)) {
        *msg = std::string(name) + ": null or struct_size too small";
        return false;
    }
    if (s->count < 0 || (s->count > 0 && (s->planes < 1 || !s->row_masks || !s->col_offsets ||
                                          !s->cols))) {
        *msg = std::string(name) + ": count < 0, planes < 1 or a null device pointer";
        return false;
    }
    return true;
}

}  // namespace

extern "C" {

ebic_status ebic_mask_rows(const uint64_t *d_masks, int32_t K, int32_t planes, int64_t n_rows,
                           int64_t *d_offsets, int32_t *d_rows, int64_t rows_capacity,
                           void *hip_stream) {
    if (K < 0 || n_rows < 0 || rows_capacity < 0) return arg_error("K, n_rows, capacity >= 0");
    if (n_rows > INT32_MAX) return arg_error("n_rows must fit int32 row indices");
    if (!d_offsets) return arg_error("d_offsets is null");
    if (K > 0 && planes < 1) return arg_error("planes must be >= 1");
    if (K > 0 && n_rows > 0 && !d_masks) return arg_error("d_masks is null");
    if (rows_capacity > 0 && !d_rows) return arg_error("d_rows is null");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int64_t W = n_rows == 0 ? 0 : (n_rows + 63) / 64;
    hipError_t e;
    if (K > 0) {
        // With no rows (W = 0) every count is 0 and the masks are not read.
        for_planes(planes, [&](auto pl) {
            hipLaunchKernelGGL((mask_count_kernel<decltype(pl)::value>), dim3((unsigned)K),
                               dim3(kBlock), 0, s, d_masks, planes, W, tail_mask(n_rows),
                               d_offsets);
        });
        if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "mask_count_kernel");
    }
    hipLaunchKernelGGL(offsets_scan_kernel, dim3(1), dim3(kBlock), 0, s, d_offsets, K);
    if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "offsets_scan_kernel");
    if (K > 0 && W > 0 && rows_capacity > 0) {
        int64_t chunk = (W + kScatterChunks - 1) / kScatterChunks;
        chunk = (chunk + kScatterWords - 1) / kScatterWords * kScatterWords;
        const dim3 grid((unsigned)K, (unsigned)((W + chunk - 1) / chunk));
        for_planes(planes, [&](auto pl) {
            hipLaunchKernelGGL((mask_scatter_kernel<decltype(pl)::value>), grid, dim3(kBlock), 0,
                               s, d_masks, planes, W, tail_mask(n_rows), d_offsets, d_rows,
                               rows_capacity, chunk);
        });
        if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "mask_scatter_kernel");
    }
    return EBIC_OK;
}

ebic_status ebic_match_scores(const ebic_bicluster_set *found, const ebic_bicluster_set *expected,
                              int64_t n_rows, double *d_jaccard, double *d_scores,
                              void *hip_stream) {
    std::string msg;
    if (!set_ok(found, "found", &msg) || !set_ok(expected, "expected", &msg))
        return arg_error(msg);
    if (n_rows < 0) return arg_error("n_rows must be >= 0");
    if (!d_scores) return arg_error("d_scores is null");
    const int64_t F = found->count, E = expected->count;
    if (F * E > 0 && !d_jaccard) return arg_error("d_jaccard is null");
    if (F * E > (int64_t)INT32_MAX * kWaves) return arg_error("too many bicluster pairs");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int64_t W = (n_rows + 63) / 64;
    hipError_t e;
    if (F * E > 0) {
        SetView fs{found->row_masks, found->planes, found->col_offsets, found->cols};
        SetView es{expected->row_masks, expected->planes, expected->col_offsets, expected->cols};
        // Four expected biclusters to a wave once that still leaves each of
        // the GPU's 1024 SIMDs a wave (120 x 60 biclusters of 50000 rows:
        // 16.0 us, 18.4 with one); one otherwise, where more waves hide more
        // latency (100 x 20 of 20000 rows: 8.3 us, 11.6 with four).
        const bool tiled = F * ((E + 3) / 4) >= 1024;
        const int64_t waves = F * (tiled ? (E + 3) / 4 : E);
        const int64_t blocks = (waves + kWaves - 1) / kWaves;
        auto launch = [&](auto type, auto te) {
            for_planes(found->planes, [&](auto fp) {
                for_planes(expected->planes, [&](auto ep) {
                    hipLaunchKernelGGL((jaccard_kernel<decltype(type), decltype(te)::value,
                                                       decltype(fp)::value, decltype(ep)::value>),
                                       dim3((unsigned)blocks), dim3(kBlock), 0, s, fs, (int32_t)F,
                                       es, (int32_t)E, W, tail_mask(n_rows), d_jaccard);
                });
            });
        };
        using one = std::integral_constant<int, 1>;
        using four = std::integral_constant<int, 4>;
        if (n_rows > INT32_MAX)
            tiled ? launch(int64_t{}, four{}) : launch(int64_t{}, one{});
        else
            tiled ? launch(int32_t{}, four{}) : launch(int32_t{}, one{});
        if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "jaccard_kernel");
    }
    hipLaunchKernelGGL(scores_kernel, dim3(1), dim3(kScoreBlock), 0, s, d_jaccard, (int32_t)F,
                       (int32_t)E, d_scores);
    if ((e = hipGetLastError()) != hipSuccess) return hip_error(e, "scores_kernel");
    return EBIC_OK;
}

}  // extern "C"
