// Device code shared by the single-run and batched evaluation kernels
// (gfx950, wave64): helpers, the Eq. (1) fitness write, and one tile of the
// index evaluator (strict, negative and approximate trend tests over the
// pairwise order index).  Included by the .hip files only.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "ebic_internal.h"

namespace ebic {
namespace {

constexpr int kWave = 64;
constexpr int kBlock = 256;
constexpr int kAlignedThreads = 320;   // largest single-run whole-candidate workgroup
constexpr int kXcds = 8;

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// Pointers read from device memory (a run table) are generic to the
// compiler; declaring them global lets it emit global (not flat) loads.
template <typename T>
using global_ptr = const __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ global_ptr<T> as_global(const T *p) {
    return (global_ptr<T>)p;
}

__device__ __forceinline__ uint64_t tail_bits(int64_t n, int64_t w, int64_t W) {
    if (w < W - 1) return ~0ull;
    const int rem = (int)(n - (W - 1) * 64);  // 1..64
    return rem == 64 ? ~0ull : ((1ull << rem) - 1ull);
}

// --------------------------------------------------------- fitness (Eq. 1) --
//
// Each part of a candidate (a workgroup's row slice, or a run of 64-row
// words) reports with ONE 64-bit atomic add on acc[c]:
//   bits  0..31  rows it accepted (|I| <= n < 2^31)
//   bit  32      set by the part that found the candidate malformed
//   bits 33..63  its share of the candidate's `parts`
// The part whose add completes the shares owns the total: a single
// read-modify-write orders everything, so no memory fence is needed.  It
// resets acc[c] for the next call and writes the count and Eq. (1).
// ln(count-1) comes from a table built on the host with the C library's
// log; L * ln is one rounded FP64 product and 2^e an exact scaling, so the
// result equals the host formula bit for bit.
constexpr int kShareShift = 33;
constexpr uint64_t kBadBit = 1ull << 32;

// Count and Eq. (1) fitness of candidate c (count -1 and NaN fitness for a
// malformed candidate).
template <typename LogPtr>
__device__ __forceinline__ void write_result(int64_t c, int32_t total, bool bad, int32_t L,
                                             int32_t sigma, LogPtr logt,
                                             int32_t *__restrict__ counts,
                                             double *__restrict__ fitness) {
    if (bad) {
        counts[c] = -1;
        fitness[c] = __builtin_nan("");
        return;
    }
    counts[c] = total;
    double f = 0.0;
    if (total > 1) {
        const int32_t e = total - sigma < 0 ? total - sigma : 0;
        f = ldexp((double)L * logt[total - 1], e);
    }
    fitness[c] = f;
}

template <typename LogPtr>
__device__ __forceinline__ void finish_part(int64_t c, uint32_t cnt, bool bad, int64_t share,
                                            int64_t parts, int32_t L, int32_t sigma,
                                            LogPtr logt,
                                            unsigned long long *__restrict__ acc,
                                            int32_t *__restrict__ counts,
                                            double *__restrict__ fitness) {
    const unsigned long long add =
        ((unsigned long long)share << kShareShift) | (bad ? kBadBit : 0ull) | cnt;
    const unsigned long long before = atomicAdd(acc + c, add);
    const unsigned long long now = before + add;
    if ((int64_t)(now >> kShareShift) != parts) return;
    atomicExch(acc + c, 0ull);
    write_result(c, (int32_t)(uint32_t)now, (now & kBadBit) != 0, L, sigma, logt, counts, fitness);
}

// -------------------------------------------------------- index evaluator --
//
// Thread = (candidate c, V consecutive 64-row words), c-major, so every
// lane has work whatever W is; the V words share the lane's column reads and
// loop, and are read with 16-byte loads when V > 1 (fewer waves, more loads
// in flight per lane, the same bytes).  The workgroup first stages the CBF
// columns of the candidates it covers in LDS.  Per consecutive pair (p, q) a
// lane reads lt(p,q) from the pairwise order index and folds the violation
// words into bit-sliced counters per direction (Violations).  A row that
// does not rise falls, unless the pair ties on it: lt(q,p) is ~lt(p,q)
// (lt(p,p) itself for a repeated column), and is read only for pairs that
// may tie (a set bit of the tie-pair bitmap).
//
// Two loops.  The fast one serves workgroups whose columns all lie in the
// matrix and of whose pairs few tie, which staging finds out: there a pair
// costs one LDS read (the two offsets of its columns, formed once per staged
// column), one address and 2 to 3 operations per half-word and direction, and
// no column is checked; the few tied pairs are counted before it.  The general
// one serves the rest (many tied pairs, malformed candidates, series past the
// staging area, whose columns it reads from memory).  Loads
// for U pairs are issued before any is consumed (the lane's latency chain is
// one order-word round trip per U pairs), and a lane stops once every row of
// its words is rejected in every enabled direction.
constexpr int kUnroll = 4;   // pairs per batch of loads (single-run default)
constexpr int kWordsPerLane = 2;   // 64-row words per lane (flattened single-run tiling)

// Any bitwise function of three words in one operation (v_bitop3_b32): T is
// its truth table, written as the same expression over kA, kB and kC.
constexpr uint32_t kA = 0xF0, kB = 0xCC, kC = 0xAA;
template <uint32_t T>
__device__ __forceinline__ uint32_t bitop3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, T & 0xFF);
}

// Violation counters of one 32-row half-word and direction, bit-sliced: bit
// b of every word belongs to row b.  For a class K = 2^BITS - 1 of
// tolerances k <= K the counter has BITS bits and starts at K - k, so the
// (k + 1)-th violation carries out of its top bit; c[OVER] collects the
// carries, the rows with more than k violations.
//
// The violations of four pairs are first added up: from the words o of "the
// row rises on this pair", r = t0 + 2 t1 + 4 t2 rising pairs (two half and
// one full adder, 6 operations) are the falling direction's violations, and
// 4 - r the rising one's (2 more), so the adder is shared by the directions
// and a pair costs 3.3 operations per half-word for k = 1 in both
// directions, 5.5 for k = 7; counted pair by pair in unary, with the
// complements formed separately, it was about 9 and 25.
template <int K>
struct Violations {
    static constexpr int bits() {
        int b = 0;
        while ((1 << b) - 1 < K) ++b;
        return b;
    }
    static constexpr int BITS = bits(), OVER = BITS, N = BITS + 1;
    static_assert(K == (1 << BITS) - 1, "tolerance classes are 2^bits - 1");
    uint32_t c[N];

    __device__ __forceinline__ void start(int32_t k) {
#pragma unroll
        for (int i = 0; i < BITS; ++i) c[i] = (((K - k) >> i) & 1) ? ~0u : 0u;
        c[OVER] = 0u;
    }
    // one violation on the rows of v
    __device__ __forceinline__ void add(uint32_t v) {
#pragma unroll
        for (int i = 0; i < BITS; ++i) {
            const uint32_t carry = c[i] & v;
            c[i] ^= v;
            v = carry;
        }
        c[OVER] |= v;
    }
    // n0 + 2 n1 + 4 n2 violations
    __device__ __forceinline__ void add(uint32_t n0, uint32_t n1, uint32_t n2) {
        uint32_t carry = 0u;
        auto digit = [&](auto bit, uint32_t d) {
            constexpr int i = decltype(bit)::value;
            if constexpr (i < BITS) {
                const uint32_t x = c[i];
                if constexpr (i == 0) {
                    c[i] = x ^ d;
                    carry = x & d;
                } else {
                    c[i] = bitop3<kA ^ kB ^ kC>(x, d, carry);
                    carry = bitop3<(kA & kB) | (kA & kC) | (kB & kC)>(x, d, carry);
                }
            } else {
                c[OVER] |= d;
            }
        };
        digit(std::integral_constant<int, 0>{}, n0);
        digit(std::integral_constant<int, 1>{}, n1);
        digit(std::integral_constant<int, 2>{}, n2);
#pragma unroll
        for (int i = 3; i < BITS; ++i) {
            const uint32_t x = c[i];
            c[i] = x ^ carry;
            carry &= x;
        }
        c[OVER] |= carry;
    }
};

// Folds four pairs of one half-word into both directions' counters.
template <int K, bool NEG>
__device__ __forceinline__ void fold4(Violations<K> &up, Violations<K> &down, uint32_t o0,
                                      uint32_t o1, uint32_t o2, uint32_t o3) {
    if constexpr (K == 0) {
        up.c[0] = bitop3<kA | ~(kB & kC)>(up.c[0], bitop3<kA & kB & kC>(o0, o1, o2), o3);
        if constexpr (NEG)
            down.c[0] = bitop3<kA | kB | kC>(down.c[0], bitop3<kA | kB | kC>(o0, o1, o2), o3);
        return;
    }
    const uint32_t s = bitop3<kA ^ kB ^ kC>(o0, o1, o2);
    const uint32_t c = bitop3<(kA & kB) | (kA & kC) | (kB & kC)>(o0, o1, o2);
    const uint32_t t0 = s ^ o3, c1 = s & o3, t1 = c ^ c1, t2 = c & c1;
    // 4 - r: its digits are t0, t0 ^ t1 and "no pair rises"
    if constexpr (K == 1) {
        // both upper digits overflow: r <= 2
        up.c[1] |= bitop3<~(kA | (kB & kC))>(t2, t1, t0);
        up.add(t0);
    } else {
        up.add(t0, t0 ^ t1, bitop3<~(kA | kB | kC)>(t0, t1, t2));
    }
    if constexpr (NEG) down.add(t0, t1, t2);
}

// A staged column x: the order row of pair (p, q) starts at
// row(p) + col(q), row = x m S and col = x S for a row stride S.  With a
// 32-bit index (OFF32) S is in bytes, otherwise in units of 128 bytes (rows
// are multiples of 128 bytes).
struct PreCol {
    uint32_t row, col;
};

// LDS of one tile: for whole-candidate tiles the per-candidate row counts and
// malformed flags, the tie-pair bitmap, and what staging found.
struct TileLds {
    int32_t rows[kBlock];
    int32_t bad[kBlock];
    uint32_t tbits[kTieWords];
    uint32_t found;                // what staging found (kFound*)
    uint32_t n_tied;               // bits set in StageLds::tied
};
// The launch's staging area of `entries` columns (a multiple of 64) behind it.
struct StageLds {
    PreCol *pre;
    uint64_t *tied;   // bit e % 64 of word e / 64: staged column e may tie with
                      // the one before it, or repeats it
    int32_t entries;
    __device__ StageLds(uint64_t *lds, int32_t n)
        : pre(reinterpret_cast<PreCol *>(lds)), tied(lds + n), entries(n) {}
};
static_assert(sizeof(PreCol) == sizeof(uint64_t), "one word of the staging area per column");
constexpr uint32_t kFoundBad = 1;    // a staged column is out of range, or a lane's
                                     // series lies outside the staged span
constexpr uint32_t kFoundTied = 2;   // a staged pair may tie

// V consecutive order words of one pair, read with 16-byte loads when V > 1
// (the caller keeps the address 16-byte aligned).
template <int V>
__device__ __forceinline__ void load_words(global_ptr<uint64_t> p, uint64_t (&o)[V]) {
    if constexpr (V == 1) {
        o[0] = p[0];
    } else {
        typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < V; i += 2) {
            const u64x2 x = *(global_ptr<u64x2>)(p + i);
            o[i] = x.x;
            o[i + 1] = x.y;
        }
    }
}

// Calls f(integral_constant<int, r>) for the run-time count r in [1, N]
// (nothing for r = 0): the last, shorter batch of a series' pairs.
template <int N>
struct ShortBatch {
    template <class F>
    __device__ __forceinline__ static void run(int32_t r, F &&f) {
        if (r == N)
            f(std::integral_constant<int, N>{});
        else
            ShortBatch<N - 1>::run(r, f);
    }
};
template <>
struct ShortBatch<0> {
    template <class F>
    __device__ __forceinline__ static void run(int32_t, F &&) {}
};

// One tile of one run.  An item is a candidate and V consecutive 64-row
// words of it (V words per lane share the lane's column reads and loop).
// Two tilings:
//   ALIGNED = false: kBlock consecutive items of the flattened (candidate,
//     item) order; a candidate may span workgroups, so each workgroup adds
//     its share of a candidate's count with one packed global atomic and the
//     last share writes the result (finish_part).  Shared by the single-run
//     kernel and the persistent multi-run kernel.
//   ALIGNED = true: the workgroup holds `cpw` whole candidates (requires
//     ceil(W / V) <= kBlock and cpw <= kBlock; the workgroup may have up to
//     kAlignedThreads lanes); counts are summed with LDS atomics and the
//     first lane of each candidate writes its result after a workgroup
//     barrier -- no global atomics and no accumulator scratch.
template <int K, bool NEG, int U, int V, bool ALIGNED, bool OFF32 = false, bool TAIL = false>
__device__ __forceinline__ void index_tile(const IndexRun &R, uint32_t tile, uint32_t cpw,
                                           const int32_t *__restrict__ offsets,
                                           const int32_t *__restrict__ cols, int64_t n_entries,
                                           int32_t sigma, uint64_t *__restrict__ masks,
                                           unsigned long long *__restrict__ acc,
                                           int32_t *__restrict__ counts,
                                           double *__restrict__ fitness, TileLds &lds,
                                           const StageLds &stage) {
    // (V <= 8 keeps a wave's per-candidate row count within 16 bits below)
    static_assert(V == 1 || V == 2 || V == 4 || V == 8, "words per lane");
    const auto idx = as_global(R.idx);
    const auto logt = as_global(R.logt);
    const int64_t n = R.n, W = R.W, wpad = R.wpad;
    const int32_t m = R.m, P = R.P;
    const int tid = threadIdx.x, lane = tid & 63;
    // The launcher guarantees P * ceil(W / V) < 2^32.
    const uint32_t Wg = (uint32_t)((W + V - 1) / V);   // items per candidate
    uint32_t cl, g, c_lo, c_hi, slot = 0;
    bool active;
    if constexpr (ALIGNED) {
        slot = (uint32_t)tid / Wg;                                // candidate slot in the tile
        c_lo = tile * cpw;
        c_hi = min(c_lo + cpw, (uint32_t)P) - 1;
        active = slot < cpw && c_lo + slot < (uint32_t)P;
        cl = active ? c_lo + slot : c_hi;
        g = active ? (uint32_t)tid - slot * Wg : 0;
    } else {
        const uint32_t item = tile * (uint32_t)kBlock + (uint32_t)tid;
        active = item < (uint32_t)P * Wg;
        cl = active ? item / Wg : (uint32_t)P - 1;               // candidate within the run
        g = active ? item - cl * Wg : 0;
        const uint32_t i0 = tile * (uint32_t)kBlock;
        c_lo = i0 / Wg;
        c_hi = min((i0 + kBlock - 1) / Wg, (uint32_t)P - 1);
    }
    const int64_t w0 = (int64_t)g * V;                           // first word of the item
    const int64_t c = R.cand_base + cl;                          // candidate in the launch

    // The tie-pair bitmap (null: no two distinct columns tie) in LDS; the
    // byte flag of a pair whose bit is set says whether it ties.
    const bool ties = NEG && R.tbits != nullptr;
    if (NEG && ties) {
        const auto tb = as_global(R.tbits);
        for (int i = tid; i < kTieWords; i += (int)blockDim.x) lds.tbits[i] = tb[i];
    }
    if (tid == 0) lds.found = lds.n_tied = 0;
    auto in_bitmap = [&](int64_t pq) -> bool {
        const uint32_t h = tie_hash((uint32_t)pq);
        return ((lds.tbits[h >> 5] >> (h & 31)) & 1u) != 0;
    };

    const int64_t start = offsets[c], end = offsets[c + 1];
    const bool ok_range = start >= 0 && end <= n_entries && end > start;
    const int32_t L = ok_range ? (int32_t)(end - start) : 0;

    // Stage the columns of candidates [c_lo, c_hi] in LDS when they fit.
    // They are used when every lane's series lies inside the staged span
    // (always, for a well-formed CBF); otherwise the whole workgroup reads
    // them from global memory.  Every choice is uniform over the workgroup.
    const int64_t b0 = offsets[R.cand_base + c_lo], b1 = offsets[R.cand_base + c_hi + 1];
    int32_t *const s_rows = lds.rows;
    int32_t *const s_bad = lds.bad;
    if (ALIGNED && (uint32_t)tid < cpw) {
        s_rows[tid] = 0;
        s_bad[tid] = 0;
    }
    // row strides of the offsets of order rows (the unit form fits 32 bits up
    // to an index of 512 GiB)
    const uint32_t col_s = OFF32 ? (uint32_t)wpad * 8u : (uint32_t)(wpad / 16);
    const uint32_t row_s = (uint32_t)m * col_s;
    const bool staged = b0 >= 0 && b1 <= n_entries && b1 >= b0 && b1 - b0 <= stage.entries;
    const int32_t span = staged ? (int32_t)(b1 - b0) : 0;
    __syncthreads();   // lds.found is cleared, the bitmap is in LDS
    bool wrong = staged && ok_range && (start < b0 || end > b1);
    uint32_t n_tied = 0;
    // N entries per lane, blockDim.x apart, whose reads are all in flight
    // together (entries past the span repeat its last one).
    auto stage_entries = [&](auto per_lane, auto look_up_ties, int32_t e0) {
        constexpr int N = decltype(per_lane)::value;
        constexpr bool TIES = decltype(look_up_ties)::value;
        int32_t x[N];
        uint32_t tie[N];   // of the pair that ends in the entry
#pragma unroll
        for (int u = 0; u < N; ++u)
            x[u] = cols[b0 + min(e0 + u * (int32_t)blockDim.x, span - 1)];
        if constexpr (NEG) {
            int64_t pq[N];   // -1: no pair
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int32_t e = min(e0 + u * (int32_t)blockDim.x, span);
                const int32_t xp = cols[b0 + max(min(e, span - 1) - 1, 0)];
                // pairs that straddle two candidates included (no series reads them)
                const bool pair = e > 0 && e < span && (uint32_t)x[u] < (uint32_t)m &&
                                  (uint32_t)xp < (uint32_t)m;
                pq[u] = pair ? (int64_t)xp * m + x[u] : -1;
                tie[u] = pair && x[u] == xp;
            }
            if constexpr (TIES) {
                bool any = false;
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    pq[u] = pq[u] >= 0 && in_bitmap(pq[u]) ? pq[u] : -1;
                    any |= pq[u] >= 0;
                }
                if (ballot(any) != 0ull) {   // (few waves, if few pairs tie)
                    uint32_t flag[N];        // (a clear bit reads flag 0, whatever it says)
#pragma unroll
                    for (int u = 0; u < N; ++u) flag[u] = as_global(R.tie)[max(pq[u], int64_t{0})];
#pragma unroll
                    for (int u = 0; u < N; ++u) tie[u] |= pq[u] >= 0 ? flag[u] : 0u;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int32_t e = e0 + u * (int32_t)blockDim.x;
            if ((e & ~63) >= span) break;   // whole waves
            wrong |= e < span && (uint32_t)x[u] >= (uint32_t)m;
            if (e < span) stage.pre[e] = PreCol{(uint32_t)x[u] * row_s, (uint32_t)x[u] * col_s};
            if constexpr (NEG) {
                const uint64_t t = ballot(tie[u] != 0u);
                n_tied += (uint32_t)__popcll(t);
                if (lane == 0) stage.tied[e >> 6] = t;
            }
        }
    };
    // Most workgroups have an entry per lane at most.  Those of few lanes and
    // many series stage several per lane at a time (fewer where ties are looked
    // up, for the registers), out of the others' way.
    auto stage_span = [&](auto look_up_ties) {
        constexpr int N = decltype(look_up_ties)::value ? 2 : 4;
        if (__builtin_expect(span <= (int32_t)blockDim.x, 1)) {
            if ((tid & ~63) < span)
                stage_entries(std::integral_constant<int, 1>{}, look_up_ties, tid);
            return;
        }
        for (int32_t e = tid; (e & ~63) < span; e += N * (int32_t)blockDim.x)
            stage_entries(std::integral_constant<int, N>{}, look_up_ties, e);
    };
    if (NEG && ties)
        stage_span(std::integral_constant<bool, NEG>{});
    else
        stage_span(std::false_type{});
    {
        const uint32_t f = (ballot(wrong) != 0ull ? kFoundBad : 0u) |
                           (n_tied != 0u ? kFoundTied : 0u);
        if (f != 0u && lane == 0) {
            atomicOr(&lds.found, f);
            if (NEG) atomicAdd(&lds.n_tied, n_tied);
        }
    }
    __syncthreads();
    const uint32_t found = __builtin_amdgcn_readfirstlane(lds.found);
    const bool good = staged && (found & kFoundBad) == 0;
    // Tied pairs cost the fast loop both their order rows again, the general
    // one the reverse's; that one has fewer pairs in flight.  2048 series,
    // k = 0, both directions, a share of the pairs tied: 20000 rows, 2 words
    // per lane, 2%: fast 7.7, general 7.9 us; 10%: 9.0 and 8.1; 20%: 10.7 and
    // 8.5; 30000 rows, 4 words, 2%: 11.0 and 11.3; 5%: 11.8 and 11.3; 10%:
    // 12.8 and 11.4 (but a launch of both kinds of workgroup lasts as long as
    // the slower one: matrices with a tie here and there stay with the fast).
    constexpr uint32_t kTiedShare = V < 4 ? 8 : 12;
    const bool many_ties = NEG && (found & kFoundTied) != 0 &&
                           __builtin_amdgcn_readfirstlane(lds.n_tied) * kTiedShare > (uint32_t)span;
    const int32_t lds0 = (int32_t)(start - b0);

    uint64_t valid[V];
    uint64_t any_valid = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        valid[v] = (active && ok_range && w0 + v < W) ? tail_bits(n, w0 + v, W) : 0ull;
        any_valid |= valid[v];
    }
    constexpr int OVER = Violations<K>::OVER;
    uint64_t up[V], down[V];   // rows of each word rejected in each direction
#pragma unroll
    for (int v = 0; v < V; ++v) up[v] = down[v] = ~0ull;
    auto half = [](uint64_t x, int h) -> uint32_t { return (uint32_t)(h ? x >> 32 : x); };
    // The lane of a candidate's first word reports whether it is malformed.
    bool bad = active && g == 0 && !ok_range;

    // The lane's words (from its v-th on) of the order row at a staged offset.
    typedef const __attribute__((address_space(1))) char *gchar;
    const auto base = OFF32 ? (gchar)idx : (gchar)(idx + w0);
    const uint32_t w_off = OFF32 ? (uint32_t)w0 * 8u : 0u;
    auto row_at = [&](uint32_t off, uint32_t v) {
        if constexpr (OFF32)
            return (global_ptr<uint64_t>)(base + (off + (w_off + v * 8u)));
        else
            return (global_ptr<uint64_t>)(base + (((uint64_t)off << 7) + v * 8u));
    };

    if (good && !many_ties) {
        if (any_valid) {
            const PreCol *const pre = stage.pre + lds0;
            constexpr bool REST_FIRST = K > 1;
            Violations<K> cu[V][2], cd[V][2];   // rising, falling; low and high half-word
#pragma unroll
            for (int v = 0; v < V; ++v)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    cu[v][h].start(R.k);
                    cd[v][h].start(R.k);
                }
            auto over = [&](const Violations<K> (&c)[V][2], int v) -> uint64_t {
                return ((uint64_t)c[v][1].c[OVER] << 32) | c[v][0].c[OVER];
            };
            // whether a row of the lane's words is still accepted in some direction
            auto undecided = [&]() -> bool {
                uint64_t live = 0;
#pragma unroll
                for (int v = 0; v < V; ++v)
                    live |= valid[v] & ~(NEG ? (over(cu, v) & over(cd, v)) : over(cu, v));
                return live != 0ull;
            };
            // The order words of N pairs, pair i(u) in slot u: the offset
            // reads and loads are all issued before any word is consumed.
            uint64_t lt[U][V];
            auto load_row = [&](uint32_t off, uint64_t (&o)[V]) { load_words<V>(row_at(off, 0), o); };
            auto load = [&](auto n_pairs, auto &&i) {
#pragma unroll
                for (int u = 0; u < decltype(n_pairs)::value; ++u)
                    load_row(pre[i(u) - 1].row + pre[i(u)].col, lt[u]);
            };
            // slot u's pair, on the rows of `in`
            auto fold1 = [&](int u, uint32_t in) {
#pragma unroll
                for (int v = 0; v < V; ++v)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t o = half(lt[u][v], h);
                        cu[v][h].add(~o & in);
                        if (NEG) cd[v][h].add(o & in);
                    }
            };
            // The (L - 1) mod U pairs that do not fill a batch, from pair t.
            const int32_t rest = (L - 1) & (U - 1);
            auto short_batch = [&](int32_t t) {
                if constexpr (TAIL) {
                    // as one shorter batch
                    ShortBatch<U - 1>::run(rest, [&](auto r) {
                        load(r, [&](int u) { return t + u; });
#pragma unroll
                        for (int u = 0; u < decltype(r)::value; ++u) fold1(u, ~0u);
                    });
                } else if (U > 1 && rest > 0) {
                    // as a batch whose surplus slots repeat the last pair and
                    // break nothing
                    load(std::integral_constant<int, U - 1>{},
                         [&](int u) { return t + min(u, rest - 1); });
#pragma unroll
                    for (int u = 0; u < U - 1; ++u) fold1(u, u < rest ? ~0u : 0u);
                }
            };
            // The loop below takes a row that does not rise for a falling one.
            // Tied rows (in neither order row; every row of a repeated
            // column) break the falling trend too, and are counted here from
            // both order rows of the pairs that may tie, two at a time.
            if (NEG && (found & kFoundTied) != 0) {
                const int32_t e0 = lds0 + 1, e1 = lds0 + L;   // pairs end in staged columns [e0, e1)
                for (int32_t wi = e0 >> 6; wi < (e1 + 63) >> 6; ++wi) {
                    uint64_t bits = stage.tied[wi];
                    if (wi == e0 >> 6) bits &= ~0ull << (e0 & 63);
                    if (wi == e1 >> 6) bits &= ~(~0ull << (e1 & 63));
                    while (bits != 0ull) {
                        int32_t e[2];
                        bool have[2];
                        uint64_t o[2][2][V];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            have[u] = bits != 0ull;
                            e[u] = have[u] ? wi * 64 + __builtin_ctzll(bits) : e0;
                            bits &= bits - 1;
                            load_row(stage.pre[e[u] - 1].row + stage.pre[e[u]].col, o[u][0]);
                            load_row(stage.pre[e[u]].row + stage.pre[e[u] - 1].col, o[u][1]);
                        }
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int v = 0; v < V; ++v)
#pragma unroll
                                for (int h = 0; h < 2; ++h)
                                    cd[v][h].add(have[u] ? ~(half(o[u][0][v], h) |
                                                             half(o[u][1][v], h)) : 0u);
                    }
                }
            }
            if constexpr (REST_FIRST) short_batch(1);
            int32_t t = REST_FIRST ? 1 + rest : 1;
            bool more = true;
            if (t + U <= L) do {
                load(std::integral_constant<int, U>{}, [&](int u) { return t + u; });
                constexpr int N4 = U / 4 * 4;   // pairs folded four at a time
#pragma unroll
                for (int u = 0; u < N4; u += 4)
#pragma unroll
                    for (int v = 0; v < V; ++v)
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            fold4<K, NEG>(cu[v][h], cd[v][h], half(lt[u][v], h),
                                          half(lt[u + 1][v], h), half(lt[u + 2][v], h),
                                          half(lt[u + 3][v], h));
#pragma unroll
                for (int u = N4; u < U; ++u) fold1(u, ~0u);
                t += U;
                more = undecided();
            } while (t + U <= L && more);
            if constexpr (!REST_FIRST)
                if (more) short_batch(t);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                up[v] = over(cu, v);
                if (NEG) down[v] = over(cd, v);
            }
        }
    } else {
        // The rising direction from the pair's order row, the falling one from
        // the reverse's where the pair may tie (with 1 word per lane always)
        // and otherwise from the same row again (it falls where it does not
        // rise); four words at a time (all 8
        // where the fast loop has two pairs of 8 in flight), so that this loop
        // needs no more registers than the fast one.  rows_at(t, pair) calls
        // pair(u, up, down, tied) for the UU pairs that end at positions t,
        // t + 1, ... with the offsets (as staged) of their order rows and of
        // their reverses' (past the series' end any row).
        constexpr int VV = V == 8 && U > 1 ? 8 : (V < 4 ? V : 4);
        constexpr int PAIRS = VV >= 4 || K > 3 ? 1 : (U < 4 / VV ? U : 4 / VV);
        auto by_words = [&](auto pairs, auto &&rows_at) {
            constexpr int UU = decltype(pairs)::value;
#pragma clang loop unroll(disable)
            for (int v0 = 0; v0 < V; v0 += VV) {
                uint64_t rows_v[VV];
#pragma unroll
                for (int v = 0; v < VV; ++v)
                    if constexpr (VV == V)
                        rows_v[v] = valid[v];
                    else
                        rows_v[v] = (active && ok_range && w0 + v0 + v < W)
                                        ? tail_bits(n, w0 + v0 + v, W) : 0ull;
                if (rows_v[0] == 0ull) break;   // no words past the last one
                Violations<K> cu[VV][2], cd[VV][2];
#pragma unroll
                for (int v = 0; v < VV; ++v)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        cu[v][h].start(R.k);
                        cd[v][h].start(R.k);
                    }
                auto over = [](const Violations<K> (&c)[2]) -> uint64_t {
                    return ((uint64_t)c[1].c[OVER] << 32) | c[0].c[OVER];
                };
                bool more = true;
                for (int32_t t = 1; t < L && more; t += UU) {
                    uint64_t lu[UU][VV], ld[UU][VV];
                    uint32_t flip[UU];
                    rows_at(t, [&](int u, uint32_t up_at, uint32_t down_at, bool tied) {
                        load_words<VV>(row_at(up_at, (uint32_t)v0), lu[u]);
                        if (NEG) load_words<VV>(row_at(tied ? down_at : up_at, (uint32_t)v0), ld[u]);
                        flip[u] = tied ? ~0u : 0u;
                    });
#pragma unroll
                    for (int u = 0; u < UU; ++u) {
                        const uint32_t in = t + u < L ? ~0u : 0u;
#pragma unroll
                        for (int v = 0; v < VV; ++v)
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                cu[v][h].add(~half(lu[u][v], h) & in);
                                if (NEG) cd[v][h].add((half(ld[u][v], h) ^ flip[u]) & in);
                            }
                    }
                    uint64_t live = 0;
#pragma unroll
                    for (int v = 0; v < VV; ++v)
                        live |= rows_v[v] & ~(NEG ? (over(cu[v]) & over(cd[v])) : over(cu[v]));
                    more = live != 0ull;
                }
#pragma unroll
                for (int x = 0; x < V; ++x)
                    if (x / VV * VV == v0) {
                        up[x] = over(cu[x % VV]);
                        if (NEG) down[x] = over(cd[x % VV]);
                    }
            }
        };
        if (good) {
            by_words(
                std::integral_constant<int, PAIRS>{}, [&](int32_t t, auto &&pair) {
#pragma unroll
                    for (int u = 0; u < PAIRS; ++u) {
                        const int32_t i = lds0 + min(t + u, L - 1);
                        const PreCol p = stage.pre[i - 1], q = stage.pre[i];
                        pair(u, p.row + q.col, q.row + p.col,
                             NEG && (V == 1 || ((stage.tied[i >> 6] >> (i & 63)) & 1ull) != 0ull));
                    }
                });
        } else {
            // columns from global memory, clamped so that no read leaves the
            // index; the lane of the candidate's first word checks them all
            if (active && g == 0) {
                constexpr int kAhead = V < 4 ? 8 : 2;   // (registers)
                for (int32_t t = 0; t < L; t += kAhead) {
                    int32_t x[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) x[u] = cols[start + min(t + u, L - 1)];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) bad |= x[u] < 0 || x[u] >= m;
                }
            }
            auto col = [&](int32_t t) -> uint32_t {
                const int32_t x = cols[start + min(t, L - 1)];
                return x < 0 || x >= m ? 0u : (uint32_t)x;
            };
            // (the columns of the next pairs are read while the rows of these
            // are under way)
            constexpr int UU = PAIRS > 1 ? PAIRS / 2 : 1;
            uint32_t p = 0, next[UU];
            by_words(
                std::integral_constant<int, UU>{}, [&](int32_t t, auto &&pair) {
                    if (t == 1) {
                        p = col(0);
#pragma unroll
                        for (int u = 0; u < UU; ++u) next[u] = col(1 + u);
                    }
#pragma unroll
                    for (int u = 0; u < UU; ++u) {
                        pair(u, p * row_s + next[u] * col_s, next[u] * row_s + p * col_s,
                             ties || p == next[u]);
                        p = next[u];
                    }
#pragma unroll
                    for (int u = 0; u < UU; ++u) next[u] = col(t + UU + u);
                });
        }
    }

    int32_t rows = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const uint64_t pos = valid[v] & ~up[v];
        const uint64_t neg = NEG ? (valid[v] & ~down[v]) : 0ull;
        rows += __popcll(pos | neg);
        if (masks && active && w0 + v < W) {
            masks[R.mask_base + ((int64_t)cl * 2 + 0) * W + w0 + v] = pos;
            masks[R.mask_base + ((int64_t)cl * 2 + 1) * W + w0 + v] = neg;
        }
    }

    if constexpr (ALIGNED) {
        // The staging barrier above ordered the zeroing of s_rows/s_bad
        // before these updates.
        if (active) {
            atomicAdd(&s_rows[slot], rows);
            if (bad) s_bad[slot] = 1;
        }
        __syncthreads();
        if (active && g == 0)
            write_result(c, s_rows[slot], s_bad[slot] != 0, L, sigma, logt, counts, fitness);
        return;
    }

    // Segmented sum over lanes of the same candidate (lanes hold consecutive
    // items, so each candidate is one contiguous run of lanes): the run's
    // head gets the run's row count (low 16 bits, <= 64*64*V) and its number
    // of words (high bits), then reports them once.
    const int32_t words = active ? (int32_t)min<int64_t>(V, W - w0) : 0;
    int32_t packed = active ? (rows | (words << 16)) : 0;
    const int32_t cc = (int32_t)cl;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int32_t x = __shfl_down(packed, off);
        const int32_t oc = __shfl_down(cc, off);
        if (lane + off < kWave && oc == cc) packed += x;
    }
    const int32_t prev_c = __shfl_up(cc, 1);
    const bool head = lane == 0 || prev_c != cc;
    // the first item of a candidate is always the first lane of its run,
    // hence a head itself.
    if (active && head)
        finish_part(c, (uint32_t)(packed & 0xFFFF), bad, packed >> 16, W, L, sigma, logt, acc,
                    counts, fitness);
}

}  // namespace
}  // namespace ebic
