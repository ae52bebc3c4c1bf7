// Fused training step of the surrogate MLP for embed_dim 32 and hidden 256
// (the configuration of the screened runs) on gfx950:
//
//   A  mlp_rows_kernel    per tile of 32 candidates: pooling, both layers,
//                         the output, the loss gradient and the whole
//                         per-candidate backward pass (dz2, dz1, dx), with
//                         the tile's activations kept in LDS; writes the
//                         BF16 operands of the weight gradients transposed
//                         (tile-major, candidates contiguous) and each
//                         tile's partial bias/output-weight gradient sums
//   B  mlp_grads_kernel   weight gradients as split-K products over the
//                         batch (one partial per 256 candidates), the bias
//                         and output-weight gradients from the tiles'
//                         partial sums, and the embedding gradients gathered
//                         by column occurrence and by series length
//   C  mlp_update_kernel  every parameter: its gradient (partials summed in
//                         a fixed order), then Adam, then the BF16 copies
//                         (row-major and transposed) of W1, W2 and w3
//
// Products run on v_mfma_f32_16x16x32_bf16 (BF16 operands, FP32
// accumulation) with 16-byte operand fragments: A and B lane l holds row or
// column (l mod 16) and 8 consecutive k from 8 (l / 16); the 16 x 16 result
// gives lane l rows 4 (l / 16) + v, column l mod 16.  The rounding points
// are those of the layer-by-layer kernels: bf16(x), bf16(relu(z1)),
// bf16(relu(z2)), bf16(dz2), bf16(dz1), weights read as BF16 copies.  Every
// sum has a fixed order, so a step is deterministic on one device.
//
// What bounds a step (B = 8192, 500 columns: A 32.5 us, B 17.8, C 4.2; 38.2,
// 34.1 and 4.2 before): the products are small, and each launch lasts as long
// as its workgroups' chains of dependent loads.  A's tile of 32 candidates is
// one workgroup of 8 waves (with 4 waves 38.2 us; with each layer's weights
// loaded whole, a phase ahead, 38.3, since 140 VGPRs leave one workgroup per
// compute unit and the loads gain nothing), B's operands are stored tile by
// tile (30.2 us with rows of the whole batch, whose fragments met in the same
// cache channels).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "ebic_mlp.h"

namespace ebic {
namespace mlp {
namespace {

constexpr int kBlock = 256;
constexpr int kRowsBlock = 512;        // lanes of a row tile's workgroup
constexpr int kTB = 32;                // candidates per row tile
constexpr int kD = 32, kD2 = 64, kH = 256;
constexpr int kLdX = kD2 + 8, kLdH = kH + 8;   // LDS row strides (bf16), 16-byte aligned rows
constexpr int kChunk = 256;            // candidates per weight-gradient partial
static_assert(kTB == 32 && kChunk % kTB == 0, "one MFMA step of candidates per tile");

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// 16 x 32 fragment of a row-major BF16 matrix (row stride ld elements):
// rows r0 + (lane mod 16), columns k0 + 8 (lane / 16) .. + 7.
__device__ __forceinline__ bf16x8 frag(const uint16_t *base, int64_t ld, int64_t r0, int64_t k0,
                                      int lane) {
    return *reinterpret_cast<const bf16x8 *>(base + (r0 + (lane & 15)) * ld + k0 + 8 * (lane >> 4));
}

// Sum over the four lane groups (l, l+16, l+32, l+48) in a fixed order.
__device__ __forceinline__ float sum_groups(float v) {
    const float a = v + __shfl_xor(v, 16);
    return a + __shfl_xor(a, 32);
}
// Sum over the 16 lanes of a group in a fixed order.
__device__ __forceinline__ float sum_row(float v) {
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    return v + __shfl_xor(v, 8);
}

constexpr int kTileCols = 2048;        // series entries of a tile staged in LDS

struct RowsLds {
    int32_t off[kTB + 1];
    int32_t cols[kTileCols];
    uint16_t x[kTB][kLdX];
    uint16_t h1[kTB][kLdH];
    uint16_t dz2[kTB][kLdH];
    uint16_t dz1[kTB][kLdH];
    uint8_t m1[kTB][kH];
    float yp[kRowsBlock / 128][kTB];
    float dy[kTB];
};

// Copies a [32][W] LDS tile to its place in a tile-major global matrix
// [tile][W][32] (features of a tile of candidates, candidates contiguous),
// 16 bytes per store, neighbouring lanes next to each other.
template <int W, int LD>
__device__ __forceinline__ void store_transposed(const uint16_t (*src)[LD], uint16_t *dst,
                                                 int64_t tile) {
    dst += tile * (W * kTB);
    for (int i = threadIdx.x; i < W * (kTB / 8); i += kRowsBlock) {
        const int w = i / (kTB / 8), c = i % (kTB / 8);
        uint16_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = src[c * 8 + j][w];
        uint4 q;
        q.x = v[0] | ((uint32_t)v[1] << 16);
        q.y = v[2] | ((uint32_t)v[3] << 16);
        q.z = v[4] | ((uint32_t)v[5] << 16);
        q.w = v[6] | ((uint32_t)v[7] << 16);
        *reinterpret_cast<uint4 *>(dst + w * kTB + c * 8) = q;
    }
}

__global__ __launch_bounds__(kRowsBlock) void mlp_rows_kernel(FusedRows a) {
    __shared__ RowsLds S;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t b0 = (int64_t)blockIdx.x * kTB;
    constexpr int kC = 2;   // 16-column blocks per wave
    // acc += A W^T for the wave's columns 32 wv .. 32 wv + 31: A (32 x K) in
    // LDS, the fragments of the weight copy W two k-steps ahead of their use.
    auto product = [&](auto k_size, const uint16_t *A, int ld, const uint16_t *W,
                       f32x4 (&acc)[2][kC]) {
        constexpr int K = decltype(k_size)::value, KS = K / 32, kAhead = KS < 2 ? KS : 2;
        bf16x8 w[kAhead][kC];
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
#pragma unroll
            for (int c = 0; c < kC; ++c) w[k][c] = frag(W, K, 32 * wv + 16 * c, 32 * k, lane);
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            bf16x8 now[kC];
#pragma unroll
            for (int c = 0; c < kC; ++c) {
                now[c] = w[k % kAhead][c];
                if (k + kAhead < KS)
                    w[k % kAhead][c] = frag(W, K, 32 * wv + 16 * c, 32 * (k + kAhead), lane);
            }
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                const bf16x8 fa = frag(A, ld, 16 * rb, 32 * k, lane);
#pragma unroll
                for (int c = 0; c < kC; ++c) acc[rb][c] = mfma(fa, now[c], acc[rb][c]);
            }
        }
    };

    // pooling: x = [mean E + Z[L] ; mean of F[c_t] * T[c_{t+1}]], bf16(x).
    // The tile's series are staged in LDS.
    if (tid <= kTB) {
        const int64_t b = b0 + tid;
        S.off[tid] = b <= a.B ? a.off[b] : a.off[a.B];
    }
    __syncthreads();
    const int32_t base = S.off[0], n_cols = S.off[kTB] - base;
    for (int i = tid; i < n_cols && i < kTileCols; i += kRowsBlock) S.cols[i] = a.cols[base + i];
    __syncthreads();
    {
        // thread = (candidate r, 4 consecutive dimensions 4q .. 4q + 3 of x):
        // q < 8 pools E, q >= 8 the pair products F * T; ten series
        // positions' loads in flight at a time, sums in series order
        const int r = tid / 16, q = tid % 16;
        const bool pair = q >= kD / 4;
        const int d0 = 4 * (pair ? q - kD / 4 : q);
        const int32_t s = S.off[r], e = S.off[r + 1], L = e - s;
        const bool staged = n_cols <= kTileCols;
        auto col = [&](int32_t t) -> int32_t { return staged ? S.cols[t - base] : a.cols[t]; };
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        const int32_t n_terms = pair ? L - 1 : L;
        constexpr int kAhead = 10;
        for (int32_t t0 = 0; t0 < n_terms; t0 += kAhead) {
            float4 v[kAhead], w[kAhead];
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const int32_t t = t0 + j;
                v[j] = w[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (t < n_terms) {
                    const int32_t c = col(s + t);
                    const float *table = pair ? a.F : a.E;
                    v[j] = *reinterpret_cast<const float4 *>(table + (int64_t)c * kD + d0);
                    if (pair)
                        w[j] = *reinterpret_cast<const float4 *>(
                            a.T + (int64_t)col(s + t + 1) * kD + d0);
                }
            }
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                if (pair) v[j] = make_float4(v[j].x * w[j].x, v[j].y * w[j].y, v[j].z * w[j].z,
                                             v[j].w * w[j].w);
                acc[0] += v[j].x;
                acc[1] += v[j].y;
                acc[2] += v[j].z;
                acc[3] += v[j].w;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float x = 0.f;
            if (b0 + r < a.B) {
                if (!pair) x = acc[u] / (float)L + a.Zl[(int64_t)L * kD + d0 + u];
                else if (L > 1) x = acc[u] / (float)(L - 1);
            }
            S.x[r][(pair ? kD : 0) + d0 + u] = to_bf16(x);
        }
    }
    __syncthreads();

    // layer 1: z1 = bf16(x) W1^T + b1 (wave wv: columns 32 wv .. 32 wv + 31)
    {
        f32x4 acc[2][kC] = {};
        product(std::integral_constant<int, kD2>{}, &S.x[0][0], kLdX, a.W1b, acc);
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            const int n = 32 * wv + 16 * c + (lane & 15);
            const float bias = a.b1[n];
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 16 * rb + 4 * (lane >> 4) + v;
                    const float z = acc[rb][c][v] + bias;
                    S.h1[r][n] = to_bf16(fmaxf(z, 0.f));
                    S.m1[r][n] = z > 0.f ? 1 : 0;
                }
        }
    }
    __syncthreads();

    // layer 2: z2 = bf16(h1) W2^T + b2; h2 = bf16(relu(z2)) kept in
    // registers, [z2 > 0] as bits of m2
    float h2[2][kC][4];
    uint32_t m2 = 0;
    auto bit2 = [](int rb, int c, int v) { return (rb * kC + c) * 4 + v; };
    {
        f32x4 acc[2][kC] = {};
        product(std::integral_constant<int, kH>{}, &S.h1[0][0], kLdH, a.W2b, acc);
        // The output product adds 64 columns per lane group, 16 apart, in
        // column order: the even wave of a pair hands its partial sums of the
        // first 32 to the odd one through LDS (dz2 is not in use yet).
        float yp[2][4] = {};
        float *const hand = reinterpret_cast<float *>(&S.dz2[0][0]) + (wv >> 1) * 8 * 64;
        auto add_columns = [&]() {
#pragma unroll
            for (int c = 0; c < kC; ++c) {
                const float w3 = from_bf16(a.w3b[32 * wv + 16 * c + (lane & 15)]);
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) yp[rb][v] += h2[rb][c][v] * w3;
            }
        };
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            const float bias = a.b2[32 * wv + 16 * c + (lane & 15)];
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float z = acc[rb][c][v] + bias;
                    h2[rb][c][v] = from_bf16(to_bf16(fmaxf(z, 0.f)));
                    m2 |= (z > 0.f ? 1u : 0u) << bit2(rb, c, v);
                }
        }
        if ((wv & 1) == 0) {
            add_columns();
#pragma unroll
            for (int i = 0; i < 8; ++i) hand[i * 64 + lane] = yp[i >> 2][i & 3];
        }
        __syncthreads();
        if (wv & 1) {
#pragma unroll
            for (int i = 0; i < 8; ++i) yp[i >> 2][i & 3] = hand[i * 64 + lane];
            add_columns();
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float s = sum_row(yp[rb][v]);
                    if ((lane & 15) == 0) S.yp[wv >> 1][16 * rb + 4 * (lane >> 4) + v] = s;
                }
        }
    }
    __syncthreads();
    if (tid < kTB) {
        const int64_t b = b0 + tid;
        const float y = ((S.yp[0][tid] + S.yp[1][tid]) + (S.yp[2][tid] + S.yp[3][tid])) + a.b3[0];
        float dy = 0.f;
        if (b < a.B) {
            a.y[b] = y;
            if (a.target) {
                const float r = y - a.target[b];
                dy = 2.f * r / (float)a.B;
                a.sq[b] = r * r;
            }
        }
        S.dy[tid] = dy;
    }
    if (!a.target) return;   // forward only (uniform)
    __syncthreads();

    // output layer backward: dz2 = dy w3 [z2 > 0]; per-tile sums of dz2
    // (b2), h2 dy (w3) and dy (b3); bf16(dz2) to LDS
    const int64_t tile = blockIdx.x;
#pragma unroll
    for (int c = 0; c < kC; ++c) {
        const int n = 32 * wv + 16 * c + (lane & 15);
        const float w3 = from_bf16(a.w3b[n]);
        float sb2 = 0.f, sw3 = 0.f;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * rb + 4 * (lane >> 4) + v;
                const float dy = S.dy[r];
                const float g = (m2 >> bit2(rb, c, v)) & 1u ? dy * w3 : 0.f;
                sb2 += g;
                sw3 += h2[rb][c][v] * dy;
                S.dz2[r][n] = to_bf16(g);
            }
        sb2 = sum_groups(sb2);
        sw3 = sum_groups(sw3);
        if (lane < 16) {
            a.pb2[tile * kH + n] = sb2;
            a.pw3[tile * kH + n] = sw3;
        }
    }
    if (tid == 0) {
        float s = 0.f;
        for (int r = 0; r < kTB; ++r) s += S.dy[r];
        a.pb3[tile] = s;
    }
    __syncthreads();

    // dz1 = (bf16(dz2) W2) [z1 > 0]; per-tile sums (b1); bf16(dz1) to LDS
    const int cb = wv & 3, rbx = wv >> 2;   // the wave's block of dx
    bf16x8 w1t[kH / 32];
    {
        f32x4 acc[2][kC] = {};
        product(std::integral_constant<int, kH>{}, &S.dz2[0][0], kLdH, a.W2bT, acc);
#pragma unroll
        for (int k = 0; k < kH / 32; ++k) w1t[k] = frag(a.W1bT, kH, 16 * cb, 32 * k, lane);
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            const int n = 32 * wv + 16 * c + (lane & 15);
            float sb1 = 0.f;
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 16 * rb + 4 * (lane >> 4) + v;
                    const float g = S.m1[r][n] ? acc[rb][c][v] : 0.f;
                    sb1 += g;
                    S.dz1[r][n] = to_bf16(g);
                }
            sb1 = sum_groups(sb1);
            if (lane < 16) a.pb1[tile * kH + n] = sb1;
        }
    }
    __syncthreads();

    // dx = bf16(dz1) W1 (wave wv: columns 16 (wv mod 4) .. + 15 of rows
    // 16 (wv / 4) .. + 15)
    {
        f32x4 acc = {};
#pragma unroll
        for (int k = 0; k < kH / 32; ++k)
            acc = mfma(frag(&S.dz1[0][0], kLdH, 16 * rbx, 32 * k, lane), w1t[k], acc);
        const int d = 16 * cb + (lane & 15);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t b = b0 + 16 * rbx + 4 * (lane >> 4) + v;
            a.dX[b * kD2 + d] = acc[v];
        }
    }
    // the weight-gradient operands
    store_transposed<kD2, kLdX>(S.x, a.XrT, tile);
    store_transposed<kH, kLdH>(S.h1, a.H1rT, tile);
    store_transposed<kH, kLdH>(S.dz2, a.dZ2rT, tile);
    store_transposed<kH, kLdH>(S.dz1, a.dZ1rT, tile);
}

// ------------------------------------------------------------- kernel B --

// One 64 x 64 tile of a split-K product over a chunk of 256 candidates:
// out[m][n] = sum_b A[m][b] Bm[n][b], A and Bm tile-major (MA and MB
// features, kTB candidates per tile: a fragment is 1 KiB of consecutive
// memory); four waves of 32 x 32.
template <int MA, int MB>
__device__ void grad_tile(const uint16_t *A, const uint16_t *Bm, int64_t m0, int64_t n0,
                          int64_t kb, float *out, int64_t ldo) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t mw = m0 + 32 * (wv >> 1), nw = n0 + 32 * (wv & 1);
    f32x4 acc[2][2] = {};
    constexpr int kSteps = kChunk / 32;
    constexpr int kAhead = 4;   // k-steps in flight (all 8 cost a wave per SIMD)
    for (int k0 = 0; k0 < kSteps; k0 += kAhead) {
        bf16x8 fa[kAhead][2], fb[kAhead][2];
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int64_t tile = kb / kTB + k0 + k;
                fa[k][i] = frag(A + tile * (MA * kTB), kTB, mw + 16 * i, 0, lane);
                fb[k][i] = frag(Bm + tile * (MB * kTB), kTB, nw + 16 * i, 0, lane);
            }
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mfma(fa[k][i], fb[k][j], acc[i][j]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                out[(mw + 16 * i + 4 * (lane >> 4) + v) * ldo + nw + 16 * j + (lane & 15)] =
                    acc[i][j][v];
}

// Embedding gradients.  A list (a column's occurrences, a length's
// candidates) is summed in a fixed order: entry o belongs to row
// (o / 32) mod 8, place o mod 32; entries of one row and place are added
// first (list order), then a row's 32 places, then the 8 rows.  Half-wave =
// row, lane = embedding dimension, so that every read of a table row is one
// 128-byte line; what the entries of the 32 places need is loaded first, a
// place per lane, and passed on by lane exchanges.  (With an entry per thread and
// its 96 sums in registers, 212 VGPRs and three reductions through LDS, whose
// rows met in two banks, these jobs took most of the kernel's 34 us.)
constexpr int kRows = kBlock / kD;     // 8
constexpr int kPlaces = 16;           // a column's places whose loads are in flight
static_assert(kRows * kD == kBlock && kD == 32, "half-waves are rows");

// The rows' sums acc of one dimension each -> out[0..kD).
__device__ void row_sums(float acc, float *red, float *out) {
    red[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < kD) {
        float s = 0.f;
        for (int k = 0; k < kRows; ++k) s += red[k * kD + threadIdx.x];
        out[threadIdx.x] = s;
    }
    __syncthreads();
}

// Column j: dE from its occurrences' dx / L, dF from the pairs it begins (times
// T of the next column) or dT from those it ends (times F of the one before).
// A job each, as a long list lasts as long as one compute unit's chain of
// entries and gathered rows; 16 places at a time, so that the entries are read
// twice.  The kernel takes 17.8 us at 8192 candidates over 500 columns (190
// entries a list), 61 us over 20 columns (3000 a list); with the three in one
// job, 8 places at a time, 18.1 and 103 us; with every place's sum kept over
// the rounds (32, 165 VGPRs) 24.2 and 62 us.
enum Table { kTabE, kTabF, kTabT };
template <Table TAB>
__device__ void column_grads(const FusedGrads &g, int32_t j, float *red) {
    constexpr bool PAIRS = TAB != kTabE;
    const int r = threadIdx.x / kD, c = threadIdx.x % kD;
    const int32_t o0 = g.occ_start[j], o1 = g.occ_start[j + 1];
    const float *const other = TAB == kTabF ? g.T : g.F;
    const float *const dx = g.dX + (PAIRS ? kD : 0) + c;
    float acc = 0.f;
    const int32_t row0 = o0 + r * kD;
    // lane c: what the entry at place c of the row's round at `o` needs: its
    // candidate, the pair's other column (-1: none) and the mean's factor
    int32_t b, col;
    float inv;
    auto entry = [&](int32_t o) {
        const int32_t mine = o + c < o1 ? o + c : o1 - 1;
        b = g.occ_b[mine];
        const int32_t s = g.off[b], e = g.off[b + 1], L = e - s;
        if (PAIRS) {
            const int32_t pos = g.occ_pos[mine] + (TAB == kTabF ? 1 : -1);
            col = pos >= s && pos < e ? g.cols[pos] : -1;
            inv = L > 1 ? 1.f / (float)(L - 1) : 0.f;
        } else {
            inv = 1.f / (float)L;
        }
    };
    if (row0 < o1) entry(row0);
    for (int p0 = 0; p0 < kD && row0 + p0 < o1; p0 += kPlaces) {
        float v[kPlaces];
#pragma unroll
        for (int u = 0; u < kPlaces; ++u) v[u] = 0.f;
        for (int32_t o = row0; o + p0 < o1; o += kBlock) {
            if (o != row0 || (p0 > 0 && row0 + kBlock < o1)) entry(o);
            float x[kPlaces], w[kPlaces];
#pragma unroll
            for (int u = 0; u < kPlaces; ++u) {
                x[u] = dx[(int64_t)__shfl(b, p0 + u, kD) * kD2];
                if (PAIRS) {
                    const int32_t cu = __shfl(col, p0 + u, kD);
                    w[u] = other[(int64_t)(cu < 0 ? 0 : cu) * kD + c];
                }
            }
#pragma unroll
            for (int u = 0; u < kPlaces; ++u) {
                const float iv = __shfl(inv, p0 + u, kD);
                const bool have = !PAIRS || __shfl(col, p0 + u, kD) >= 0;
                if (have && o + p0 + u < o1) v[u] += PAIRS ? x[u] * w[u] * iv : x[u] * iv;
            }
        }
#pragma unroll
        for (int u = 0; u < kPlaces; ++u) acc += v[u];
    }
    float *const out = TAB == kTabE ? g.gE : (TAB == kTabF ? g.gF : g.gT);
    row_sums(acc, red, out + (int64_t)j * kD);
}

// Length l: dZ from its candidates' dx; every place's sum stays in registers,
// and the next round's candidates are read ahead (8192 candidates of one
// length: 55 us, 85 with 8 places at a time).
__device__ void length_grads(const FusedGrads &g, int32_t l, float *red) {
    const int r = threadIdx.x / kD, c = threadIdx.x % kD;
    const int32_t o0 = g.len_start[l], o1 = g.len_start[l + 1];
    const int32_t row0 = o0 + r * kD;
    float acc = 0.f, v[kD] = {};
    auto owner = [&](int32_t o) { return g.len_b[o + c < o1 ? o + c : o1 - 1]; };
    int32_t b = row0 < o1 ? owner(row0) : 0;   // lane c: place c
    for (int32_t o = row0; o < o1; o += kBlock) {
        const int32_t now = b;
        if (o + kBlock < o1) b = owner(o + kBlock);
        float x[kD];
#pragma unroll
        for (int u = 0; u < kD; ++u) x[u] = g.dX[(int64_t)__shfl(now, u, kD) * kD2 + c];
#pragma unroll
        for (int u = 0; u < kD; ++u)
            if (o + u < o1) v[u] += x[u];
    }
#pragma unroll
    for (int u = 0; u < kD; ++u) acc += v[u];
    row_sums(acc, red, g.gZ + (int64_t)l * kD);
}

__global__ __launch_bounds__(kBlock) void mlp_grads_kernel(FusedGrads g) {
    __shared__ float red[kBlock];
    const int tid = threadIdx.x;
    const int64_t nS = g.Bp / kChunk;
    const int64_t nT = g.Bp / kTB;
    int64_t job = blockIdx.x;
    // dW2 partials: 16 tiles per chunk
    if (job < 16 * nS) {
        const int64_t s = job / 16, t = job % 16;
        grad_tile<kH, kH>(g.dZ2rT, g.H1rT, 64 * (t / 4), 64 * (t % 4), s * kChunk,
                          g.ws2 + s * (int64_t)kH * kH, kH);
        return;
    }
    job -= 16 * nS;
    // dW1 partials: 4 tiles per chunk
    if (job < 4 * nS) {
        const int64_t s = job / 4, t = job % 4;
        grad_tile<kH, kD2>(g.dZ1rT, g.XrT, 64 * t, 0, s * kChunk,
                           g.ws1 + s * (int64_t)kH * kD2, kD2);
        return;
    }
    job -= 4 * nS;
    // b1, b2, w3: the row tiles' partial sums, 32 columns per job
    if (job < 3 * (kH / 32)) {
        const int v = (int)(job / (kH / 32));
        const int h = (int)(job % (kH / 32)) * 32 + tid % 32, r = tid / 32;
        const float *src = v == 0 ? g.pb1 : (v == 1 ? g.pb2 : g.pw3);
        float *dst = v == 0 ? g.gb1 : (v == 1 ? g.gb2 : g.gw3);
        float acc = 0.f;
        for (int64_t t = r; t < nT; t += kBlock / 32) acc += src[t * kH + h];
        red[r * 32 + tid % 32] = acc;
        __syncthreads();
        if (r == 0) {
            float sum = 0.f;
            for (int k = 0; k < kBlock / 32; ++k) sum += red[k * 32 + tid];
            dst[h] = sum;
        }
        return;
    }
    job -= 3 * (kH / 32);
    if (job == 0) {   // b3
        float acc = 0.f;
        for (int64_t t = tid; t < nT; t += kBlock) acc += g.pb3[t];
        red[tid] = acc;
        __syncthreads();
        if (tid == 0) {
            float sum = 0.f;
            for (int k = 0; k < kBlock; ++k) sum += red[k];
            g.gb3[0] = sum;
        }
        return;
    }
    job -= 1;
    if (job < 3 * (int64_t)g.M) {
        const int32_t col = (int32_t)(job % g.M), t = (int32_t)(job / g.M);
        if (t == 0)
            column_grads<kTabF>(g, col, red);
        else if (t == 1)
            column_grads<kTabT>(g, col, red);
        else
            column_grads<kTabE>(g, col, red);
        return;
    }
    job -= 3 * (int64_t)g.M;
    if (job <= g.M) length_grads(g, (int32_t)job, red);
}

// ------------------------------------------------------------- kernel C --

__global__ __launch_bounds__(kBlock) void mlp_update_kernel(FusedUpdate u) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= u.n_params) return;
    float p = u.p[i];
    if (u.mode != kUpdateCast) {
        float g;
        if (i < u.oW1 || (i >= u.ob1 && i < u.oW2) || i >= u.ob2) {
            g = u.g[i];                        // embeddings, b1, b2, w3, b3 (kernel B)
        } else if (i < u.ob1) {
            const int64_t k = i - u.oW1;
            g = 0.f;
#pragma unroll 8
            for (int64_t s = 0; s < u.nS; ++s) g += u.ws1[s * (int64_t)kH * kD2 + k];
        } else {
            const int64_t k = i - u.oW2;
            g = 0.f;
#pragma unroll 8
            for (int64_t s = 0; s < u.nS; ++s) g += u.ws2[s * (int64_t)kH * kH + k];
        }
        u.g[i] = g;
        if (u.mode == kUpdateGradients) return;
        const float m1 = u.beta1 * u.m1[i] + (1.f - u.beta1) * g;
        const float m2 = u.beta2 * u.m2[i] + (1.f - u.beta2) * g * g;
        u.m1[i] = m1;
        u.m2[i] = m2;
        p -= u.lr * (m1 / u.c1) / (sqrtf(m2 / u.c2) + u.eps);
        u.p[i] = p;
    }
    // BF16 copies
    if (i >= u.oW1 && i < u.ob1) {
        const int64_t k = i - u.oW1, h = k / kD2, d = k % kD2;
        const uint16_t q = to_bf16(p);
        u.W1b[k] = q;
        u.W1bT[d * kH + h] = q;
    } else if (i >= u.oW2 && i < u.ob2) {
        const int64_t k = i - u.oW2, n = k / kH, c = k % kH;
        const uint16_t q = to_bf16(p);
        u.W2b[k] = q;
        u.W2bT[c * kH + n] = q;
    } else if (i >= u.ow3 && i < u.ob3) {
        u.w3b[i - u.ow3] = to_bf16(p);
    }
}

}  // namespace

bool fused_shape(int32_t D, int32_t H) { return D == kD && H == kH; }
int32_t fused_tile_rows() { return kTB; }
int32_t fused_chunk() { return kChunk; }

hipError_t fused_rows(const FusedRows &a, hipStream_t s) {
    hipLaunchKernelGGL(mlp_rows_kernel, dim3((unsigned)(a.Bp / kTB)), dim3(kRowsBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t fused_grads(const FusedGrads &g, hipStream_t s) {
    const int64_t nS = g.Bp / kChunk;
    const int64_t jobs = 20 * nS + 3 * (kH / 32) + 1 + 3 * (int64_t)g.M + (g.M + 1);
    hipLaunchKernelGGL(mlp_grads_kernel, dim3((unsigned)jobs), dim3(kBlock), 0, s, g);
    return hipGetLastError();
}

hipError_t fused_update(const FusedUpdate &u, hipStream_t s) {
    hipLaunchKernelGGL(mlp_update_kernel, dim3((unsigned)((u.n_params + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, s, u);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace ebic
