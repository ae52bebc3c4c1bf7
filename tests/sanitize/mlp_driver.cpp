// Sanitizer driver for the surrogate network's host side (ebic_mlp.cpp) with
// host memory in place of the device's and kernels that only check that every
// buffer they are given is alive and large enough.  Every allocation of a
// growing batch fails once; a batch that fitted before has to be evaluated
// from whole buffers afterwards.  Built by tests/test_mlp_memory_cpu.py; exits
// non-zero on any mismatch.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

#include "ebic.h"
#include "ebic_mlp.h"

// ------------------------------------------------------------ memory ----

static std::map<const char *, size_t> g_live;
static int g_calls = 0, g_fail_at = 0;   // the g_fail_at-th allocation fails (0: none)
static hipError_t g_last = hipSuccess;
static const char *g_where = "";

#define CHECK(x)                                                        \
    do {                                                                \
        if (!(x)) {                                                     \
            std::printf("%s: line %d: %s\n", g_where, __LINE__, #x);    \
            std::exit(1);                                               \
        }                                                               \
    } while (0)

static hipError_t allocate(void **p, size_t n) {
    *p = nullptr;
    if (++g_calls == g_fail_at) return g_last = hipErrorOutOfMemory;
    *p = std::calloc(n, 1);
    g_live[(const char *)*p] = n;
    return hipSuccess;
}
static hipError_t release(void *p) {
    CHECK(g_live.erase((const char *)p) == 1);
    std::free(p);
    return hipSuccess;
}
// [p, p + n) lies in one live allocation.
static bool whole(const void *p, size_t n) {
    auto it = g_live.upper_bound((const char *)p);
    if (it == g_live.begin()) return false;
    --it;
    return (const char *)p + n <= it->first + it->second;
}
template <typename T>
static void need(const T *p, int64_t n) {
    CHECK(p != nullptr && whole(p, sizeof(T) * (size_t)n));
}
// A launch: reports an error that is left over, as a launch check would.
static hipError_t launched() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return allocate(p, n); }
hipError_t hipFree(void *p) { return release(p); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return allocate(p, n); }
hipError_t hipHostFree(void *p) { return release(p); }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
    CHECK(whole(k == hipMemcpyHostToDevice ? d : s, n));
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) {
    CHECK(whole(d, n) && whole(s, n));   // either way through the pinned room
    return hipMemcpy(d, s, n, k);
}
hipError_t hipMemset(void *d, int v, size_t n) {
    CHECK(whole(d, n));
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetLastError() { return launched(); }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
}

// ----------------------------------------------------------- kernels ----

namespace ebic {
void set_thread_error(const char *) {}
namespace mlp {
static int64_t g_L = 0;   // entries of the batch at hand

bool fused_shape(int32_t D, int32_t H) { return D == 32 && H == 256; }
int32_t fused_tile_rows() { return 32; }
int32_t fused_chunk() { return 256; }
bool lists_on_device(int32_t M) { return M < 8192; }
int64_t lists_workspace(int64_t B, int64_t L, int32_t M) { return B + L + M; }

hipError_t build_lists(const int32_t *off, const int32_t *cols, int32_t B, int64_t L, int32_t M,
                       int32_t *ws, int32_t *occ_start, int32_t *occ_pos, int32_t *occ_b,
                       int32_t *len_start, int32_t *len_b, hipStream_t) {
    need(off, B + 1);
    need(cols, L);
    need(ws, lists_workspace(B, L, M));
    need(occ_start, M + 1);
    need(occ_pos, L);
    need(occ_b, L);
    need(len_start, M + 2);
    need(len_b, B);
    return launched();
}
hipError_t fused_rows(const FusedRows &a, hipStream_t) {
    need(a.off, a.B + 1);
    need(a.cols, g_L);
    need(a.y, a.B);
    if (!a.target) return launched();
    need(a.target, a.B);
    need(a.sq, a.B);
    need(a.XrT, 64 * a.Bp);
    need(a.H1rT, 256 * a.Bp);
    need(a.dZ2rT, 256 * a.Bp);
    need(a.dZ1rT, 256 * a.Bp);
    need(a.dX, 64 * a.Bp);
    need(a.pw3, a.Bp / 32 * 256);
    need(a.pb2, a.Bp / 32 * 256);
    need(a.pb1, a.Bp / 32 * 256);
    need(a.pb3, a.Bp / 32);
    return launched();
}
hipError_t fused_grads(const FusedGrads &g, hipStream_t) {
    need(g.ws1, g.Bp / 256 * 256 * 64);
    need(g.ws2, g.Bp / 256 * 256 * 256);
    need(g.occ_start, g.M + 1);
    need(g.occ_pos, g_L);
    need(g.occ_b, g_L);
    need(g.len_start, g.M + 2);
    return launched();
}
hipError_t fused_update(const FusedUpdate &u, hipStream_t) {
    need(u.p, u.n_params);
    return launched();
}
hipError_t pool_fwd(const float *, const float *, const float *, const float *, int32_t D,
                    const int32_t *off, const int32_t *cols, int32_t B, float *X, uint16_t *Xb,
                    hipStream_t) {
    need(off, B + 1);
    need(cols, g_L);
    need(X, (int64_t)B * 2 * D);
    need(Xb, (int64_t)B * 2 * D);
    return launched();
}
hipError_t len_bwd(const float *dX, int32_t, const int32_t *len_start, const int32_t *len_b,
                   int32_t n_len, float *, hipStream_t) {
    need(dX, 1);
    need(len_start, n_len + 1);
    need(len_b, 1);
    return launched();
}
hipError_t pool_bwd(const float *dX, int32_t, const float *, const float *, const int32_t *,
                    const int32_t *, const int32_t *occ_start, const int32_t *occ_pos,
                    const int32_t *occ_b, int32_t M, float *, float *, float *, hipStream_t) {
    need(dX, 1);
    need(occ_start, M + 1);
    need(occ_pos, g_L);
    need(occ_b, g_L);
    return launched();
}
hipError_t gemm(const Gemm &g, hipStream_t) {
    need(g.A, (int64_t)g.M * g.K);
    need(g.B, (int64_t)g.N * g.K);
    if (g.out_f32) need(g.out_f32, (int64_t)g.M * g.N);
    if (g.out_bf16) need(g.out_bf16, (int64_t)g.M * g.N);
    if (g.splits > 1) need(g.ws, (int64_t)g.splits * g.M * g.N);
    return launched();
}
hipError_t colsum(const float *X, const float *, int32_t B, int32_t N, int32_t, float *ws,
                  float *, hipStream_t) {
    need(X, (int64_t)B * N);
    need(ws, 1);
    return launched();
}
hipError_t dw3(const uint16_t *H2b, const float *dy, int32_t B, int32_t N, int32_t, float *,
               float *, hipStream_t) {
    need(H2b, (int64_t)B * N);
    need(dy, B);
    return launched();
}
hipError_t out_fwd(const uint16_t *H2b, const uint16_t *, const float *, int32_t B, int32_t H,
                   float *y, hipStream_t) {
    need(H2b, (int64_t)B * H);
    need(y, B);
    return launched();
}
hipError_t loss(const float *y, const float *t, int32_t B, float *dy, float *sq, hipStream_t) {
    need(y, B);
    need(t, B);
    need(dy, B);
    need(sq, B);
    return launched();
}
hipError_t out_bwd(const float *, const uint16_t *, const float *Z2, int32_t B, int32_t H,
                   float *dZ2, uint16_t *dZ2b, hipStream_t) {
    need(Z2, (int64_t)B * H);
    need(dZ2, (int64_t)B * H);
    need(dZ2b, (int64_t)B * H);
    return launched();
}
hipError_t relu_bwd(const float *G, const float *Z, int64_t n, float *dZ, uint16_t *dZb,
                    hipStream_t) {
    need(G, n);
    need(Z, n);
    need(dZ, n);
    need(dZb, n);
    return launched();
}
hipError_t adam(float *, const float *, float *, float *, int64_t, float, float, float, float,
                float, float, hipStream_t) {
    return launched();
}
hipError_t cast_bf16(const float *src, int64_t n, uint16_t *dst, hipStream_t) {
    need(src, n);
    need(dst, n);
    return launched();
}
}  // namespace mlp
}  // namespace ebic

// -------------------------------------------------------------- calls ----

enum Call { kPredict, kGradients, kTrain, kTrainQueued };

// One call on B series of three columns.
static ebic_status call(ebic_mlp *m, Call what, int32_t B) {
    std::vector<int32_t> off((size_t)B + 1), cols((size_t)B * 3);
    for (int32_t b = 0; b <= B; ++b) off[(size_t)b] = 3 * b;
    for (size_t i = 0; i < cols.size(); ++i) cols[i] = (int32_t)(i % 7);
    std::vector<float> t((size_t)B, 1.f), y((size_t)B), g((size_t)ebic_mlp_param_count(m));
    float l = 0.f;
    ebic::mlp::g_L = (int64_t)cols.size();
    switch (what) {
    case kPredict: return ebic_mlp_predict(m, off.data(), cols.data(), B, y.data());
    case kGradients:
        return ebic_mlp_gradients(m, off.data(), cols.data(), B, t.data(), g.data(), &l);
    case kTrain: return ebic_mlp_train(m, off.data(), cols.data(), B, t.data(), 2, &l);
    default: return ebic_mlp_train(m, off.data(), cols.data(), B, t.data(), 2, nullptr);
    }
}

int main() {
    const Call calls[] = {kPredict, kGradients, kTrain, kTrainQueued};
    int failures = 0;
    for (int hidden : {256, 64}) {   // the fused step, the layer-by-layer one
        for (int round = 0; round < 8; ++round) {
            const Call grow = calls[round / 2];
            const bool trained = round % 2 != 0;   // before the failure
            for (int n = 1;; ++n) {
                g_where = "create";
                g_fail_at = 0;
                ebic_mlp_config cfg{};
                cfg.struct_size = sizeof(cfg);
                cfg.embed_dim = 32;
                cfg.hidden = hidden;
                cfg.lr = 1e-3f;
                cfg.beta1 = 0.9f;
                cfg.beta2 = 0.999f;
                cfg.eps = 1e-8f;
                ebic_mlp *m = nullptr;
                CHECK(ebic_mlp_create(9, &cfg, 1, 0, &m) == EBIC_OK);
                g_where = "small batch";
                for (Call c : calls)
                    if (trained || c == kPredict) CHECK(call(m, c, 40) == EBIC_OK);
                g_where = "growing batch";
                g_calls = 0;
                g_fail_at = n;
                const ebic_status st = call(m, grow, 3000);
                const bool failed = g_calls >= n;
                CHECK(st == (failed ? EBIC_E_NOMEM : EBIC_OK));
                failures += failed;
                g_fail_at = 0;
                // what fitted before the failure, from whole buffers
                g_where = "small batch after the failure";
                float l = 0.f;
                const ebic_status last = ebic::mlp_last_loss(m, &l);
                CHECK(last == EBIC_OK || last == EBIC_E_STATE);   // the loss may have gone with its buffer
                for (Call c : calls) CHECK(call(m, c, 40) == EBIC_OK);
                CHECK(ebic::mlp_last_loss(m, &l) == EBIC_OK);
                g_where = "growing batch after the failure";
                for (Call c : calls) CHECK(call(m, c, 3000) == EBIC_OK);
                CHECK(ebic_mlp_destroy(m) == EBIC_OK);
                CHECK(g_live.empty());
                if (!failed) break;
            }
        }
    }
    CHECK(failures > 40);
    std::printf("mlp driver ok: %d failed allocations\n", failures);
    return 0;
}
