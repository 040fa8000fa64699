// Host entry points that do not belong to a single kernel file: version,
// workspace query, the expert-FFN dispatcher (fp32, bf16 and its fast shapes), and the layer in one call.
#include "c2r_internal.h"

namespace c2r {
size_t route_workspace_bytes(int64_t T, int d, int E);
size_t permute_workspace_bytes(int64_t T, int E, int K);
size_t dedup_workspace_bytes(int64_t T, int n_dev);
int launch_ffn_f32_pass(int pass, const float *a, const int32_t *offsets, int E_local, int64_t A_cap, int d,
                        int F, const float *b0, const float *b1, float *out, hipStream_t st);
int launch_ffn_bf16_pass(int pass, const uint16_t *a, const int32_t *offsets, int E_local, int64_t A_cap, int d,
                         int F, const uint16_t *b0, const uint16_t *b1, uint16_t *out, hipStream_t st);
int launch_ffn_bf16_dma_pass(int pass, const uint16_t *a, int lda, const int32_t *offsets, int E_local,
                             int64_t A_cap, int d, int F, const uint16_t *b0, const uint16_t *b1,
                             uint16_t *out, int ldo, const int32_t *gather, int gather_div, int gather_rows,
                             hipStream_t st);
struct FfnProblem;
}  // namespace c2r
#include "ffn_common.h"
#include "route_few.h"
namespace c2r {
FfnProblem ffn_bf16_dma_problem(int pass, const uint16_t *a, int lda, const int32_t *offsets, int E_local,
                                int64_t A_cap, int d, int F, const uint16_t *b0, const uint16_t *b1, uint16_t *out,
                                int ldo, const int32_t *gather, int gather_div, int gather_rows);
int launch_ffn_bf16_dma(int pass, const FfnProblem &first, const FfnProblem *second, int likely, hipStream_t st);
int launch_ffn_bf16_dma_both(const FfnProblem (&first)[2], const FfnProblem *const (&second)[2], int likely, hipStream_t st);
bool ffn_few_takes(const FfnProblem &routed, const FfnProblem *shared);
int launch_ffn_few(const FfnProblem &routed, const FfnProblem *shared, const FewRoute &few, hipStream_t st);
}  // namespace c2r

using namespace c2r;

// Row pitch of the hidden activation h inside the library's own workspace: padded to the
// k-slice of the fast bf16 path (the padding is kept at zero by the first pass).
static bool fast_bf16(c2r_dtype dt, int d, int F) {
    // the copy-engine kernel: bf16 and a model width of whole 64-element k-slices (F is
    // padded to such slices inside the workspace)
    (void)F;
    return dt == C2R_BF16 && d % 64 == 0;
}

static int h_pitch(c2r_dtype dt, int d, int F) { return fast_bf16(dt, d, F) ? (F + 63) / 64 * 64 : F; }

extern "C" int c2r_version(void) { return 100; }

extern "C" size_t c2r_workspace_bytes(int stage, int64_t T, int d, int E, int K, int F, c2r_dtype dt) {
    switch (stage) {
        case C2R_STAGE_COACTIVATION:
            return 0;
        case C2R_STAGE_ROUTE:
            return route_workspace_bytes(T, d, E);
        case C2R_STAGE_PERMUTE:
            return permute_workspace_bytes(T, E, K);
        case C2R_STAGE_EXPERT_FFN: {
            if (T <= 0 || F <= 0) return 0;
            const size_t sz = dt == C2R_BF16 ? 2 : 4;
            return round_up((size_t)T * (size_t)(K > 0 ? K : 1) * (size_t)h_pitch(dt, d, F) * sz, 256);
        }
        case C2R_STAGE_DEDUP_DISPATCH:
            return dedup_workspace_bytes(T, E);  // E: number of devices
        default:
            return 0;
    }
}

static int check_ffn(c2r_dtype dt, int E_local, int64_t A_cap, int d, int F) {
    if (E_local < 1 || A_cap < 0 || d < 1 || F < 1) return C2R_ERR_INVALID_ARG;
    if (dt != C2R_F32 && dt != C2R_BF16) return C2R_ERR_INVALID_ARG;
    if (E_local > C2R_MAX_E) return C2R_ERR_UNSUPPORTED;
    if (A_cap >= (1ll << 31)) return C2R_ERR_UNSUPPORTED;
    if (d % 8 != 0 || F % 8 != 0) return C2R_ERR_UNSUPPORTED;
    const size_t sz = dt == C2R_BF16 ? 2 : 4;
    // 32-bit byte offsets are used inside one tile's rows and inside one expert's weights
    if ((size_t)d * F * sz >= (1ull << 32) || 256ull * (d > F ? d : F) * sz >= (1ull << 32))
        return C2R_ERR_UNSUPPORTED;
    return C2R_OK;
}

// ldh: pitch of h (output of pass 0, input of pass 1).  The copy-engine path needs the
// contraction rows of A padded to a multiple of 64 elements.
static int ffn_pass(int pass, c2r_dtype dt, const void *a, const int32_t *offsets, int E_local, int64_t A_cap,
                    int d, int F, int ldh, const void *b0, const void *b1, void *out, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (fast_bf16(dt, d, F) && ldh % 64 == 0)
        return launch_ffn_bf16_dma_pass(pass, static_cast<const uint16_t *>(a), pass == 0 ? d : ldh, offsets,
                                        E_local, A_cap, d, F, static_cast<const uint16_t *>(b0),
                                        static_cast<const uint16_t *>(b1), static_cast<uint16_t *>(out),
                                        pass == 0 ? ldh : d, nullptr, 1, 1, st);
    if (ldh != F) return C2R_ERR_UNSUPPORTED;
    if (dt == C2R_BF16)
        return launch_ffn_bf16_pass(pass, static_cast<const uint16_t *>(a), offsets, E_local, A_cap, d, F,
                                    static_cast<const uint16_t *>(b0), static_cast<const uint16_t *>(b1),
                                    static_cast<uint16_t *>(out), st);
    return launch_ffn_f32_pass(pass, static_cast<const float *>(a), offsets, E_local, A_cap, d, F,
                               static_cast<const float *>(b0), static_cast<const float *>(b1),
                               static_cast<float *>(out), st);
}

// Both passes of routed groups on the copy-engine kernel: h of pitch ldh in between; gather: rows of x by perm.
static void both_problems(const void *a, const int32_t *offsets, int E_local, int64_t A_cap, int d, int F, int ldh,
                          const void *w_gate, const void *w_up, const void *w_down, void *h, void *y_perm, const int32_t *gather,
                          int gather_div, int gather_rows, FfnProblem (&p)[2]) {
    uint16_t *const hb = static_cast<uint16_t *>(h);
    p[0] = ffn_bf16_dma_problem(0, static_cast<const uint16_t *>(a), d, offsets, E_local, A_cap, d, F,
                                static_cast<const uint16_t *>(w_gate), static_cast<const uint16_t *>(w_up), hb, ldh, gather,
                                gather_div, gather_rows);
    p[1] = ffn_bf16_dma_problem(1, hb, ldh, offsets, E_local, A_cap, d, F, static_cast<const uint16_t *>(w_down), nullptr,
                                static_cast<uint16_t *>(y_perm), d, nullptr, 1, 1);
}

extern "C" int c2r_expert_ffn_gate_up(const void *x_perm, c2r_dtype dt, const int32_t *offsets, int E_local,
                                      int64_t A_cap, int d, int F, const void *w_gate, const void *w_up,
                                      void *h, void *stream) {
    const int rc = check_ffn(dt, E_local, A_cap, d, F);
    if (rc != C2R_OK) return rc;
    if (A_cap == 0) return C2R_OK;
    if (!x_perm || !offsets || !w_gate || !w_up || !h) return C2R_ERR_INVALID_ARG;
    if (!aligned(x_perm, 16) || !aligned(w_gate, 16) || !aligned(w_up, 16) || !aligned(h, 16))
        return C2R_ERR_INVALID_ARG;
    return ffn_pass(0, dt, x_perm, offsets, E_local, A_cap, d, F, F, w_gate, w_up, h, stream);
}

static int check_gate_up_gather(const void *x, c2r_dtype dt, const int32_t *perm, int64_t T, int K, const int32_t *offsets,
                                int E_local, int64_t A_cap, int d, int F, const void *w_gate, const void *w_up, const void *h) {
    const int rc = check_ffn(dt, E_local, A_cap, d, F);
    if (rc != C2R_OK) return rc;
    if (T < 1 || K < 1) return C2R_ERR_INVALID_ARG;
    if (A_cap == 0) return C2R_OK;
    if (!x || !perm || !offsets || !w_gate || !w_up || !h) return C2R_ERR_INVALID_ARG;
    if (!aligned(x, 16) || !aligned(w_gate, 16) || !aligned(w_up, 16) || !aligned(h, 16))
        return C2R_ERR_INVALID_ARG;
    // only the copy-engine kernel folds the gather into its addresses (32-bit row offsets into x)
    if (!fast_bf16(dt, d, F) || F % 64 != 0 || (uint64_t)T * d * 2 >= (1ull << 32)) return C2R_ERR_UNSUPPORTED;
    return C2R_OK;
}

extern "C" int c2r_expert_ffn_gate_up_gather(const void *x, c2r_dtype dt, const int32_t *perm, int64_t T, int K,
                                             const int32_t *offsets, int E_local, int64_t A_cap, int d, int F,
                                             const void *w_gate, const void *w_up, void *h, void *stream) {
    const int rc = check_gate_up_gather(x, dt, perm, T, K, offsets, E_local, A_cap, d, F, w_gate, w_up, h);
    if (rc != C2R_OK || A_cap == 0) return rc;
    return launch_ffn_bf16_dma_pass(0, static_cast<const uint16_t *>(x), d, offsets, E_local, A_cap, d, F,
                                    static_cast<const uint16_t *>(w_gate), static_cast<const uint16_t *>(w_up),
                                    static_cast<uint16_t *>(h), F, perm, K, (int)T, static_cast<hipStream_t>(stream));
}

static int check_down(const void *h, c2r_dtype dt, const int32_t *offsets, int E_local, int64_t A_cap, int d, int F,
                      const void *w_down, const void *y_perm) {
    const int rc = check_ffn(dt, E_local, A_cap, d, F);
    if (rc != C2R_OK) return rc;
    if (A_cap == 0) return C2R_OK;
    if (!h || !offsets || !w_down || !y_perm) return C2R_ERR_INVALID_ARG;
    if (!aligned(h, 16) || !aligned(w_down, 16) || !aligned(y_perm, 16)) return C2R_ERR_INVALID_ARG;
    return C2R_OK;
}

extern "C" int c2r_expert_ffn_down(const void *h, c2r_dtype dt, const int32_t *offsets, int E_local,
                                   int64_t A_cap, int d, int F, const void *w_down, void *y_perm,
                                   void *stream) {
    const int rc = check_down(h, dt, offsets, E_local, A_cap, d, F, w_down, y_perm);
    if (rc != C2R_OK || A_cap == 0) return rc;
    return ffn_pass(1, dt, h, offsets, E_local, A_cap, d, F, F, w_down, nullptr, y_perm, stream);
}

extern "C" int c2r_expert_ffn(const void *x_perm, c2r_dtype dt, const int32_t *offsets, int E_local,
                              int64_t A_cap, int d, int F, const void *w_gate, const void *w_up,
                              const void *w_down, void *y_perm, void *ws, size_t ws_bytes,
                              void *stream) {
    int rc = check_ffn(dt, E_local, A_cap, d, F);
    if (rc != C2R_OK) return rc;
    if (A_cap == 0) return C2R_OK;
    if (!x_perm || !offsets || !w_gate || !w_up || !w_down || !y_perm) return C2R_ERR_INVALID_ARG;
    if (!aligned(x_perm, 16) || !aligned(w_gate, 16) || !aligned(w_up, 16) || !aligned(w_down, 16) ||
        !aligned(y_perm, 16))
        return C2R_ERR_INVALID_ARG;
    const int ldh = h_pitch(dt, d, F);
    const size_t need = round_up((size_t)A_cap * ldh * (dt == C2R_BF16 ? 2 : 4), 256);
    if (!ws || ws_bytes < need || !aligned(ws, 256)) return C2R_ERR_WORKSPACE;
    if (fast_bf16(dt, d, F)) {
        FfnProblem p[2];
        both_problems(x_perm, offsets, E_local, A_cap, d, F, ldh, w_gate, w_up, w_down, ws, y_perm, nullptr, 1, 1, p);
        return launch_ffn_bf16_dma_both(p, {nullptr, nullptr}, (int)A_cap, static_cast<hipStream_t>(stream));
    }
    rc = ffn_pass(0, dt, x_perm, offsets, E_local, A_cap, d, F, ldh, w_gate, w_up, ws, stream);
    if (rc != C2R_OK) return rc;
    return ffn_pass(1, dt, ws, offsets, E_local, A_cap, d, F, ldh, w_down, nullptr, y_perm, stream);
}

// The arguments of c2r_expert_ffn_gather, checked; p: its two passes (A_cap > 0).
static int gather_problems(const void *x, c2r_dtype dt, const int32_t *perm, int64_t T, int K, const int32_t *offsets, int E_local,
                           int64_t A_cap, int d, int F, const void *w_gate, const void *w_up, const void *w_down, void *y_perm,
                           void *ws, size_t ws_bytes, FfnProblem (&p)[2]) {
    const int rc = check_ffn(dt, E_local, A_cap, d, F);
    if (rc != C2R_OK) return rc;
    if (T < 1 || K < 1) return C2R_ERR_INVALID_ARG;
    if (A_cap == 0) return C2R_OK;
    if (!x || !perm || !offsets || !w_gate || !w_up || !w_down || !y_perm) return C2R_ERR_INVALID_ARG;
    if (!aligned(x, 16) || !aligned(w_gate, 16) || !aligned(w_up, 16) || !aligned(w_down, 16) || !aligned(y_perm, 16))
        return C2R_ERR_INVALID_ARG;
    // only the copy-engine kernel folds the gather into its addresses (32-bit row offsets into x)
    if (!fast_bf16(dt, d, F) || (uint64_t)T * d * 2 >= (1ull << 32)) return C2R_ERR_UNSUPPORTED;
    const int ldh = h_pitch(dt, d, F);
    const size_t need = round_up((size_t)A_cap * ldh * 2, 256);
    if (!ws || ws_bytes < need || !aligned(ws, 256)) return C2R_ERR_WORKSPACE;
    both_problems(x, offsets, E_local, A_cap, d, F, ldh, w_gate, w_up, w_down, ws, y_perm, perm, K, (int)T, p);
    return C2R_OK;
}

extern "C" int c2r_expert_ffn_gather(const void *x, c2r_dtype dt, const int32_t *perm, int64_t T, int K,
                                     const int32_t *offsets, int E_local, int64_t A_cap, int d, int F,
                                     const void *w_gate, const void *w_up, const void *w_down, void *y_perm,
                                     void *ws, size_t ws_bytes, void *stream) {
    FfnProblem p[2];
    const int rc = gather_problems(x, dt, perm, T, K, offsets, E_local, A_cap, d, F, w_gate, w_up, w_down, y_perm, ws, ws_bytes, p);
    if (rc != C2R_OK || A_cap == 0) return rc;
    return launch_ffn_bf16_dma_both(p, {nullptr, nullptr}, (int)A_cap, static_cast<hipStream_t>(stream));
}

// ---- routed groups and an always-on shared expert in ONE launch per pass ----
static int check_with_shared(c2r_dtype dt, int64_t T, int E_local, int64_t A_cap, int d, int F, int F_shared) {
    int rc = check_ffn(dt, E_local, A_cap, d, F);
    if (rc != C2R_OK) return rc;
    if (T < 1 || F_shared < 1) return C2R_ERR_INVALID_ARG;
    rc = check_ffn(dt, 1, T, d, F_shared);
    if (rc != C2R_OK) return rc;
    if (dt != C2R_BF16 || d % 64 != 0 || F % 64 != 0 || F_shared % 64 != 0) return C2R_ERR_UNSUPPORTED;
    if ((uint64_t)T * d * 2 >= (1ull << 32)) return C2R_ERR_UNSUPPORTED;
    return C2R_OK;
}

static int gate_up_with_shared_problems(const void *x, c2r_dtype dt, const int32_t *perm, int64_t T, int K, const int32_t *offsets,
                                        int E_local, int64_t A_cap, int d, int F, const void *w_gate, const void *w_up, void *h,
                                        int F_shared, const void *ws_gate, const void *ws_up, void *h_shared,
                                        FfnProblem &routed, FfnProblem &shared) {
    const int rc = check_with_shared(dt, T, E_local, A_cap, d, F, F_shared);
    if (rc != C2R_OK) return rc;
    if (K < 1) return C2R_ERR_INVALID_ARG;
    if (!x || !ws_gate || !ws_up || !h_shared) return C2R_ERR_INVALID_ARG;
    if (A_cap > 0 && (!perm || !offsets || !w_gate || !w_up || !h)) return C2R_ERR_INVALID_ARG;
    if (!aligned(x, 16) || !aligned(w_gate, 16) || !aligned(w_up, 16) || !aligned(h, 16) || !aligned(ws_gate, 16) ||
        !aligned(ws_up, 16) || !aligned(h_shared, 16))
        return C2R_ERR_INVALID_ARG;
    const uint16_t *xs = static_cast<const uint16_t *>(x);
    shared = ffn_bf16_dma_problem(0, xs, d, nullptr, 1, T, d, F_shared, static_cast<const uint16_t *>(ws_gate),
                                  static_cast<const uint16_t *>(ws_up), static_cast<uint16_t *>(h_shared), F_shared, nullptr, 1, 1);
    routed = ffn_bf16_dma_problem(0, xs, d, offsets, E_local, A_cap, d, F, static_cast<const uint16_t *>(w_gate),
                                  static_cast<const uint16_t *>(w_up), static_cast<uint16_t *>(h), F, perm, K, (int)T);
    return C2R_OK;
}

static int down_with_shared_problems(const void *h, c2r_dtype dt, const int32_t *offsets, int E_local, int64_t A_cap, int d, int F,
                                     const void *w_down, void *y_perm, int64_t T, int F_shared, const void *h_shared,
                                     const void *ws_down, void *y_shared, FfnProblem &routed, FfnProblem &shared) {
    const int rc = check_with_shared(dt, T, E_local, A_cap, d, F, F_shared);
    if (rc != C2R_OK) return rc;
    if (!h_shared || !ws_down || !y_shared) return C2R_ERR_INVALID_ARG;
    if (A_cap > 0 && (!h || !offsets || !w_down || !y_perm)) return C2R_ERR_INVALID_ARG;
    if (!aligned(h, 16) || !aligned(w_down, 16) || !aligned(y_perm, 16) || !aligned(h_shared, 16) ||
        !aligned(ws_down, 16) || !aligned(y_shared, 16))
        return C2R_ERR_INVALID_ARG;
    shared = ffn_bf16_dma_problem(1, static_cast<const uint16_t *>(h_shared), F_shared, nullptr, 1, T, d, F_shared,
                                  static_cast<const uint16_t *>(ws_down), nullptr, static_cast<uint16_t *>(y_shared), d, nullptr, 1, 1);
    routed = ffn_bf16_dma_problem(1, static_cast<const uint16_t *>(h), F, offsets, E_local, A_cap, d, F,
                                  static_cast<const uint16_t *>(w_down), nullptr, static_cast<uint16_t *>(y_perm), d, nullptr, 1, 1);
    return C2R_OK;
}

extern "C" int c2r_expert_ffn_gate_up_with_shared(const void *x, c2r_dtype dt, const int32_t *perm, int64_t T, int K,
                                                  const int32_t *offsets, int E_local, int64_t A_cap, int d, int F,
                                                  const void *w_gate, const void *w_up, void *h, int F_shared,
                                                  const void *ws_gate, const void *ws_up, void *h_shared,
                                                  void *stream) {
    FfnProblem routed, shared;
    const int rc = gate_up_with_shared_problems(x, dt, perm, T, K, offsets, E_local, A_cap, d, F, w_gate, w_up, h, F_shared,
                                                ws_gate, ws_up, h_shared, routed, shared);
    if (rc != C2R_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return A_cap == 0 ? launch_ffn_bf16_dma(0, shared, nullptr, (int)T, st) : launch_ffn_bf16_dma(0, routed, &shared, (int)A_cap, st);
}

extern "C" int c2r_expert_ffn_down_with_shared(const void *h, c2r_dtype dt, const int32_t *offsets, int E_local,
                                               int64_t A_cap, int d, int F, const void *w_down, void *y_perm,
                                               int64_t T, int F_shared, const void *h_shared, const void *ws_down,
                                               void *y_shared, void *stream) {
    FfnProblem routed, shared;
    const int rc = down_with_shared_problems(h, dt, offsets, E_local, A_cap, d, F, w_down, y_perm, T, F_shared, h_shared, ws_down,
                                             y_shared, routed, shared);
    if (rc != C2R_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    return A_cap == 0 ? launch_ffn_bf16_dma(1, shared, nullptr, (int)T, st) : launch_ffn_bf16_dma(1, routed, &shared, (int)A_cap, st);
}

// ---- the layer in one host call ----
extern "C" int c2r_layer_forward(const c2r_layer *layer, const void *x, void *stream) {
    if (!layer || (layer->h && layer->x_perm)) return C2R_ERR_INVALID_ARG;
    const c2r_layer &L = *layer;
    if (L.dtype != C2R_F32 && L.dtype != C2R_BF16) return C2R_ERR_INVALID_ARG;
    for (int64_t v : {L.d, L.E, L.K, L.F, L.Tc, L.E_local, L.F_shared})  // (the stages take them as int)
        if (v != (int64_t)(int)v) return C2R_ERR_UNSUPPORTED;
    for (int64_t v : {L.ws_route_bytes, L.ws_permute_bytes, L.ws_ffn_bytes, L.ws_shared_bytes})
        if (v < 0) return C2R_ERR_WORKSPACE;
    const c2r_dtype dt = static_cast<c2r_dtype>(L.dtype);
    const int d = (int)L.d, E = (int)L.E, K = (int)L.K, F = (int)L.F, El = (int)L.E_local, Fs = (int)L.F_shared;
    const int64_t T = L.T, A = T * K;
    const bool shared = Fs > 0, rides = shared && L.fuse_shared != 0 && L.h && L.h_shared;  // (else it runs by itself)
    if (shared && !rides) {
        int rc;
        if (L.h_shared)
            rc = c2r_expert_ffn_gate_up(x, dt, L.off_shared, 1, T, d, Fs, L.ws_gate, L.ws_up, L.h_shared, stream);
        else
            rc = c2r_expert_ffn(x, dt, L.off_shared, 1, T, d, Fs, L.ws_gate, L.ws_up, L.ws_down, L.y_shared, L.ws_shared,
                                (size_t)L.ws_shared_bytes, stream);
        if (rc != C2R_OK) return rc;
    }
    // The forms whose first pass reads rows of x: the passes' arguments first, so that the gate/up launch of a few tokens can finish the
    // routing (an error in them is still reported after one in the routing's, and one in the down pass's after the gate/up pass).
    const bool own_h = L.h && !shared, gathers = rides || own_h || (!L.h && !L.x_perm);
    FfnProblem routed[2], with[2];
    int ffn_rc = C2R_OK, down_rc = C2R_OK;
    if (rides) {
        ffn_rc = gate_up_with_shared_problems(x, dt, L.perm, T, K, L.offsets, El, A, d, F, L.w_gate, L.w_up, L.h, Fs, L.ws_gate, L.ws_up,
                                              L.h_shared, routed[0], with[0]);
        if (ffn_rc == C2R_OK)
            down_rc = down_with_shared_problems(L.h, dt, L.offsets, El, A, d, F, L.w_down, L.y_perm, T, Fs, L.h_shared, L.ws_down,
                                                L.y_shared, routed[1], with[1]);
    } else if (own_h) {
        ffn_rc = check_gate_up_gather(x, dt, L.perm, T, K, L.offsets, El, A, d, F, L.w_gate, L.w_up, L.h);
        if (ffn_rc == C2R_OK) down_rc = check_down(L.h, dt, L.offsets, El, A, d, F, L.w_down, L.y_perm);
        if (ffn_rc == C2R_OK && A > 0)
            both_problems(x, L.offsets, El, A, d, F, F, L.w_gate, L.w_up, L.w_down, L.h, L.y_perm, L.perm, K, (int)T, routed);
    } else if (gathers) {
        ffn_rc = gather_problems(x, dt, L.perm, T, K, L.offsets, El, A, d, F, L.w_gate, L.w_up, L.w_down, L.y_perm, L.ws_ffn,
                                 (size_t)L.ws_ffn_bytes, routed);
    }
    // (a device that holds a part of the experts)
    const int likely = gathers && ffn_rc == C2R_OK && A > 0 ? (int)(El <= E ? A * El / E : A) : 0;
    const FfnProblem *const beside[2] = {rides ? &with[0] : nullptr, rides ? &with[1] : nullptr};
    FewRoute few;
    bool later = gathers && ffn_rc == C2R_OK && down_rc == C2R_OK && A > 0 && route_may_finish_later(T, d, E, K) && ffn_few_takes(routed[0], beside[0]);
    if (later) {
        // (every workgroup of that launch reads what the selection is made from, while others write h)
        const size_t a4 = (size_t)A * 4, up = (size_t)El * F * d * 2, up_shared = rides ? (size_t)Fs * d * 2 : 0;
        later = all_apart({{L.topk_idx, a4}, {L.gates, a4}, {L.counts, (size_t)El * 4}, {L.offsets, (size_t)(El + 1) * 4}, {L.perm, a4},
                           {L.inv_perm, a4}, {routed[0].out, (size_t)A * routed[0].ldo * 2}, {L.h_shared, rides ? (size_t)T * Fs * 2 : 0}},
                          {{L.ws_route, route_workspace_bytes(T, d, E)}, {L.bias, (size_t)E * 4}, {L.collab_idx, (size_t)E * L.Tc * 4},
                           {L.local_slot, (size_t)E * 4}, {x, (size_t)T * d * 2}, {L.w_gate, up}, {L.w_up, up}, {L.ws_gate, up_shared},
                           {L.ws_up, up_shared}});
    }
    int rc = route_and_permute(x, dt, L.Wg, L.bias, T, d, E, K, L.collab_idx, (int)L.Tc, L.topk_idx, L.gates, L.ws_route,
                               (size_t)L.ws_route_bytes, L.local_slot, El, L.counts, L.offsets, L.perm, L.inv_perm, L.x_perm,
                               L.ws_permute, (size_t)L.ws_permute_bytes, later ? &few : nullptr, stream);
    if (rc != C2R_OK) return rc;
    if (gathers) {
        hipStream_t st = static_cast<hipStream_t>(stream);
        rc = ffn_rc;
        if (later) {
            rc = launch_ffn_few(routed[0], beside[0], few, st);
            if (rc == C2R_OK) rc = launch_ffn_bf16_dma(1, routed[1], beside[1], likely, st);
        } else if (rc == C2R_OK && A > 0) {
            rc = down_rc == C2R_OK ? launch_ffn_bf16_dma_both(routed, beside, likely, st)
                                  : launch_ffn_bf16_dma(0, routed[0], beside[0], likely, st);
            if (rc == C2R_OK) rc = down_rc;
        }
    } else if (L.h) {
        rc = c2r_expert_ffn_gate_up_gather(x, dt, L.perm, T, K, L.offsets, El, A, d, F, L.w_gate, L.w_up, L.h, stream);
    } else {
        rc = c2r_expert_ffn(L.x_perm, dt, L.offsets, El, A, d, F, L.w_gate, L.w_up, L.w_down, L.y_perm, L.ws_ffn,
                            (size_t)L.ws_ffn_bytes, stream);
    }
    if (rc != C2R_OK) return rc;
    if (shared && !rides && L.h_shared) {
        rc = c2r_expert_ffn_down(L.h_shared, dt, L.off_shared, 1, T, d, Fs, L.ws_down, L.y_shared, stream);
        if (rc != C2R_OK) return rc;
    }
    if (L.h && !gathers) {
        rc = c2r_expert_ffn_down(L.h, dt, L.offsets, El, A, d, F, L.w_down, L.y_perm, stream);
        if (rc != C2R_OK) return rc;
    }
    return c2r_combine(L.y_perm, dt, L.gates, L.inv_perm, T, d, K, shared ? L.y_shared : nullptr, L.y, stream);
}
