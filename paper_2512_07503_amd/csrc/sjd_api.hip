// Host side of the sjd library: the C ABI of include/sjd.h, the context, the paged KV cache and the
// fixed kernel sequence of one speculative Jacobi iteration (Sec. 4.1 of the paper, Steps 1-4).
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "common.hip.h"
#include "decide.h"
#include "kernels_attention.hip.h"
#include "kernels_f32.hip.h"
#include "kernels_forward.hip.h"
#include "kernels_gemm.hip.h"
#include "kernels_skinny.hip.h"
#include "kernels_few.hip.h"
#include "kernels_tile.hip.h"
#include "kernels_lds.hip.h"

void sjd_set_error(char *buf, const char *fmt, ...) {
    if (!buf) return;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, 512, fmt, ap);
    va_end(ap);
}

namespace {

char g_create_error[512] = "";

enum KernelClass {
    KC_STAGE = 0, KC_EMBED, KC_ADDNORM, KC_GEMM_QKV, KC_ROPE_KV, KC_ATTENTION, KC_GEMM_O, KC_GEMM_GATEUP, KC_SWIGLU,
    KC_GEMM_DOWN, KC_GEMM_HEAD, KC_SAMPLE_ROWS, KC_VERIFY, KC_DRAW, KC_COMMIT, KC_COUNT
};
const char *const kKernelClassName[KC_COUNT] = {
    "stage_rows", "embed", "addnorm", "gemm_qkv", "rope_kv_write", "window_attention", "gemm_out", "gemm_gate_up", "swiglu",
    "gemm_down", "gemm_head", "sample_rows", "verify", "draw", "commit"};

struct Tracer {
    bool on = false;
    std::vector<hipEvent_t> pool;   // pairs: start, stop
    std::vector<int> cls;           // class of each recorded pair
    size_t used = 0;
    int64_t launches[KC_COUNT] = {0};
    double total_ms[KC_COUNT] = {0};
};

struct LayerWeights {
    float *attn_norm = nullptr, *mlp_norm = nullptr;
    void *wqkv = nullptr, *wo = nullptr, *wgu = nullptr, *wdown = nullptr;
};

// The rows of one forward: a decoding step's (L per segment; prompts in the same form where the context asks for the
// chunked attention) or a packed piece of the prompts (L = 0).
struct FwdRows {
    int M = 0, n_segs = 0;
    int L = 0;       // rows per segment; 0: packed
    int n_qt = 0;    // query tiles of 32 rows of the longest segment
    RowMap rm{};
    StageRows stage{};   // a step's rows are worked out by the embedding kernel
};

// Rows of a prefill forward at most.  A prompt's forward is as wide as the prompts allow, not as the window: 120 prompt
// tokens with a window of 1 used to be 119 forwards of two rows (131 ms on the 36 x 1280 shape, 2.1 ms as one forward of
// 238).  2 000-token prompts on the 8 x 4096 shape with 14336-wide MLPs, rows per forward 64 / 1024 / 2048 / 4096: 62.8 /
// 16.1 / 14.4 / 14.0 ms; from 2048 on the buffers only grow.  The reference kernels re-read a weight every 8 rows whatever
// the forward's size: 512 rows fill the chip.
constexpr int kPrefillRows = 2048, kPrefillRowsGeneric = 512;

}  // namespace

struct sjd_ctx {
    sjd_model_desc md;
    sjd_sampling sampling;
    SamplingParams sp;
    hipStream_t stream = nullptr;
    char err[512] = "";
    int hd = 0, Vs = 0, L = 0, S = 0, n_seqs = 0, pt = 0, pps = 0, n_pages = 0, max_visible = 0;
    int n_cus = 256, n_xcds = 8;   // compute units and XCDs (L2 domains) of the device, read at create
    bool prefilled = false, all_done = false;
    // one sjd_step = the same launch sequence with the same arguments every time (what changes lives in device
    // memory): captured once per batch size into a HIP graph and replayed
    bool use_graph = false;
    // ... one graph per attention regime (below)
    hipGraph_t graph[2] = {nullptr, nullptr};
    hipGraphExec_t graph_exec[2] = {nullptr, nullptr};
    int graph_n_seqs[2] = {0, 0};
    bool attn_mfma = false;
    int attn_chunk = 0, attn_nchunks = 0;
    // Window attention runs as one workgroup per (segment, head) while that is the faster of the two kernels (enough
    // such workgroups to fill the chip, or a context of up to a few thousand tokens), and as chunks over workgroups
    // plus a merge kernel beyond: chosen per step from the cache lengths, which the host follows from the verdicts
    // it reads back anyway.
    bool attn_onepass_ok = false;          // the context may use the one-pass kernel at all
    bool attn_onepass = false;             // regime of the launches being enqueued
    std::vector<int32_t> kv_host;          // committed cache positions per segment (sequence * 2 + branch)
    float *part_o = nullptr, *part_ml = nullptr;
    // Partial sums of squares of the residual stream's rows, [partial][M]: up to ceil(d / 32) of them per row, 2 ceil(d / 32) where the few-row kernels
    // leave them (M <= 64), so max(M, 128) x ceil(d / 32) hold both
    float *row_ssq = nullptr;
    QkvRow *row_meta = nullptr;            // per-row tables of the fused path, rewritten by every forward
    float2 *row_rot = nullptr;
    bool l2_warm = true;                   // projection launches touch the next projection's weights
    uint32_t *pf_sink = nullptr;
    float *skinny_part = nullptr;          // partial tiles of K-split fused projections
    size_t skinny_part_elems = 0;
    ProjShape shape{};   // what the choice of the fused projections' kernels depends on
    bool fused = false;  // bf16 path of fused projection kernels
    bool fold_gain = false;  // ... with the RMSNorm gains multiplied into the packed weights, else into the rows
    // weights (owned)
    void *tok_emb = nullptr, *lm_head = nullptr;
    float *final_norm = nullptr;
    std::vector<LayerWeights> layers;
    float *rope_cos = nullptr, *rope_sin = nullptr;
    // KV pages
    void *kpool = nullptr, *vpool = nullptr;
    size_t pool_layer_bytes = 0;
    int32_t *page_table = nullptr;
    std::vector<int32_t> page_table_host;  // what sjd_prefill uploaded (snapshots carry it)
    std::vector<int32_t> n_image_host;     // image tokens wanted per sequence of the current batch
    // workspaces
    float *x = nullptr, *partial = nullptr, *logits = nullptr;
    float *z = nullptr;                    // [S][L][V_s] guided logits written by the fused vocabulary head
    bool z_used = false;                   // the last forward's head wrote z (and the logits only if they are kept)
    bool keep_logits = false;
    void *xn = nullptr, *q = nullptr, *attn = nullptr, *h = nullptr;
    size_t partial_elems = 0;
    int32_t *win_row_tok = nullptr, *win_row_pos = nullptr, *win_seg_kv = nullptr, *win_seg_n = nullptr;  // a step's row map
    DecideState ds{};
    // what a prefill sends to the device, in one copy: the page table, the sequences' scalars, the packed rows and the
    // segment tables of every prefill forward
    int32_t *pre_dev = nullptr;
    size_t pre_elems = 0;
    std::vector<int32_t> pre_host;         // its source: stays until the copy has run
    int pre_rows = 0;                      // rows of a prefill forward at most
    int max_rows = 0;                      // rows the forward's buffers are sized for
    sjd_step_result *res_host = nullptr;
    std::vector<void *> allocations;
    Tracer tracer;
};

namespace {

template <typename P> int dev_alloc(sjd_ctx *c, P **out, size_t bytes, bool zero = true) {
    void *p = nullptr;
    if (bytes == 0) bytes = 16;
    hipError_t e = hipMalloc(&p, bytes);
    if (e != hipSuccess) {
        sjd_set_error(c->err, "hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e));
        return SJD_ENOMEM;
    }
    c->allocations.push_back(p);
    if (zero) {
        e = hipMemsetAsync(p, 0, bytes, c->stream);
        if (e != hipSuccess) {
            sjd_set_error(c->err, "hipMemsetAsync failed: %s", hipGetErrorString(e));
            return SJD_EDEVICE;
        }
    }
    *out = reinterpret_cast<P *>(p);
    return SJD_OK;
}

void trace_begin(sjd_ctx *c, int cls) {
    Tracer &t = c->tracer;
    if (!t.on) return;
    if (t.used + 2 > t.pool.size()) {
        hipEvent_t a, b;
        if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) { t.on = false; return; }
        t.pool.push_back(a);
        t.pool.push_back(b);
    }
    t.cls.push_back(cls);
    (void)hipEventRecord(t.pool[t.used], c->stream);
}
void trace_end(sjd_ctx *c) {
    Tracer &t = c->tracer;
    if (!t.on) return;
    (void)hipEventRecord(t.pool[t.used + 1], c->stream);
    t.used += 2;
}
// after the stream has been synchronised
void trace_collect(sjd_ctx *c) {
    Tracer &t = c->tracer;
    for (size_t i = 0; i + 1 < t.used; i += 2) {
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, t.pool[i], t.pool[i + 1]) == hipSuccess) {
            t.total_ms[t.cls[i / 2]] += ms;
            t.launches[t.cls[i / 2]] += 1;
        }
    }
    t.used = 0;
    t.cls.clear();
}

#define SJD_LAUNCH(c, cls, expr)                                                                   \
    do {                                                                                           \
        trace_begin(c, cls);                                                                       \
        hipError_t e__ = (expr);                                                                   \
        trace_end(c);                                                                              \
        if (e__ != hipSuccess) {                                                                   \
            sjd_set_error((c)->err, "launch of %s failed: %s", kKernelClassName[cls], hipGetErrorString(e__)); \
            return SJD_EDEVICE;                                                                    \
        }                                                                                          \
    } while (0)

template <typename F> hipError_t after(F &&f) {
    f();
    return hipGetLastError();
}

bool use_reference(const sjd_ctx *c) { return c->md.dtype == SJD_F32 || (c->md.kernel_flags & SJD_KERNELS_REFERENCE); }

// ------------------------------------------------------------------------------------- GEMM dispatch
// C_partial[splits][M][N]; returns the number of splits written.
template <typename T>
int run_gemm(sjd_ctx *c, int cls, const T *A, const T *W, float *C, int M, int N, int K, int force_splits, int *splits_out);

template <>
int run_gemm<float>(sjd_ctx *c, int cls, const float *A, const float *W, float *C, int M, int N, int K, int, int *splits_out) {
    *splits_out = 1;
    SJD_LAUNCH(c, cls, launch_gemm_reference<float>(c->stream, A, W, C, M, N, K));
    return SJD_OK;
}

template <>
int run_gemm<bf16_t>(sjd_ctx *c, int cls, const bf16_t *A, const bf16_t *W, float *C, int M, int N, int K, int force_splits,
                     int *splits_out) {
    if (c->md.kernel_flags & SJD_KERNELS_REFERENCE) {
        *splits_out = 1;
        SJD_LAUNCH(c, cls, launch_gemm_reference<bf16_t>(c->stream, A, W, C, M, N, K));
        return SJD_OK;
    }
    GemmPlan p = plan_gemm_bf16(M, N, K, force_splits);
    if ((size_t)p.splits * M * N > c->partial_elems && C == c->partial) {
        // never happens: the workspace is sized with the same plan at create
        sjd_set_error(c->err, "split-K workspace too small");
        return SJD_EINVAL;
    }
    *splits_out = p.splits;
    SJD_LAUNCH(c, cls, launch_gemm_bf16(c->stream, p, A, W, C, M, N, K));
    return SJD_OK;
}

// ---------------------------------------------------------------------------------------- attention
template <typename T> int run_attention(sjd_ctx *c, const KvPool &pool, const FwdRows &fr);

template <> int run_attention<float>(sjd_ctx *c, const KvPool &pool, const FwdRows &fr) {
    SJD_LAUNCH(c, KC_ATTENTION, launch_attention_reference<float>(c->stream, (const float *)c->q, pool, fr.rm, (float *)c->attn, nullptr,
                                                                  fr.M, fr.L, c->md.n_heads, c->md.n_kv_heads, c->hd, c->max_visible));
    return SJD_OK;
}

template <> int run_attention<bf16_t>(sjd_ctx *c, const KvPool &pool, const FwdRows &fr) {
    if (!c->attn_mfma) {
        SJD_LAUNCH(c, KC_ATTENTION, launch_attention_reference<bf16_t>(c->stream, (const bf16_t *)c->q, pool, fr.rm, (bf16_t *)c->attn,
                                                                       nullptr, fr.M, fr.L, c->md.n_heads, c->md.n_kv_heads, c->hd,
                                                                       c->max_visible));
        return SJD_OK;
    }
    AttnArgs a;
    a.q = (const bf16_t *)c->q;
    a.pool = pool;
    a.rm = fr.rm;
    a.part_o = c->part_o;
    a.part_ml = c->part_ml;
    a.out_act = (bf16_t *)c->attn;
    a.out_plain = nullptr;
    a.L = fr.L; a.H = c->md.n_heads; a.Hkv = c->md.n_kv_heads; a.hd = c->hd;
    a.chunk = c->attn_chunk;
    a.n_chunks = c->attn_nchunks;
    a.n_qt = fr.n_qt;
    a.scale_log2e = (float)(1.4426950408889634 / sqrt((double)c->hd));
    // packed prompt rows: a workgroup per (query tile, head) is plenty of them, whatever the context
    SJD_LAUNCH(c, KC_ATTENTION, launch_attention_mfma(c->stream, a, fr.n_segs, c->attn_onepass || fr.L == 0, c->n_cus));
    return SJD_OK;
}

// ------------------------------------------------------------------------------------------ forward
// Runs the rows of fr through the model.  Keys and values of active rows are written to their pages; with_head also
// produces fp32 logits [M][V_s].  Without the head the forward ends with the last layer's keys and values: nothing reads
// what its attention and MLP would add to the rows.
template <typename T> int forward(sjd_ctx *c, const FwdRows &fr, bool with_head) {
    const sjd_model_desc &md = c->md;
    const int M = fr.M, d = md.d_model, H = md.n_heads, Hkv = md.n_kv_heads, hd = c->hd, F = md.d_ff;
    const int Nqkv = (H + 2 * Hkv) * hd;
    hipStream_t st = c->stream;
    SJD_LAUNCH(c, KC_EMBED, after([&] { embed_kernel<T><<<M, 256, 0, st>>>((const T *)c->tok_emb, fr.rm.row_tok, c->x, d, fr.stage); }));
    int down_splits = 0;
    for (int l = 0; l < md.n_layers; ++l) {
        const LayerWeights &lw = c->layers[l];
        KvPool pool;
        pool.k = (char *)c->kpool + c->pool_layer_bytes * l;
        pool.v = (char *)c->vpool + c->pool_layer_bytes * l;
        pool.page_table = c->page_table;
        pool.pages_per_seg = c->pps;
        pool.page_tokens = c->pt;

        SJD_LAUNCH(c, KC_ADDNORM, after([&] {
                       addnorm_kernel<T><<<M, 256, 0, st>>>(c->x, l == 0 ? nullptr : c->partial, down_splits, M, lw.attn_norm,
                                                            (T *)c->xn, d, md.rms_eps);
                   }));
        int splits = 1;
        int rc = run_gemm<T>(c, KC_GEMM_QKV, (const T *)c->xn, (const T *)lw.wqkv, c->partial, M, Nqkv, d, 0, &splits);
        if (rc) return rc;
        SJD_LAUNCH(c, KC_ROPE_KV, after([&] {
                       rope_kv_kernel<T><<<M, 256, 0, st>>>(c->partial, splits, M, fr.rm, c->rope_cos, c->rope_sin, (T *)c->q, pool, fr.L,
                                                            H, Hkv, hd);
                   }));
        if (!with_head && l + 1 == md.n_layers) return SJD_OK;
        if ((rc = run_attention<T>(c, pool, fr))) return rc;
        rc = run_gemm<T>(c, KC_GEMM_O, (const T *)c->attn, (const T *)lw.wo, c->partial, M, d, H * hd, 0, &splits);
        if (rc) return rc;
        SJD_LAUNCH(c, KC_ADDNORM, after([&] {
                       addnorm_kernel<T><<<M, 256, 0, st>>>(c->x, c->partial, splits, M, lw.mlp_norm, (T *)c->xn, d, md.rms_eps);
                   }));
        rc = run_gemm<T>(c, KC_GEMM_GATEUP, (const T *)c->xn, (const T *)lw.wgu, c->partial, M, 2 * F, d, 0, &splits);
        if (rc) return rc;
        SJD_LAUNCH(c, KC_SWIGLU, after([&] { swiglu_kernel<T><<<M, 256, 0, st>>>(c->partial, splits, M, (T *)c->h, F); }));
        rc = run_gemm<T>(c, KC_GEMM_DOWN, (const T *)c->h, (const T *)lw.wdown, c->partial, M, d, F, 0, &down_splits);
        if (rc) return rc;
    }
    if (with_head) {
        SJD_LAUNCH(c, KC_ADDNORM, after([&] {
                       addnorm_kernel<T><<<M, 256, 0, st>>>(c->x, c->partial, down_splits, M, c->final_norm, (T *)c->xn, d,
                                                            md.rms_eps);
                   }));
        int splits = 1;
        int rc = run_gemm<T>(c, KC_GEMM_HEAD, (const T *)c->xn, (const T *)c->lm_head, c->logits, M, c->Vs, d, 1, &splits);
        if (rc) return rc;
    }
    return SJD_OK;
}

// fp32 path: five kernels per layer, the same sums bit for bit as forward<float> (nine), which SJD_KERNELS_REFERENCE selects; QKV, gate/up
// and head of more results leave their norm, rotation and SwiGLU to forward<float>'s kernels (f32_inside).
// 2 layers of 256, window 16, a step: 26 launches, now 16.
int forward_f32(sjd_ctx *c, const FwdRows &fr, bool with_head) {
    const sjd_model_desc &md = c->md;
    const int d = md.d_model, H = md.n_heads, Hkv = md.n_kv_heads, hd = c->hd;
    hipStream_t st = c->stream;
    SJD_LAUNCH(c, KC_EMBED, after([&] { embed_kernel<float><<<fr.M, 256, 0, st>>>((const float *)c->tok_emb, fr.rm.row_tok, c->x, d, fr.stage); }));
    F32Args a{};
    a.M = fr.M;
    a.eps = md.rms_eps;
    a.rm = fr.rm;
    a.rope_cos = c->rope_cos; a.rope_sin = c->rope_sin;
    a.q_out = (float *)c->q;
    a.L = fr.L; a.H = H; a.Hkv = Hkv; a.hd = hd;
    // a projection behind a norm whose element-wise steps run on their own: the norm here, the product into `out`
    auto apart = [&](int cls, const void *W, int N, const float *gain, float *out) -> int {
        SJD_LAUNCH(c, KC_ADDNORM, after([&] { addnorm_kernel<float><<<fr.M, 256, 0, st>>>(c->x, nullptr, 0, fr.M, gain, (float *)c->xn, d, md.rms_eps); }));
        int splits;
        return run_gemm<float>(c, cls, (const float *)c->xn, (const float *)W, out, fr.M, N, d, 1, &splits);
    };
    auto gemm = [&](auto epi, int cls, const void *A, const void *W, int N, int K, const float *gain, float *out) -> int {
        a.N = N; a.K = K; a.gain = gain; a.out = out;
        SJD_LAUNCH(c, cls, launch_gemm_f32<decltype(epi)::value>(st, (const float *)A, (const float *)W, a));
        return SJD_OK;
    };
    constexpr std::integral_constant<int, F32_QKV> kQkv{};
    constexpr std::integral_constant<int, F32_RESID> kResid{};
    constexpr std::integral_constant<int, F32_SWIGLU> kSwiglu{};
    constexpr std::integral_constant<int, F32_LOGITS> kLogits{};
    for (int l = 0; l < md.n_layers; ++l) {
        const LayerWeights &lw = c->layers[l];
        KvPool &pool = a.pool;
        pool.k = (char *)c->kpool + c->pool_layer_bytes * l;
        pool.v = (char *)c->vpool + c->pool_layer_bytes * l;
        pool.page_table = c->page_table;
        pool.pages_per_seg = c->pps;
        pool.page_tokens = c->pt;
        const int n_qkv = (H + 2 * Hkv) * hd;
        int rc;
        if (f32_inside(fr.M, n_qkv, F32_QKV_INSIDE)) {
            if ((rc = gemm(kQkv, KC_GEMM_QKV, c->x, lw.wqkv, n_qkv, d, lw.attn_norm, nullptr))) return rc;
        } else {
            if ((rc = apart(KC_GEMM_QKV, lw.wqkv, n_qkv, lw.attn_norm, c->partial))) return rc;
            SJD_LAUNCH(c, KC_ROPE_KV, after([&] {
                           rope_kv_kernel<float><<<fr.M, 256, 0, st>>>(c->partial, 1, fr.M, fr.rm, c->rope_cos, c->rope_sin, (float *)c->q, pool, fr.L, H,
                                                                       Hkv, hd);
                       }));
        }
        if (!with_head && l + 1 == md.n_layers) return SJD_OK;
        if ((rc = run_attention<float>(c, pool, fr))) return rc;
        if ((rc = gemm(kResid, KC_GEMM_O, c->attn, lw.wo, d, H * hd, nullptr, c->x))) return rc;
        if (f32_inside(fr.M, 2 * md.d_ff, F32_GATE_UP_INSIDE)) {
            if ((rc = gemm(kSwiglu, KC_GEMM_GATEUP, c->x, lw.wgu, 2 * md.d_ff, d, lw.mlp_norm, (float *)c->h))) return rc;
        } else {
            if ((rc = apart(KC_GEMM_GATEUP, lw.wgu, 2 * md.d_ff, lw.mlp_norm, c->partial))) return rc;
            SJD_LAUNCH(c, KC_SWIGLU, after([&] { swiglu_kernel<float><<<fr.M, 256, 0, st>>>(c->partial, 1, fr.M, (float *)c->h, md.d_ff); }));
        }
        if ((rc = gemm(kResid, KC_GEMM_DOWN, c->h, lw.wdown, d, md.d_ff, nullptr, c->x))) return rc;
    }
    if (!with_head) return SJD_OK;
    if (!f32_inside(fr.M, c->Vs, F32_HEAD_INSIDE)) return apart(KC_GEMM_HEAD, c->lm_head, c->Vs, c->final_norm, c->logits);
    return gemm(kLogits, KC_GEMM_HEAD, c->x, c->lm_head, c->Vs, d, c->final_norm, c->logits);
}

// Small-M bf16 path: five kernels per layer (QKV+RoPE+KV write, attention, out+residual, gate/up+SwiGLU,
// down+residual); c->xn holds the bf16 copy of the residual stream.
int forward_fused(sjd_ctx *c, const FwdRows &fr, bool with_head) {
    const sjd_model_desc &md = c->md;
    const int M = fr.M, d = md.d_model, H = md.n_heads, Hkv = md.n_kv_heads, hd = c->hd, F = md.d_ff;
    // up to 64 rows: one row group; more: row groups of 64 over the same weights, the last one as ragged as it comes (the
    // activation buffers hold whole groups; rows past M are computed from whatever they hold and never stored)
    const int m_groups = ceil_div(M, 64);
    const int MT = M <= 64 ? ceil_div(M, 32) : 2;
    const int n_cus = c->n_cus;
    hipStream_t st = c->stream;
    SJD_LAUNCH(c, KC_EMBED, after([&] {
                   RowTables rt;
                   rt.rm = fr.rm; rt.rope_cos = c->rope_cos; rt.rope_sin = c->rope_sin;
                   rt.page_table = c->page_table; rt.pages_per_seg = c->pps; rt.page_tokens = c->pt;
                   rt.L = fr.L; rt.H = H; rt.hd = hd; rt.meta = c->row_meta; rt.rot = c->row_rot;
                   rt.ssq_part = c->row_ssq;
                   rt.gain = c->layers[0].attn_norm;
                   rt.stage = fr.stage;
                   embed_dual_kernel<<<M, 256, 0, st>>>((const bf16_t *)c->tok_emb, c->x, (bf16_t *)c->xn, d, rt);
               }));
    SkinnyArgs a;
    memset(&a, 0, sizeof a);
    a.M = M;
    a.n_cus = n_cus;
    a.m_groups = m_groups;
    a.eps = md.rms_eps;
    a.row_meta = c->row_meta;
    a.k_rot = (md.kernel_flags & SJD_NO_K_ROTATION) ? 0 : 1;
    a.row_rot = c->row_rot;
    a.q_out = (bf16_t *)c->q;
    a.H = H; a.Hkv = Hkv; a.hd = hd; a.F = F;
    a.x = c->x;
    a.xb = (bf16_t *)c->xn;
    a.h = (bf16_t *)c->h;
    a.logits = c->logits;
    const int nbw_d = resid_nbw(d);
    a.part = c->skinny_part;
    auto whole_k = [&]() { a.ksplit = 1; a.kb_per_split = a.KB; };
    auto no_room = [&]() { sjd_set_error(c->err, "split-K workspace too small"); return SJD_EINVAL; };
    // Wavefronts per workgroup, measured: 8 pull a workgroup's share through the CU's L1 faster than 4 and halve
    // the epilogue's elements per thread; once a launch fills most CUs with weights that come from HBM (the 7B
    // shapes' gate/up and head) a CU's outstanding misses are the limit either way, the second wavefront of a SIMD
    // only queues behind the first, and 4 win by the cheaper LDS reduction.
    auto nw_for = [](int groups) { return groups >= 200 ? 4 : 8; };
    const bool want_z = c->z && !(md.kernel_flags & SJD_NO_HEAD_FUSION);
    const ForwardPlan plan = forward_plan(c->shape, M, want_z && fr.L == 32);
    const bool tile = plan.tile;
    // output / down projection: x += A W^T.  One kernel when a workgroup's share is small, else K split over
    // grid.y with the partial sums added by resid_reduce_kernel after the kernel boundary.
    // Launches of row groups and LDS tiles touch the weights of the projection behind them (touch, plans.h).
    struct Proj { const void *W; Slabs slabs; };
    const int groups_d = ceil_div(ceil_div(d, 32), nbw_d), groups_qkv = (H + 2 * Hkv) * (hd / 64);
    // More than 32 rows and so few column groups that a workgroup per group and 32-row tile still finds a CU of its
    // own: row groups of 32 rows instead of 64 (all row groups of a column group on one XCD, whose L2 serves the
    // later readers of the weights).  Each workgroup pulls half the activations, twice as many CUs work.
    auto rows2_for = [&](int groups) { return rows_of_32(c->shape, M, groups); };
    auto proj_of = [&](const void *W, int n_blocks, int KB, int nbw, const ProjPlan &p) { return Proj{W, slabs_of(p, n_blocks, KB, nbw)}; };
    const int groups_v = c->shape.head_groups();
    const ProjPlan &plan_qkv = plan.qkv, &plan_o = plan.o, &plan_gu = plan.gate_up, &plan_down = plan.down, &plan_head = plan.head;
    auto warm = [&](int cur_wgs, double cur_us, const Proj &nx) {
        a.pf_wgs = 0;
        if (!c->l2_warm || tile || !nx.W) return;
        const Touch t = touch(c->shape, M, cur_wgs, cur_us, nx.slabs);
        if (!t.wgs) return;
        a.pf_base = (const char *)nx.W; a.pf_slab_bytes = (uint32_t)nx.slabs.nbw * nx.slabs.KB * 1024; a.pf_groups = t.slabs; a.pf_wgs = t.wgs; a.pf_sink = c->pf_sink;
    };
    // The same for the keys and values of the next one-pass attention launch (one workgroup per (head, segment), in
    // that order); call after warm(): takes what is left of the CUs.
    auto warm_kv = [&](int cur_groups, const KvPool &pool) {
        a.kv_wgs = 0;
        if (!c->l2_warm || tile || m_groups > 1 || !c->attn_mfma || !c->attn_onepass || fr.L < 1 || fr.L > 32) return;
        const size_t kv_bytes = (size_t)fr.n_segs * Hkv * md.max_ctx * hd * 2 * sizeof(bf16_t);
        const int room = (n_cus - cur_groups - a.pf_wgs) / 8 * 8;
        a.kv_wgs = std::max(0, std::min(room, (int)((kv_bytes / (48 << 10) + 7) / 8 * 8)));
        a.kv_pairs = fr.n_segs * H;
        a.kv_seg_kv = fr.rm.seg_kv;
        a.kv_pool = pool;
        a.pf_sink = c->pf_sink;
    };
    const Proj none = {nullptr, {}};
    const bool mixed_ok = !(md.kernel_flags & SJD_NO_MIXED_WIDTH);
    // LDS-tile and tile kernels (and row groups with the gains in the rows) take the RMSNorm row sums of squares from the kernel
    // that wrote the residual stream: embedding gather, whole-K output / down projection or split-K reduction
    const int tile_rows = (md.kernel_flags & SJD_TILES_256_ROWS) ? 256 : 0;  // 0: chosen per launch
    int ssq_n = 1;   // partial sums per row that the last writer left; the embedding kernel wrote one
    float *ssq_out = nullptr;   // where the coming output / down projection leaves them: set if its reader takes them (tile kernels: always)
    auto use_ssq = [&]() { a.row_ssq_part = c->row_ssq; a.row_ssq_n = ssq_n; };
    auto takes_ssq = [&](const ProjPlan &p) { return p.tile || p.lds >= 0 || !c->fold_gain; };
    // The row-group kernels sum the squares of their operands, which are the stream only while the gains are in the weights
    auto skinny_ssq = [&]() { if (!c->fold_gain) use_ssq(); };
    auto reduce = [&]() -> int {
        SJD_LAUNCH(c, KC_ADDNORM, after([&] {
                       const int grid = reduce_grid(M, d);
                       if (a.gain) resid_reduce_kernel<true><<<grid, 256, 0, st>>>(c->skinny_part, a.ksplit, M, d, c->x, (bf16_t *)c->xn, ssq_out, a.gain);
                       else resid_reduce_kernel<false><<<grid, 256, 0, st>>>(c->skinny_part, a.ksplit, M, d, c->x, (bf16_t *)c->xn, ssq_out, nullptr);
                   }));
        ssq_n = ceil_div(d, 256);
        return SJD_OK;
    };
    auto resid = [&](int cls, const void *A, const void *W, int K, const ProjPlan &plan, const Proj &nx, const KvPool *kv_next) -> int {
        a.A = (const bf16_t *)A; a.W = (const bf16_t *)W; a.KB = K / 16; a.N = d;
        a.pf_wgs = 0;
        a.row_ssq_part = nullptr;
        a.ssq_out = ssq_out;
        if (plan.lds >= 0) {
            const int nb = ceil_div(d, 32);
            a.kb_per_split = ceil_div(a.KB, 2 * plan.ks) * 2;
            a.ksplit = ceil_div(a.KB, a.kb_per_split);
            if (a.ksplit == 1) {
                ssq_n = ceil_div(nb, lds_tile(plan.lds).cb);
                warm(lds_wgs(plan.lds, M, nb), plan.us, nx);
                SJD_LAUNCH(c, cls, launch_lds<EPI_RESID>(st, a, nb, plan.lds));
                a.pf_wgs = 0;
                return SJD_OK;
            }
            if ((size_t)a.ksplit * M * d > c->skinny_part_elems) return no_room();
            SJD_LAUNCH(c, cls, launch_lds<EPI_PARTIAL>(st, a, nb, plan.lds));
            return reduce();
        }
        if (plan.tile) {
            const int n_blocks = ceil_div(d, 64) * 2;
            a.ksplit = plan.ks;
            a.kb_per_split = ceil_div(a.KB, a.ksplit);
            if (a.ksplit == 1) {
                a.ssq_out = c->row_ssq;   // also where the reader sums for itself: the kernel always leaves them
                ssq_n = ceil_div(n_blocks, 4);
                SJD_LAUNCH(c, cls, launch_tile<EPI_RESID>(st, a, n_blocks, tile_rows, mixed_ok));
                return SJD_OK;
            }
            if ((size_t)a.ksplit * M * d > c->skinny_part_elems) return no_room();
            SJD_LAUNCH(c, cls, launch_tile<EPI_PARTIAL>(st, a, n_blocks, tile_rows, mixed_ok));
            return reduce();
        }
        const int groups = ceil_div(ceil_div(d, 32), nbw_d);
        if (plan.ks == 1) {
            whole_k();
            // (few rows: no weights are touched ahead, kernels_few.hip.h)
            if (const int rt = nbw_d == 1 ? few_rows(c->shape, M, groups) : 0) {
                if (kv_next) warm_kv(few_wgs(M, groups, rt), *kv_next);
                ssq_n = 2 * groups;
                SJD_LAUNCH(c, cls, launch_few<EPI_RESID>(st, a, rt, groups));
                a.kv_wgs = 0;
                return SJD_OK;
            }
            const bool r2 = rows2_for(groups);
            a.m_groups = r2 ? 2 * m_groups : m_groups;
            const int n_compute = row_group_wgs(M, groups, r2);
            warm(n_compute, plan.us, nx);
            if (kv_next) warm_kv(n_compute, *kv_next);
            ssq_n = groups;
            SJD_LAUNCH(c, cls, launch_skinny<EPI_RESID>(st, a, r2 ? 1 : MT, groups, nbw_d, nw_for(groups)));
            a.pf_wgs = a.kv_wgs = 0;
            a.m_groups = m_groups;
            return SJD_OK;
        }
        a.ksplit = plan.ks;
        a.kb_per_split = ceil_div(a.KB, a.ksplit);
        if ((size_t)a.ksplit * M * d > c->skinny_part_elems) return no_room();
        SJD_LAUNCH(c, cls, launch_skinny<EPI_PARTIAL>(st, a, MT, groups, nbw_d, nw_for(groups * a.ksplit)));
        return reduce();
    };
    const Proj proj_o0 = proj_of(nullptr, groups_d * nbw_d, H * hd / 16, nbw_d, plan_o), proj_down0 = proj_of(nullptr, groups_d * nbw_d, F / 16, nbw_d, plan_down);
    auto with_w = [](Proj p, const void *W) { p.W = W; return p; };
    for (int l = 0; l < md.n_layers; ++l) {
        const LayerWeights &lw = c->layers[l];
        KvPool pool;
        pool.k = (char *)c->kpool + c->pool_layer_bytes * l;
        pool.v = (char *)c->vpool + c->pool_layer_bytes * l;
        pool.page_table = c->page_table;
        pool.pages_per_seg = c->pps;
        pool.page_tokens = c->pt;
        a.pool = pool;
        a.A = (const bf16_t *)c->xn; a.W = (const bf16_t *)lw.wqkv; a.KB = d / 16;
        if (plan_qkv.tile) {
            whole_k();
            use_ssq();
            SJD_LAUNCH(c, KC_GEMM_QKV, launch_tile<EPI_QKV>(st, a, (H + 2 * Hkv) * (hd / 64) * 2, tile_rows, mixed_ok));
        } else if (plan_qkv.lds >= 0) {
            whole_k();
            use_ssq();
            warm(lds_wgs(plan_qkv.lds, M, groups_qkv * 2), plan_qkv.us, with_head || l + 1 < md.n_layers ? with_w(proj_o0, lw.wo) : none);
            SJD_LAUNCH(c, KC_GEMM_QKV, launch_lds<EPI_QKV>(st, a, groups_qkv * 2, plan_qkv.lds));
            a.pf_wgs = 0;
        } else if (const int rt = few_rows(c->shape, M, groups_qkv)) {
            whole_k();
            skinny_ssq();
            if (l == 0) warm_kv(few_wgs(M, groups_qkv, rt), pool);
            SJD_LAUNCH(c, KC_GEMM_QKV, launch_few<EPI_QKV>(st, a, rt, groups_qkv));
            a.kv_wgs = 0;
        } else {
            whole_k();
            skinny_ssq();
            const bool r2 = rows2_for(groups_qkv);
            a.m_groups = r2 ? 2 * m_groups : m_groups;
            const int n_compute = row_group_wgs(M, groups_qkv, r2);
            warm(n_compute, plan_qkv.us, with_head || l + 1 < md.n_layers ? with_w(proj_o0, lw.wo) : none);
            if (l == 0) warm_kv(n_compute, pool);  // later layers: requested by the down projection before them
            SJD_LAUNCH(c, KC_GEMM_QKV, launch_skinny<EPI_QKV>(st, a, r2 ? 1 : MT, groups_qkv, 2, nw_for(groups_qkv)));
            a.pf_wgs = a.kv_wgs = 0;
            a.m_groups = m_groups;
        }
        if (!with_head && l + 1 == md.n_layers) return SJD_OK;
        { int rc = run_attention<bf16_t>(c, pool, fr); if (rc) return rc; }
        ssq_out = takes_ssq(plan_gu) ? c->row_ssq : nullptr;
        a.gain = lw.mlp_norm;
        { int rc = resid(KC_GEMM_O, c->attn, lw.wo, H * hd, plan_o, proj_of(lw.wgu, F / 32 * 2, d / 16, 2, plan_gu), nullptr); if (rc) return rc; }
        a.A = (const bf16_t *)c->xn; a.W = (const bf16_t *)lw.wgu; a.KB = d / 16;
        if (plan_gu.tile) {
            whole_k();
            use_ssq();
            SJD_LAUNCH(c, KC_GEMM_GATEUP, launch_tile<EPI_SWIGLU>(st, a, F / 32 * 2, tile_rows, mixed_ok));
        } else if (plan_gu.lds >= 0) {
            whole_k();
            use_ssq();
            warm(lds_wgs(plan_gu.lds, M, F / 32 * 2), plan_gu.us, with_w(proj_down0, lw.wdown));
            SJD_LAUNCH(c, KC_GEMM_GATEUP, launch_lds<EPI_SWIGLU>(st, a, F / 32 * 2, plan_gu.lds));
            a.pf_wgs = 0;
        } else if (const int rt = few_rows(c->shape, M, F / 32)) {
            whole_k();
            skinny_ssq();
            SJD_LAUNCH(c, KC_GEMM_GATEUP, launch_few<EPI_SWIGLU>(st, a, rt, F / 32));
        } else {
            whole_k();
            skinny_ssq();
            const bool r2 = rows2_for(F / 32);
            a.m_groups = r2 ? 2 * m_groups : m_groups;
            const int n_compute = row_group_wgs(M, F / 32, r2);
            warm(n_compute, plan_gu.us, with_w(proj_down0, lw.wdown));
            if (mixed_ok && skinny_mixed_applies(a, F / 32, 2, nw_for(F / 32))) SJD_LAUNCH(c, KC_GEMM_GATEUP, launch_skinny_mixed<EPI_SWIGLU>(st, a, MT, F / 32));
            else SJD_LAUNCH(c, KC_GEMM_GATEUP, launch_skinny<EPI_SWIGLU>(st, a, r2 ? 1 : MT, F / 32, 2, nw_for(F / 32)));
            a.pf_wgs = 0;
            a.m_groups = m_groups;
        }
        const Proj after_down = l + 1 < md.n_layers ? proj_of(c->layers[l + 1].wqkv, groups_qkv * 2, d / 16, 2, plan_qkv)
                                : with_head         ? proj_of(c->lm_head, groups_v * 2, d / 16, 2, plan_head)
                                                    : none;
        KvPool pool_next = pool;
        pool_next.k = (char *)c->kpool + c->pool_layer_bytes * (l + 1);
        pool_next.v = (char *)c->vpool + c->pool_layer_bytes * (l + 1);
        ssq_out = takes_ssq(l + 1 < md.n_layers ? plan_qkv : plan_head) ? c->row_ssq : nullptr;
        a.gain = l + 1 < md.n_layers ? c->layers[l + 1].attn_norm : c->final_norm;
        { int rc = resid(KC_GEMM_DOWN, c->h, lw.wdown, F, plan_down, after_down, l + 1 < md.n_layers ? &pool_next : nullptr); if (rc) return rc; }
    }
    if (with_head) {
        a.A = (const bf16_t *)c->xn; a.W = (const bf16_t *)c->lm_head; a.KB = d / 16; a.N = c->Vs;
        // Guidance fused into the head where a position's conditional and unconditional rows meet in one thread of the
        // epilogue: windows of 32 (row tiles alternate conditional / unconditional) and one sequence with a window of 16
        const bool head_mixed = !tile && mixed_ok && skinny_mixed_applies(a, groups_v, 2, nw_for(groups_v));
        const bool head_r2 = !tile && !head_mixed && rows2_for(groups_v);
        int z_mode = 0;
        if (want_z) {
            if (c->L == 32 && (tile || plan_head.lds >= 0 || (MT == 2 && !head_r2))) z_mode = 1;
            else if (c->L == 16 && M == 32 && !tile) z_mode = 2;
        }
        a.z_out = c->z; a.z_mode = z_mode; a.cfg_scale = c->sp.cfg_scale; a.inv_t = c->sp.inv_temperature;
        a.logits = z_mode == 0 || c->keep_logits ? c->logits : nullptr;
        c->z_used = z_mode != 0;
        if (tile) {
            whole_k();
            use_ssq();
            SJD_LAUNCH(c, KC_GEMM_HEAD, launch_tile<EPI_HEAD>(st, a, ceil_div(c->Vs, 64) * 2, z_mode ? 256 : tile_rows));
        } else if (plan_head.lds >= 0) {
            whole_k();
            use_ssq();
            SJD_LAUNCH(c, KC_GEMM_HEAD, launch_lds<EPI_HEAD>(st, a, groups_v * 2, plan_head.lds));
        } else {
            whole_k();
            skinny_ssq();
            if (head_mixed) SJD_LAUNCH(c, KC_GEMM_HEAD, launch_skinny_mixed<EPI_HEAD>(st, a, MT, groups_v));
            else {
                const bool r2 = head_r2;
                a.m_groups = r2 ? 2 * m_groups : m_groups;
                SJD_LAUNCH(c, KC_GEMM_HEAD, launch_skinny<EPI_HEAD>(st, a, r2 ? 1 : MT, groups_v, 2, nw_for(groups_v)));
                a.m_groups = m_groups;
            }
        }
    }
    return SJD_OK;
}

int forward_any(sjd_ctx *c, const FwdRows &fr, bool with_head) {
    if (c->fused) return forward_fused(c, fr, with_head);
    if (c->md.dtype == SJD_F32) return c->md.kernel_flags & SJD_KERNELS_REFERENCE ? forward<float>(c, fr, with_head) : forward_f32(c, fr, with_head);
    return forward<bf16_t>(c, fr, with_head);
}

// ------------------------------------------------------------------------------------------ create
template <typename T> int copy_weights(sjd_ctx *c, const sjd_weights *w) {
    const sjd_model_desc &md = c->md;
    const int d = md.d_model, H = md.n_heads, Hkv = md.n_kv_heads, hd = c->hd, F = md.d_ff;
    hipStream_t st = c->stream;
    int rc;
    T *emb;
    if ((rc = dev_alloc(c, &emb, (size_t)md.vocab * d * sizeof(T), false))) return rc;
    SJD_HIP_TRY(c->err, hipMemcpyAsync(emb, w->tok_emb, (size_t)md.vocab * d * sizeof(T), hipMemcpyDeviceToDevice, st));
    c->tok_emb = emb;
    auto gain = [&](const void *src, float **dst) -> int {
        int r = dev_alloc(c, dst, (size_t)d * sizeof(float));
        if (r) return r;
        to_float_kernel<T><<<ceil_div(d, 256), 256, 0, st>>>((const T *)src, *dst, d);
        return hipGetLastError() == hipSuccess ? SJD_OK : SJD_EDEVICE;
    };
    auto pack = [&](T *dst, const void *src, int N, int K, int row0) -> int {
        if (!src) { sjd_set_error(c->err, "null weight pointer"); return SJD_EINVAL; }
        pack_weight_kernel<T><<<1024, 256, 0, st>>>((const T *)src, dst, N, K, row0);
        return hipGetLastError() == hipSuccess ? SJD_OK : SJD_EDEVICE;
    };
    if ((rc = gain(w->final_norm, &c->final_norm))) return rc;
    T *head;
    if ((rc = dev_alloc(c, &head, Layout<T>::w_elems(c->Vs, d) * sizeof(T)))) return rc;
    if ((rc = pack(head, (const T *)w->lm_head + (size_t)md.sample_lo * d, c->Vs, d, 0))) return rc;
    c->lm_head = head;
    c->layers.resize(md.n_layers);
    for (int l = 0; l < md.n_layers; ++l) {
        LayerWeights &lw = c->layers[l];
        if (!w->attn_norm[l] || !w->mlp_norm[l]) { sjd_set_error(c->err, "null weight pointer"); return SJD_EINVAL; }
        if ((rc = gain(w->attn_norm[l], &lw.attn_norm))) return rc;
        if ((rc = gain(w->mlp_norm[l], &lw.mlp_norm))) return rc;
        T *qkv, *o, *gu, *down;
        const int Nqkv = (H + 2 * Hkv) * hd;
        if ((rc = dev_alloc(c, &qkv, Layout<T>::w_elems(Nqkv, d) * sizeof(T)))) return rc;
        if ((rc = pack(qkv, w->wq[l], H * hd, d, 0))) return rc;
        if ((rc = pack(qkv, w->wk[l], Hkv * hd, d, H * hd))) return rc;
        if ((rc = pack(qkv, w->wv[l], Hkv * hd, d, (H + Hkv) * hd))) return rc;
        if ((rc = dev_alloc(c, &o, Layout<T>::w_elems(d, H * hd) * sizeof(T)))) return rc;
        if ((rc = pack(o, w->wo[l], d, H * hd, 0))) return rc;
        if ((rc = dev_alloc(c, &gu, Layout<T>::w_elems(2 * F, d) * sizeof(T)))) return rc;
        if ((rc = pack(gu, w->w_gate[l], F, d, 0))) return rc;
        if ((rc = pack(gu, w->w_up[l], F, d, F))) return rc;
        if ((rc = dev_alloc(c, &down, Layout<T>::w_elems(d, F) * sizeof(T)))) return rc;
        if ((rc = pack(down, w->w_down[l], d, F, 0))) return rc;
        lw.wqkv = qkv; lw.wo = o; lw.wgu = gu; lw.wdown = down;
    }
    return SJD_OK;
}

// Weights of the fused path: gains folded in or kept beside (the context's pointers to them stay NULL where they are in the
// weights), QKV rows in (head, rotary pair) order, gate and up interleaved by blocks of 32.
int copy_weights_fused(sjd_ctx *c, const sjd_weights *w) {
    typedef bf16_t T;
    const sjd_model_desc &md = c->md;
    const int d = md.d_model, H = md.n_heads, Hkv = md.n_kv_heads, hd = c->hd, F = md.d_ff;
    hipStream_t st = c->stream;
    int rc;
    T *emb;
    if ((rc = dev_alloc(c, &emb, (size_t)md.vocab * d * sizeof(T), false))) return rc;
    SJD_HIP_TRY(c->err, hipMemcpyAsync(emb, w->tok_emb, (size_t)md.vocab * d * sizeof(T), hipMemcpyDeviceToDevice, st));
    c->tok_emb = emb;
    float *gain;  // scratch, reused per matrix (stream order keeps it safe)
    if ((rc = dev_alloc(c, &gain, (size_t)d * sizeof(float)))) return rc;
    auto pack = [&](T *dst, const void *s0, const void *s1, const void *s2, int n0, int n1, int N, int K, const void *g,
                    PackMap pm) -> int {
        if (!s0 || (n0 < N && !s1) || (n1 < N && !s2)) { sjd_set_error(c->err, "null weight pointer"); return SJD_EINVAL; }
        const bool fold = g && c->fold_gain;
        if (fold) to_float_kernel<T><<<ceil_div(K, 256), 256, 0, st>>>((const T *)g, gain, K);
        pack_weight_fused_kernel<<<2048, 256, 0, st>>>((const T *)s0, (const T *)s1, (const T *)s2, n0, n1, fold ? gain : nullptr, dst,
                                                       N, K, pm);
        return hipGetLastError() == hipSuccess ? SJD_OK : SJD_EDEVICE;
    };
    float *gains = nullptr;   // final, then attention and MLP norm of every layer
    if (!c->fold_gain && (rc = dev_alloc(c, &gains, (size_t)d * (1 + 2 * md.n_layers) * sizeof(float), false))) return rc;
    auto keep_gain = [&](const void *src, float **dst) -> int {
        if (c->fold_gain) return SJD_OK;
        to_float_kernel<T><<<ceil_div(d, 256), 256, 0, st>>>((const T *)src, gains, d);
        *dst = gains;
        gains += d;
        return hipGetLastError() == hipSuccess ? SJD_OK : SJD_EDEVICE;
    };
    const PackMap ident{0, hd, F}, qkvmap{1, hd, F}, gumap{2, hd, F};
    if ((rc = keep_gain(w->final_norm, &c->final_norm))) return rc;
    T *head;
    if ((rc = dev_alloc(c, &head, Layout<T>::w_elems(ceil_div(c->Vs, 64) * 64, d) * sizeof(T)))) return rc;
    if ((rc = pack(head, (const T *)w->lm_head + (size_t)md.sample_lo * d, nullptr, nullptr, c->Vs, c->Vs, c->Vs, d, w->final_norm, ident)))
        return rc;
    c->lm_head = head;
    c->layers.resize(md.n_layers);
    const int Nqkv = (H + 2 * Hkv) * hd, dpad = ceil_div(d, 64) * 64;
    for (int l = 0; l < md.n_layers; ++l) {
        LayerWeights &lw = c->layers[l];
        if (!w->attn_norm[l] || !w->mlp_norm[l]) { sjd_set_error(c->err, "null weight pointer"); return SJD_EINVAL; }
        if ((rc = keep_gain(w->attn_norm[l], &lw.attn_norm)) || (rc = keep_gain(w->mlp_norm[l], &lw.mlp_norm))) return rc;
        T *qkv, *o, *gu, *down;
        if ((rc = dev_alloc(c, &qkv, Layout<T>::w_elems(Nqkv, d) * sizeof(T)))) return rc;
        if ((rc = pack(qkv, w->wq[l], w->wk[l], w->wv[l], H * hd, (H + Hkv) * hd, Nqkv, d, w->attn_norm[l], qkvmap))) return rc;
        if ((rc = dev_alloc(c, &o, Layout<T>::w_elems(dpad, H * hd) * sizeof(T)))) return rc;
        if ((rc = pack(o, w->wo[l], nullptr, nullptr, d, d, d, H * hd, nullptr, ident))) return rc;
        if ((rc = dev_alloc(c, &gu, Layout<T>::w_elems(2 * F, d) * sizeof(T)))) return rc;
        if ((rc = pack(gu, w->w_gate[l], w->w_up[l], nullptr, F, 2 * F, 2 * F, d, w->mlp_norm[l], gumap))) return rc;
        if ((rc = dev_alloc(c, &down, Layout<T>::w_elems(dpad, F) * sizeof(T)))) return rc;
        if ((rc = pack(down, w->w_down[l], nullptr, nullptr, d, d, d, F, nullptr, ident))) return rc;
        lw.wqkv = qkv; lw.wo = o; lw.wgu = gu; lw.wdown = down;
    }
    return SJD_OK;
}

template <typename T> int alloc_buffers(sjd_ctx *c) {
    const sjd_model_desc &md = c->md;
    const int S = c->S, L = c->L, d = md.d_model, H = md.n_heads, Hkv = md.n_kv_heads, hd = c->hd, F = md.d_ff;
    const int Nqkv = (H + 2 * Hkv) * hd;
    int rc;
    // Rows of a forward: S * 2 windows, or as much of the prompts as one prefill forward takes (whole 32-row tiles)
    const size_t prompt_rows = (size_t)S * 2 * (md.max_ctx - 1);
    c->pre_rows = (int)std::min<size_t>(c->fused ? kPrefillRows : kPrefillRowsGeneric, (prompt_rows + 31) / 32 * 32);
    const int M = c->max_rows = std::max(S * 2 * L, c->pre_rows);
    // KV pages
    c->pps = ceil_div(md.max_ctx, c->pt);
    c->n_pages = S * 2 * c->pps;
    c->pool_layer_bytes = (size_t)c->n_pages * Hkv * c->pt * hd * sizeof(T);
    if ((rc = dev_alloc(c, &c->kpool, c->pool_layer_bytes * md.n_layers))) return rc;
    if ((rc = dev_alloc(c, &c->vpool, c->pool_layer_bytes * md.n_layers))) return rc;
    const size_t packed = 3 * prompt_rows + (prompt_rows / c->pre_rows + 1) * 8 * (size_t)S;
    const size_t windows = md.kernel_flags & SJD_ATTENTION_CHUNKED ? (size_t)ceil_div(md.max_ctx - 1, L) * 4 * S * (L + 1) : 0;
    c->pre_elems = (size_t)S * 2 * c->pps + 5 * (size_t)S + std::max(packed, windows);
    if ((rc = dev_alloc(c, &c->pre_dev, c->pre_elems * sizeof(int32_t)))) return rc;
    c->page_table = c->pre_dev;
    // workspaces
    if ((rc = dev_alloc(c, &c->x, (size_t)M * d * sizeof(float)))) return rc;
    const bool generic = !c->fused && (md.dtype == SJD_BF16 || (md.kernel_flags & SJD_KERNELS_REFERENCE));
    const bool f32_apart = md.dtype == SJD_F32 && !(f32_inside(M, Nqkv, F32_QKV_INSIDE) && f32_inside(M, 2 * F, F32_GATE_UP_INSIDE));
    if (generic || f32_apart) {   // the generic path's GEMM outputs, with their K splits
        const int shapes[4][2] = {{Nqkv, d}, {d, H * hd}, {2 * F, d}, {d, F}};
        for (auto &s : shapes) {
            size_t need = (size_t)M * s[0];
            if (md.dtype == SJD_BF16 && !(md.kernel_flags & SJD_KERNELS_REFERENCE)) {
                // worst case over the number of sequences actually decoded (M = n * 2 * L) and the rows of a prefill forward
                // (the plan of M rows is that of its 32-row tiles)
                auto cover = [&](int m) {
                    GemmPlan p = plan_gemm_bf16(m, s[0], s[1], 0);
                    need = std::max(need, (size_t)p.splits * m * s[0]);
                };
                for (int n = 1; n <= S; ++n) cover(n * 2 * L);
                for (int m = 32; m <= c->pre_rows; m += 32) cover(m);
            }
            c->partial_elems = std::max(c->partial_elems, need);
        }
        if ((rc = dev_alloc(c, &c->partial, c->partial_elems * sizeof(float)))) return rc;
    }
    if ((rc = dev_alloc(c, &c->logits, (size_t)S * 2 * L * c->Vs * sizeof(float)))) return rc;
    const int Mpad = ceil_div(M, 64) * 64;   // whole 64-row groups: the row-group projections read every row of the last one
    if ((c->fused || generic || f32_apart || !f32_inside(S * 2 * L, c->Vs, F32_HEAD_INSIDE)) &&
        (rc = dev_alloc(c, &c->xn, Layout<T>::a_elems(Mpad, d) * sizeof(T)))) return rc;
    if ((rc = dev_alloc(c, &c->attn, Layout<T>::a_elems(Mpad, H * hd) * sizeof(T)))) return rc;
    if ((rc = dev_alloc(c, &c->h, Layout<T>::a_elems(Mpad, F) * sizeof(T)))) return rc;
    // queries: 32-row tiles of one segment each (packed segments leave a ragged tile each at most)
    const size_t q_tiles = std::max((size_t)S * 2 * ceil_div(L, 32), (size_t)c->pre_rows / 32 + 2 * (size_t)S);
    if ((rc = dev_alloc(c, &c->q, q_tiles * H * 32 * hd * sizeof(T)))) return rc;
    if (c->fused) {
        if ((rc = dev_alloc(c, &c->z, (size_t)S * L * c->Vs * sizeof(float)))) return rc;
        // partial sums of the output and down projections where they split K, over the rows a step or a prefill forward can have
        auto cover = [&](int m) {
            for (int K : {H * hd, F}) {
                const int ks = max_splits(c->shape, m, K);
                if (ks > 1) c->skinny_part_elems = std::max(c->skinny_part_elems, (size_t)ks * m * d);
            }
        };
        for (int n = 1; n <= S; ++n) cover(n * 2 * L);
        for (int m = 1; m <= c->pre_rows; ++m) cover(m);
        if ((rc = dev_alloc(c, &c->skinny_part, c->skinny_part_elems * sizeof(float)))) return rc;
        if ((rc = dev_alloc(c, &c->pf_sink, 256))) return rc;
        if ((rc = dev_alloc(c, &c->row_ssq, (size_t)std::max(M, 128) * ceil_div(d, 32) * sizeof(float)))) return rc;
        if ((rc = dev_alloc(c, &c->row_meta, (size_t)M * sizeof(QkvRow)))) return rc;
        if ((rc = dev_alloc(c, &c->row_rot, (size_t)M * (hd / 2) * sizeof(float2)))) return rc;
        c->l2_warm = !(md.kernel_flags & SJD_NO_L2_WARM);
    }
    if (c->attn_mfma) {
        // chunk length: about 640 wavefronts at full context (measured: every chunk costs a partial result of
        // 32 x hd floats per head, written and read back, which at 128-token chunks is as many bytes as the keys and
        // values themselves; fewer, longer chunks win until the workgroups no longer fill the chip), at least 128
        // tokens, a multiple of 64
        long want = (long)md.max_ctx * S * 2 * H * ceil_div(L, 32) / 640;
        int chunk = (int)((want + 63) / 64) * 64;
        if (chunk < 128) chunk = 128;
        c->attn_chunk = chunk;
        c->attn_onepass_ok = !(md.kernel_flags & SJD_ATTENTION_CHUNKED);
        c->attn_nchunks = ceil_div(md.max_ctx, chunk);
        const size_t slots = (size_t)S * 2 * H * ceil_div(L, 32) * c->attn_nchunks;
        if ((rc = dev_alloc(c, &c->part_o, slots * 32 * hd * sizeof(float)))) return rc;
        if ((rc = dev_alloc(c, &c->part_ml, slots * 64 * sizeof(float)))) return rc;
    }
    return SJD_OK;
}

int alloc_state(sjd_ctx *c) {
    const int S = c->S, L = c->L, M = S * 2 * L;
    int rc;
    if ((rc = dev_alloc(c, &c->win_row_tok, (size_t)M * 4))) return rc;
    if ((rc = dev_alloc(c, &c->win_row_pos, (size_t)M * 4))) return rc;
    if ((rc = dev_alloc(c, &c->win_seg_kv, (size_t)S * 2 * 4))) return rc;
    if ((rc = dev_alloc(c, &c->win_seg_n, (size_t)S * 2 * 4))) return rc;
    DecideState &d = c->ds;
    d.L = L; d.V = c->Vs; d.lo = c->md.sample_lo; d.max_img = c->md.max_ctx;
    if ((rc = dev_alloc(c, &d.win_tok, (size_t)S * L * 4))) return rc;
    if ((rc = dev_alloc(c, &d.anchor, (size_t)S * 2 * 4))) return rc;
    if ((rc = dev_alloc(c, &d.ref_row, (size_t)S * L * 4))) return rc;
    if ((rc = dev_alloc(c, &d.n_img, (size_t)S * 4))) return rc;
    if ((rc = dev_alloc(c, &d.n_image, (size_t)S * 4))) return rc;
    if ((rc = dev_alloc(c, &d.kv_len, (size_t)S * 2 * 4))) return rc;
    if ((rc = dev_alloc(c, &d.Le, (size_t)S * 4))) return rc;
    if ((rc = dev_alloc(c, &d.out_tok, (size_t)S * d.max_img * 4))) return rc;
    if ((rc = dev_alloc(c, &d.acc_len, (size_t)S * 4))) return rc;
    if ((rc = dev_alloc(c, &d.cand, (size_t)S * L * 4))) return rc;
    if ((rc = dev_alloc(c, &d.cand_new, (size_t)S * L * 4))) return rc;
    d.cap = c->Vs;   // room for a whole row of kept pairs (ties at the K-th value can keep everything); pages that are never
                     // written are never touched
    if (c->sp.init_mode == 4) {
        const size_t rows = (size_t)S * c->sp.row_width;
        if ((rc = dev_alloc(c, &d.hist_ids, rows * d.cap * sizeof(int32_t), false))) return rc;
        if ((rc = dev_alloc(c, &d.hist_e, rows * d.cap * sizeof(float), false))) return rc;
        if ((rc = dev_alloc(c, &d.hist_cnt, rows * sizeof(int32_t)))) return rc;
        if ((rc = dev_alloc(c, &d.hist_Z, rows * sizeof(uint64_t)))) return rc;
    }
    if ((rc = dev_alloc(c, &d.step, 4))) return rc;
    for (int b = 0; b < 2; ++b) {
        if ((rc = dev_alloc(c, &d.ids_buf[b], (size_t)S * L * d.cap * sizeof(int32_t), false))) return rc;
        if ((rc = dev_alloc(c, &d.e_buf[b], (size_t)S * L * d.cap * sizeof(float), false))) return rc;
        if ((rc = dev_alloc(c, &d.cnt_buf[b], (size_t)S * L * sizeof(int32_t)))) return rc;
        if ((rc = dev_alloc(c, &d.Z_buf[b], (size_t)S * L * sizeof(uint64_t)))) return rc;
    }
    if ((rc = dev_alloc(c, &d.allow_lo, (size_t)S * d.max_img * 4))) return rc;
    if ((rc = dev_alloc(c, &d.allow_hi, (size_t)S * d.max_img * 4))) return rc;
    hipError_t e = hipHostMalloc((void **)&c->res_host, (size_t)S * sizeof(sjd_step_result), hipHostMallocMapped | hipHostMallocCoherent);
    if (e != hipSuccess) { sjd_set_error(c->err, "hipHostMalloc failed: %s", hipGetErrorString(e)); return SJD_ENOMEM; }
    d.res_host = c->res_host;   // (host and device share the address)
    return SJD_OK;
}

int make_rope_tables(sjd_ctx *c) {
    const int half = c->hd / 2, n = c->md.max_ctx;
    std::vector<float> cs((size_t)n * half), sn((size_t)n * half);
    for (int pos = 0; pos < n; ++pos)
        for (int i = 0; i < half; ++i) {
            const double angle = (double)pos * pow((double)c->md.rope_theta, -2.0 * i / c->hd);
            cs[(size_t)pos * half + i] = (float)cos(angle);
            sn[(size_t)pos * half + i] = (float)sin(angle);
        }
    int rc;
    if ((rc = dev_alloc(c, &c->rope_cos, cs.size() * 4, false))) return rc;
    if ((rc = dev_alloc(c, &c->rope_sin, sn.size() * 4, false))) return rc;
    SJD_HIP_TRY(c->err, hipMemcpy(c->rope_cos, cs.data(), cs.size() * 4, hipMemcpyHostToDevice));
    SJD_HIP_TRY(c->err, hipMemcpy(c->rope_sin, sn.data(), sn.size() * 4, hipMemcpyHostToDevice));
    return SJD_OK;
}

int validate_desc(const sjd_model_desc *md, const sjd_weights *w, const sjd_sampling *sp, char *err) {
    if (!md || !w || !sp) { sjd_set_error(err, "null argument"); return SJD_EINVAL; }
    if (md->n_layers < 1 || md->d_model < 1 || md->n_heads < 1 || md->n_kv_heads < 1 || md->d_ff < 1 || md->vocab < 1) {
        sjd_set_error(err, "non-positive model dimension"); return SJD_EINVAL;
    }
    if (md->d_model % md->n_heads || md->n_heads % md->n_kv_heads) { sjd_set_error(err, "heads do not divide"); return SJD_EINVAL; }
    const int hd = md->d_model / md->n_heads;
    if (hd % 2) { sjd_set_error(err, "odd head dimension"); return SJD_EINVAL; }
    if (md->sample_lo < 0 || md->sample_hi > md->vocab || md->sample_hi <= md->sample_lo) {
        sjd_set_error(err, "bad sampled id range"); return SJD_EINVAL;
    }
    if (md->dtype != SJD_F32 && md->dtype != SJD_BF16) { sjd_set_error(err, "unknown dtype"); return SJD_EINVAL; }
    if (md->max_seqs < 1 || md->max_ctx < 2 || md->window < 1 || md->window > 1024) {
        sjd_set_error(err, "bad capacity (max_seqs >= 1, max_ctx >= 2, 1 <= window <= 1024)"); return SJD_EINVAL;
    }
    if (md->kv_page_tokens < 0 || md->kv_page_tokens % 32) { sjd_set_error(err, "kv_page_tokens must be a multiple of 32"); return SJD_EINVAL; }
    if (md->dtype == SJD_BF16 && (hd % 32 || md->d_model % 16 || md->d_ff % 16)) {
        sjd_set_error(err, "bf16 needs head_dim %% 32 == 0, d_model %% 16 == 0, d_ff %% 16 == 0"); return SJD_EINVAL;
    }
    if (!(md->rms_eps > 0.0f) || !(md->rope_theta > 0.0f)) { sjd_set_error(err, "bad rms_eps / rope_theta"); return SJD_EINVAL; }
    if (sp->top_k < 1 || !(sp->temperature > 0.0f) || sp->init_mode < 0 || sp->init_mode > 4 ||
        ((sp->init_mode == 2 || sp->init_mode == 4) && sp->row_width < 1) || sp->reuse_tau != sp->reuse_tau || sp->reuse_tau < 0.0f) {
        sjd_set_error(err, "bad sampling parameters (top_k >= 1, temperature > 0, tau >= 0, init_mode 0..4, row_width >= 1 for init_mode 2 and 4)"); return SJD_EINVAL;
    }
    if (!w->tok_emb || !w->final_norm || !w->lm_head || !w->attn_norm || !w->wq || !w->wk || !w->wv || !w->wo || !w->mlp_norm ||
        !w->w_gate || !w->w_up || !w->w_down) {
        sjd_set_error(err, "null weight pointer"); return SJD_EINVAL;
    }
    return SJD_OK;
}

// from_logits: the logits buffer was filled by the caller (no forward ran): the guided logits are computed from it
int run_decide(sjd_ctx *c, bool from_logits) {
    SJD_LAUNCH(c, KC_SAMPLE_ROWS, launch_sample_rows(c->stream, c->ds, c->sp, c->logits, c->n_seqs, c->z_used && !from_logits ? c->z : nullptr));
    SJD_LAUNCH(c, KC_VERIFY, launch_verify(c->stream, c->ds, c->sp, c->n_seqs));
    SJD_LAUNCH(c, KC_DRAW, launch_draw(c->stream, c->ds, c->sp, c->n_seqs));
    if (c->sp.init_mode == 4) SJD_LAUNCH(c, KC_COMMIT, launch_keep_rows(c->stream, c->ds, c->sp, c->n_seqs));
    SJD_LAUNCH(c, KC_COMMIT, launch_commit(c->stream, c->ds, c->sp, c->n_seqs));
    return SJD_OK;
}

int finish_step(sjd_ctx *c, sjd_step_result *out) {
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));   // the verdicts are in host memory then
    trace_collect(c);
    bool all = true;
    for (int s = 0; s < c->n_seqs; ++s) {
        out[s] = c->res_host[s];
        all = all && out[s].done;
        c->kv_host[s * 2] += out[s].n_finalized;
        c->kv_host[s * 2 + 1] += out[s].n_finalized;
    }
    c->all_done = all;
    return SJD_OK;
}

// everything one decoding step launches, in stream order (the host reads the verdicts back afterwards)
int enqueue_step(sjd_ctx *c) {
    FwdRows fr;
    fr.stage = stage_rows(c->ds, c->win_row_tok, c->win_row_pos, c->win_seg_kv, c->win_seg_n);
    fr.n_segs = c->n_seqs * 2;
    fr.L = c->L;
    fr.M = fr.n_segs * c->L;
    fr.n_qt = ceil_div(c->L, 32);
    fr.rm = {c->win_row_tok, c->win_row_pos, c->win_seg_kv, c->win_seg_n, nullptr, nullptr, nullptr};
    int rc = forward_any(c, fr, true);
    if (rc) return rc;
    return run_decide(c, false);
}

void drop_graph(sjd_ctx *c, int g) {
    if (c->graph_exec[g]) (void)hipGraphExecDestroy(c->graph_exec[g]);
    if (c->graph[g]) (void)hipGraphDestroy(c->graph[g]);
    c->graph_exec[g] = nullptr;
    c->graph[g] = nullptr;
    c->graph_n_seqs[g] = 0;
}

// Records the launches of a step, which have been enqueued already, as graph g; false where that fails.
bool record_step(sjd_ctx *c, int g) {
    hipGraph_t gr = nullptr;
    hipGraphExec_t ex = nullptr;
    bool ok = hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal) == hipSuccess;
    if (ok) {
        ok = enqueue_step(c) == SJD_OK;
        ok = hipStreamEndCapture(c->stream, &gr) == hipSuccess && gr && ok;   // always end the capture, also after a failed launch
        ok = ok && hipGraphInstantiate(&ex, gr, nullptr, nullptr, 0) == hipSuccess;
    }
    if (!ok) {
        if (gr) (void)hipGraphDestroy(gr);
        (void)hipGetLastError();   // not the error of a launch to come
        return false;
    }
    c->graph[g] = gr;
    c->graph_exec[g] = ex;
    c->graph_n_seqs[g] = c->n_seqs;
    return true;
}

// one-pass attention for a step's launches iff the longest visible context (cache + rows) is short
void choose_attention(sjd_ctx *c, int max_kv) {
    c->attn_onepass = c->attn_mfma && c->attn_onepass_ok && attention_onepass_pays(max_kv + c->L, c->hd, c->n_seqs * 2 * c->md.n_heads, c->n_cus);
}

}  // namespace

// =================================================================================================
extern "C" {

const char *sjd_last_error(const sjd_ctx *ctx) { return ctx ? ctx->err : g_create_error; }

void sjd_destroy(sjd_ctx *c) {
    if (!c) return;
    (void)hipStreamSynchronize(c->stream);
    drop_graph(c, 0);
    drop_graph(c, 1);
    for (void *p : c->allocations) (void)hipFree(p);
    if (c->res_host) (void)hipHostFree(c->res_host);
    for (hipEvent_t e : c->tracer.pool) (void)hipEventDestroy(e);
    delete c;
}

int sjd_create(const sjd_model_desc *desc, const sjd_weights *weights, const sjd_sampling *sampling, void *hip_stream,
               sjd_ctx **out) {
    if (!out) { sjd_set_error(g_create_error, "null output pointer"); return SJD_EINVAL; }
    *out = nullptr;
    int rc = validate_desc(desc, weights, sampling, g_create_error);
    if (rc) return rc;
    sjd_ctx *c = new (std::nothrow) sjd_ctx();
    if (!c) { sjd_set_error(g_create_error, "out of host memory"); return SJD_ENOMEM; }
    c->md = *desc;
    c->sampling = *sampling;
    c->stream = (hipStream_t)hip_stream;
    c->hd = desc->d_model / desc->n_heads;
    c->Vs = desc->sample_hi - desc->sample_lo;
    c->L = desc->window;
    c->S = desc->max_seqs;
    c->pt = desc->kv_page_tokens ? desc->kv_page_tokens : 64;
    c->md.kv_page_tokens = c->pt;
    c->max_visible = desc->max_ctx + 1;
    c->sp.cfg_scale = sampling->cfg_scale;
    c->sp.inv_temperature = 1.0f / sampling->temperature;
    c->sp.tau = sampling->reuse_tau;
    c->sp.top_k = sampling->top_k;
    c->sp.seed = sampling->seed;
    c->sp.init_mode = sampling->init_mode;
    c->sp.row_width = sampling->row_width;
    {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess) {
            if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) c->n_cus = v;
            if (hipDeviceGetAttribute(&v, hipDeviceAttributeNumberOfXccs, dev) == hipSuccess && v > 0) c->n_xcds = v;
        }
        (void)hipGetLastError();
    }
    c->shape = {desc->d_model, desc->n_heads, desc->n_kv_heads, desc->d_ff, c->Vs, c->n_cus, desc->kernel_flags};
    c->keep_logits = (desc->kernel_flags & SJD_KEEP_LOGITS) != 0;
    const bool f32 = desc->dtype == SJD_F32;
    c->use_graph = !(desc->kernel_flags & SJD_NO_GRAPH) && hip_stream != nullptr;  // the default stream cannot be captured
    c->attn_mfma = !f32 && !(desc->kernel_flags & SJD_KERNELS_REFERENCE) &&
                   attention_mfma_supported(c->L, desc->n_heads, desc->n_kv_heads, c->hd, c->pt);
    // Every bf16 model whose heads are 64 or 128 wide (and whose matrices are whole 32-row tiles) takes the fused projections,
    // whatever the number of rows: against the generic split-K GEMMs with their element-wise kernels, a forward of the 36 x 1280
    // shape measured 5.9 -> 3.9 ms at 500 rows and 5.4 -> 1.9 ms at 192.
    c->fused = !f32 && !(desc->kernel_flags & SJD_KERNELS_REFERENCE) && c->hd % 64 == 0 &&
               desc->d_model % 32 == 0 && desc->d_ff % 32 == 0;
    // Windows that fill one row group or whole ones have the gains in the weights: their row-group kernels need no sums of
    // squares from the kernel before.  All others keep the caller's weights as they are, as the generic GEMMs did for them.
    c->fold_gain = c->S * 2 * c->L <= 64 || (2 * c->L) % 64 == 0;
    rc = f32 ? copy_weights<float>(c, weights) : (c->fused ? copy_weights_fused(c, weights) : copy_weights<bf16_t>(c, weights));
    if (!rc) rc = f32 ? alloc_buffers<float>(c) : alloc_buffers<bf16_t>(c);
    if (!rc) rc = alloc_state(c);
    if (!rc) rc = make_rope_tables(c);
    if (!rc && hipStreamSynchronize(c->stream) != hipSuccess) {
        sjd_set_error(c->err, "device error while copying the weights: %s", hipGetErrorString(hipGetLastError()));
        rc = SJD_EDEVICE;
    }
    if (rc) {
        memcpy(g_create_error, c->err, sizeof g_create_error);
        sjd_destroy(c);
        return rc;
    }
    *out = c;
    return SJD_OK;
}

int sjd_prefill(sjd_ctx *c, int32_t n_seqs, const int32_t *const *cond_ids, const int32_t *cond_len,
                const int32_t *const *uncond_ids, const int32_t *uncond_len, const int32_t *n_image_tokens) {
    if (!c) return SJD_EINVAL;
    if (!cond_ids || !cond_len || !uncond_ids || !uncond_len || !n_image_tokens || n_seqs < 1) {
        sjd_set_error(c->err, "null argument or n_seqs < 1");
        return SJD_EINVAL;
    }
    if (n_seqs > c->S) { sjd_set_error(c->err, "n_seqs %d > max_seqs %d", n_seqs, c->S); return SJD_ECAPACITY; }
    size_t total_rows = 0;   // every prompt token but the last
    for (int s = 0; s < n_seqs; ++s) {
        if (!cond_ids[s] || !uncond_ids[s] || cond_len[s] < 1 || uncond_len[s] < 1 || n_image_tokens[s] < 1) {
            sjd_set_error(c->err, "sequence %d: null prompt, empty prompt or no image tokens", s);
            return SJD_EINVAL;
        }
        if (cond_len[s] + n_image_tokens[s] > c->md.max_ctx || uncond_len[s] + n_image_tokens[s] > c->md.max_ctx) {
            sjd_set_error(c->err, "sequence %d: prompt + image tokens exceed max_ctx %d", s, c->md.max_ctx);
            return SJD_ECAPACITY;
        }
        for (int i = 0; i < cond_len[s]; ++i)
            if (cond_ids[s][i] < 0 || cond_ids[s][i] >= c->md.vocab) { sjd_set_error(c->err, "token id outside the vocabulary"); return SJD_EINVAL; }
        for (int i = 0; i < uncond_len[s]; ++i)
            if (uncond_ids[s][i] < 0 || uncond_ids[s][i] >= c->md.vocab) { sjd_set_error(c->err, "token id outside the vocabulary"); return SJD_EINVAL; }
        total_rows += (size_t)(cond_len[s] - 1) + (uncond_len[s] - 1);
    }
    c->prefilled = false;
    c->n_seqs = n_seqs;
    const int n_segs = n_seqs * 2;
    hipStream_t st = c->stream;
    SJD_HIP_TRY(c->err, hipStreamSynchronize(st));   // (after a failed call its copy may still be under way)
    std::vector<int32_t> table((size_t)c->S * 2 * c->pps, 0);
    // Pages are handed out round-robin over the segments, so that the pages of one segment are not
    // contiguous in the pool; a segment takes only the pages its prompt + image need.
    {
        std::vector<int> need((size_t)n_seqs * 2), got((size_t)n_seqs * 2, 0);
        int next = 0, pending = 0;
        for (int s = 0; s < n_seqs; ++s) {
            need[s * 2] = ceil_div(cond_len[s] + n_image_tokens[s], c->pt);
            need[s * 2 + 1] = ceil_div(uncond_len[s] + n_image_tokens[s], c->pt);
            pending += need[s * 2] + need[s * 2 + 1];
        }
        if (pending > c->n_pages) { sjd_set_error(c->err, "KV page pool exhausted"); return SJD_ECAPACITY; }
        while (pending > 0)
            for (int seg = 0; seg < n_seqs * 2; ++seg)
                if (got[seg] < need[seg]) { table[(size_t)seg * c->pps + got[seg]++] = next++; --pending; }
    }
    c->page_table_host = table;
    c->n_image_host.assign(n_image_tokens, n_image_tokens + n_seqs);
    c->kv_host.assign((size_t)n_segs, 0);
    std::vector<int32_t> &up = c->pre_host;
    up.assign(table.size() + 5 * (size_t)n_seqs, 0);
    std::copy(table.begin(), table.end(), up.begin());
    const size_t o_len = table.size(), o_last = o_len + n_segs, o_img = o_last + n_segs;
    auto prompt = [&](int seg) { return seg & 1 ? uncond_ids[seg >> 1] : cond_ids[seg >> 1]; };
    auto prompt_len = [&](int seg) { return seg & 1 ? uncond_len[seg >> 1] : cond_len[seg >> 1]; };
    int max_len = 1;
    for (int seg = 0; seg < n_segs; ++seg) {
        up[o_len + seg] = prompt_len(seg);
        up[o_last + seg] = prompt(seg)[prompt_len(seg) - 1];
        c->kv_host[seg] = prompt_len(seg) - 1;
        max_len = std::max(max_len, prompt_len(seg));
    }
    std::copy(n_image_tokens, n_image_tokens + n_seqs, up.begin() + o_img);
    std::vector<FwdRows> fwds;
    if (c->attn_mfma && (c->md.kernel_flags & SJD_ATTENTION_CHUNKED)) {
        // the chunk kernels take windows of L rows per segment, as in a step
        const int L = c->L, M = n_segs * L;
        for (int start = 0; start < max_len - 1; start += L) {
            const size_t o = up.size();
            up.resize(o + 2 * (size_t)M + 2 * n_segs, 0);
            int32_t *tok = &up[o], *pos = tok + M, *kv = pos + M, *n = kv + n_segs;
            for (int seg = 0; seg < n_segs; ++seg) {
                kv[seg] = start;
                n[seg] = std::min(std::max(prompt_len(seg) - 1 - start, 0), L);
                for (int i = 0; i < L; ++i) {
                    tok[seg * L + i] = i < n[seg] ? prompt(seg)[start + i] : -1;
                    pos[seg * L + i] = start + i;
                }
            }
            FwdRows f;
            f.M = M; f.n_segs = n_segs; f.L = L; f.n_qt = ceil_div(L, 32);
            const int32_t *dev = c->pre_dev + o;
            f.rm = {dev, dev + M, dev + 2 * (size_t)M, dev + 2 * (size_t)M + n_segs, nullptr, nullptr, nullptr};
            fwds.push_back(f);
        }
    } else {
        // The rows of all prompts one after the other, cut into forwards of about equal size (whole tiles of 256 rows while
        // there are several); a segment may start in one forward and go on in the next.
        const size_t n_fwd_max = ceil_div_sz(total_rows, c->pre_rows);
        const int per_fwd = n_fwd_max < 2 ? c->pre_rows : (int)std::min<size_t>(c->pre_rows, ceil_div_sz(ceil_div_sz(total_rows, n_fwd_max), 256) * 256);
        const size_t o_tok = up.size(), o_pos = o_tok + total_rows, o_seg = o_pos + total_rows;
        up.resize(o_seg + total_rows, 0);
        size_t row = 0, o_tab = 0;
        int q_next = 0;   // next free query tile of the forward
        for (int seg = 0; seg < n_segs; ++seg) {
            const int len = prompt_len(seg);
            for (int pos = 0; pos < len - 1;) {
                if (fwds.empty() || fwds.back().M == per_fwd) {
                    o_tab = up.size();   // seg_kv, seg_n, seg_row0, seg_q0
                    up.resize(o_tab + 4 * (size_t)n_segs, 0);
                    FwdRows f;
                    f.n_segs = n_segs;
                    const int32_t *dev = c->pre_dev, *tab = dev + o_tab;
                    f.rm = {dev + o_tok + row, dev + o_pos + row, tab, tab + n_segs, dev + o_seg + row, tab + 2 * n_segs, tab + 3 * n_segs};
                    fwds.push_back(f);
                    q_next = 0;
                }
                FwdRows &f = fwds.back();
                const int n = std::min(len - 1 - pos, per_fwd - f.M);
                int32_t *tab = &up[o_tab];
                tab[seg] = pos;
                tab[n_segs + seg] = n;
                tab[2 * n_segs + seg] = f.M;
                tab[3 * n_segs + seg] = q_next;
                for (int i = 0; i < n; ++i, ++row, ++pos) {
                    up[o_tok + row] = prompt(seg)[pos];
                    up[o_pos + row] = pos;
                    up[o_seg + row] = seg;
                }
                f.M += n;
                f.n_qt = std::max(f.n_qt, ceil_div(n, 32));
                q_next += ceil_div(n, 32);
            }
        }
    }
    if (up.size() > c->pre_elems) { sjd_set_error(c->err, "prompt staging too small"); return SJD_EINVAL; }   // cannot happen: sized at create
    SJD_HIP_TRY(c->err, hipMemcpyAsync(c->pre_dev, up.data(), up.size() * 4, hipMemcpyHostToDevice, st));
    for (const FwdRows &f : fwds) {
        int rc = forward_any(c, f, false);
        if (rc) return rc;
    }
    SJD_LAUNCH(c, KC_STAGE, launch_init_window(st, c->ds, c->sp, n_seqs, c->S, c->pre_dev + o_last, c->pre_dev + o_len, c->pre_dev + o_img));
    SJD_HIP_TRY(c->err, hipStreamSynchronize(st));
    trace_collect(c);
    c->prefilled = true;
    c->all_done = false;
    return SJD_OK;
}

int sjd_step(sjd_ctx *c, sjd_step_result *out) {
    if (!c) return SJD_EINVAL;
    if (!out) { sjd_set_error(c->err, "null result pointer"); return SJD_EINVAL; }
    if (!c->prefilled) { sjd_set_error(c->err, "sjd_step before sjd_prefill"); return SJD_ESTATE; }
    int rc;
    int max_kv = 0;
    for (int32_t kv : c->kv_host) max_kv = std::max(max_kv, (int)kv);
    choose_attention(c, max_kv);
    const int g = c->attn_onepass ? 1 : 0;
    if (c->use_graph && !c->tracer.on) {   // per-kernel event timing needs the kernels one by one
        if (c->graph_exec[g] && c->graph_n_seqs[g] != c->n_seqs) drop_graph(c, g);
        if (!c->graph_exec[g]) {
            // The first step of a graph is launched kernel by kernel and recorded while the device works on it: recorded and
            // instantiated ahead of it, its launches kept the device idle for half a millisecond (a new context's first prefill and
            // step, 36 layers of 1280, window 16: 1800 -> 1260 us; with a 120-token prompt, window 32: 4310 -> 3370)
            if ((rc = enqueue_step(c))) return rc;
            const bool recorded = record_step(c, g);
            rc = finish_step(c, out);
            if (!rc && !recorded) c->use_graph = false;   // the step is the step; those after it are launched one by one
            return rc;
        }
        SJD_HIP_TRY(c->err, hipGraphLaunch(c->graph_exec[g], c->stream));
    } else if ((rc = enqueue_step(c))) {
        return rc;
    }
    return finish_step(c, out);
}

int sjd_debug_step_from_logits(sjd_ctx *c, const float *logits_host, sjd_step_result *out) {
    if (!c) return SJD_EINVAL;
    if (!out || !logits_host) { sjd_set_error(c->err, "null pointer"); return SJD_EINVAL; }
    if (!c->prefilled) { sjd_set_error(c->err, "step before sjd_prefill"); return SJD_ESTATE; }
    SJD_HIP_TRY(c->err, hipMemcpyAsync(c->logits, logits_host, (size_t)c->n_seqs * 2 * c->L * c->Vs * sizeof(float),
                                       hipMemcpyHostToDevice, c->stream));
    SJD_LAUNCH(c, KC_STAGE, launch_stage_window(c->stream, stage_rows(c->ds, c->win_row_tok, c->win_row_pos, c->win_seg_kv, c->win_seg_n), c->n_seqs));
    int rc = run_decide(c, true);
    if (rc) return rc;
    return finish_step(c, out);
}

int sjd_debug_copy_logits(sjd_ctx *c, float *dst_host) {
    if (!c || !dst_host) return SJD_EINVAL;
    if (!c->prefilled) { sjd_set_error(c->err, "no step yet"); return SJD_ESTATE; }
    if (c->z_used && !c->keep_logits) {
        sjd_set_error(c->err, "the logits are not kept: this context's vocabulary head writes guided logits only (create it with SJD_KEEP_LOGITS)");
        return SJD_ESTATE;
    }
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));
    SJD_HIP_TRY(c->err, hipMemcpy(dst_host, c->logits, (size_t)c->n_seqs * 2 * c->L * c->Vs * sizeof(float), hipMemcpyDeviceToHost));
    return SJD_OK;
}

int sjd_get_tokens(sjd_ctx *c, int32_t seq, int32_t *dst, int32_t cap, int32_t *n_out) {
    if (!c || !n_out) return SJD_EINVAL;
    if (!c->prefilled) { sjd_set_error(c->err, "no prefill yet"); return SJD_ESTATE; }
    if (seq < 0 || seq >= c->n_seqs || cap < 0 || (cap > 0 && !dst)) { sjd_set_error(c->err, "bad sequence index or buffer"); return SJD_EINVAL; }
    int32_t n = 0;
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));
    SJD_HIP_TRY(c->err, hipMemcpy(&n, c->ds.n_img + seq, 4, hipMemcpyDeviceToHost));
    const int32_t k = n < cap ? n : cap;
    if (k > 0) SJD_HIP_TRY(c->err, hipMemcpy(dst, c->ds.out_tok + (size_t)seq * c->ds.max_img, (size_t)k * 4, hipMemcpyDeviceToHost));
    *n_out = n;
    return SJD_OK;
}

int sjd_get_window(sjd_ctx *c, int32_t seq, int32_t *tokens, int32_t *ref_rows, int32_t *n_slots) {
    if (!c || !tokens || !ref_rows || !n_slots) return SJD_EINVAL;
    if (!c->prefilled) { sjd_set_error(c->err, "no prefill yet"); return SJD_ESTATE; }
    if (seq < 0 || seq >= c->n_seqs) { sjd_set_error(c->err, "bad sequence index"); return SJD_EINVAL; }
    const int L = c->L;
    int32_t le = 0;
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));
    SJD_HIP_TRY(c->err, hipMemcpy(tokens, c->ds.win_tok + (size_t)seq * L, (size_t)L * 4, hipMemcpyDeviceToHost));
    SJD_HIP_TRY(c->err, hipMemcpy(ref_rows, c->ds.ref_row + (size_t)seq * L, (size_t)L * 4, hipMemcpyDeviceToHost));
    SJD_HIP_TRY(c->err, hipMemcpy(tokens, c->ds.anchor + (size_t)seq * 2, 4, hipMemcpyDeviceToHost));
    SJD_HIP_TRY(c->err, hipMemcpy(&le, c->ds.Le + seq, 4, hipMemcpyDeviceToHost));
    ref_rows[0] = -1;
    *n_slots = le;
    return SJD_OK;
}

int sjd_set_token_ranges(sjd_ctx *c, int32_t seq, const int32_t *first_id, const int32_t *end_id, int32_t n_positions) {
    if (!c) return SJD_EINVAL;
    if (!c->prefilled) { sjd_set_error(c->err, "sjd_set_token_ranges before sjd_prefill"); return SJD_ESTATE; }
    if (seq < 0 || seq >= c->n_seqs || !first_id || !end_id || n_positions < 0 || (size_t)seq >= c->n_image_host.size() ||
        n_positions > c->n_image_host[seq]) {
        sjd_set_error(c->err, "bad sequence index, null array or more positions than image tokens");
        return SJD_EINVAL;
    }
    std::vector<int32_t> lo(n_positions), hi(n_positions);
    for (int i = 0; i < n_positions; ++i) {
        if (first_id[i] < c->md.sample_lo || end_id[i] > c->md.sample_hi || first_id[i] >= end_id[i]) {
            sjd_set_error(c->err, "position %d: id range [%d, %d) is empty or leaves the sampled ids", i, first_id[i], end_id[i]);
            return SJD_EINVAL;
        }
        lo[i] = first_id[i] - c->md.sample_lo;
        hi[i] = end_id[i] - c->md.sample_lo;
    }
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));
    if (n_positions > 0) {
        SJD_HIP_TRY(c->err, hipMemcpy(c->ds.allow_lo + (size_t)seq * c->ds.max_img, lo.data(), (size_t)n_positions * 4, hipMemcpyHostToDevice));
        SJD_HIP_TRY(c->err, hipMemcpy(c->ds.allow_hi + (size_t)seq * c->ds.max_img, hi.data(), (size_t)n_positions * 4, hipMemcpyHostToDevice));
    }
    return SJD_OK;
}

int sjd_trace_enable(sjd_ctx *c, int32_t on) {
    if (!c) return SJD_EINVAL;
    c->tracer.on = on != 0;
    return SJD_OK;
}
int sjd_trace_reset(sjd_ctx *c) {
    if (!c) return SJD_EINVAL;
    for (int i = 0; i < KC_COUNT; ++i) { c->tracer.launches[i] = 0; c->tracer.total_ms[i] = 0.0; }
    return SJD_OK;
}
int sjd_trace_read(sjd_ctx *c, sjd_trace_entry *dst, int32_t cap, int32_t *n_out) {
    if (!c || !n_out || (cap > 0 && !dst)) return SJD_EINVAL;
    for (int i = 0; i < KC_COUNT && i < cap; ++i) {
        dst[i].name = kKernelClassName[i];
        dst[i].launches = c->tracer.launches[i];
        dst[i].total_ms = c->tracer.total_ms[i];
    }
    *n_out = KC_COUNT;
    return SJD_OK;
}

}  // extern "C"

// ------------------------------------------------------------------------------------------ snapshots
// The state that Sec. 4.1 carries from one iteration to the next: the accepted tokens, the window's drafts with the
// rows they were drawn from (the previous iteration's distributions), and the cache of the accepted prefix.
namespace {

struct SnapshotHeader {
    uint64_t magic, total_bytes;
    int32_t version, n_seqs, all_done;
    // the context a snapshot fits: same model, capacities and sampling set-up
    int32_t n_layers, d_model, n_heads, n_kv_heads, hd, Vs, L, S, max_ctx, pt, pps, dtype, init_mode, row_width;
    uint64_t seed;
    float cfg_scale, temperature, reuse_tau;
    int32_t top_k;
    int32_t pages_used[1];  // [n_seqs * 2] follows (flexible; the struct is written with its real length)
};
constexpr uint64_t kSnapshotMagic = 0x31544e53444a53ull;  // "SJDSNT1"

// the per-sequence device arrays of the decoding state: pointer, bytes per sequence (NULL: a place of the format that nothing uses any
// more - the last verdicts - written as zeros and not read)
struct StateArray { void *p; size_t per_seq; };
std::vector<StateArray> state_arrays(sjd_ctx *c) {
    const DecideState &d = c->ds;
    const size_t L = c->L, V = c->Vs;
    const size_t cap = d.cap;
    std::vector<StateArray> a = {
        {d.win_tok, L * 4}, {d.anchor, 8}, {d.ref_row, L * 4}, {d.n_img, 4}, {d.n_image, 4}, {d.kv_len, 8}, {d.Le, 4},
        {d.out_tok, (size_t)d.max_img * 4}, {d.acc_len, 4}, {d.cand, L * 4}, {d.cand_new, L * 4},
        {d.ids_buf[0], L * cap * 4}, {d.ids_buf[1], L * cap * 4}, {d.e_buf[0], L * cap * 4}, {d.e_buf[1], L * cap * 4},
        {d.cnt_buf[0], L * 4}, {d.cnt_buf[1], L * 4}, {d.Z_buf[0], L * 8}, {d.Z_buf[1], L * 8},
        {d.allow_lo, (size_t)d.max_img * 4}, {d.allow_hi, (size_t)d.max_img * 4}, {nullptr, sizeof(sjd_step_result)}};
    if (c->sp.init_mode == 4) {
        a.push_back({d.hist_ids, (size_t)c->sp.row_width * cap * 4});
        a.push_back({d.hist_e, (size_t)c->sp.row_width * cap * 4});
        a.push_back({d.hist_cnt, (size_t)c->sp.row_width * 4});
        a.push_back({d.hist_Z, (size_t)c->sp.row_width * 8});
    }
    (void)V;
    return a;
}
size_t snapshot_header_bytes(int n_seqs) { return (sizeof(SnapshotHeader) + (size_t)(2 * n_seqs) * 4 + 15) / 16 * 16; }

// pages in use per segment (committed positions only: the window's entries are rewritten by every step)
int snapshot_pages(sjd_ctx *c, std::vector<int32_t> &pages) {
    std::vector<int32_t> kv((size_t)c->n_seqs * 2);
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));
    SJD_HIP_TRY(c->err, hipMemcpy(kv.data(), c->ds.kv_len, kv.size() * 4, hipMemcpyDeviceToHost));
    pages.resize(kv.size());
    for (size_t i = 0; i < kv.size(); ++i) pages[i] = ceil_div(kv[i], c->pt);
    return SJD_OK;
}
size_t snapshot_bytes(sjd_ctx *c, int n_seqs, const std::vector<int32_t> &pages) {
    size_t n = snapshot_header_bytes(n_seqs) + (size_t)c->S * 2 * c->pps * 4 + 16 /* step counter */;
    for (const StateArray &a : state_arrays(c)) n += a.per_seq * n_seqs;
    size_t total_pages = 0;
    for (int32_t p : pages) total_pages += p;
    const size_t page_bytes = c->pool_layer_bytes / c->n_pages;  // one page of one layer's key (or value) pool, all kv heads
    return n + total_pages * page_bytes * 2 * c->md.n_layers;
}
bool snapshot_fits(const sjd_ctx *c, const SnapshotHeader &h) {
    return h.n_layers == c->md.n_layers && h.d_model == c->md.d_model && h.n_heads == c->md.n_heads &&
           h.n_kv_heads == c->md.n_kv_heads && h.hd == c->hd && h.Vs == c->Vs && h.L == c->L && h.S == c->S &&
           h.max_ctx == c->md.max_ctx && h.pt == c->pt && h.pps == c->pps && h.dtype == c->md.dtype &&
           h.init_mode == c->sp.init_mode && h.row_width == c->sp.row_width && h.seed == c->sp.seed &&
           h.cfg_scale == c->sampling.cfg_scale && h.temperature == c->sampling.temperature &&
           (h.reuse_tau == c->sampling.reuse_tau || (h.reuse_tau != h.reuse_tau && c->sampling.reuse_tau != c->sampling.reuse_tau)) &&
           h.top_k == c->sampling.top_k;
}

}  // namespace

extern "C" {

int sjd_snapshot_size(sjd_ctx *c, uint64_t *bytes) {
    if (!c || !bytes) return SJD_EINVAL;
    if (!c->prefilled) { sjd_set_error(c->err, "no prefill yet"); return SJD_ESTATE; }
    std::vector<int32_t> pages;
    int rc = snapshot_pages(c, pages);
    if (rc) return rc;
    *bytes = snapshot_bytes(c, c->n_seqs, pages);
    return SJD_OK;
}

int sjd_snapshot_save(sjd_ctx *c, void *dst_host, uint64_t cap, uint64_t *written) {
    if (!c || !dst_host || !written) return SJD_EINVAL;
    if (!c->prefilled) { sjd_set_error(c->err, "no prefill yet"); return SJD_ESTATE; }
    std::vector<int32_t> pages;
    int rc = snapshot_pages(c, pages);
    if (rc) return rc;
    const size_t total = snapshot_bytes(c, c->n_seqs, pages);
    if (cap < total) { sjd_set_error(c->err, "snapshot needs %zu bytes, buffer has %llu", total, (unsigned long long)cap); return SJD_ECAPACITY; }
    char *w = (char *)dst_host;
    const size_t hb = snapshot_header_bytes(c->n_seqs);
    memset(w, 0, hb);
    SnapshotHeader *h = (SnapshotHeader *)w;
    h->magic = kSnapshotMagic; h->total_bytes = total; h->version = 1; h->n_seqs = c->n_seqs; h->all_done = c->all_done;
    h->n_layers = c->md.n_layers; h->d_model = c->md.d_model; h->n_heads = c->md.n_heads; h->n_kv_heads = c->md.n_kv_heads;
    h->hd = c->hd; h->Vs = c->Vs; h->L = c->L; h->S = c->S; h->max_ctx = c->md.max_ctx; h->pt = c->pt; h->pps = c->pps;
    h->dtype = c->md.dtype; h->init_mode = c->sp.init_mode; h->row_width = c->sp.row_width; h->seed = c->sp.seed;
    h->cfg_scale = c->sampling.cfg_scale; h->temperature = c->sampling.temperature; h->reuse_tau = c->sampling.reuse_tau;
    h->top_k = c->sampling.top_k;
    memcpy(h->pages_used, pages.data(), pages.size() * 4);
    w += hb;
    memcpy(w, c->page_table_host.data(), c->page_table_host.size() * 4);
    w += c->page_table_host.size() * 4;
    SJD_HIP_TRY(c->err, hipMemcpy(w, c->ds.step, 4, hipMemcpyDeviceToHost));
    w += 16;
    for (const StateArray &a : state_arrays(c)) {
        if (a.p) SJD_HIP_TRY(c->err, hipMemcpy(w, a.p, a.per_seq * c->n_seqs, hipMemcpyDeviceToHost));
        else memset(w, 0, a.per_seq * c->n_seqs);
        w += a.per_seq * c->n_seqs;
    }
    const size_t page_bytes = c->pool_layer_bytes / c->n_pages;  // one page of one layer's key (or value) pool, all kv heads
    for (int l = 0; l < c->md.n_layers; ++l)
        for (int kv = 0; kv < 2; ++kv) {
            const char *pool = (const char *)(kv ? c->vpool : c->kpool) + c->pool_layer_bytes * l;
            for (int seg = 0; seg < c->n_seqs * 2; ++seg)
                for (int i = 0; i < pages[seg]; ++i) {
                    const int page = c->page_table_host[(size_t)seg * c->pps + i];
                    SJD_HIP_TRY(c->err, hipMemcpyAsync(w, pool + (size_t)page * page_bytes, page_bytes, hipMemcpyDeviceToHost, c->stream));
                    w += page_bytes;
                }
        }
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));
    *written = (uint64_t)(w - (char *)dst_host);
    return SJD_OK;
}

int sjd_snapshot_restore(sjd_ctx *c, const void *src_host, uint64_t bytes) {
    if (!c || !src_host) return SJD_EINVAL;
    if (bytes < sizeof(SnapshotHeader)) { sjd_set_error(c->err, "snapshot truncated"); return SJD_EINVAL; }
    const SnapshotHeader *h = (const SnapshotHeader *)src_host;
    if (h->magic != kSnapshotMagic || h->version != 1) { sjd_set_error(c->err, "not a snapshot of this library version"); return SJD_EINVAL; }
    if (!snapshot_fits(c, *h)) { sjd_set_error(c->err, "snapshot was taken from a context with another model, capacity or sampling set-up"); return SJD_EINVAL; }
    if (h->n_seqs < 1 || h->n_seqs > c->S || h->total_bytes != bytes) { sjd_set_error(c->err, "snapshot truncated or corrupt"); return SJD_EINVAL; }
    const int n_seqs = h->n_seqs;
    std::vector<int32_t> pages(h->pages_used, h->pages_used + 2 * n_seqs);
    for (int32_t p : pages)
        if (p < 0 || p > c->pps) { sjd_set_error(c->err, "snapshot corrupt (page count)"); return SJD_EINVAL; }
    if (bytes < snapshot_header_bytes(n_seqs) || snapshot_bytes(c, n_seqs, pages) != bytes) {
        sjd_set_error(c->err, "snapshot truncated or corrupt");
        return SJD_EINVAL;
    }
    const char *r = (const char *)src_host + snapshot_header_bytes(n_seqs);
    const size_t table_n = (size_t)c->S * 2 * c->pps;
    std::vector<int32_t> table((const int32_t *)r, (const int32_t *)r + table_n);
    for (int seg = 0; seg < n_seqs * 2; ++seg)
        for (int i = 0; i < pages[seg]; ++i)
            if (table[(size_t)seg * c->pps + i] < 0 || table[(size_t)seg * c->pps + i] >= c->n_pages) {
                sjd_set_error(c->err, "snapshot corrupt (page table)");
                return SJD_EINVAL;
            }
    // The decoding state: the kernels index memory with these values, so every one of them is checked against the
    // context's capacities before anything is uploaded (a buffer of the right size with wrong contents must be an
    // error here, not an out-of-bounds access in the next step).
    {
        const std::vector<StateArray> arrays = state_arrays(c);
        std::vector<const char *> at(arrays.size());
        const char *q = r + table_n * 4 + 16;
        for (size_t i = 0; i < arrays.size(); ++i) { at[i] = q; q += arrays[i].per_seq * n_seqs; }
        enum { A_WIN, A_ANCHOR, A_REF, A_NIMG, A_NIMAGE, A_KV, A_LE, A_OUT, A_ACC, A_CAND, A_CANDNEW, A_IDS0, A_IDS1, A_E0, A_E1,
               A_CNT0, A_CNT1, A_Z0, A_Z1, A_ALO, A_AHI, A_RES, A_HIDS, A_HE, A_HCNT, A_HZ };
        auto i32 = [&](int which, size_t idx) { return ((const int32_t *)at[which])[idx]; };
        const int L = c->L, V = c->Vs, cap = c->ds.cap, max_img = c->ds.max_img, lo = c->md.sample_lo, hi = c->md.sample_hi;
        const int rw = c->sp.init_mode == 4 ? c->sp.row_width : 0;
        auto bad = [&](const char *what, int s) { sjd_set_error(c->err, "snapshot corrupt (%s of sequence %d)", what, s); return SJD_EINVAL; };
        for (int s = 0; s < n_seqs; ++s) {
            const int n_image = i32(A_NIMAGE, s), n_img = i32(A_NIMG, s), Le = i32(A_LE, s);
            if (n_image < 0 || n_image > max_img || n_img < 0 || n_img > n_image) return bad("token counts", s);
            if (Le < 0 || Le > L || Le > n_image - n_img) return bad("window length", s);
            for (int b = 0; b < 2; ++b) {
                const int kv = i32(A_KV, (size_t)s * 2 + b);
                if (kv < 0 || (long)kv + (n_image - n_img) > c->md.max_ctx) return bad("cache length", s);
                // every page the rest of the decode will read or write
                const int need = ceil_div(kv + (n_image - n_img), c->pt);
                for (int i = 0; i < need; ++i) {
                    const int32_t pg = table[((size_t)s * 2 + b) * c->pps + i];
                    if (pg < 0 || pg >= c->n_pages) return bad("page table", s);
                }
                const int anchor = i32(A_ANCHOR, (size_t)s * 2 + b);
                if (anchor < 0 || anchor >= c->md.vocab) return bad("window tokens", s);
            }
            if (i32(A_ACC, s) < -1 || i32(A_ACC, s) >= L) return bad("accept count", s);
            for (int k = 1; k < Le; ++k) {
                const int tok = i32(A_WIN, (size_t)s * L + k), ref = i32(A_REF, (size_t)s * L + k);
                if (tok < lo || tok >= hi) return bad("window tokens", s);
                if (ref >= L || ref < -2 - rw) return bad("reference rows", s);
            }
            for (int k = 0; k < L; ++k) {
                const int t0 = i32(A_CAND, (size_t)s * L + k), t1 = i32(A_CANDNEW, (size_t)s * L + k);
                if (t0 < 0 || t0 >= c->md.vocab || t1 < 0 || t1 >= c->md.vocab) return bad("drawn tokens", s);
            }
            for (int i = 0; i < n_image; ++i) {
                const int a0 = i32(A_ALO, (size_t)s * max_img + i), a1 = i32(A_AHI, (size_t)s * max_img + i);
                if (a0 < 0 || a1 > V || a0 >= a1) return bad("token ranges", s);
            }
            auto rows_ok = [&](int ids_arr, int cnt_arr, size_t row0, int n_rows) {
                for (int k = 0; k < n_rows; ++k) {
                    const int n = i32(cnt_arr, row0 + k);
                    if (n < 0 || n > cap) return false;
                    const int32_t *ids = (const int32_t *)at[ids_arr] + (row0 + k) * cap;
                    for (int i = 0; i < n; ++i)
                        if (ids[i] < 0 || ids[i] >= V || (i > 0 && ids[i] <= ids[i - 1])) return false;
                }
                return true;
            };
            if (!rows_ok(A_IDS0, A_CNT0, (size_t)s * L, L) || !rows_ok(A_IDS1, A_CNT1, (size_t)s * L, L)) return bad("stored rows", s);
            if (rw > 0 && !rows_ok(A_HIDS, A_HCNT, (size_t)s * rw, rw)) return bad("kept rows", s);
        }
    }
    // everything checked: from here on the context's batch is replaced
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));
    c->prefilled = false;
    c->n_seqs = n_seqs;
    c->page_table_host = table;
    SJD_HIP_TRY(c->err, hipMemcpy(c->page_table, table.data(), table_n * 4, hipMemcpyHostToDevice));
    r += table_n * 4;
    SJD_HIP_TRY(c->err, hipMemcpy(c->ds.step, r, 4, hipMemcpyHostToDevice));
    r += 16;
    for (const StateArray &a : state_arrays(c)) {
        if (a.p) SJD_HIP_TRY(c->err, hipMemcpy(a.p, r, a.per_seq * n_seqs, hipMemcpyHostToDevice));
        r += a.per_seq * n_seqs;
    }
    const size_t page_bytes = c->pool_layer_bytes / c->n_pages;  // one page of one layer's key (or value) pool, all kv heads
    for (int l = 0; l < c->md.n_layers; ++l)
        for (int kv = 0; kv < 2; ++kv) {
            char *pool = (char *)(kv ? c->vpool : c->kpool) + c->pool_layer_bytes * l;
            for (int seg = 0; seg < n_seqs * 2; ++seg)
                for (int i = 0; i < pages[seg]; ++i) {
                    const int page = table[(size_t)seg * c->pps + i];
                    SJD_HIP_TRY(c->err, hipMemcpyAsync(pool + (size_t)page * page_bytes, r, page_bytes, hipMemcpyHostToDevice, c->stream));
                    r += page_bytes;
                }
        }
    SJD_HIP_TRY(c->err, hipStreamSynchronize(c->stream));
    c->all_done = h->all_done != 0;
    c->prefilled = true;
    {   // host copy of the image lengths (sjd_set_token_ranges checks against it)
        const std::vector<StateArray> arrays = state_arrays(c);
        const char *q = (const char *)src_host + snapshot_header_bytes(n_seqs) + table_n * 4 + 16;
        for (int i = 0; i < 4; ++i) q += arrays[i].per_seq * n_seqs;
        c->n_image_host.assign((const int32_t *)q, (const int32_t *)q + n_seqs);
        q += arrays[4].per_seq * n_seqs;   // the cache lengths follow the image lengths
        c->kv_host.assign((const int32_t *)q, (const int32_t *)q + 2 * n_seqs);
    }
    return SJD_OK;
}

}  // extern "C"

#include "sjd_ops.hip.h"
