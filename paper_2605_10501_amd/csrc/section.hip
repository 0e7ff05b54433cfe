// Section executor: validates a call, carves the caller's workspace, and sequences the kernels
// of a layer stack forward (teacher) or forward + backward (student / vision encoder).
//
// Tensors that live between kernels are stored in the section dtype, except the forward residual
// stream (layer inputs, post-attention sums, last layer output), which is the running sum of all
// branch outputs and is kept in fp32; norm statistics, log-sum-exps, weight gradients and the loss
// are fp32 too.  The first layer's input of a bf16 section is bf16 already (x_in, or rows of the embedding table) and is
// read as it is: the same numbers, without a conversion pass and with half the bytes for the norm, the residual and the
// norm backward that read it.  In forward+backward mode every layer keeps its
// input, both normed activations, the (rotated) qkv, the attention output and log-sum-exp, the
// post-attention residual, the FFN pre-activation and activation: nothing is recomputed.
#include <vector>

#include "common.h"
#include "launch.h"

namespace {

struct LayerBuf {
    void *x, *h1, *qkv, *o, *x2, *h2, *up, *act;
    float *lse, *rstd1, *mean1, *rstd2, *mean2;
};

struct Plan {
    std::vector<LayerBuf> layers;  // n_layers entries (backward) or 1 shared entry (forward only)
    void *xa, *xb;                 // forward-only residual ping-pong
    void *y_last;
    float *rstd_f, *mean_f;
    int32_t *pos;
    float *rope;
    // backward temporaries
    void *dy0, *dy1, *dx2, *dh, *d_o, *dqkv, *da, *dup, *dhs;
    void *norm_scratch, *attn_scratch;
    size_t norm_scratch_bytes, bytes;
    bool bwd;                      // layers keep their activations for a backward pass
};

struct Dims {
    int n, d, dqkv, dattn, dup, f, nq, nkv, hd, max_seqlen;
    size_t es;
    bool dec;
};

Dims dims_of(const ms_section_config *c, int n, int max_seqlen) {
    Dims m;
    m.n = n; m.d = c->d_model; m.nq = c->n_q_heads; m.nkv = c->n_kv_heads; m.hd = c->head_dim;
    m.dqkv = (c->n_q_heads + 2 * c->n_kv_heads) * c->head_dim;
    m.dattn = c->n_q_heads * c->head_dim;
    m.dec = c->arch == MS_DECODER;
    m.f = c->d_ffn;
    m.dup = m.dec ? 2 * c->d_ffn : c->d_ffn;
    m.es = ms_dtype_size(c->dtype);
    m.max_seqlen = max_seqlen;
    return m;
}

Plan make_plan(const ms_section_config *c, int n, int max_seqlen, bool bwd, void *ws) {
    const Dims m = dims_of(c, n, max_seqlen);
    Arena a(ws);
    Plan p = {};
    const size_t N = (size_t)n;
    auto act = [&](size_t cols) { return a.take<void>(N * cols * m.es); };
    auto res = [&](size_t cols) { return a.take<void>(N * cols * 4); };   // residual stream: fp32
    auto f32 = [&](size_t cnt) { return a.take<float>(cnt * 4); };
    const int nbuf = bwd ? c->n_layers : 1;
    p.bwd = bwd;
    p.layers.resize(nbuf);
    for (auto &l : p.layers) {
        l.x = bwd ? res(m.d) : nullptr;
        l.h1 = act(m.d); l.qkv = act(m.dqkv); l.o = act(m.dattn); l.x2 = res(m.d); l.h2 = act(m.d);
        l.up = act(m.dup); l.act = act(m.f);
        l.lse = f32(N * m.nq); l.rstd1 = f32(N); l.mean1 = f32(N); l.rstd2 = f32(N); l.mean2 = f32(N);
    }
    if (!bwd) { p.xa = res(m.d); p.xb = res(m.d); }
    p.y_last = res(m.d);
    p.rstd_f = f32(N); p.mean_f = f32(N);
    p.pos = a.take<int32_t>(N * 4);
    p.rope = f32((size_t)max_seqlen * m.hd);  // [max_seqlen, hd/2] (cos, sin)
    if (bwd) {
        p.dy0 = act(m.d); p.dy1 = act(m.d); p.dx2 = act(m.d); p.dh = act(m.d); p.d_o = act(m.dattn);
        p.dqkv = act(m.dqkv); p.da = act(m.f); p.dup = act(m.dup); p.dhs = act(m.d);
        const int widest = m.dup > m.dqkv ? (m.dup > m.d ? m.dup : m.d) : (m.dqkv > m.d ? m.dqkv : m.d);
        p.norm_scratch_bytes = ms_k_norm_backward_scratch_bytes(widest);
        p.norm_scratch = a.take<void>(p.norm_scratch_bytes);
        p.attn_scratch = a.take<void>(ms_k_attention_backward_scratch_bytes(c->dtype, m.nq, m.nkv, m.hd, n));
    }
    p.bytes = a.off;
    return p;
}

ms_status validate_config(const ms_section_config *c) {
    if (!c) return ms_fail(MS_ERR_INVALID_ARG, "section: null config");
    if (c->arch != MS_DECODER && c->arch != MS_ENCODER) return ms_fail(MS_ERR_INVALID_ARG, "section: bad arch %d", c->arch);
    if (c->dtype != MS_BF16 && c->dtype != MS_F32) return ms_fail(MS_ERR_INVALID_ARG, "section: bad dtype %d", c->dtype);
    if (c->n_layers <= 0 || c->d_model <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0 || c->head_dim <= 0 ||
        c->d_ffn <= 0 || c->vocab < 0)
        return ms_fail(MS_ERR_SHAPE, "section: sizes must be positive");
    if (c->n_q_heads % c->n_kv_heads)
        return ms_fail(MS_ERR_SHAPE, "section: n_q_heads=%d is not a multiple of n_kv_heads=%d", c->n_q_heads, c->n_kv_heads);
    if (c->head_dim != 64 && c->head_dim != 80 && c->head_dim != 128)
        return ms_fail(MS_ERR_UNSUPPORTED, "section: head_dim=%d (supported: 64, 80, 128)", c->head_dim);
    if (c->d_model % 8 || c->d_ffn % 8)
        return ms_fail(MS_ERR_UNSUPPORTED, "section: d_model=%d and d_ffn=%d must be multiples of 8", c->d_model, c->d_ffn);
    if (!(c->norm_eps >= 0.f) || (c->arch == MS_DECODER && !(c->rope_base > 1.f)))
        return ms_fail(MS_ERR_INVALID_ARG, "section: norm_eps / rope_base out of range");
    return MS_OK;
}

// Limits of the kernels this call will launch, so that nothing fails after the first launch.
ms_status validate_limits(const ms_section_config *c, int n_tokens, bool backward) {
    if (backward && c->d_model > ms_norm_backward_max_d(c->dtype))
        return ms_fail(MS_ERR_UNSUPPORTED, "section: d_model=%d above %d, the widest row the norm backward kernel holds",
                       c->d_model, ms_norm_backward_max_d(c->dtype));
    if (c->dtype == MS_BF16 && !ms_attn_offsets_fit(n_tokens, c->n_q_heads, c->n_kv_heads, c->head_dim))
        return ms_fail(MS_ERR_UNSUPPORTED, "section: %d tokens x %d qkv columns exceed the 4 GiB the attention kernels address",
                       n_tokens, (c->n_q_heads + 2 * c->n_kv_heads) * c->head_dim);
    return MS_OK;
}

ms_status validate_batch(const ms_batch *b, int *max_seqlen) {
    if (!b) return ms_fail(MS_ERR_INVALID_ARG, "section: null batch");
    if (b->n_tokens < 0 || b->n_seqs < 0) return ms_fail(MS_ERR_INVALID_ARG, "section: negative batch size");
    *max_seqlen = 0;
    if (b->n_tokens == 0) return MS_OK;
    if (!b->cu_seqlens_host || !b->cu_seqlens_dev || b->n_seqs == 0)
        return ms_fail(MS_ERR_INVALID_ARG, "section: tokens without cu_seqlens");
    const int32_t *cu = b->cu_seqlens_host;
    if (cu[0] != 0 || cu[b->n_seqs] != b->n_tokens)
        return ms_fail(MS_ERR_INVALID_ARG, "section: cu_seqlens must start at 0 and end at n_tokens=%d", b->n_tokens);
    for (int i = 0; i < b->n_seqs; ++i) {
        if (cu[i + 1] < cu[i]) return ms_fail(MS_ERR_INVALID_ARG, "section: cu_seqlens decreases at %d", i);
        if (cu[i + 1] - cu[i] > *max_seqlen) *max_seqlen = cu[i + 1] - cu[i];
    }
    return MS_OK;
}

ms_status validate_ptrs(const ms_section_config *c, const ms_section_ptrs *w, const char *what) {
    if (!w || !w->layers) return ms_fail(MS_ERR_INVALID_ARG, "section: null %s", what);
    const bool enc = c->arch == MS_ENCODER;
    if ((c->vocab > 0 && !w->embedding) || !w->final_norm_g || (enc && !w->final_norm_b))
        return ms_fail(MS_ERR_INVALID_ARG, "section: %s: null embedding / final norm pointer", what);
    for (int i = 0; i < c->n_layers; ++i) {
        const ms_layer_ptrs &l = w->layers[i];
        if (!l.norm1_g || !l.w_qkv || !l.w_o || !l.norm2_g || !l.w_up || !l.w_down)
            return ms_fail(MS_ERR_INVALID_ARG, "section: %s: null pointer in layer %d", what, i);
        if (enc && (!l.norm1_b || !l.b_qkv || !l.b_o || !l.norm2_b || !l.b_up || !l.b_down))
            return ms_fail(MS_ERR_INVALID_ARG, "section: %s: null bias pointer in encoder layer %d", what, i);
    }
    return MS_OK;
}

struct Exec {
    const ms_section_config *c;
    Dims m;
    const ms_batch *b;
    Plan *p;
    hipStream_t s;
    int dt, kind;
    ColumnWork cols;              // column reductions of the backward pass
    const void *x0;               // first layer's input in the storage type, null if it is in the fp32 stream like the others'

    bool fp32_stream(const void *x) const { return x != x0; }
    ms_status gemm(int ta, int tb, int M, int N, int K, const void *A, long lda, const void *B, long ldb, void *C,
                   long ldc, bool c_fp32, bool acc, const void *bias, const void *res, long ldr) {
        return ms_k_gemm(dt, ta, tb, M, N, K, 1.f, A, lda, B, ldb, C, ldc, c_fp32, acc, bias, res, ldr, res && fp32_stream(res),
                         acc ? 0 : 1, s);
    }
    // y[n, out] = x[n, in] W[out, in]^T (+ bias) (+ res); with a residual, y is the fp32 stream
    ms_status linear(const void *x, int in, const void *W, const void *bias, int out, void *y, const void *res) {
        return gemm(0, 0, m.n, out, in, x, in, W, in, y, out, res != nullptr, false, bias, res, out);
    }
    // The biases' column sums: all four of a layer in one launch at its end, when the four output gradients are still there, up
    // to 8192 tokens (encoder layer d 1280, each behind its products -> at the end: 64 tokens 215 -> 206 us, 1031 393 -> 383, 2048 553 ->
    // 546; even from 3000 to 10000); above, each behind the products that read its matrix, while a part of that is in the Infinity Cache
    // (at the end 0.3-0.6 % slower from 12000 tokens on; 46173 tokens: the sums 177 us against 203).
    bool sums_at_end() const { return m.n <= 8192; }
    // dx[n, in] = dy[n, out] W[out, in];  dW[out, in] += dy[n, out]^T x[n, in];  db[out] += colsum(dy)
    ms_status linear_backward(const void *dy, int out, const void *W, int in, const void *x, void *dx, void *dW, void *db) {
        MS_TRY(ms_k_linear_backward(dt, m.n, out, in, dy, out, W, x, dx, 0, 0, dW, s));
        const ColSum sum = {dy, (float *)db, out};
        return db && !m.dec && !sums_at_end() ? column_sums_pending(dt, m.n, &sum, 1, &cols, s) : MS_OK;
    }

    ms_status prologue() {
        if (!m.dec) return MS_OK;
        return launch_rope_setup(m.n, b->n_seqs, b->cu_seqlens_dev, p->pos, m.max_seqlen, m.hd, c->rope_base, p->rope, s);
    }

    // The first layer's input: x_in itself, rows of the embedding table in `buf`, or, where x_in cannot be read in place (its
    // rows are not 16-byte aligned, or the call writes h_out or d_x_in over it before the backward pass is done with it), a
    // copy in the fp32 stream.
    ms_status first_input(const void *x_in, const ms_section_ptrs *weights, void *buf, const void *h_out, const void *d_x_in, const void **x) {
        const size_t bytes = (size_t)m.n * m.d * m.es;
        auto overlaps = [&](const void *q) { return q && (const char *)q < (const char *)x_in + bytes && (const char *)x_in < (const char *)q + bytes; };
        if (c->vocab > 0) {
            MS_TRY(ms_k_embedding_forward(dt, 0, m.n, m.d, c->vocab, (const int32_t *)x_in, weights->embedding, buf, s));
            x0 = *x = buf;
        } else if (dt == MS_F32) {
            x0 = *x = x_in;
        } else if (((uintptr_t)x_in & 15) == 0 && !overlaps(h_out) && !overlaps(d_x_in)) {
            x0 = *x = x_in;
        } else {
            MS_TRY(launch_convert_bf16_to_f32(x_in, (float *)buf, (long)m.n * m.d, s));
            *x = buf;
        }
        return MS_OK;
    }

    ms_status layer_forward(const ms_layer_ptrs &w, const void *x, LayerBuf &l, void *y) {
        bool done = false;
        if (m.dec && dt == MS_F32)
            MS_TRY(norm_qkv_rope_f32(m.n, m.d, m.nq + 2 * m.nkv, m.nq + m.nkv, m.hd, c->norm_eps, (const float *)x, (const float *)w.norm1_g,
                                     (const float *)w.w_qkv, p->pos, p->rope, (float *)l.qkv, p->bwd ? (float *)l.h1 : nullptr, l.rstd1, &done, s));
        if (!done) {
            MS_TRY(ms_k_norm_forward(kind, dt, fp32_stream(x), m.n, m.d, c->norm_eps, x, w.norm1_g, w.norm1_b, l.h1, l.mean1, l.rstd1, s));
            MS_TRY(linear(l.h1, m.d, w.w_qkv, m.dec ? nullptr : w.b_qkv, m.dqkv, l.qkv, nullptr));
            if (m.dec) MS_TRY(ms_k_rope(dt, m.n, m.nq + m.nkv, m.hd, m.dqkv, l.qkv, p->pos, p->rope, 0, s));
        }
        MS_TRY(ms_k_attention_forward(dt, m.dec, m.nq, m.nkv, m.hd, m.n, b->n_seqs, m.max_seqlen, b->cu_seqlens_dev,
                                      l.qkv, l.o, l.lse, s));
        MS_TRY(linear(l.o, m.dattn, w.w_o, m.dec ? nullptr : w.b_o, m.d, l.x2, x));
        // decoder, fp32: norm, gate/up and SwiGLU are one launch.  bf16: SwiGLU runs in the epilogue of the gate/up GEMM.  (The
        // pre-activations are only written when a backward pass will read them.)
        void *gu = p->bwd ? l.up : nullptr;
        done = false;
        if (m.dec && dt == MS_F32)
            MS_TRY(norm_swiglu_f32(m.n, m.d, m.f, c->norm_eps, (const float *)l.x2, (const float *)w.norm2_g, (const float *)w.w_up, (float *)l.act,
                                   (float *)gu, p->bwd ? (float *)l.h2 : nullptr, l.rstd2, &done, s));
        if (!done) {
            MS_TRY(ms_k_norm_forward(kind, dt, 1, m.n, m.d, c->norm_eps, l.x2, w.norm2_g, w.norm2_b, l.h2, l.mean2, l.rstd2, s));
            if (m.dec && dt == MS_BF16 && gemm_swiglu_supported(m.n, m.f, m.d, l.h2, m.d, w.w_up, m.d, l.act, m.f, gu, m.dup)) {
                MS_TRY(gemm_swiglu(m.n, m.f, m.d, l.h2, m.d, w.w_up, m.d, l.act, m.f, gu, m.dup, s));
            } else {
                MS_TRY(linear(l.h2, m.d, w.w_up, m.dec ? nullptr : w.b_up, m.dup, l.up, nullptr));
                MS_TRY(ms_k_act_forward(m.dec ? 0 : 1, dt, m.n, m.f, l.up, l.act, s));
            }
        }
        MS_TRY(linear(l.act, m.f, w.w_down, m.dec ? nullptr : w.b_down, m.d, y, l.x2));
        return MS_OK;
    }

    // dy: gradient of the layer output; dx: gradient of the layer input (distinct buffers)
    ms_status layer_backward(const ms_layer_ptrs &w, const ms_layer_ptrs &g, const LayerBuf &l, const void *dy, void *dx) {
        if (m.dec) {
            MS_TRY(ms_k_swiglu_linear_backward(dt, m.n, m.d, m.f, dy, w.w_down, l.act, l.up, p->da, p->dup, g.w_down, s));
        } else {
            MS_TRY(linear_backward(dy, m.d, w.w_down, m.f, l.act, p->da, g.w_down, g.b_down));
            MS_TRY(ms_k_act_backward(1, dt, m.n, m.f, p->da, l.up, p->dup, s));
        }
        MS_TRY(linear_backward(p->dup, m.dup, w.w_up, m.d, l.h2, p->dh, g.w_up, g.b_up));
        MS_TRY(norm_backward_pending(kind, dt, 1, m.n, m.d, p->dh, l.x2, w.norm2_g, l.mean2, l.rstd2, dy, p->dx2,
                                     (float *)g.norm2_g, (float *)g.norm2_b, &cols, s));
        MS_TRY(linear_backward(p->dx2, m.d, w.w_o, m.dattn, l.o, p->d_o, g.w_o, g.b_o));
        MS_TRY(ms_k_attention_backward(dt, m.dec, m.nq, m.nkv, m.hd, m.n, b->n_seqs, m.max_seqlen, b->cu_seqlens_dev,
                                       l.qkv, l.o, l.lse, p->d_o, p->dqkv, p->attn_scratch, s));
        if (m.dec) MS_TRY(ms_k_rope(dt, m.n, m.nq + m.nkv, m.hd, m.dqkv, p->dqkv, p->pos, p->rope, 1, s));
        MS_TRY(linear_backward(p->dqkv, m.dqkv, w.w_qkv, m.d, l.h1, p->dh, g.w_qkv, g.b_qkv));
        MS_TRY(norm_backward_pending(kind, dt, fp32_stream(l.x), m.n, m.d, p->dh, l.x, w.norm1_g, l.mean1, l.rstd1, p->dx2, dx,
                                     (float *)g.norm1_g, (float *)g.norm1_b, &cols, s));
        if (!m.dec && sums_at_end()) {
            const ColSum sums[4] = {{dy, (float *)g.b_down, m.d}, {p->dup, (float *)g.b_up, m.dup}, {p->dx2, (float *)g.b_o, m.d},
                                    {p->dqkv, (float *)g.b_qkv, m.dqkv}};
            MS_TRY(column_sums_pending(dt, m.n, sums, 4, &cols, s));
        }
        MS_TRY(column_work_finish(&cols, s));
        return MS_OK;
    }
};

}  // namespace

extern "C" size_t ms_section_workspace_bytes(const ms_section_config *cfg, int32_t max_tokens, int32_t max_seqlen,
                                             int32_t need_backward) {
    if (validate_config(cfg) != MS_OK || max_tokens < 0 || max_seqlen < 0) return 0;
    return make_plan(cfg, max_tokens, max_seqlen, need_backward != 0, nullptr).bytes;
}

extern "C" ms_status ms_section_forward(const ms_section_config *cfg, const ms_section_ptrs *weights,
                                        const ms_batch *batch, const void *x_in, void *h_out, void *workspace_dev,
                                        size_t workspace_bytes, void *stream) {
    MS_TRY(validate_config(cfg));
    int max_seqlen = 0;
    MS_TRY(validate_batch(batch, &max_seqlen));
    if (batch->n_tokens == 0) return MS_OK;
    MS_TRY(validate_limits(cfg, batch->n_tokens, false));
    MS_TRY(validate_ptrs(cfg, weights, "weights"));
    if (!x_in || !h_out || !workspace_dev) return ms_fail(MS_ERR_INVALID_ARG, "section_forward: null pointer");
    Plan p = make_plan(cfg, batch->n_tokens, max_seqlen, false, workspace_dev);
    if (workspace_bytes < p.bytes)
        return ms_fail(MS_ERR_WORKSPACE, "section_forward: workspace %zu < %zu bytes", workspace_bytes, p.bytes);
    Exec e{cfg, dims_of(cfg, batch->n_tokens, max_seqlen), batch, &p, (hipStream_t)stream, cfg->dtype,
           cfg->arch == MS_ENCODER ? 1 : 0, {}, nullptr};
    MS_TRY(e.prologue());
    const void *x = nullptr;
    MS_TRY(e.first_input(x_in, weights, p.xa, nullptr, nullptr, &x));
    for (int li = 0; li < cfg->n_layers; ++li) {
        void *y = li + 1 == cfg->n_layers ? p.y_last : (x == p.xa ? p.xb : p.xa);
        MS_TRY(e.layer_forward(weights->layers[li], x, p.layers[0], y));
        e.x0 = nullptr;                       // (its buffer takes a later layer's fp32 stream)
        x = y;
    }
    return ms_k_norm_forward(e.kind, e.dt, 1, e.m.n, e.m.d, cfg->norm_eps, x, weights->final_norm_g, weights->final_norm_b,
                             h_out, p.mean_f, p.rstd_f, e.s);
}

extern "C" ms_status ms_section_forward_backward(const ms_section_config *cfg, const ms_section_ptrs *weights,
                                                 const ms_section_ptrs *grads, const ms_batch *batch, const void *x_in,
                                                 void *h_out, const void *d_h_out, const ms_kd_config *kd,
                                                 const void *h_teacher, void *d_w_student, float *loss_dev,
                                                 float *kl_per_token_dev, void *d_x_in, void *workspace_dev,
                                                 size_t workspace_bytes, void *stream) {
    MS_TRY(validate_config(cfg));
    int max_seqlen = 0;
    MS_TRY(validate_batch(batch, &max_seqlen));
    hipStream_t s = (hipStream_t)stream;
    if (batch->n_tokens == 0) return (kd && loss_dev) ? launch_fill_f32(loss_dev, 1, 0.f, s) : MS_OK;
    if ((d_h_out != nullptr) == (kd != nullptr))
        return ms_fail(MS_ERR_INVALID_ARG, "section_forward_backward: give exactly one of d_h_out and kd");
    if (kd) {
        MS_TRY(validate_kd(kd, batch->n_tokens));
        if (kd->h_student != cfg->d_model || kd->dtype != cfg->dtype)
            return ms_fail(MS_ERR_SHAPE, "section_forward_backward: kd->h_student / dtype do not match the section");
        if (!loss_dev) return ms_fail(MS_ERR_INVALID_ARG, "section_forward_backward: loss_dev is null");
    }
    MS_TRY(validate_limits(cfg, batch->n_tokens, true));
    MS_TRY(validate_ptrs(cfg, weights, "weights"));
    MS_TRY(validate_ptrs(cfg, grads, "grads"));
    if (!x_in || !h_out || !workspace_dev || (kd && !h_teacher))
        return ms_fail(MS_ERR_INVALID_ARG, "section_forward_backward: null pointer");
    Plan p = make_plan(cfg, batch->n_tokens, max_seqlen, true, workspace_dev);
    const size_t kd_bytes = kd ? ms_kd_workspace_bytes(kd, batch->n_tokens) : 0;
    if (workspace_bytes < p.bytes + kd_bytes)
        return ms_fail(MS_ERR_WORKSPACE, "section_forward_backward: workspace %zu < %zu bytes", workspace_bytes, p.bytes + kd_bytes);
    Exec e{cfg, dims_of(cfg, batch->n_tokens, max_seqlen), batch, &p, s, cfg->dtype, cfg->arch == MS_ENCODER ? 1 : 0,
           {(char *)p.norm_scratch, p.norm_scratch_bytes, 0, 0, {}}, nullptr};
    MS_TRY(e.prologue());
    const int L = cfg->n_layers;
    const void *x = nullptr;
    MS_TRY(e.first_input(x_in, weights, p.layers[0].x, h_out, d_x_in, &x));
    for (int li = 0; li < L; ++li) {
        void *y = li + 1 == L ? p.y_last : p.layers[li + 1].x;
        p.layers[li].x = const_cast<void *>(x);
        MS_TRY(e.layer_forward(weights->layers[li], x, p.layers[li], y));
        x = y;
    }
    MS_TRY(ms_k_norm_forward(e.kind, e.dt, 1, e.m.n, e.m.d, cfg->norm_eps, p.y_last, weights->final_norm_g,
                             weights->final_norm_b, h_out, p.mean_f, p.rstd_f, s));
    const void *dh = d_h_out;
    if (kd) {
        MS_TRY(kd_forward_backward(kd, e.m.n, h_teacher, h_out, loss_dev, kl_per_token_dev, p.dhs, d_w_student,
                                   (char *)workspace_dev + p.bytes, workspace_bytes - p.bytes, s));
        dh = p.dhs;
    }
    void *dy = p.dy0;
    MS_TRY(norm_backward_pending(e.kind, e.dt, 1, e.m.n, e.m.d, dh, p.y_last, weights->final_norm_g, p.mean_f, p.rstd_f, nullptr,
                                 dy, (float *)grads->final_norm_g, (float *)grads->final_norm_b, &e.cols, s));
    for (int li = L - 1; li >= 0; --li) {
        void *dx = (li == 0 && cfg->vocab == 0 && d_x_in) ? d_x_in : (dy == p.dy0 ? p.dy1 : p.dy0);
        MS_TRY(e.layer_backward(weights->layers[li], grads->layers[li], p.layers[li], dy, dx));
        dy = dx;
    }
    if (cfg->vocab > 0)
        MS_TRY(ms_k_embedding_backward(e.dt, e.m.n, e.m.d, cfg->vocab, (const int32_t *)x_in, dy, (float *)grads->embedding, s));
    return MS_OK;
}
