"""The workloads whose speed is tracked: one training micro-batch's work in each kind of section.

Every case is a call a training program makes once per micro-batch (or per optimizer step) through the binding:
a frozen teacher's forward pass, a student's or vision encoder's forward and backward pass, the distillation
loss with both lm_heads, the vision -> language hand-off and the parameter update.  Widths are those of the
workload configurations c1 .. c5 (workloads.py); sections are one layer deep, except in the two whole
distillation steps, because a stack repeats its layer.  Token counts run from a single short sample to the
largest packed micro-batch of those workloads, with ragged lengths throughout.
"""
import math
import random

import torch
from torch.utils.checkpoint import checkpoint

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl

DEV = "cuda"
BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64

# d_model, query heads, key/value heads, head_dim, d_ffn
DECODERS = {"c1_teacher": (256, 4, 4, 64, 688), "c1_student": (128, 2, 2, 64, 344),
            "c2_teacher": (2048, 16, 4, 128, 5504), "c2_student": (1024, 8, 2, 128, 2816),
            "c5_teacher": (4096, 32, 8, 128, 11008), "c5_student": (1536, 12, 2, 128, 8960),
            "hd64": (1024, 16, 4, 64, 2816)}
ENCODER = (1280, 16, 16, 80, 5120)                                   # c4
HEADS = {"c2": (32000, 2048, 1024, 2.0), "c3": (151936, 4096, 2048, 2.0), "c5": (151936, 4096, 1536, 1.0)}
STEPS = {"c1": ("fp32", 2, 1, 1024, 1.0), "c2": ("bf16", 8, 4, 32000, 2.0)}   # dtype, teacher / student layers, vocab, T
# range of sequence lengths; "lognormal" and "long" as the workloads draw them
MIXES = {"short": (16, 128), "patches": (256, 4096)}


def listed():
    return [
        # c1: the whole fp32 distillation step on four short samples; launches and latency are what it costs
        dict(name="step_fp32", kind="step", cfg="c1", tokens=293, mix="short"),
        # c2 at a teacher micro-batch of one 4096-token pack: the whole bf16 step, embedding to gradients
        dict(name="step_bf16", kind="step", cfg="c2", tokens=4096, mix="lognormal"),
        # teacher layer on a single sample of odd length: the smallest call of a teacher worker
        dict(name="teacher_small", kind="forward", cfg="c2_teacher", tokens=777, mix="lognormal"),
        # teacher layer on the largest micro-batch (half short, half long documents)
        dict(name="teacher_large", kind="forward", cfg="c5_teacher", tokens=32768, mix="long"),
        # student layer forward + backward on a small micro-batch
        dict(name="student_small", kind="train", cfg="c2_student", tokens=2053, mix="lognormal"),
        # student layer forward + backward on the largest micro-batch
        dict(name="student_large", kind="train", cfg="c5_student", tokens=32768, mix="long"),
        # vision-encoder layer forward + backward on one image
        dict(name="encoder_small", kind="encoder", tokens=1031, mix="patches"),
        # vision-encoder layer forward + backward on a full image micro-batch
        dict(name="encoder_large", kind="encoder", tokens=46173, mix="patches"),
        # distillation loss on one short sample and on the c3 micro-batch
        dict(name="kd_small", kind="kd", cfg="c2", tokens=1024, chunk=8192, token_block=0, grads=True),
        dict(name="kd_large", kind="kd", cfg="c3", tokens=8192, chunk=8192, token_block=0, grads=True),
        # 4:1 merger + projector into the language model's stream, forward + backward
        dict(name="merger", kind="merger", d_llm=1536, groups=5771, text=4099),
        # AdamW over the parameters of the c2 student
        dict(name="adamw", kind="adamw", n=110_600_192, zero_grad=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "forward", "forward", "train", "train", "encoder", "encoder", "kd", "kd", "merger", "adamw"])
    if kind == "step":
        if rng.random() < 0.6:
            return dict(kind=kind, cfg="c1", tokens=_log_int(rng, 64, 2048), mix="short")
        return dict(kind=kind, cfg="c2", tokens=_log_int(rng, 512, 8192), mix="lognormal")
    if kind == "forward":
        cfg = rng.choice(["c2_teacher", "c5_teacher"])
        return dict(kind=kind, cfg=cfg, tokens=_log_int(rng, 256, 32768), mix="long" if cfg == "c5_teacher" else "lognormal")
    if kind == "train":
        cfg = rng.choice(["c2_student", "c5_student", "hd64"])
        return dict(kind=kind, cfg=cfg, tokens=_log_int(rng, 256, 32768), mix="long" if cfg == "c5_student" else "lognormal")
    if kind == "encoder":
        return dict(kind=kind, tokens=_log_int(rng, 256, 46173), mix="patches")
    if kind == "kd":
        grads = rng.random() < 0.8                                    # without: an evaluation pass
        block = rng.choice([0, 0, 1024]) if grads else 0              # 1024: teacher logits kept between the passes
        return dict(kind=kind, cfg=rng.choice(list(HEADS)), tokens=_log_int(rng, 128, 8192), chunk=rng.choice([4096, 8192]),
                    token_block=block, grads=grads)
    if kind == "merger":
        return dict(kind=kind, d_llm=rng.choice([1024, 1536, 2048]), groups=_log_int(rng, 64, 11543), text=_log_int(rng, 16, 8192))
    return dict(kind=kind, n=4 * _log_int(rng, 25_000, 27_650_048), zero_grad=rng.random() < 0.5)


# ------------------------------------------------------------------ shapes
def _lengths(case):
    """The case's sequence lengths: drawn from its mix until the token budget is full, the last one cut."""
    rng = random.Random("%(mix)s %(tokens)d" % case)
    out, left = [], case["tokens"]
    while left > 0:
        if case["mix"] == "lognormal":
            n = min(4096, max(64, round(1024 * math.exp(rng.gauss(0.0, 1.0)))))
        elif case["mix"] == "long":
            n = rng.randint(128, 1024) if rng.random() < 0.5 else rng.randint(4096, 16384)
        else:
            n = rng.randint(*MIXES[case["mix"]])
        out.append(min(n, left))
        left -= out[-1]
    return out


def _decoder(name, dtype="bf16", layers=1, vocab=0):
    d, nq, nkv, hd, f = DECODERS[name]
    return wl.SectionConfig("decoder", dtype, layers, d, nq, nkv, hd, f, vocab)


def _section(case):
    if case["kind"] == "encoder":
        d, nq, nkv, hd, f = ENCODER
        return wl.SectionConfig("encoder", "bf16", 1, d, nq, nkv, hd, f, 0)
    return _decoder(case["cfg"])


def _step(case):
    dtype, lt, ls, vocab, temp = STEPS[case["cfg"]]
    teacher = _decoder(case["cfg"] + "_teacher", dtype, lt, vocab)
    student = _decoder(case["cfg"] + "_student", dtype, ls, vocab)
    return teacher, student, wl.KDConfig(vocab, teacher.d_model, student.d_model, temp, 8192, dtype)


def _head(case):
    vocab, ht, hs, temp = HEADS[case["cfg"]]
    return wl.KDConfig(vocab, ht, hs, temp, case["chunk"], "bf16", case["token_block"])


# ------------------------------------------------------------------ inputs
class _Gen:
    """Normal and integer tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(seed)

    def normal(self, shape, std, mean=0.0, dtype=BF16):
        t = torch.empty(shape, dtype=F32, device=DEV).normal_(mean, std, generator=self.g)
        return t.to(dtype)

    def ints(self, n, hi):
        return torch.randint(0, hi, (n,), device=DEV, generator=self.g).to(torch.int32)


def _weights(cfg, gen):
    """Matrices, embedding and biases N(0, 0.02), norm gains 1 + N(0, 0.02)."""
    dt, d, dup = cfg.torch_dtype, cfg.d_model, cfg.d_up

    def mat(*shape):
        return gen.normal(shape, 0.02, dtype=dt)

    def layer():
        w = dict(norm1_g=gen.normal((d,), 0.02, 1.0, dt), w_qkv=mat(cfg.d_qkv, d), w_o=mat(d, cfg.n_q_heads * cfg.head_dim),
                 norm2_g=gen.normal((d,), 0.02, 1.0, dt), w_up=mat(dup, d), w_down=mat(d, cfg.d_ffn))
        if cfg.arch == "encoder":
            w.update(norm1_b=mat(d), b_qkv=mat(cfg.d_qkv), b_o=mat(d), norm2_b=mat(d), b_up=mat(dup), b_down=mat(d))
        return w

    w = dict(embedding=mat(cfg.vocab, d) if cfg.vocab else None, layers=[layer() for _ in range(cfg.n_layers)],
             final_norm_g=gen.normal((d,), 0.02, 1.0, dt))
    if cfg.arch == "encoder":
        w["final_norm_b"] = mat(d)
    return w


def _flat_grads(tensors):
    """fp32 gradient views of one flat buffer (a training program clears it with one fill), each 256-byte aligned."""
    sizes = [(t.numel() + 63) // 64 * 64 for t in tensors]
    flat = torch.zeros(sum(sizes), dtype=F32, device=DEV)
    views, at = [], 0
    for t, n in zip(tensors, sizes):
        views.append(flat[at:at + t.numel()].view(t.shape))
        at += n
    return flat, views


def _section_grads(w, extra=()):
    keys = [(None, k) for k in w if k != "layers" and w[k] is not None]
    keys += [(i, k) for i, lw in enumerate(w["layers"]) for k in lw]
    flat, views = _flat_grads([w[k] if i is None else w["layers"][i][k] for i, k in keys] + list(extra))
    g = dict(layers=[{} for _ in w["layers"]])
    for (i, k), v in zip(keys, views):
        (g if i is None else g["layers"][i])[k] = v
    return flat, g, views[len(keys):]


def prepare(case, seed):
    gen, kind = _Gen(seed), case["kind"]
    s = dict(case=case, kind=kind)
    if kind == "step":
        s["teacher"], s["student"], s["kd"] = _step(case)
        dt = s["teacher"].torch_dtype
        s["batch"] = B.Batch(wl.cu_seqlens_of(_lengths(case)))
        s["ids"] = gen.ints(case["tokens"], s["kd"].vocab)
        s["tw"], s["sw"] = _weights(s["teacher"], gen), _weights(s["student"], gen)
        s["w_t"] = gen.normal((s["kd"].vocab, s["kd"].h_teacher), 0.02, dtype=dt)
        s["w_s"] = gen.normal((s["kd"].vocab, s["kd"].h_student), 0.02, dtype=dt)
        s["flat"], s["grads"], (s["d_w_s"],) = _section_grads(s["sw"], [s["w_s"]])
    elif kind in ("forward", "train", "encoder"):
        s["cfg"] = cfg = _section(case)
        s["batch"] = B.Batch(wl.cu_seqlens_of(_lengths(case)))
        s["w"] = _weights(cfg, gen)
        s["x"] = gen.normal((case["tokens"], cfg.d_model), 1.0)
        if kind != "forward":
            s["dh"] = gen.normal((case["tokens"], cfg.d_model), 1.0)
            s["flat"], s["grads"], _ = _section_grads(s["w"])
    elif kind == "kd":
        s["kd"] = kd = _head(case)
        s["w_t"], s["w_s"] = gen.normal((kd.vocab, kd.h_teacher), 0.02), gen.normal((kd.vocab, kd.h_student), 0.02)
        s["h_t"], s["h_s"] = gen.normal((case["tokens"], kd.h_teacher), 1.0), gen.normal((case["tokens"], kd.h_student), 1.0)
        if case["grads"]:
            s["d_w_s"] = torch.zeros((kd.vocab, kd.h_student), dtype=F32, device=DEV)
    elif kind == "merger":
        d_vit, d_llm, n = ENCODER[0], case["d_llm"], case["groups"]
        hidden = 4 * d_vit
        s["w"] = dict(w1=gen.normal((hidden, hidden), 0.02), b1=gen.normal((hidden,), 0.02),
                      w2=gen.normal((d_llm, hidden), 0.02), b2=gen.normal((d_llm,), 0.02))
        s["h_vit"] = gen.normal((4 * n, d_vit), 1.0)
        order = torch.randperm(n + case["text"], device=DEV, generator=gen.g)[:n]
        s["pos"] = order.sort().values.to(torch.int32)
        s["x_llm"] = gen.normal((n + case["text"], d_llm), 0.02)
        s["d_x_llm"] = gen.normal((n + case["text"], d_llm), 1.0)
        s["flat"], views = _flat_grads([s["w"][k] for k in ("w1", "b1", "w2", "b2")])
        s["grads"] = dict(zip(("w1", "b1", "w2", "b2"), views))
        s["ws"] = torch.empty(B.merger_workspace_bytes(s["w"], n), dtype=torch.uint8, device=DEV)
    else:
        n = case["n"]
        s["master"] = gen.normal((n,), 0.02, dtype=F32)
        s["weight"] = s["master"].to(BF16)
        s["grad"] = gen.normal((n,), 1e-3, dtype=F32)
        s["m"] = gen.normal((n,), 1e-3, dtype=F32)
        s["v"] = gen.normal((n,), 1e-3, dtype=F32).square_()
    return s


# ------------------------------------------------------------------ one pass
ADAMW = dict(step=100, lr=1e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1, grad_scale=0.5)


def _tree(d):
    return {k: v for k, v in d.items() if v is not None}


def run(s):
    kind = s["kind"]
    if kind == "step":
        s["flat"].zero_()
        h_t = B.section_forward(s["teacher"], s["tw"], s["batch"], s["ids"])
        out = B.section_forward_backward(s["student"], s["sw"], s["grads"], s["batch"], s["ids"], kd=s["kd"],
                                         w_teacher=s["w_t"], w_student=s["w_s"], h_teacher=h_t, d_w_student=s["d_w_s"])
        return dict(_tree(out), h_teacher=h_t, grads=s["grads"], d_w_student=s["d_w_s"])
    if kind == "forward":
        return B.section_forward(s["cfg"], s["w"], s["batch"], s["x"])
    if kind in ("train", "encoder"):
        s["flat"].zero_()
        out = B.section_forward_backward(s["cfg"], s["w"], s["grads"], s["batch"], s["x"], d_h_out=s["dh"], want_d_x_in=True)
        return dict(_tree(out), grads=s["grads"])
    if kind == "kd":
        if not s["case"]["grads"]:
            return _tree(B.kd_loss_forward_backward(s["kd"], s["w_t"], s["w_s"], s["h_t"], s["h_s"], need_d_h=False))
        s["d_w_s"].zero_()
        out = B.kd_loss_forward_backward(s["kd"], s["w_t"], s["w_s"], s["h_t"], s["h_s"], d_w_student=s["d_w_s"])
        return dict(out, d_w_student=s["d_w_s"])
    if kind == "merger":
        s["flat"].zero_()
        B.merger_forward(s["w"], s["h_vit"], s["pos"], s["x_llm"], s["ws"])
        d_h = B.merger_backward(s["w"], s["grads"], s["h_vit"], s["pos"], s["d_x_llm"], s["ws"])
        return dict(x_llm=s["x_llm"], d_h_vit=d_h, grads=s["grads"])
    B.adamw_step(s["grad"], s["master"], s["m"], s["v"], s["weight"], zero_grad=s["case"]["zero_grad"], **ADAMW)
    return dict(master=s["master"], m=s["m"], v=s["v"], weight=s["weight"], grad=s["grad"])


# ------------------------------------------------------------------ necessary work
def _pairs(case, causal):
    return sum(n * (n + 1) // 2 if causal else n * n for n in _lengths(case))


def _section_work(cfg, n, pairs, bwd, es):
    """(flops, bytes): linears and attention products; weights and ends of the section once."""
    linear = 2.0 * n * cfg.layer_params() * cfg.n_layers
    attn = 4.0 * cfg.n_q_heads * cfg.head_dim * pairs * cfg.n_layers
    params = cfg.layer_params() * cfg.n_layers
    flops = linear * (3 if bwd else 1) + attn * (3.5 if bwd else 1)      # S, PV; backward S, dP, dV, dK, dQ
    ends = n * cfg.d_model * es * (4 if bwd else 2) if not cfg.vocab else n * (cfg.d_model * es * (2 + 2 * bwd) + 4)
    return flops, params * (es + (4 if bwd else 0)) + ends


def _kd_work(kd, n, grads, es):
    flops = 2.0 * n * kd.vocab * (kd.h_teacher + kd.h_student * (3 if grads else 1))
    size = kd.vocab * (kd.h_teacher + kd.h_student) * es + n * (kd.h_teacher + kd.h_student * (2 if grads else 1)) * es + 4 * n
    return flops, size + (4 * kd.vocab * kd.h_student if grads else 0)


def work(case):
    kind = case["kind"]
    if kind == "step":
        teacher, student, kd = _step(case)
        es, n, pairs = 4 if kd.dtype == "fp32" else 2, case["tokens"], _pairs(case, True)
        parts = [_section_work(teacher, n, pairs, False, es), _section_work(student, n, pairs, True, es), _kd_work(kd, n, True, es)]
        extra = 4.0 * kd.vocab * student.d_model                         # the embedding gradient is cleared and returned
        return dict(flops=sum(p[0] for p in parts), bytes=sum(p[1] for p in parts) + extra)
    if kind in ("forward", "train", "encoder"):
        flops, size = _section_work(_section(case), case["tokens"], _pairs(case, kind != "encoder"), kind != "forward", 2)
        return dict(flops=flops, bytes=size)
    if kind == "kd":
        flops, size = _kd_work(_head(case), case["tokens"], case["grads"], 2)
        return dict(flops=flops, bytes=size)
    if kind == "merger":
        n, hidden, d_llm = case["groups"], 4 * ENCODER[0], case["d_llm"]
        params = hidden * hidden + d_llm * hidden
        return dict(flops=6.0 * n * params, bytes=params * 6.0 + n * (2 * hidden + 2 * d_llm) * 2.0)
    return dict(flops=15.0 * case["n"], bytes=(30.0 + 4 * case["zero_grad"]) * case["n"])


def tolerance(case):
    """About four times the error of the path against `exact`, for each kind and precision."""
    if case["kind"] == "adamw":
        return {"rel": 2e-3, "max": 1e-2}                               # the bf16 weights: a rounding tie; fp32 state 1e-6
    if case["kind"] == "step":
        return {"rel": 1e-5, "max": 1e-3} if case["cfg"] == "c1" else {"rel": 0.03, "max": 0.9}
    if case["kind"] in ("kd", "merger"):
        return {"rel": 0.01, "max": 0.3}
    return {"rel": 0.02, "max": 0.5}


# ------------------------------------------------------------------ the same in 64 bits
def _norm(x, g, b, eps):
    if b is None:
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g
    mu = x.mean(-1, keepdim=True)
    return (x - mu) * torch.rsqrt((x - mu).square().mean(-1, keepdim=True) + eps) * g + b


def _head_attention(q, k, v, causal):
    s = q @ k.T / math.sqrt(q.shape[1])
    if causal:
        s = s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), -math.inf)
    return s.softmax(-1) @ v


def _attention(qkv, cu, cfg):
    nq, nkv, hd = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    causal, x = cfg.arch == "decoder", qkv.view(-1, nq + 2 * nkv, hd)
    rows = []
    for a, b in zip(cu[:-1], cu[1:]):
        if causal:
            ang = torch.arange(b - a, device=DEV, dtype=F64)[:, None] * cfg.rope_base ** (
                -2.0 * torch.arange(hd // 2, device=DEV, dtype=F64) / hd)
            c, s = ang.cos()[:, None], ang.sin()[:, None]
            lo, hi = x[a:b, :nq + nkv].split(hd // 2, -1)
            qk = torch.cat([lo * c - hi * s, hi * c + lo * s], -1)
        else:
            qk = x[a:b, :nq + nkv]
        heads = [checkpoint(_head_attention, qk[:, h], qk[:, nq + h * nkv // nq], x[a:b, nq + nkv + h * nkv // nq], causal,
                            use_reentrant=False) for h in range(nq)]
        rows.append(torch.cat(heads, -1))
    return torch.cat(rows)


def _exact_section(cfg, w, cu, x):
    dec = cfg.arch == "decoder"
    for lw in w["layers"]:
        def lin(t, name):
            y = t @ lw["w_" + name].T
            return y if dec else y + lw["b_" + name]
        h = _norm(x, lw["norm1_g"], lw.get("norm1_b"), cfg.norm_eps)
        x = x + lin(_attention(lin(h, "qkv"), cu, cfg), "o")
        up = lin(_norm(x, lw["norm2_g"], lw.get("norm2_b"), cfg.norm_eps), "up")
        if dec:
            gate, up = up.split(cfg.d_ffn, -1)
            act = torch.nn.functional.silu(gate) * up
        else:
            act = torch.nn.functional.gelu(up)
        x = x + lin(act, "down")
    return _norm(x, w["final_norm_g"], w.get("final_norm_b"), cfg.norm_eps)


def _double(t, grad=False):
    if isinstance(t, dict):
        return {k: _double(v, grad) for k, v in t.items() if v is not None}
    if isinstance(t, list):
        return [_double(v, grad) for v in t]
    return t.double().requires_grad_(grad)


def _grads_of(w):
    if isinstance(w, dict):
        return {k: _grads_of(v) for k, v in w.items()}
    return [_grads_of(v) for v in w] if isinstance(w, list) else w.grad


def _exact_kd(kd, w_t, w_s, h_t, h_s):
    lt = torch.log_softmax(h_t @ w_t.T / kd.temperature, -1)
    ls = torch.log_softmax(h_s @ w_s.T / kd.temperature, -1)
    return (lt.exp() * (lt - ls)).sum(-1)


def exact(case, seed):
    s, kind = prepare(case, seed), case["kind"]
    if kind == "forward":
        with torch.no_grad():
            return _exact_section(s["cfg"], _double(s["w"]), s["batch"].cu, s["x"].double())
    if kind in ("train", "encoder"):
        w, x = _double(s["w"], True), s["x"].double().requires_grad_()
        h = _exact_section(s["cfg"], w, s["batch"].cu, x)
        h.backward(s["dh"].double())
        return dict(h_out=h.detach(), d_x_in=x.grad, grads=_grads_of(w))
    if kind == "step":
        ids = s["ids"].long()
        with torch.no_grad():
            tw = _double(s["tw"])
            h_t = _exact_section(s["teacher"], tw, s["batch"].cu, tw["embedding"][ids])
        sw, w_s = _double(s["sw"], True), s["w_s"].double().requires_grad_()
        h_s = _exact_section(s["student"], sw, s["batch"].cu, sw["embedding"][ids])
        kl = _exact_kd(s["kd"], s["w_t"].double(), w_s, h_t, h_s)
        kl.mean().backward()
        return dict(h_out=h_s.detach(), loss=kl.mean().detach(), kl_tok=kl.detach(), h_teacher=h_t, grads=_grads_of(sw),
                    d_w_student=w_s.grad)
    if kind == "kd":
        out = dict(loss=0.0, kl_tok=[], d_h_s=[], d_w_student=0.0)
        w_t, w_s, n = s["w_t"].double(), s["w_s"].double(), case["tokens"]
        for a in range(0, n, 2048):                                     # rows are independent; a block at a time
            h_t, h_s = s["h_t"][a:a + 2048].double(), s["h_s"][a:a + 2048].double()
            h_s.requires_grad_(case["grads"])
            w_s.requires_grad_(case["grads"])
            kl = _exact_kd(s["kd"], w_t, w_s, h_t, h_s)
            if case["grads"]:
                (kl.sum() / n).backward()
                out["d_h_s"].append(h_s.grad)
            out["kl_tok"].append(kl.detach())
        out["kl_tok"] = torch.cat(out["kl_tok"])
        out["loss"] = out["kl_tok"].mean()
        if not case["grads"]:
            return dict(loss=out["loss"], kl_tok=out["kl_tok"])
        return dict(out, d_h_s=torch.cat(out["d_h_s"]), d_w_student=w_s.grad)
    if kind == "merger":
        w, h, pos = _double(s["w"], True), s["h_vit"].double().requires_grad_(), s["pos"].long()
        y = torch.nn.functional.gelu(h.view(case["groups"], -1) @ w["w1"].T + w["b1"]) @ w["w2"].T + w["b2"]
        y.backward(s["d_x_llm"].double()[pos])
        x = s["x_llm"].double()
        x[pos] = y.detach()
        return dict(x_llm=x, d_h_vit=h.grad, grads=_grads_of(w))
    a, step = ADAMW, ADAMW["step"]
    g = a["grad_scale"] * s["grad"].double()
    m = a["beta1"] * s["m"].double() + (1 - a["beta1"]) * g
    v = a["beta2"] * s["v"].double() + (1 - a["beta2"]) * g * g
    master = s["master"].double() * (1 - a["lr"] * a["weight_decay"]) - a["lr"] * (m / (1 - a["beta1"] ** step)) / (
        (v / (1 - a["beta2"] ** step)).sqrt() + a["eps"])
    return dict(master=master, m=m, v=v, weight=master, grad=torch.zeros_like(g) if case["zero_grad"] else s["grad"].double())
