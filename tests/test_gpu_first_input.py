"""The first layer reads a bf16 input where it is: the same bits as through the copy that is made of an input that cannot be
read in place (rows not 16-byte aligned, or h_out written over it), and as through the embedding table."""
import ctypes as C

import pytest
import torch

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl

pytestmark = pytest.mark.gpu
LENGTHS = [70, 1, 129]


def _section(arch, vocab):
    cfg = wl.SectionConfig(arch, "bf16", 3, 256, 4, 4, 64, 512, vocab)
    g = torch.Generator(device="cuda").manual_seed(7)
    rand = lambda *shape, std=0.05, mean=0.0: torch.empty(shape, device="cuda").normal_(mean, std, generator=g).bfloat16()
    d, dup = cfg.d_model, cfg.d_up
    def layer():
        w = dict(norm1_g=rand(d, mean=1.0), w_qkv=rand(cfg.d_qkv, d), w_o=rand(d, 256), norm2_g=rand(d, mean=1.0), w_up=rand(dup, d),
                 w_down=rand(d, cfg.d_ffn))
        return dict(w, norm1_b=rand(d), b_qkv=rand(cfg.d_qkv), b_o=rand(d), norm2_b=rand(d), b_up=rand(dup), b_down=rand(d)) if arch == "encoder" else w
    w = dict(embedding=rand(vocab, d, std=1.0) if vocab else None, layers=[layer() for _ in range(3)], final_norm_g=rand(d, mean=1.0))
    if arch == "encoder":
        w["final_norm_b"] = rand(d)
    return cfg, w, rand(sum(LENGTHS), d, std=1.0), rand(sum(LENGTHS), d, std=1.0)


@pytest.mark.parametrize("arch", ["encoder", "decoder"])
def test_in_place_copied_and_embedded_inputs_agree(arch):
    cfg, w, x, dh = _section(arch, 0)
    batch, n = B.Batch(wl.cu_seqlens_of(LENGTHS)), sum(LENGTHS)
    def both(c, wt, inp):
        out = B.section_forward_backward(c, wt, B.zero_grads(wt), batch, inp, d_h_out=dh, want_d_x_in=True)
        return [B.section_forward(c, wt, batch, inp), out["h_out"], out["d_x_in"]]
    ref = both(cfg, w, x)
    assert torch.equal(ref[0], ref[1])
    shifted = torch.empty(n * cfg.d_model + 8, dtype=torch.bfloat16, device="cuda")[1:n * cfg.d_model + 1].view(n, -1)
    shifted.copy_(x)
    assert all(torch.equal(a, b) for a, b in zip(ref, both(cfg, w, shifted)))
    # h_out over x_in
    io, d_x, c, b, g = x.clone(), torch.empty_like(x), B._cfg_c(cfg), batch.c(), B.zero_grads(w)
    ws = B.workspace(B.section_workspace_bytes(cfg, n, batch.max_seqlen, True), "cuda")
    null = C.c_void_p(0)
    B._check(B.lib().ms_section_forward_backward(C.byref(c), C.byref(B._ptrs_c(cfg, w)), C.byref(B._ptrs_c(cfg, g)), C.byref(b), B._p(io), B._p(io), B._p(dh),
                                                 null, null, null, null, null, B._p(d_x), B._p(ws), C.c_size_t(ws.numel()), B._stream()))
    assert torch.equal(io, ref[1]) and torch.equal(d_x, ref[2])
    # the same rows out of an embedding table (all three layers of the forward-only ping-pong)
    cfg_e = wl.scaled(cfg, vocab=n)
    out = B.section_forward(cfg_e, dict(w, embedding=x), batch, torch.arange(n, dtype=torch.int32, device="cuda"))
    assert torch.equal(out, ref[0])
