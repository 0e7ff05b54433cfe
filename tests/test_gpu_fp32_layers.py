"""fp32 decoder layers through the fused launches (norm + QKV + rotary embedding, norm + gate / up + SwiGLU) and, where these do not
apply (head_dim 80, rows not 16-byte aligned), the kernels one by one; against the oracle, forward and backward."""
import pytest
import torch

from oracle import identity
from oracle.section import section_backward, section_forward
from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl
from parity import TOL_F32, assert_parity
from test_gpu_section import check_grads, spec_of

pytestmark = pytest.mark.gpu


# widths below, at and above the 16-deep slices of K and the 16-column blocks; one token, tiles of 32 rows with remainders
@pytest.mark.parametrize("lengths", [[1], [31, 1, 33], [64, 0, 70]])
@pytest.mark.parametrize("d,nq,nkv,hd,f", [(8, 1, 1, 64, 8), (72, 2, 1, 64, 24), (136, 2, 2, 128, 344), (64, 1, 1, 80, 40), (520, 3, 1, 64, 136)])
def test_layers_against_the_oracle(lengths, d, nq, nkv, hd, f):
    cfg = wl.SectionConfig("decoder", "fp32", 2, d, nq, nkv, hd, f, 0)
    cu = wl.cu_seqlens_of(lengths)
    n = cu[-1]
    w = wl.section_weights(cfg, 3, "s", "cuda")
    x, d_h = wl.normal(3, "x", (n, d), 1.0, 0.0, torch.float32, "cuda"), wl.normal(3, "dh", (n, d), 1.0, 0.0, torch.float32, "cuda")
    grads = B.zero_grads(w)
    out = B.section_forward_backward(cfg, w, grads, B.Batch(cu), x, d_h_out=d_h, want_d_x_in=True)
    h, cache = section_forward(spec_of(cfg), wl.to_f64(w), cu, wl.to_f64(x), identity, keep=True)
    g_ref, dx_ref = section_backward(spec_of(cfg), wl.to_f64(w), cu, cache, wl.to_f64(d_h), identity)
    assert_parity(out["h_out"], h, TOL_F32, "h_out")
    assert_parity(out["d_x_in"], dx_ref, TOL_F32, "d_x_in")
    check_grads(grads, g_ref, 2e-4)
    assert torch.equal(B.section_forward(cfg, w, B.Batch(cu), x), out["h_out"])      # nothing is kept for a backward pass


def test_unaligned_weights_take_the_separate_kernels():
    cfg = wl.SectionConfig("decoder", "fp32", 1, 64, 1, 1, 64, 48, 0)
    w = wl.section_weights(cfg, 4, "s", "cuda")
    x, batch = wl.normal(4, "x", (50, 64), 1.0, 0.0, torch.float32, "cuda"), B.Batch([0, 20, 50])
    ref = B.section_forward(cfg, w, batch, x)
    shifted = dict(w, layers=[dict(w["layers"][0])])
    for k in ("w_qkv", "w_up"):
        t = w["layers"][0][k]
        buf = torch.empty(t.numel() + 4, device="cuda")[1:t.numel() + 1].view(t.shape)      # 4 bytes off
        shifted["layers"][0][k] = buf.copy_(t)
    out = B.section_forward(cfg, shifted, batch, x)
    assert ((out - ref).norm() / ref.norm()).item() < 8 * 64 ** 0.5 * 2 ** -24       # sums of 64 .. in another order


def test_an_infinite_value_column_stays_alone():
    """Values are not rotated: an infinite column of V leaves the column half a head away as it is."""
    cfg = wl.SectionConfig("decoder", "fp32", 1, 64, 2, 1, 64, 48, 0)
    w = wl.section_weights(cfg, 5, "s", "cuda")
    x, batch, n = wl.normal(5, "x", (50, 64), 1.0, 0.0, torch.float32, "cuda"), B.Batch([0, 20, 50]), 50
    ws = torch.zeros(B.section_workspace_bytes(cfg, n, 30, False), dtype=torch.uint8, device="cuda")
    qkv = ws[(n * 64 * 4 + 255) // 256 * 256:][:n * cfg.d_qkv * 4].view(torch.float32).view(n, cfg.d_qkv)    # behind the normed rows
    B.section_forward(cfg, w, batch, x, ws=ws)
    ref = qkv.clone()
    for col in (3 * 64 + 5, 3 * 64 + 32 + 20):                     # one in each half of the value head
        bad = dict(w, layers=[dict(w["layers"][0])])
        bad["layers"][0]["w_qkv"] = w["layers"][0]["w_qkv"].clone()
        bad["layers"][0]["w_qkv"][col, 7] = float("inf")
        B.section_forward(cfg, bad, batch, x, ws=ws)
        assert not torch.isfinite(qkv[:, col]).any()
        keep = [c for c in range(cfg.d_qkv) if c != col]
        assert torch.equal(qkv[:, keep], ref[:, keep])
