"""Row statistics of the student-logits product's epilogue (max, sums of exponentials, cross term over strips of 64 columns): vocabulary
widths around the edges of a strip, rows around the 16 and 32 of a block, logits far apart and single columns
with nearly the type's lowest value (a masked vocabulary entry), on every tile and both matrix instructions."""
import pytest
import torch

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,mfma", [(256, -1), (128, -1), (128128, -1), (128256, -1), (64128, -1), (64064, -1), (256, 0), (128, 0)])
@pytest.mark.parametrize("n,vocab", [(1, 8), (15, 56), (16, 64), (17, 72), (33, 248), (257, 264), (31, 328), (130, 8)])
def test_statistics_at_the_edges(tile, mfma, n, vocab):
    h = 64
    g = torch.Generator(device="cuda").manual_seed(vocab)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(0, 1, generator=g).bfloat16()
    w_t, w_s, h_t, h_s = rand(vocab, h), rand(vocab, h), rand(n, h), rand(n, h)                # logits of about +-8, up to +-30
    h_t[:, 0] = 1
    w_t[3::64, 0] = -3e37
    kd = wl.KDConfig(vocab, h, h, 1.0, vocab, "bf16", 0)
    try:
        B.k_gemm_config(tile, mfma)
        out = B.kd_loss_forward_backward(kd, w_t, w_s, h_t, h_s, need_d_h=False)
    finally:
        B.k_gemm_config(0, -1)
    lt, ls = (torch.log_softmax(a.double() @ w.double().T, -1) for a, w in ((h_t, w_t), (h_s, w_s)))
    p = lt.exp()
    kl = (p * torch.where(p > 0, lt - ls, 0)).sum(-1)
    # fp32 logits of 64 products (2^-24 x 64 x |z| <= 1.2e-4 at |z| = 30) enter as differences, weighted by probabilities that sum to 1,
    # four times: as lt, ls and in both normalisations
    assert torch.isfinite(out["kl_tok"]).all()
    assert ((out["kl_tok"].double() - kl).abs() <= 5e-4 + 1e-5 * kl.abs()).all()
    assert abs(out["loss"].item() - kl.mean().item()) <= 5e-4 + 1e-5 * kl.mean().item()
