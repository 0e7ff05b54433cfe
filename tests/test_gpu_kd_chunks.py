"""The distillation loss over few and many vocabulary chunks: which logits of the first pass are still there in the second
(the last two chunks' on the fused path, the last one's otherwise) depends on the number of chunks and on their width."""
import pytest
import torch

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl
from test_gpu_section import _kd_loss_standalone

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,ht,hs", [("bf16", 128, 64), ("bf16", 72, 40), ("fp32", 72, 40)])   # fused, not fused, fp32
@pytest.mark.parametrize("vocab,chunk", [(256, 512), (256, 256), (256, 128), (328, 128), (648, 128), (40, 8), (64, 16), (296, 72)])
def test_chunk_counts_and_widths(dtype, ht, hs, vocab, chunk):
    _kd_loss_standalone(dtype, vocab, chunk, 45, ht, hs, 1.5, 0)


# bf16 heads whose student and teacher products share launches: every tile, ragged rows and columns, chunks of unequal width, a
# round of tiles of one kind and more (kinds take turns in runs of 256 workgroups)
@pytest.mark.parametrize("n,vocab,chunk,ht,hs", [(45, 648, 128, 128, 64), (300, 1000, 264, 64, 192), (130, 3 * 8192 + 520, 8192, 64, 64), (2100, 6 * 2048, 2048, 64, 64)])
@pytest.mark.parametrize("tile", [0, 256, 128, 128128, 128256, 64064])
def test_shared_launches_on_every_tile(tile, n, vocab, chunk, ht, hs):
    g = torch.Generator(device="cuda").manual_seed(n)
    rand = lambda *s, std=1.0: torch.empty(s, device="cuda").normal_(0, std, generator=g).bfloat16()
    w_t, w_s, h_t, h_s = rand(vocab, ht, std=0.1), rand(vocab, hs, std=0.1), rand(n, ht), rand(n, hs)
    d_ws = torch.zeros(vocab, hs, device="cuda")
    kd = wl.KDConfig(vocab, ht, hs, 2.0, chunk, "bf16", 0)
    try:
        B.k_gemm_config(tile, -1)
        out = B.kd_loss_forward_backward(kd, w_t, w_s, h_t, h_s, d_w_student=d_ws)
        ev = B.kd_loss_forward_backward(kd, w_t, w_s, h_t, h_s, need_d_h=False)
    finally:
        B.k_gemm_config(0, -1)
    lt, ls = (torch.log_softmax(h.double() @ w.double().T / 2.0, -1) for h, w in ((h_t, w_t), (h_s, w_s)))
    kl = (lt.exp() * (lt - ls)).sum(-1)
    dz = (ls.exp() - lt.exp()) / (2.0 * n)
    # fp32 log-sum-exps of about 8 in kl; bf16 dz (2^-9 relative, independent) in the gradients, with a margin of 4
    assert ((out["kl_tok"].double() - kl).norm() / kl.norm()).item() < 1e-4 and torch.equal(ev["kl_tok"], out["kl_tok"])
    for got, ref in ((out["d_h_s"], dz @ w_s.double()), (d_ws, dz.T @ h_s.double())):
        assert ((got.double() - ref).norm() / ref.norm()).item() < 2 ** -7
