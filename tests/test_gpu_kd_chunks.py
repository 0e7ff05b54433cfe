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
# round of tiles of one kind and more (kinds take turns in runs of 256 or 512 workgroups), the longer ones first: teacher or student
@pytest.mark.parametrize("n,vocab,chunk,ht,hs", [(45, 648, 128, 128, 64), (300, 1000, 264, 64, 192), (130, 3 * 8192 + 520, 8192, 64, 64), (2100, 6 * 2048, 2048, 64, 64),
                                                 (2100, 3 * 2048, 2048, 64, 192)])
@pytest.mark.parametrize("tile", [0, 256, 128, 128128, 128256, 64128, 64064])
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


@pytest.mark.parametrize("token_block", [0, 40])
@pytest.mark.parametrize("over", ["h_s", "h_t"])
def test_fp32_gradient_over_an_input(over, token_block):
    """d_h_student may be the tensor that holds the student's (or an equally wide teacher's) states: the same bits as apart from it, where
    the gradient adds up in the result itself.  97 tokens: three token blocks of 40, one without."""
    n, vocab, h = 97, 296, 40
    g = torch.Generator(device="cuda").manual_seed(4)
    rand = lambda *s, std=1.0: torch.empty(s, device="cuda").normal_(0, std, generator=g)
    w_t, w_s, h_t, h_s = rand(vocab, h, std=0.1), rand(vocab, h, std=0.1), rand(n, h), rand(n, h)
    kd = wl.KDConfig(vocab, h, h, 1.5, 72, "fp32", token_block)
    def run(h_t, h_s, d_h):
        loss, kl, d_w = torch.zeros((), device="cuda"), torch.empty(n, device="cuda"), torch.zeros(vocab, h, device="cuda")
        B.kd_loss_forward_backward_static(kd, w_t, w_s, h_t, h_s, loss, kl, d_h, d_w)
        return loss, kl, d_h, d_w
    ref = run(h_t, h_s, torch.empty(n, h, device="cuda"))
    ins = dict(h_t=h_t.clone(), h_s=h_s.clone())
    assert all(torch.equal(a, b) for a, b in zip(run(**ins, d_h=ins[over]), ref))
    # fp64: 72 (or 296) fp32 products of each logit and sum, 2^-24 each, with a margin of 8 and the probabilities' own 1e-6
    lt, ls = (torch.log_softmax(a.double() @ w.double().T / 1.5, -1) for a, w in ((h_t, w_t), (h_s, w_s)))
    dz = (ls.exp() - lt.exp()) / (1.5 * n)
    for got, want in ((ref[2], dz @ w_s.double()), (ref[3], dz.T @ h_s.double())):
        assert ((got.double() - want).norm() / want.norm()).item() < 8 * 296 ** 0.5 * 2 ** -24 + 1e-5
