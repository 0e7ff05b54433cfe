"""Every workgroup tile of the bf16 GEMM (two-stage and ring kernels) at the edges of tiles and of the stage ring:
against the matrix product in fp64, and bit-identical between tiles (all add up K in the same order)."""
import pytest
import torch

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl
from parity import TOL_BF16, TOL_F32, assert_parity

pytestmark = pytest.mark.gpu
TILES = [128, 256, 256256, 128128, 128256, 64128, 64064]


@pytest.fixture
def any_tile():
    yield B.k_gemm_config
    B.k_gemm_config(0, -1)


def f64(t):
    return t.detach().cpu().to(torch.float64).numpy()


def dev(name, shape, std=1.0):
    return wl.normal(23, name, shape, std, 0.0, torch.bfloat16, "cuda")


# M, N: one row, one past and one short of a tile edge; K: 1, 2, 3, 4, 5 tiles (fewer than, as many as and more than the
# ring's stages); K-major operands also with a ragged K
@pytest.mark.parametrize("ta,tb,M,N,K", [(0, 0, 1, 8, 64), (0, 0, 65, 136, 128), (0, 0, 127, 264, 192), (0, 0, 257, 72, 256),
                                         (0, 1, 129, 264, 320), (0, 1, 63, 64, 64), (1, 0, 72, 129, 192), (1, 1, 136, 264, 77),
                                         (1, 1, 64, 64, 1), (1, 1, 264, 72, 321)])
def test_every_tile_matches_and_agrees(ta, tb, M, N, K, any_tile):
    a, b = dev(f"ta{M}.{K}", (K, M) if ta else (M, K)), dev(f"tb{N}.{K}", (K, N) if tb else (N, K))
    ref = (f64(a).T if ta else f64(a)) @ (f64(b) if tb else f64(b).T)
    res = dev(f"tr{M}.{N}", (M, N))
    first = None
    for tile in TILES:
        any_tile(tile, -1)
        c = B.k_gemm(a, b, ta, tb, c_fp32=True)
        assert_parity(c, ref, TOL_F32, f"tile {tile}")
        assert_parity(B.k_gemm(a, b, ta, tb, residual=res), ref + f64(res), TOL_BF16, f"tile {tile} residual")
        acc = torch.ones((M, N), dtype=torch.float32, device="cuda")
        B.k_gemm(a, b, ta, tb, c=acc, c_fp32=True, accumulate=True, split_k=2 if K > 128 else 1)
        assert_parity(acc, ref + 1.0, TOL_F32, f"tile {tile} split")
        first = c if first is None else first
        assert torch.equal(c, first), f"tile {tile} adds up in another order"


@pytest.mark.parametrize("M,F,K", [(1, 4, 64), (65, 36, 192), (300, 344, 320)])
def test_swiglu_epilogue_on_every_tile(M, F, K, any_tile):
    a, w = dev(f"sa{M}", (M, K)), dev(f"sw{F}", (2 * F, K), 0.1)
    outs = []
    for tile in TILES:
        any_tile(tile, -1)
        outs.append(B.k_gemm_swiglu(a, w))
    gu = f64(a) @ f64(w).T
    assert_parity(outs[0][1], gu, TOL_BF16, "gate_up")
    for act, up in outs[1:]:
        assert torch.equal(act, outs[0][0]) and torch.equal(up, outs[0][1])


# (the last one is wide enough for another order of K to show through the bf16 roundings)
@pytest.mark.parametrize("n,vocab,chunk,h", [(1, 72, 64, 192), (65, 328, 136, 192), (300, 1032, 512, 192), (520, 4480, 4480, 1024)])
def test_kd_epilogues_on_every_tile(n, vocab, chunk, h, any_tile):
    kd = wl.KDConfig(vocab, 128, h, 1.5, chunk)
    std = 0.2 * (192 / h) ** 0.5
    wt, ws, ht, hs = dev("kt", (vocab, 128), 0.2), dev("ks", (vocab, h), std), dev("kht", (n, 128)), dev("khs", (n, h))
    lt = torch.log_softmax(ht.double() @ wt.double().T / 1.5, -1)
    ls = torch.log_softmax(hs.double() @ ws.double().T / 1.5, -1)
    kl, dz = (lt.exp() * (lt - ls)).sum(-1), (ls.exp() - lt.exp()) / (1.5 * n)
    first = None
    for tile in TILES:
        any_tile(tile, -1)
        dw = torch.zeros((vocab, h), dtype=torch.float32, device="cuda")
        out = B.kd_loss_forward_backward(kd, wt, ws, ht, hs, d_w_student=dw)
        assert_parity(out["kl_tok"], kl.cpu().numpy(), 1e-3, f"kl tile {tile}")
        assert_parity(out["d_h_s"], f64(dz @ ws.double()), TOL_BF16, f"d_h tile {tile}")
        assert_parity(dw, f64(dz.T @ hs.double()), TOL_BF16, f"d_w tile {tile}")
        first = out if first is None else first               # one token's results do not depend on how many come with it
        assert torch.equal(out["kl_tok"], first["kl_tok"]) and torch.equal(out["d_h_s"], first["d_h_s"]), f"tile {tile}"
