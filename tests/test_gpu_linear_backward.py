"""Backward pass of a linear layer in one grid (ms_k_linear_backward) against fp64 and against the two products one by one."""
import ctypes as C

import pytest
import torch

from paper_2605_10501_amd import binding as B

pytestmark = pytest.mark.gpu


def _run(dy, W, x, dx, acc, dW):
    n, (out, inn) = dy.shape[0], W.shape
    B._check(B.lib().ms_k_linear_backward(int(dy.dtype == torch.bfloat16), n, out, inn, B._p(dy), C.c_int64(dy.stride(0)), B._p(W), B._p(x), B._p(dx),
                                          int(dx.dtype == torch.float32), int(acc), B._p(dW), B._stream()))


# tile 0: chosen by size (-1 would be the generic kernel); out = 72: no full K tile, so the products stay apart
@pytest.mark.parametrize("tile", [0, 256, 128, 128128, 128256, 64128, 64064])
@pytest.mark.parametrize("n,out,inn,pad,f32", [(1, 64, 8, 0, 0), (70, 64, 64, 0, 1), (257, 128, 264, 64, 1), (513, 320, 256, 0, 0),
                                               (1100, 192, 520, 8, 0), (130, 72, 40, 0, 0)])
def test_bf16(tile, n, out, inn, pad, f32):
    g = torch.Generator(device="cuda").manual_seed(n + out)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=g).bfloat16()
    dy, W, x = rand(n, out + pad)[:, :out], rand(out, inn), rand(n, inn)
    old, dw0 = torch.empty(n, inn, device="cuda").normal_(generator=g), torch.empty(out, inn, device="cuda").normal_(generator=g)
    dx = old.clone() if f32 else torch.full((n, inn), float("nan"), device="cuda", dtype=torch.bfloat16)
    dW = dw0.clone()
    try:
        B.k_gemm_config(tile, -1)
        _run(dy, W, x, dx, f32, dW)
    finally:
        B.k_gemm_config(0, -1)
    one = old.clone() if f32 else torch.empty_like(dx)
    B.k_gemm(dy, W, trans_b=True, c=one, c_fp32=bool(f32), accumulate=bool(f32))
    assert torch.equal(dx, one)                                     # the same K order whatever the grid
    # fp32 sums of K products of bf16 numbers: sqrt(K) roundings of 2^-24 on a sum of size sqrt(K), with a margin of 8
    ref = dw0.double() + dy.double().T @ x.double()
    assert ((dW.double() - ref).norm() / ref.norm()).item() < 8 * n ** 0.5 * 2 ** -24 + 2 ** -23
    ref = (old.double() if f32 else 0.0) + dy.double() @ W.double()
    assert ((dx.double() - ref).norm() / ref.norm()).item() < (8 * out ** 0.5 * 2 ** -24 + 2 ** -23 if f32 else 2 ** -8)


# 31, 65: rows not 16-byte aligned; n > out: the weight gradient's workgroups come first
@pytest.mark.parametrize("n,out,inn", [(1, 4, 4), (293, 688, 128), (33, 31, 65), (64, 32, 32), (65, 64, 40), (4000, 688, 256)])
def test_fp32(n, out, inn):
    g = torch.Generator(device="cuda").manual_seed(n + out)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=g)
    dy, W, x, dw0, old = rand(n, out), rand(out, inn), rand(n, inn), rand(out, inn), rand(n, inn)
    for acc in (False, True):
        dx, dW = old.clone(), dw0.clone()
        _run(dy, W, x, dx, acc, dW)
        for got, ref, k in ((dx, (old.double() if acc else 0.0) + dy.double() @ W.double(), out), (dW, dw0.double() + dy.double().T @ x.double(), n)):
            assert ((got.double() - ref).norm() / ref.norm()).item() < 8 * k ** 0.5 * 2 ** -24 + 2 ** -23


@pytest.mark.parametrize("tile", [0, 256, 128, 128128, 128256, 64128, 64064])
@pytest.mark.parametrize("n,out,f", [(1, 64, 8), (70, 64, 64), (257, 128, 264), (513, 320, 256), (130, 72, 40)])   # 72: the products stay apart
def test_swiglu_derivative_in_the_epilogue(tile, n, out, f):
    g = torch.Generator(device="cuda").manual_seed(n + out + f)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=g).bfloat16()
    dy, W, act, up, dw0 = rand(n, out), rand(out, f), rand(n, f), 3 * rand(n, 2 * f), rand(out, f).float()
    one = {k: torch.full((n, c), float("nan"), device="cuda", dtype=torch.bfloat16) for k, c in (("da", f), ("dup", 2 * f))}
    dW, dW1 = dw0.clone(), dw0.clone()
    try:
        B.k_gemm_config(tile, -1)
        B._check(B.lib().ms_k_swiglu_linear_backward(1, n, out, f, B._p(dy), B._p(W), B._p(act), B._p(up), B._p(one["da"]), B._p(one["dup"]), B._p(dW), B._stream()))
        da = torch.empty(n, f, device="cuda", dtype=torch.bfloat16)
        _run(dy, W, act, da, False, dW1)
    finally:
        B.k_gemm_config(0, -1)
    if tile:                                                        # a pass of its own, and da stored, only where the products stay apart
        assert torch.isnan(one["da"]).all() if out % 64 == 0 else torch.equal(one["da"], da)
    two = torch.empty(n, 2 * f, device="cuda", dtype=torch.bfloat16)
    B._check(B.lib().ms_k_act_backward(0, 1, n, f, B._p(da), B._p(up), B._p(two), B._stream()))
    assert torch.equal(one["dup"], two)                             # the same roundings of the same da
    assert ((dW - dW1).norm() / dW1.norm()).item() < 8 * n ** 0.5 * 2 ** -24 + 2 ** -23


def test_swiglu_derivative_does_not_depend_on_the_batch():
    """64 tokens take the epilogue; together with 3072 others they take the kernel of its own (where one grid is not estimated
    faster): the same bits either way."""
    n, out, f = 3136, 1024, 4096
    g = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *s: torch.empty(s, device="cuda").normal_(generator=g).bfloat16()
    dy, W, act, up = rand(n, out), rand(out, f), rand(n, f), 3 * rand(n, 2 * f)
    got = {}
    for m in (64, n):
        da, dup, dW = (torch.full(s, float("nan"), device="cuda", dtype=t) for s, t in (((m, f), torch.bfloat16), ((m, 2 * f), torch.bfloat16), ((out, f), torch.float32)))
        B._check(B.lib().ms_k_swiglu_linear_backward(1, m, out, f, B._p(dy), B._p(W), B._p(act), B._p(up), B._p(da), B._p(dup), B._p(dW), B._stream()))
        assert torch.isnan(da).all() == (m == 64)
        got[m] = dup
    assert torch.equal(got[64], got[n][:64])
    # fp64 of the same rounded da (now stored): a few fp32 roundings, then one of bf16
    G, U, D = up[:, :f].double(), up[:, f:].double(), da.double()
    s = torch.sigmoid(G)
    for have, ref in ((got[n][:, :f], D * U * s * (1 + G * (1 - s))), (got[n][:, f:], D * G * s)):
        assert ((have.double() - ref).norm() / ref.norm()).item() < 2 ** -8
