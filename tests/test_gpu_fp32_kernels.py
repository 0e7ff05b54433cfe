"""fp32 GEMM (K split over the waves of a workgroup) and fp32 attention (16-row tiles, waves over every fourth block) at
the edges of their tiles and splits, against fp64."""
import ctypes as C
import math

import pytest
import torch

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl
from parity import TOL_F32, assert_parity

pytestmark = pytest.mark.gpu


def f64(t):
    return t.detach().cpu().to(torch.float64).numpy()


def dev(name, shape, std=1.0):
    return wl.normal(29, name, shape, std, 0.0, torch.float32, "cuda")


# K: one element, below one 16-deep slice, one slice short of / at / past the four waves, several rounds of slices;
# K % 4 and odd leading dimensions take the scalar loads
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (31, 33, 15), (32, 32, 48), (33, 70, 64), (64, 31, 65), (5, 129, 260), (97, 40, 1027)])
def test_gemm_fp32_edges(ta, tb, M, N, K):
    a, b = dev(f"a{M}.{K}", (K, M) if ta else (M, K)), dev(f"b{N}.{K}", (K, N) if tb else (N, K))
    ref = (f64(a).T if ta else f64(a)) @ (f64(b) if tb else f64(b).T)
    assert_parity(B.k_gemm(a, b, ta, tb), ref, TOL_F32)
    c = dev("c", (M, N))
    out = c.clone()
    B.k_gemm(a, b, ta, tb, c=out, accumulate=True, c_fp32=True, alpha=0.5)
    assert_parity(out, f64(c) + 0.5 * ref, TOL_F32, "accumulate")


# nothing to contract: bias, residual and what C holds remain; leading dimensions past the row length, as a slice has them
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,pad", [(1, 1, 0), (33, 70, 2), (64, 31, 1023)])
def test_gemm_fp32_without_a_contraction(ta, tb, M, N, pad):
    a = torch.ones((1, (M if ta else 0) + pad + 1), device="cuda")
    b = torch.ones((1, (N if tb else 0) + pad + 1), device="cuda")
    bias, res, c = dev("kb", (N,)), dev("kr", (M, N)), dev("kc", (M, N))
    for accumulate in (0, 1):
        out = c.clone()
        B._check(B.lib().ms_k_gemm(B.MS_F32, ta, tb, M, N, 0, C.c_float(2.0), B._p(a), C.c_int64(a.shape[1]), B._p(b), C.c_int64(b.shape[1]),
                                   B._p(out), C.c_int64(N), 1, accumulate, B._p(bias), B._p(res), C.c_int64(N), 0, 1, B._stream()))
        assert torch.equal(out, c + (bias + res) if accumulate else bias + res)


# rows of A that lie backwards in memory: not for the descriptor
def test_gemm_fp32_negative_leading_dimension():
    M, N, K = 37, 20, 24
    a, b = dev("na", (M, K)), dev("nb", (N, K))
    out = torch.empty((M, N), device="cuda")
    last = a[M - 1:]
    B._check(B.lib().ms_k_gemm(B.MS_F32, 0, 0, M, N, K, C.c_float(1.0), B._p(last), C.c_int64(-K), B._p(b), C.c_int64(K), B._p(out), C.c_int64(N),
                               1, 0, None, None, C.c_int64(0), 0, 1, B._stream()))
    assert_parity(out, f64(a)[::-1] @ f64(b).T, TOL_F32)


# more than 2^24 output tiles, along either side: beyond what one launch takes
@pytest.mark.parametrize("along_n", [True, False])
def test_gemm_fp32_with_very_many_tiles(along_n):
    n = 32 * (1 << 24) + 40
    long = torch.arange(n, device="cuda").remainder_(8191).to(torch.float32).view(1, n)
    three, bias = torch.full((1, 1), 3.0, device="cuda"), long.add(1.0).view(n) if along_n else torch.ones(1, device="cuda")
    out = B.k_gemm(three, long, False, True, bias=bias) if along_n else B.k_gemm(long, three, True, True, bias=bias)
    assert torch.equal(out.view(1, n), long.mul_(3.0).add_(bias.view(1, -1)))


# very many sequences under a large bound on their length: more 16-row tiles than one launch holds
def test_attention_fp32_very_many_sequences():
    ones, tail, hd = 100_000, 70, 64
    batch, n = B.Batch(list(range(ones + 1)) + [ones + tail]), ones + tail
    batch.max_seqlen = 4096
    qkv, d_o = dev("vm", (n, 3 * hd)), dev("vmo", (n, hd))
    o, lse = B.k_attention_forward(qkv, batch, 1, 1, hd, True)
    q, k, v = qkv.split(hd, 1)
    assert torch.equal(o[:ones], v[:ones])                    # a sequence of one token returns its value
    assert_parity(lse[0, :ones], f64((q * k).sum(1)[:ones]) / 8.0, TOL_F32)
    dqkv = B.k_attention_backward(qkv, o, lse, d_o, batch, 1, 1, hd, True)
    assert float(dqkv[:ones, :2 * hd].abs().max()) < 1e-4 and float((dqkv[:ones, 2 * hd:] - d_o[:ones]).abs().max()) < 1e-4
    small = B.Batch([0, tail])
    xt, dt = qkv[ones:].contiguous(), d_o[ones:].contiguous()
    o2, lse2 = B.k_attention_forward(xt, small, 1, 1, hd, True)
    assert_parity(o[ones:], f64(o2), TOL_F32)
    assert_parity(dqkv[ones:], f64(B.k_attention_backward(xt, o2, lse2, dt, small, 1, 1, hd, True)), TOL_F32)


@pytest.mark.parametrize("hd,nq,nkv", [(64, 4, 4), (80, 2, 1), (128, 6, 2)])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("lens", [[1], [15, 16, 17], [64, 0, 65, 130]])
def test_attention_fp32_edges(hd, nq, nkv, causal, lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    batch, n = B.Batch(cu), cu[-1]
    qkv = dev(f"qkv{hd}{n}", (n, (nq + 2 * nkv) * hd))
    d_o = dev(f"do{hd}{n}", (n, nq * hd))
    x = qkv.cpu().double().requires_grad_()
    heads, outs, lses = x.view(n, nq + 2 * nkv, hd), [], []
    for a, b in zip(cu[:-1], cu[1:]):
        if a == b:
            continue
        q, k, v = heads[a:b, :nq], heads[a:b, nq:nq + nkv], heads[a:b, nq + nkv:]
        k, v = (t.repeat_interleave(nq // nkv, 1).transpose(0, 1) for t in (k, v))
        s = q.transpose(0, 1) @ k.transpose(1, 2) / math.sqrt(hd)
        if causal:
            s = s.masked_fill(torch.ones(b - a, b - a, dtype=torch.bool).triu(1), -math.inf)
        outs.append((s.softmax(-1) @ v).transpose(0, 1).reshape(b - a, nq * hd))
        lses.append(s.logsumexp(-1))
    ref = torch.cat(outs)
    ref.backward(d_o.cpu().double())
    o, lse = B.k_attention_forward(qkv, batch, nq, nkv, hd, causal)
    assert_parity(o, ref.detach().numpy(), TOL_F32, "o")
    assert_parity(lse, torch.cat(lses, 1).detach().numpy(), TOL_F32, "lse")
    dqkv = B.k_attention_backward(qkv, o, lse, d_o, batch, nq, nkv, hd, causal)
    assert_parity(dqkv, x.grad.numpy(), TOL_F32, "dqkv")
    assert torch.equal(dqkv, B.k_attention_backward(qkv, o, lse, d_o, batch, nq, nkv, hd, causal))   # no atomics


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_causal_masked_pairs_never_meet(hd, bad):
    """A non-finite key, value, query or output gradient only reaches the tokens that see it, tile mates or not."""
    n, nq, t = 40, 2, 21
    # a tile that holds such an element adds up in another order: at most 40 terms, |w x| summed below 40: 40 * 2^-24 * 40
    same = lambda a, c: bool(torch.isfinite(a).all()) and float((a - c).abs().max()) <= 1e-4
    batch = B.Batch([0, n])
    qkv, d_o = dev(f"mq{hd}", (n, 3 * nq * hd)), dev(f"md{hd}", (n, nq * hd))
    o, lse = B.k_attention_forward(qkv, batch, nq, nq, hd, True)
    dqkv = B.k_attention_backward(qkv, o, lse, d_o, batch, nq, nq, hd, True)
    x = qkv.clone()
    x[t, nq * hd:] = bad                                      # key and value of token t: earlier tokens do not see them
    o1, lse1 = B.k_attention_forward(x, batch, nq, nq, hd, True)
    assert same(o1[:t], o[:t]) and same(lse1[:, :t], lse[:, :t]) and not torch.isfinite(o1[t:]).all()
    d1 = B.k_attention_backward(x, o1, lse1, d_o, batch, nq, nq, hd, True)
    assert same(d1[:t, :nq * hd], dqkv[:t, :nq * hd])
    x = qkv.clone()
    x[t, :nq * hd] = bad                                      # query and output gradient of token t: later keys are not seen
    d2o = d_o.clone()
    d2o[t] = bad
    o2, lse2 = B.k_attention_forward(x, batch, nq, nq, hd, True)
    d2 = B.k_attention_backward(x, o2, lse2, d2o, batch, nq, nq, hd, True)
    assert same(o2[:t], o[:t]) and same(o2[t + 1:], o[t + 1:])
    assert same(d2[t + 1:], dqkv[t + 1:]) and same(d2[:t, :nq * hd], dqkv[:t, :nq * hd])
