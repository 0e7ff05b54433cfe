"""Grouped-query attention backward on small batches (key block walks cut into chunks, dQ with its keys split over wave
pairs) against the same sequences inside a batch large enough for the unsplit kernels, and against fp64."""
import math

import pytest
import torch

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl

pytestmark = pytest.mark.gpu


def reference(qkv, d_o, cu, nq, nkv, hd, causal):
    x = qkv.double().requires_grad_()
    heads, outs = x.view(-1, nq + 2 * nkv, hd), []
    for a, b in zip(cu[:-1], cu[1:]):
        q, k, v = heads[a:b, :nq], heads[a:b, nq:nq + nkv], heads[a:b, nq + nkv:]
        for h in range(nq):
            s = q[:, h] @ k[:, h * nkv // nq].T / math.sqrt(hd)
            if causal:
                s = s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), -math.inf)
            outs.append((a, h, s.softmax(-1) @ v[:, h * nkv // nq]))
    o = torch.cat([torch.cat([t for a2, _, t in outs if a2 == a], -1) for a in cu[:-1] if any(a2 == a for a2, _, _ in outs)])
    o.backward(d_o.double())
    return x.grad


# one token; ends of the 64-query and 128-key tiles; several chunks of 8 query tiles with a ragged last one; head counts
# whose split grids differ
@pytest.mark.parametrize("hd,nq,nkv", [(64, 4, 2), (80, 6, 2), (128, 8, 2)])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("lens", [[1], [63, 65], [1031], [300, 1, 785]])
def test_small_batches_match_large_ones(hd, nq, nkv, causal, lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    n, ncol = cu[-1], (nq + 2 * nkv) * hd
    pad = 128 * 800 // nq                                     # fills the chip: the unsplit kernels run
    g = lambda tag, shape: wl.normal(31, f"{tag}{hd}.{n}", shape, 1.0, 0.0, torch.bfloat16, "cuda")
    qkv, d_o = g("qkv", (n + pad, ncol)), g("do", (n + pad, nq * hd))
    small, large = B.Batch(cu), B.Batch(cu + [n + i * 64 for i in range(1, pad // 64)] + [n + pad])
    out = []
    for b in (small, large):
        x, d = qkv[:b.n_tokens].contiguous(), d_o[:b.n_tokens].contiguous()
        o, lse = B.k_attention_forward(x, b, nq, nkv, hd, causal)
        out.append((o[:n], B.k_attention_backward(x, o, lse, d, b, nq, nkv, hd, causal)[:n]))
    assert torch.equal(out[0][0], out[1][0])                  # the forward pass does not depend on the batch
    ref = reference(qkv[:n], d_o[:n], cu, nq, nkv, hd, causal)
    err = [((t[1].double() - ref).norm() / ref.norm()).item() for t in out]
    # same bf16 operands, different order of the fp32 sums: the errors against fp64 agree within 2 %
    assert err[0] < 1.02 * err[1] + 1e-4 and err[0] < 1e-2, err
