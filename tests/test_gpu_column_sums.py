"""Norm and bias gradients of a layer are added up in shared launches: ragged row counts, gradients that share a row, and more
partial rows than the scratch holds at once."""
import pytest
import torch

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl

pytestmark = pytest.mark.gpu
ROWS = ("norm1_g", "norm1_b", "b_qkv", "b_o", "norm2_g", "norm2_b", "b_up", "b_down")


def _encoder(d, d_ffn, layers=2):
    cfg = wl.SectionConfig("encoder", "bf16", layers, d, d // 64, d // 64, 64, d_ffn, 0)
    g = torch.Generator(device="cuda").manual_seed(5)
    rand = lambda *s, mean=0.0: torch.empty(s, device="cuda").normal_(mean, 0.05, generator=g).bfloat16()
    layer = lambda: dict(norm1_g=rand(d, mean=1.0), norm1_b=rand(d), w_qkv=rand(3 * d, d), b_qkv=rand(3 * d), w_o=rand(d, d), b_o=rand(d),
                         norm2_g=rand(d, mean=1.0), norm2_b=rand(d), w_up=rand(d_ffn, d), b_up=rand(d_ffn), w_down=rand(d, d_ffn), b_down=rand(d))
    return cfg, dict(embedding=None, layers=[layer() for _ in range(layers)], final_norm_g=rand(d, mean=1.0), final_norm_b=rand(d)), rand


def _close(a, b, n):
    # fp32 sums of n terms in two orders: each is off by up to about sqrt(n) roundings of the running sum
    assert ((a - b).norm() / b.norm()).item() < 8 * n ** 0.5 * 2 ** -24


# d_ffn = 3 d: wide scratch; d_ffn = d: the partial rows of the norms fill it and the biases have to wait
@pytest.mark.parametrize("lengths,d_ffn", [([1, 2], 384), ([63, 70], 384), ([300, 17], 128), ([2050, 2047], 128), ([4100, 4099], 384)])
def test_one_batch_equals_two(lengths, d_ffn):
    cfg, w, rand = _encoder(128, d_ffn)
    n = sum(lengths)
    x, dh = rand(n, 128), rand(n, 128)
    one, two = B.zero_grads(w), B.zero_grads(w)
    B.section_forward_backward(cfg, w, one, B.Batch(wl.cu_seqlens_of(lengths)), x, d_h_out=dh)
    for a, b in ((0, lengths[0]), (lengths[0], n)):
        B.section_forward_backward(cfg, w, two, B.Batch([0, b - a]), x[a:b].contiguous(), d_h_out=dh[a:b].contiguous())
    for k in ("final_norm_g", "final_norm_b"):
        _close(one[k], two[k], n)
    for la, lb in zip(one["layers"], two["layers"]):
        for k in ROWS:
            _close(la[k], lb[k], n)


def test_gradients_that_share_a_row():
    cfg, w, rand = _encoder(128, 256)
    x, dh, batch = rand(333, 128), rand(333, 128), B.Batch([0, 100, 333])
    one, tied = B.zero_grads(w), B.zero_grads(w)
    B.section_forward_backward(cfg, w, one, batch, x, d_h_out=dh)
    row = tied["layers"][1]["b_o"]
    for k in ("b_down", "norm1_b", "norm2_b"):
        tied["layers"][1][k] = row
    tied["final_norm_b"] = row
    B.section_forward_backward(cfg, w, tied, batch, x, d_h_out=dh)
    l1 = one["layers"][1]
    _close(row, l1["b_o"] + l1["b_down"] + l1["norm1_b"] + l1["norm2_b"] + one["final_norm_b"], 333 * 5)
    _close(tied["layers"][1]["b_up"], l1["b_up"], 333)
