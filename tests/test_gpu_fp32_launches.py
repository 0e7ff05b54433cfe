"""fp32 products that share a launch: one of them whose operands cannot be read 16 bytes at a time does not slow the other one down
(it has a launch of its own then), and results are the same."""
import ctypes as C
import os

import pytest
import torch

from paper_2605_10501_amd import binding as B
from paper_2605_10501_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _launches(fn):
    """Kernels that a call enqueues: the nodes of its graph (which is not run)."""
    graph, n = torch.cuda.CUDAGraph(keep_graph=True), C.c_size_t(0)
    fn()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        fn()
    hip = C.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    assert hip.hipGraphGetNodes(C.c_void_p(graph.raw_cuda_graph()), None, C.byref(n)) == 0
    return n.value


def _rand(rows, cols, off=0):
    return torch.randn(rows * cols + 4, device="cuda")[off:off + rows * cols].view(rows, cols)      # off floats past a 16-byte boundary


def test_student_logits_beside_unaligned_teacher_states():
    n, V, ht, hs = 70, 96, 64, 32
    torch.manual_seed(2)
    kd, wt, ws, h_t, h_s = wl.KDConfig(V, ht, hs, 2.0, V, "fp32", 0), _rand(V, ht) * 0.1, _rand(V, hs) * 0.1, _rand(n, ht), _rand(n, hs)
    got = {}
    for off_t, off_s in ((0, 0), (1, 0), (0, 1), (1, 1)):
        a, b = _rand(n, ht, off_t).copy_(h_t), _rand(n, hs, off_s).copy_(h_s)
        loss, kl, d_h, d_w = torch.zeros((), device="cuda"), torch.empty(n, device="cuda"), torch.empty(n, hs, device="cuda"), torch.zeros(V, hs, device="cuda")
        call = lambda: B.kd_loss_forward_backward_static(kd, wt, ws, a, b, loss, kl, d_h, d_w)
        got[off_t, off_s] = (_launches(call), kl, d_h)
    assert got[1, 0][0] == got[0, 1][0] == got[0, 0][0] + 1 and got[1, 1][0] == got[0, 0][0]
    for k in got:
        assert torch.equal(got[k][1], got[0, 0][1]) and torch.equal(got[k][2], got[0, 0][2])


def test_weight_gradient_beside_an_unaligned_output_gradient():
    n, out, inn = 70, 64, 40
    torch.manual_seed(3)
    W, x, dy = _rand(out, inn), _rand(n, inn), _rand(n, out)
    got = {}
    for off in (0, 1):
        g = _rand(n, out, off).copy_(dy)
        dx, dW = torch.empty(n, inn, device="cuda"), torch.empty(out, inn, device="cuda")
        def call():
            dW.zero_()
            B._check(B.lib().ms_k_linear_backward(0, n, out, inn, B._p(g), C.c_int64(out), B._p(W), B._p(x), B._p(dx), 1, 0, B._p(dW), B._stream()))
        got[off] = (_launches(call), dx, dW)
        call()
    assert got[1][0] == got[0][0] + 1
    assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2])
