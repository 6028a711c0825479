"""Whole metric matrices of very many particles on very short records take the coordinate
form (a workgroup per four particles), their diagonal blocks the grouped one; the
blocks are bitwise those of the matrices."""
import ctypes

import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


class _Params(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint32 * 3), ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def _grid(call):
    path = next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64.so" in ln)
    hip = ctypes.CDLL(path)
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    graph, n = ctypes.c_void_p(g.raw_cuda_graph()), ctypes.c_size_t(1)
    node, p = ctypes.c_void_p(), _Params()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0 and n.value == 1
    assert hip.hipGraphGetNodes(graph, ctypes.byref(node), ctypes.byref(n)) == 0
    assert hip.hipGraphKernelNodeGetParams(node, ctypes.byref(p)) == 0
    return p.grid[0]


@pytest.mark.parametrize("cfg,N,k_lo,k_hi,T,coordinates", [
    ("gb_grad", 40000, 1, 8, 138, True),    # more than 0.4 of the block filled
    ("gb_grad", 20000, 1, 8, 224, False),
    ("gb_grad", 14000, 0, 10, 119, True),   # less
    ("gb_grad", 14000, 0, 10, 120, False),
    ("pulse_batch", 12000, 0, 20, 150, True),
    ("pulse_batch", 19000, 0, 10, 230, False),
])
def test_dense_route(lib, cfg, N, k_lo, k_hi, T, coordinates):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the line counts compute units")
    print("[case] metric_dense_route", cfg, N, k_lo, k_hi, T, flush=True)
    w = wl.make_config(cfg, N=N, k_lo=k_lo, k_hi=k_hi, T=T, beta="uniform", seed=12)
    dev = pm.to_dev
    prob = lib.Problem(w.model, dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, k_hi, N, w.M)
    off, th, be = dev(w.offsets), dev(w.theta), dev(w.beta)
    fo, F = lib.gauss_newton_metric(prob, off, th, be)
    B = lib.gauss_newton_metric_blocks(prob, off, th, be)
    torch.cuda.synchronize()
    prob.device_status()

    def dense():
        p = lambda t: ctypes.c_void_p(t.data_ptr())
        assert lib.load_library().smcx_gauss_newton_metric(
            prob.handle, N, p(off), w.M, p(th), p(be), p(fo), F.numel(), p(F),
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0

    assert (_grid(dense) == -(-N // 4)) == coordinates
    assert _grid(lambda: lib.gauss_newton_metric_blocks(prob, off, th, be, out=B)) < N // 4
    f, F, B, P = fo.cpu().numpy(), F.cpu().numpy(), B.cpu().numpy(), w.P
    for i in list(range(0, N, 97)) + [N - 1]:
        n = int(w.offsets[i + 1] - w.offsets[i])
        m = F[f[i]:f[i + 1]].reshape(n * P, n * P)
        for k in range(n):
            assert np.array_equal(m[k * P:(k + 1) * P, k * P:(k + 1) * P], B[int(w.offsets[i]) + k])
