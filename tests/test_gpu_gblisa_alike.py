"""Frequency-domain calls of between two and four particles per compute unit: a workgroup
each where their source counts differ, a wave each where they are about the same and
small. The launch that is recorded, and results that are bitwise those of a few."""
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


def _grids(call):
    path = next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64.so" in ln)
    hip = ctypes.CDLL(path)
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    graph, n = ctypes.c_void_p(g.raw_cuda_graph()), ctypes.c_size_t(8)
    nodes = (ctypes.c_void_p * 8)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for i in range(n.value):
        p = _Params()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(nodes[i]), ctypes.byref(p)) == 0
        out.append(p.grid[0])
    return out


@pytest.mark.parametrize("N,lo,hi,wide,each", [
    (800, 1, 1, 0, ()), (513, 5, 5, 0, ()), (1024, 0, 3, 200, ()), (640, 0, 3, 0, ("logl", "grad", "delta")),
    (1024, 7, 7, 0, ("logl", "grad")), (1024, 4, 4, 200, ("grad",)), (1024, 0, 10, 0, ("logl", "grad", "delta")),
    (512, 2, 2, 0, ("logl", "grad", "delta")), (1025, 0, 10, 0, ())])
@pytest.mark.parametrize("bridge", [False, True])
def test_route_and_bits(lib, N, lo, hi, wide, each, bridge):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines count compute units")
    print("[case] gblisa_alike", N, lo, hi, wide, bridge, flush=True)
    w = wl.make_gblisa(N=N, k_lo=lo, k_hi=hi, n_inj=4, beta="uniform", noise=True, seed=31)
    d = np.pad(w.noise, ((0, 0), (0, wide - w.B))) if wide else w.noise
    n = 20  # the first particles alone: a workgroup each
    rows = int(w.offsets[n])
    res = []
    for count, m in ((N, w.M), (n, rows)):
        prob, part = (lib.Problem.frequency_domain(wl.GBLISA, pm.to_dev(x), w.k0, w.T_obs, s, hi, count, m)
                      for x, s in ((d, w.S), (0.7 * d, 1.3 * w.S)))
        if bridge:
            prob.set_bridge_partner(part)
        o, t, b, tb, di = (pm.to_dev(x) for x in (
            w.offsets[:count + 1], w.theta[:m], w.beta[:count], w.extra["theta_birth"][:count],
            w.extra["death_idx"][:count]))
        l, x, y = (torch.empty_like(b) for _ in range(3))
        g = torch.empty_like(t)
        calls = {"logl": lambda: lib.logl_batch(prob, o, t, b, l),
                 "grad": lambda: lib.logl_grad_batch(prob, o, t, b, logl=l, grad=g),
                 "delta": lambda: lib.delta_logl_birth_death(prob, o, t, b, tb, di, x, y)}
        out = []
        for name, call in calls.items():
            call()
            torch.cuda.synchronize()
            out += [v.cpu().numpy() for v in ((l,) if name == "logl" else (l, g) if name == "grad" else (x, y))]
            if count == N:
                grids = _grids(call)
                assert grids[-1] == (N if name in each else -(-N // 4)), (name, grids)
        prob.device_status()
        res.append(out)
    for u, v in zip(*res):
        assert np.array_equal(u[:len(v)], v)
