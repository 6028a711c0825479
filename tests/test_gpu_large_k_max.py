"""Handles made for many components (k_max in the hundreds), whose constants fill the
LDS: how a call is laid out, by the kernels that it records, and that its results
are bitwise those of a handle made for few."""
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


def _kernels(call):
    """(workgroups, threads of one) of the kernels that a call records."""
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
        out.append((p.grid[0], p.block[0]))
    return out


@pytest.mark.parametrize("cfg,N,T,k_hi,k_max,kind,ordered,tiles", [
    # many items for the LDS: a wave each, although the waves alone would fit
    ("pulse_batch", 4000, 2000, 10, 400, "grad", True, 1),
    ("pulse_batch", 4000, 2000, 10, 60, "grad", True, 2),
    ("gb_grad", 4000, 2000, 10, 300, "delta", True, 1),
    # few items, but more than the LDS holds at once: ordered
    ("gb_grad", 1000, 4000, 10, 512, "grad", True, 1),
    ("gb_grad", 1000, 4000, 10, 60, "grad", False, 4),
    # workgroups of more than 64 KiB, each with its place
    ("pulse_batch", 300, 4096, 10, 512, "delta", False, 4),
])
def test_layout_and_bits(lib, cfg, N, T, k_hi, k_max, kind, ordered, tiles):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines count compute units")
    print("[case] large_k_max", cfg, N, T, k_max, kind, flush=True)
    w = wl.make_config(cfg, N=N, k_lo=0, k_hi=k_hi, T=T, beta="uniform", seed=17)
    dev = pm.to_dev
    off, th, be = dev(w.offsets), dev(w.theta), dev(w.beta)
    rng = np.random.default_rng(18)
    tb = dev(wl.draw_components(w.model, N, rng))
    di = dev(np.minimum(w.K - 1, 2).astype(np.int32))
    res = []
    for km in (k_max, k_hi):
        prob = lib.Problem(w.model, dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, km, N, w.M)
        a = torch.full((N,), 7.0, dtype=torch.float64, device="cuda")
        b = torch.full_like(a if kind == "delta" else th, 7.0)
        call = {"grad": lambda: lib.logl_grad_batch(prob, off, th, be, logl=a, grad=b),
                "delta": lambda: lib.delta_logl_birth_death(prob, off, th, be, tb, di, a, b)}[kind]
        call()
        torch.cuda.synchronize()
        prob.device_status()
        if km == k_max:
            ks = _kernels(call)
            assert len(ks) == 1 + ordered
            grid, threads = ks[-1]
            assert (grid >= N and threads == 64 * tiles) if tiles > 1 else grid * (threads // 64) < N + 8
        res.append((a.cpu().numpy(), b.cpu().numpy()))
    for x, y in zip(*res):
        assert np.array_equal(x, y)
