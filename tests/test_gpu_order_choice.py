"""Which calls run the ordering pass, by the kernels a captured call records: a
handle that was asked for sorted = 1 always does; left at its default it leaves
the pass out where every work item has a SIMD to itself. Same bits either way."""
import ctypes

import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _hip():
    path = next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64.so" in ln)
    f = ctypes.CDLL(path).hipGraphGetNodes
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    f.restype = ctypes.c_int
    return f


def _nodes(call):
    """Nodes of the graph that a call records (its outputs passed in)."""
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    n = ctypes.c_size_t()
    assert _hip()(g.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("N", [40, 300])
def test_explicit_order_is_kept(lib, N):
    print("[case] order_choice", N, flush=True)
    w = wl.make_config("pulse_mutate", N=N, k_lo=0, k_hi=6, T=1024, seed=9)
    dev = pm.to_dev
    off, th, be = dev(w.offsets), dev(w.theta), dev(w.beta)
    prob = lib.Problem(w.model, dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, w.k_max, N, w.M)
    tb, di = dev(w.extra["theta_birth"]), dev(w.extra["death_idx"])
    mom = torch.zeros_like(th)
    new = lambda *s: torch.full(s, 7.0, dtype=torch.float64, device="cuda")  # noqa: E731
    out = {k: [new(N), new(*th.shape)] for k in ("logl", "grad", "delta", "leap")}
    out["delta"] = [new(N), new(N)]
    out["leap"] = [new(*th.shape), new(*th.shape), new(*th.shape), new(N)]
    g0 = lib.logl_grad_batch(prob, off, th, be)[1]
    calls = {
        "logl": lambda: lib.logl_batch(prob, off, th, be, logl=out["logl"][0]),
        "grad": lambda: lib.logl_grad_batch(prob, off, th, be, logl=out["grad"][0], grad=out["grad"][1]),
        "delta": lambda: lib.delta_logl_birth_death(prob, off, th, be, tb, di, *out["delta"]),
        "leap": lambda: lib.leapfrog(prob, off, be, 1e-5, th, mom, g0, out=tuple(out["leap"])),
    }
    default = {k: _nodes(c) for k, c in calls.items()}
    first = {k: [x.clone() for x in v] for k, v in out.items()}
    assert default["logl"] == default["grad"] == default["delta"] == 1
    assert default["leap"] == 2  # the drift by itself
    for kind in (lib.KIND_LOGL, lib.KIND_GRAD, lib.KIND_DELTA):
        S, chunk, order = prob.get_tiling(kind)
        assert order == 1
        prob.set_tiling(kind, S, chunk, 1)
    asked = {k: _nodes(c) for k, c in calls.items()}
    assert asked == {"logl": 2, "grad": 2, "delta": 2, "leap": 2}
    torch.cuda.synchronize()
    prob.device_status()
    for k in calls:
        for a, b in zip(first[k], out[k]):
            assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
