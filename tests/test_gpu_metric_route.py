"""Which form of the time-domain metric a call takes, by the grid of the kernel that a
captured call records: the coordinate form has a workgroup per four particles.
Many particles on a short record keep it (the grouped form was up to 1.6 times
slower there). Halves of the population, which are below the line, give the same
bits: the whole matrices, their blocks, masked ones, and around a block that does
not fit."""
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
    """Workgroups of the one kernel that a call records."""
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


def _problem(lib, cfg, N, k_lo, k_hi, T, split):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the line counts compute units")
    print("[case] metric_route", cfg, N, k_lo, k_hi, T, split, flush=True)
    w = wl.make_config(cfg, N=N, k_lo=k_lo, k_hi=k_hi, T=T, beta="uniform", seed=8)
    dev = pm.to_dev
    prob = lib.Problem(w.model, dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, k_hi, N, w.M)
    prob.set_bridge_split(split)
    return w, prob, dev(w.offsets), dev(w.theta), dev(w.beta)


@pytest.mark.parametrize("cfg,N,k_lo,k_hi,T,split,coordinates", [
    ("pulse_batch", 4096, 0, 7, 500, 0, True),
    ("pulse_batch", 4096, 0, 10, 1100, 0, False),
    ("pulse_batch", 2048, 0, 20, 500, 0, True),
    ("pulse_batch", 2048, 0, 10, 2500, 0, True),
    ("gb_grad", 4096, 0, 8, 500, 0, True),
    ("pulse_batch", 4201, 0, 10, 1027, 0, False),   # last step ragged, last block of 41
    ("pulse_batch", 2100, 19, 21, 700, 0, False),   # one particle per wave, a slot for each
    ("pulse_batch", 4300, 1, 1, 1001, 0, False),    # 32 particles per wave
    ("pulse_batch", 4200, 0, 10, 1500, 700, False),  # two windows
    ("gb_grad", 4100, 0, 16, 500, 333, False),
])
def test_route(lib, cfg, N, k_lo, k_hi, T, split, coordinates):
    w, prob, off, th, be = _problem(lib, cfg, N, k_lo, k_hi, T, split)
    dev = pm.to_dev
    fo = lib.metric_offsets(prob, off)
    size = int(fo[-1])
    F = torch.full((size,), 7.0, dtype=torch.float64, device="cuda")
    lib.gauss_newton_metric(prob, off, th, be, f_offsets=fo, out=F)
    B = lib.gauss_newton_metric_blocks(prob, off, th, be)
    mask = np.random.default_rng(6).integers(0, 2, N).astype(np.uint8)
    Fm = lib.gauss_newton_metric(prob, off, th, be, f_offsets=fo, mask=dev(mask),
                                 out=torch.full_like(F, 7.0))[1].cpu().numpy()
    torch.cuda.synchronize()
    if split == 0 or coordinates:
        grid = _grid(lambda: lib.gauss_newton_metric_blocks(prob, off, th, be, out=B))
        assert (grid == -(-N // 4)) == coordinates
    F, f, B = F.cpu().numpy(), fo.cpu().numpy(), B.cpu().numpy()
    for a, b in ((0, N // 2), (N // 2, N)):
        o = w.offsets[a:b + 1] - w.offsets[a]
        r = slice(int(w.offsets[a]), int(w.offsets[b]))
        half = (dev(o), th[r].contiguous(), be[a:b].contiguous())
        part = lib.gauss_newton_metric(prob, *half)[1].cpu().numpy()[:f[b] - f[a]]
        assert np.array_equal(F[f[a]:f[b]], part)
        assert np.array_equal(B[r], lib.gauss_newton_metric_blocks(prob, *half).cpu().numpy()[:r.stop - r.start])
    keep = np.repeat(mask, np.diff(f)).astype(bool)
    assert np.array_equal(Fm, np.where(keep, F, 0.0))
    prob.device_status()


def test_a_block_that_does_not_fit(lib):
    w, prob, off, th, be = _problem(lib, "pulse_batch", 4200, 1, 6, 1024, 0)
    fo, F = lib.gauss_newton_metric(prob, off, th, be)
    bad = fo.clone()
    bad[-1] += 1  # the last block no longer matches (K P)^2
    guard = torch.full((F.numel() + 2,), 7.0, dtype=torch.float64, device="cuda")
    lib.gauss_newton_metric(prob, off, th, be, f_offsets=bad, out=guard)
    with pytest.raises(lib.SmcxError, match="metric block offsets"):
        prob.device_status()
    last = int(fo[-2])
    assert torch.equal(guard[:last], F[:last]) and torch.all(guard[last:] == 7.0)
