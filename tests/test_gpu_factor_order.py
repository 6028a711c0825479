"""Factors of more particles than the device holds at once, which are taken
largest first, against the same particles in small calls (particle order):
bitwise, with masked, empty and invalid particles among them, at and around the
ordering's slices."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra,k_max", [(1, 20), (1025, 21), (3000, 5)])
def test_order_does_not_change_the_factors(lib, extra, k_max):
    N = 12 * torch.cuda.get_device_properties(0).multi_processor_count + extra
    print("[case] factor_order", N, k_max, flush=True)
    rng = np.random.default_rng(N)
    K = rng.integers(0, k_max + 1, size=N)
    n = 3 * K
    off = np.concatenate([[0], np.cumsum(K)]).astype(np.int64)
    fo = np.concatenate([[0], np.cumsum(n * n)]).astype(np.int64)
    M = int(off[-1])
    F = np.empty(int(fo[-1]))
    for i in range(N):  # identity plus a rank-one part: positive definite
        v = rng.normal(size=n[i])
        F[fo[i]:fo[i + 1]] = (np.eye(n[i]) + np.outer(v, v)).ravel()
    mask = rng.integers(0, 4, size=N).astype(np.uint8)
    w = wl.make_config("pulse_small", N=1, T=64)
    prob = lib.Problem(w.model, pm.to_dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, k_max, N, max(M, 1))
    Fd, ridge = pm.to_dev(F), [1e-3, 0.0, 1e-3]

    def factor(lo, hi, foff):
        a, b = int(off[lo]), int(off[hi])
        out = torch.full((int(fo[hi] - fo[lo]),), 7.0, dtype=torch.float64, device="cuda")
        lib.metric_factor(prob, pm.to_dev(off[lo:hi + 1] - a), pm.to_dev(foff), Fd[fo[lo]:fo[hi]], ridge,
                          out=out, M=b - a, mask=pm.to_dev(mask[lo:hi]))
        torch.cuda.synchronize()
        return out.cpu().numpy()

    full = factor(0, N, fo)
    prob.device_status()
    parts = [factor(lo, min(lo + 900, N), fo[lo:min(lo + 900, N) + 1] - fo[lo]) for lo in range(0, N, 900)]
    prob.device_status()
    assert np.array_equal(full, np.concatenate(parts))
    for i in range(0, N, 97):
        if not mask[i]:
            assert np.all(full[fo[i]:fo[i + 1]] == 7.0)
    bad = fo.copy()  # particle 5's block does not match its size: flagged, the others unchanged
    i = 5 + int(np.argmax((K[5:] > 0) & (mask[5:] > 0)))
    shift = np.zeros(N + 1, dtype=np.int64)
    shift[i] = 1
    again = factor(0, N, bad + shift)
    with pytest.raises(lib.SmcxError):
        prob.device_status()
    keep = np.ones(len(full), dtype=bool)
    keep[fo[i - 1]:fo[i + 1]] = False
    assert np.array_equal(again[keep], full[keep])
