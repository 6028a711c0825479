"""The leapfrog's drift inside the ordering launch against the drift alone
(particle order), bitwise: particles that move, inactive ones, ones without
components and ones beyond k_max, at and around the workgroups' four particles
and the ordering's slices."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1025, 2047, 2049, 5002])
def test_drift_in_the_ordering_launch(lib, N):
    print("[case] leapfrog_launch", N, flush=True)
    rng = np.random.default_rng(N)
    K = rng.integers(0, 7, size=N)
    off = np.concatenate([[0], np.cumsum(K)]).astype(np.int64)
    w = wl.make_config("pulse_batch", N=N, k_lo=6, k_hi=6, T=256, beta="uniform", seed=5)
    M, k_max = int(off[-1]), 5
    th, p, g = w.theta[:M], rng.normal(size=(M, 3)), rng.normal(size=(M, 3))
    act = rng.integers(0, 2, size=N).astype(np.uint8)
    dirs = rng.choice(np.array([-1, 1], dtype=np.int8), N)
    res = []
    for order in (1, 0):
        prob = lib.Problem(w.model, pm.to_dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, k_max, N, M)
        S, chunk, _ = prob.get_tiling(lib.KIND_GRAD)
        prob.set_tiling(lib.KIND_GRAD, S, chunk, order)
        out = tuple(torch.full((M, 3), 7.0, dtype=torch.float64, device="cuda") for _ in range(3))
        out += (torch.full((N,), 7.0, dtype=torch.float64, device="cuda"),)
        lib.leapfrog(prob, pm.to_dev(off), pm.to_dev(w.beta), 1e-4, pm.to_dev(th), pm.to_dev(p),
                     pm.to_dev(g), dir=pm.to_dev(dirs), active=pm.to_dev(act), out=out)
        torch.cuda.synchronize()
        with pytest.raises(lib.SmcxError, match="k_max"):
            prob.device_status()
        res.append([x.cpu().numpy() for x in out])
    Ki = np.repeat(K, K)
    on = np.repeat(act, K).astype(bool)
    q1, p1, g1, l1 = res[0]
    for a, b in zip(res[0][:2], res[1][:2]):  # positions and, of valid particles, momenta
        keep = Ki <= k_max
        assert np.array_equal(a[keep], b[keep])
    assert np.array_equal(q1, res[1][0])
    assert np.array_equal(q1[~on], th[~on]) and np.array_equal(p1[~on], p[~on])
    assert np.all(np.isnan(g1[Ki > k_max]))
    ok = Ki <= k_max
    assert np.array_equal(g1[ok & ~on], g[ok & ~on])
    assert np.array_equal(g1[ok], res[1][2][ok])
    assert np.all(np.isnan(l1[K > k_max]))
    live = (K <= k_max) & ((act == 1) | (K == 0))
    assert np.array_equal(l1[live], res[1][3][live])
