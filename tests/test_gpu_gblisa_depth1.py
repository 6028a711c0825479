"""Frequency-domain NUTS of depth 1: one leapfrog step and the choice between its ends,
restated over the library's leapfrog; with and without a graph, masked particles, steps
that diverge, a population of one and of thousands."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,hi,wide", [(1, 4, 0), (40, 12, 0), (3000, 3, 200)])
def test_depth_one(lib, N, hi, wide):
    print("[case] gblisa_depth1", N, hi, wide, flush=True)
    w = wl.make_gblisa(N=N, k_lo=1, k_hi=hi, n_inj=4, noise=True, seed=81, beta="uniform")
    d = np.pad(w.noise, ((0, 0), (0, wide - w.B))) if wide else w.noise
    dev = pm.to_dev
    prob = lib.Problem.frequency_domain(wl.GBLISA, dev(d), w.k0, w.T_obs, w.S, hi, N, w.M)
    lib.nuts_reserve(prob, 3)
    o, t, b = dev(w.offsets), dev(w.theta), dev(w.beta)
    mom, dirs, ul, ut = wl.nuts_draws(N, w.M, 8, 1, seed=82)
    mask = (np.arange(N) % 5 != 3).astype(np.uint8)
    l0, g0 = lib.logl_grad_batch(prob, o, t, b)
    l0n, m = l0.cpu().numpy(), mask.astype(bool)
    part = np.repeat(np.arange(N), w.K)
    for eps in (4e-18, 3e-17):
        q1, p1, _, l1 = (x.cpu().numpy() for x in lib.leapfrog(prob, o, b, eps, t, dev(mom), g0, dir=dev(dirs[:, 0].copy())))
        dot = lambda x, y: np.bincount(part, (x * y).sum(1), minlength=N)
        H0, H1 = -l0n + 0.5 * dot(mom, mom), -l1 + 0.5 * dot(p1, p1)
        ok = H1 - H0 <= 1000.0
        turn = (dot(mom + p1, mom) <= 0) | (dot(mom + p1, p1) <= 0)
        take = m & ok & (ut[:, 0] < np.exp(np.minimum(H0 - H1, 0.0)))
        status = np.where(~m, 0, np.where(~ok, 2, np.where(turn, 1, 3)))
        runs = []
        for graph in (False, True):
            q, l, g = t.clone(), l0.clone(), g0.clone()
            out = lib.nuts_transition(prob, o, b, eps, 1, q, l, g, dev(mom), dev(dirs), dev(ul), dev(ut),
                                      use_graph=graph, mask=dev(mask))
            torch.cuda.synchronize()
            prob.device_status()
            runs.append([x.cpu().numpy() for x in (*out, q, l, g)])
        depth, steps, stat, q, l, _ = runs[0]
        assert all(np.array_equal(x, y) for x, y in zip(*runs))
        assert np.array_equal(stat, status) and np.array_equal(steps, m.astype(int)) and np.array_equal(depth, m & ok)
        assert np.array_equal(l, np.where(take, l1, l0n))
        assert np.array_equal(q, np.where(take[part][:, None], q1, w.theta))
