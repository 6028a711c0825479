"""Resampling and birth/death rebuild where their prefix sums change tile: a
population of one, at and around a tile, of the most tiles of one pass, of two
passes; weights packed into few particles. Integers and copies: the oracle's
exactly."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu
PULSE = wl.PULSE


@pytest.mark.parametrize("N", [1, 15, 255, 256, 257, 4097, 262144, 262145, 600011])
def test_rebuild_tiles(lib, orc, N):
    print("[case] rebuild_tiles", N, flush=True)
    rng = np.random.default_rng(N)
    K = rng.integers(0, 4, size=N)
    off = np.concatenate([[0], np.cumsum(K)]).astype(np.int64)
    M = int(off[-1])
    theta = rng.normal(size=(M, 3))
    w = wl.make_config("pulse_small", N=1, T=64)
    prob = lib.Problem(PULSE, pm.to_dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, 4, N, max(M, 1))
    o, th = pm.to_dev(off), pm.to_dev(theta)
    few = np.zeros(N)
    few[[0, N // 2, N - 1]] = [0.2, 0.5, 0.3]
    for W, u in ((rng.dirichlet(np.ones(N)), 0.3), (few, 0.0), (np.eye(1, N, N - 1)[0], 0.999)):
        ref = orc.resample_systematic(PULSE, off, theta, W, u, m_cap=4 * N)
        out = lib.resample_systematic(prob, o, th, pm.to_dev(W), u)
        torch.cuda.synchronize()
        prob.device_status()
        anc, off1, th1 = (x.cpu().numpy() for x in out)
        assert np.array_equal(anc, ref[0]) and np.array_equal(off1, ref[1])
        assert np.array_equal(th1[:off1[-1]], ref[2])
    move = rng.integers(0, 3, size=N).astype(np.int8)
    death = rng.integers(-1, 3, size=N).astype(np.int32)
    birth, db, dd = rng.normal(size=(N, 3)), rng.normal(size=N), rng.normal(size=N)
    lu = np.log(rng.random(N))
    ref = orc.rj_apply(PULSE, off, theta, move, birth, death, db, dd, lu, 0, 4)
    cap = max(int(ref[1][-1]) - 5, 0)  # too small by five rows: flagged, the rows before it written
    for m_cap in (None, cap):
        out = lib.rj_apply(prob, o, th, pm.to_dev(move), pm.to_dev(birth), pm.to_dev(death),
                           pm.to_dev(db), pm.to_dev(dd), pm.to_dev(lu), 0, 4, m_cap=m_cap)
        torch.cuda.synchronize()
        if m_cap is None or cap == int(ref[1][-1]):
            prob.device_status()
        else:
            with pytest.raises(lib.SmcxError, match="m_cap"):
                prob.device_status()
        acc, off2, th2 = (x.cpu().numpy() for x in out)
        n = int(ref[1][-1]) if m_cap is None else cap
        assert np.array_equal(acc, ref[0]) and np.array_equal(off2, ref[1])
        assert np.array_equal(th2[:n], ref[2][:n])
