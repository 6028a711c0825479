"""Birth/death on the truncation support, with the residual that birth and
death share up to the dying component: the first, a middle and the last
component dying, none, only a birth, only a death, pulses across and outside
the record, one chunk and several. Against the oracle (which evaluates every
sample) with the condition-scaled bound of parity.py."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,T,split", [("pulse_batch", 63, 0), ("pulse_batch", 1025, 0),
                                         ("pulse_batch", 4096, 1000), ("pulse_batch", 4097, 0),
                                         ("pulse_batch", 140000, 0), ("gb_grad", 4097, 100)])
def test_delta_support(lib, orc, cfg, T, split):
    print("[case] delta_support", cfg, T, split, flush=True)
    w = wl.make_config(cfg, N=24, k_lo=4, k_hi=4, T=T, beta="uniform", rj=True)
    if w.model == wl.PULSE:  # narrow, on the edges, outside and as wide as the record
        w.theta[0::8] = [3.0, 0.5, 0.3 / T]
        w.theta[1::8] = [4.0, 0.0, 0.02]
        w.theta[2::8] = [4.0, 1.3, 0.02]
        w.theta[3::8] = [2.0, 0.4, 2.0]
        w.extra["theta_birth"][0::4] = [3.0, 1.0, 0.01]
    tb = w.extra["theta_birth"]
    di = np.tile(np.array([0, 1, 2, 3, -1, 3], dtype=np.int32), 4)
    d = pm.data_of(w)
    prob = lib.Problem(w.model, pm.to_dev(d), w.t_start, w.dt, w.sigma, w.k_max, w.N, w.M)
    prob.set_bridge_split(split)
    off, th, be = pm.to_dev(w.offsets), pm.to_dev(w.theta), pm.to_dev(w.beta)
    db, dd = lib.delta_logl_birth_death(prob, off, th, be, pm.to_dev(tb), pm.to_dev(di))
    only_b, _ = lib.delta_logl_birth_death(prob, off, th, be, pm.to_dev(tb), None)
    _, only_d = lib.delta_logl_birth_death(prob, off, th, be, None, pm.to_dev(di))
    torch.cuda.synchronize()
    prob.device_status()
    assert torch.equal(db, only_b) and torch.equal(dd, only_d)
    db, dd = db.cpu().numpy(), dd.cpu().numpy()
    rb, rd = orc.delta_split(w.model, d, w.t_start, w.dt, w.sigma, w.offsets, w.theta, w.beta, tb,
                             di, split)
    if w.model == wl.PULSE:  # 15 |w| outside: exp(-112) of the peak, zero in FP32 and exactly zero here
        assert np.all(dd[2::6] == 0.0) and np.all(np.abs(rd[2::6]) < 1e-45)
        rd[2::6] = 0.0
    one = np.ones(w.N) if split else w.beta  # samples before the split count untempered
    sb = pm.delta_scale(w.model, w, list(tb), one, w.sigma, rb)
    rows = [w.theta[w.offsets[i] + di[i]] if di[i] >= 0 else None for i in range(w.N)]
    sd = pm.delta_scale(w.model, w, rows, one, w.sigma, rd)
    assert np.all(np.abs(db - rb) <= 1e-6 * sb)
    assert np.all(np.abs(dd - rd) <= 1e-6 * sd)
    assert np.all(dd[di < 0] == 0.0)
