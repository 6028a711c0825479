"""A broken offset makes the rows of an invalid particle run into those of valid
ones. Their gradients are what they are without it, and the invalid particle's
own rows NaN, in the default schedule of few particles as with the ordering
pass."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("at,value", [(3, 40), (6, 0)])  # runs forward, runs back
def test_rows_of_valid_particles(lib, at, value):
    print("[case] overlapping_rows", at, value, flush=True)
    N, k_max = 8, 6
    w = wl.make_config("pulse_small", N=N, k_lo=5, k_hi=5, T=1500, seed=21)
    off = w.offsets.copy()
    off[at] = value
    K = np.diff(off)
    ok = (K >= 0) & (K <= k_max)
    assert ok.sum() == N - 2
    rows = np.zeros(w.M, dtype=bool)
    for i in np.flatnonzero(ok):
        rows[off[i]:off[i + 1]] = True
    dev = pm.to_dev
    got = []
    for asked in (False, True):
        prob = lib.Problem(w.model, dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, k_max, N, w.M)
        ref_l, ref_g = lib.logl_grad_batch(prob, dev(w.offsets), dev(w.theta))
        if asked:
            S, chunk, _ = prob.get_tiling(lib.KIND_GRAD)
            prob.set_tiling(lib.KIND_GRAD, S, chunk, 1)
        grad = torch.full((w.M, 3), 7.0, dtype=torch.float64, device="cuda")
        logl, _ = lib.logl_grad_batch(prob, dev(off), dev(w.theta), grad=grad)
        torch.cuda.synchronize()
        with pytest.raises(lib.SmcxError):
            prob.device_status()
        logl, grad = logl.cpu().numpy(), grad.cpu().numpy()
        assert np.array_equal(logl[ok], ref_l.cpu().numpy()[ok]) and np.all(np.isnan(logl[~ok]))
        assert np.array_equal(grad[rows], ref_g.cpu().numpy()[rows])
        got.append(grad)
    own = np.zeros(w.M, dtype=bool)  # of no valid particle, but of an invalid one
    for i in np.flatnonzero(~ok & (K > 0)):
        own[off[i]:off[i + 1]] = True
    own &= ~rows
    assert own.any()
    for grad in got:
        assert np.all(np.isnan(grad[own]))
    assert np.array_equal(got[0], got[1], equal_nan=True)
