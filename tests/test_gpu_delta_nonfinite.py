"""Birth/death scores of pulses with values that FP32 does not hold: a NaN sample, a NaN
centre, a width of zero or an amplitude beyond its range make the particle's scores
NaN wherever on the record the candidates lie, and leave the other particles alone.
Few particles, many, and handles made for hundreds of components (also with particles
of more than a batch of constants)."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _scores(lib, d, k_max, K, theta, tb, beta=None, split=0):
    N, dev = len(K), pm.to_dev
    off = np.concatenate([[0], np.cumsum(K)]).astype(np.int64)
    prob = lib.Problem(wl.PULSE, dev(d), 0.0, 1.0 / (len(d) - 1), 1.0, k_max, N, len(theta))
    prob.set_bridge_split(split)
    out = lib.delta_logl_birth_death(prob, dev(off), dev(theta), dev(np.ones(N) if beta is None else beta), dev(tb),
                                     dev(np.zeros(N, dtype=np.int32)))
    torch.cuda.synchronize()
    prob.device_status()
    return [x.cpu().numpy() for x in out]


@pytest.mark.parametrize("N,T,k_max,k_bad", [(6, 3000, 4, 2), (9000, 2500, 4, 2), (6, 9001, 4, 2), (6, 3000, 300, 2),
                                             (6, 3000, 300, 140), (9000, 2500, 300, 2)])
def test_nonfinite(lib, N, T, k_max, k_bad):
    print("[case] delta_nonfinite", N, T, k_max, k_bad, flush=True)
    rng = np.random.default_rng(61)
    K = np.full(N, 2)
    K[1] = k_bad
    off = np.concatenate([[0], np.cumsum(K)])
    theta = np.tile([3.0, 0.25, 0.004], (K.sum(), 1))  # the death candidates, and the births, lie near 0.2
    theta[:, 0] += rng.random(len(theta))
    tb = np.tile([2.0, 0.2, 0.004], (N, 1))
    d = rng.normal(size=T)
    good = _scores(lib, d, k_max, K, theta, tb)
    assert all(np.all(np.isfinite(x)) for x in good)
    other = np.arange(N) != 1
    for row in ([3.0, np.nan, 0.01], [1e39, 0.8, 0.004], [3.0, 0.4, 0.0], [np.inf, 0.8, 0.004]):
        bad = theta.copy()
        bad[off[2] - 1] = row  # the last component of particle 1
        for x, ref in zip(_scores(lib, d, k_max, K, bad, tb), good):
            assert np.isnan(x[1]) and np.array_equal(x[other], ref[other]), row
    for value in (np.nan, np.inf, 1e39):
        odd = d.copy()
        odd[T - 5] = value
        for x in _scores(lib, odd, k_max, K, theta, tb):
            assert np.all(np.isnan(x)), value
    far = tb.copy()
    far[:, 1] = 3.0  # a birth wholly off the record
    bad = theta.copy()
    bad[off[2] - 1, 1] = np.nan
    x = _scores(lib, d, k_max, K, bad, far)[0]
    assert np.isnan(x[1]) and np.all(np.isfinite(x[other]))
    # the weight of the samples after a split, which no candidate meets
    for value in (np.nan, np.inf, -np.inf):
        beta = np.ones(N)
        beta[1] = value
        for x in _scores(lib, d, k_max, K, theta, tb, beta, T // 2):
            assert np.isnan(x[1]) and np.all(np.isfinite(x[other])), value
        for x in _scores(lib, d, k_max, K, theta, tb, beta, T):
            assert np.all(np.isfinite(x)), value
