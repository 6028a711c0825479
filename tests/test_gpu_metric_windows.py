"""The grouped form of the time-domain metric over several windows of 4096 samples
against the coordinate form, bitwise.

Where both forms are open (k_max P <= 64) they accumulate the same FP16 products
in the same order and scale them alike, so that a particle's matrix does not
depend on how many others are in the call. A long record always takes the
grouped form. The reference for pulses therefore takes a handle per window,
which a few particles run in the coordinate form, and adds the windows' matrices
in order, as the grouped form's flush does; the sample times and pulse centres
are dyadic numbers, so that a window's own time origin changes no bit of the
templates. The sinusoids' natural scales hold the record's length (and FP16
values too small to be normal do not scale), so for them the reference is a few
particles on the whole record, of two windows.
"""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu
WINDOW = 4096


def _windows(T, split):
    """[start, end), weighted by beta or not; none across the split."""
    out = []
    for a, b, tempered in ((0, split, False), (split, T, True)):
        while a < b:
            out.append((a, min(a + WINDOW, b), tempered))
            a = out[-1][1]
    return out


def _population(model, N, k_lo, k_hi, T, rng):
    K = rng.integers(k_lo, k_hi + 1, N)
    off = np.concatenate([[0], np.cumsum(K)]).astype(np.int64)
    M = int(off[-1])
    if model == wl.PULSE:
        dt = 2.0 ** -14
        theta = np.stack([rng.normal(size=M), rng.integers(0, T * 64, M) * dt / 64.0,
                          dt * T * rng.uniform(0.002, 0.2, M)], 1)
    else:
        dt = 15.0
        theta = wl.draw_components(model, M, rng)
    return K, off, theta, dt


@pytest.mark.parametrize("model,N,k_lo,k_hi,T,split", [
    (wl.PULSE, 40, 0, 10, 16384, 0),         # four windows, coordinates in one block
    (wl.PULSE, 40, 0, 21, 12289, 0),         # the last window one sample; two blocks
    (wl.PULSE, 40, 0, 7, 9000, 4100),        # four windows, cut at the split
    (wl.PULSE, 1, 3, 3, 20480, 0),           # five windows, one group
    (wl.PULSE, 4200, 0, 5, 8192, 0),         # two windows
    (wl.PULSE, 4200, 0, 5, 4300, 4200),      # two before the split, one after
    (wl.GBSINE, 4200, 0, 5, 8192, 0),
    (wl.GBSINE, 2100, 9, 16, 4300, 4000),
])
def test_windows_add_in_order(lib, model, N, k_lo, k_hi, T, split):
    print("[case] metric_windows", model, N, k_lo, k_hi, T, split, flush=True)
    rng = np.random.default_rng(T + N)
    K, off, theta, dt = _population(model, N, k_lo, k_hi, T, rng)
    beta = rng.random(N)
    dev, M = pm.to_dev, len(theta)
    data = rng.normal(size=T)
    prob = lib.Problem(model, dev(data), 0.0, dt, 0.5, k_hi, N, M)
    prob.set_bridge_split(split)
    fo, F = lib.gauss_newton_metric(prob, dev(off), dev(theta), dev(beta))
    torch.cuda.synchronize()
    prob.device_status()
    fo, F = fo.cpu().numpy(), F.cpu().numpy()
    idx = np.unique(np.concatenate([np.arange(min(N, 24)), np.argsort(K)[-8:]]))
    rows = np.concatenate([np.arange(off[i], off[i + 1]) for i in idx]).astype(int)
    soff = np.concatenate([[0], np.cumsum(K[idx])]).astype(np.int64)
    ref = None
    for a, b, tempered in _windows(T, split) if model == wl.PULSE else [(0, T, True)]:
        w = lib.Problem(model, dev(data[a:b]), a * dt, dt, 0.5, k_hi, len(idx), len(rows))
        w.set_bridge_split(split if (a, b) == (0, T) else 0)
        sfo, sF = lib.gauss_newton_metric(w, dev(soff), dev(theta[rows]), dev(beta[idx]) if tempered else None)
        torch.cuda.synchronize()
        w.device_status()
        sfo, sF = sfo.cpu().numpy(), sF.cpu().numpy()
        ref = sF if ref is None else ref + sF
    for x, i in enumerate(idx):
        assert np.array_equal(F[fo[i]:fo[i + 1]], ref[sfo[x]:sfo[x + 1]]), i
