"""The grouped form of the time-domain metric (many particles, or a long
record): particles packed into waves of 32 component rows.

Against the oracle with the bound of test_gpu_metric.py, and against the
coordinate form, which a call with a few of the same particles takes: both
accumulate the same FP16 products in the same order and differ at most in
the order of two FP64 scalings, 4 units in the last place.
"""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 2.0 ** -10 + 512 * 2.0 ** -24 + 1e-5
ULP4 = 4 * 2.0 ** -52


def problem(lib, w):
    return lib.Problem(w.model, pm.to_dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, w.k_max, w.N, w.M)


@pytest.mark.parametrize("cfg,N,k_lo,k_hi,T,split", [
    ("pulse_batch", 4200, 0, 10, 67, 0),      # last step ragged, K = 0, two packings per block
    ("pulse_batch", 2100, 19, 21, 64, 0),     # one particle per wave
    ("pulse_batch", 4200, 1, 1, 9, 0),        # 32 particles per wave
    ("pulse_batch", 70, 0, 7, 9000, 4100),    # three windows, one cut at the split
    ("pulse_batch", 1, 1, 3, 16390, 0),       # five windows, one group
    ("gb_grad", 2100, 0, 16, 70, 33),
    ("gb_grad", 40, 0, 8, 12289, 0),          # four windows, the last one sample
])
def test_grouped_metric(lib, orc, cfg, N, k_lo, k_hi, T, split):
    print("[case] metric_groups", cfg, N, k_lo, k_hi, T, split, flush=True)
    w = wl.make_config(cfg, N=N, k_lo=k_lo, k_hi=k_hi, T=T)
    beta = np.random.default_rng(5).random(N)
    prob = problem(lib, w)
    prob.set_bridge_split(split)
    off, th, b = pm.to_dev(w.offsets), pm.to_dev(w.theta), pm.to_dev(beta)
    fo, F = lib.gauss_newton_metric(prob, off, th, b)
    B = lib.gauss_newton_metric_blocks(prob, off, th, b)
    mask = np.random.default_rng(6).integers(0, 2, N).astype(np.uint8)
    _, Fm = lib.gauss_newton_metric(prob, off, th, b, mask=pm.to_dev(mask))
    torch.cuda.synchronize()
    prob.device_status()
    fo, F, B, Fm = fo.cpu().numpy(), F.cpu().numpy(), B.cpu().numpy(), Fm.cpu().numpy()
    idx = np.unique(np.concatenate([np.arange(min(N, 24)), np.argsort(w.K)[-8:], [N - 1]]))
    s = wl.subsample(w, idx)
    ref = orc.fisher(w.model, w.T, w.t_start, w.dt, w.sigma, s.offsets, s.theta, beta[idx],
                     split=split if split else None)
    small = problem(lib, s)
    small.set_bridge_split(split)
    sfo, sF = lib.gauss_newton_metric(small, pm.to_dev(s.offsets), pm.to_dev(s.theta), pm.to_dev(beta[idx]))
    sfo, sF = sfo.cpu().numpy(), sF.cpu().numpy()
    P = w.P
    for x, i in enumerate(idx):
        n = int(w.K[i]) * P
        got = F[fo[i]:fo[i + 1]].reshape(n, n)
        if n == 0:
            continue
        d = np.sqrt(np.diag(ref[x]))
        assert np.all(np.abs(got - ref[x]) <= TOL * np.outer(d, d) + 1e-300), i
        assert np.array_equal(got, got.T)
        alone = sF[sfo[x]:sfo[x + 1]].reshape(n, n)
        assert np.all(np.abs(got - alone) <= ULP4 * np.abs(alone)), i
        for k in range(int(w.K[i])):
            assert np.array_equal(B[w.offsets[i] + k], got[k * P:(k + 1) * P, k * P:(k + 1) * P])
    for i in range(N):
        a, e = fo[i], fo[i + 1]
        assert np.array_equal(Fm[a:e], F[a:e] if mask[i] else np.zeros(e - a))


def test_grouped_metric_skips_bad_particles(lib):
    """A block that does not fit its particle is left alone, with the flag;
    the other particles of its group are as without it."""
    w = wl.make_config("pulse_batch", N=4200, k_hi=6, k_lo=1, T=64)
    prob = problem(lib, w)
    off, th = pm.to_dev(w.offsets), pm.to_dev(w.theta)
    fo, F = lib.gauss_newton_metric(prob, off, th)
    size = F.numel()
    bad = fo.clone()
    bad[-1] += 1  # the last block no longer matches (K P)^2
    guard = torch.full((size + 2,), 7.0, dtype=torch.float64, device="cuda")
    lib.gauss_newton_metric(prob, off, th, f_offsets=bad, out=guard)
    with pytest.raises(lib.SmcxError, match="metric block offsets"):
        prob.device_status()
    last = int(fo[-2])
    assert torch.equal(guard[:last], F[:last])
    assert torch.all(guard[last:] == 7.0)
