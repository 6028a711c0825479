"""Chunk sums of logL, a thread per particle: at and around a workgroup's 256
particles, with particles without components, inactive tails beyond k_max and
broken offsets, in sorted and in particle order. Against the oracle with the
logL bound of parity.py; the two orders bitwise."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 255, 256, 257])
@pytest.mark.parametrize("cfg", ["pulse_batch", "gb_grad"])
def test_chunk_sums(lib, orc, cfg, N):
    print("[case] chunk_sums", cfg, N, flush=True)
    K = np.random.default_rng(N).integers(0, 5, size=N)
    K[0] = 4
    off = np.concatenate([[0], np.cumsum(K)]).astype(np.int64)
    w = wl.make_config(cfg, N=N, k_lo=4, k_hi=4, T=5000, beta="uniform", seed=7)
    M = int(off[-1])
    th, d = w.theta[:M], pm.data_of(w)
    got = []
    for order in (1, 0):
        prob = lib.Problem(w.model, pm.to_dev(d), w.t_start, w.dt, w.sigma, 3, N, M)
        S, _, _ = prob.get_tiling(lib.KIND_LOGL)
        prob.set_tiling(lib.KIND_LOGL, S, max(64 * S, 1024), order)
        out = lib.logl_batch(prob, pm.to_dev(off), pm.to_dev(th), pm.to_dev(w.beta))
        torch.cuda.synchronize()
        with pytest.raises(lib.SmcxError, match="k_max"):
            prob.device_status()
        got.append(out.cpu().numpy())
        broken = off.copy()
        broken[0] = 1
        out = lib.logl_batch(prob, pm.to_dev(broken), pm.to_dev(th), pm.to_dev(w.beta))
        torch.cuda.synchronize()
        with pytest.raises(lib.SmcxError):
            prob.device_status()
        if order:
            assert np.all(np.isnan(out.cpu().numpy()))
    assert np.array_equal(got[0], got[1], equal_nan=True)
    assert np.all(np.isnan(got[0][K > 3]))
    ref = orc.logl(w.model, d, w.t_start, w.dt, w.sigma, off, th, w.beta)
    ok = K <= 3
    if ok.any():
        pm.assert_logl(got[0][ok], ref[ok])
