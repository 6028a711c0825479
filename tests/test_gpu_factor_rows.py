"""The register form of the metric factor (k_max P <= 64) at every block size
it has, against numpy in float64, with failing pivots among the blocks.

Tolerance as in test_gpu_metric_nuts.py: both sides are float64 with
cond(C) < 1e3 (C the correlation matrix), so an entry of W D (D =
sqrt(diag M)) agrees to a small multiple of cond(C) * 2^-52; the bound is
1e-10 of the row's largest entry.
"""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,k_max", [(wl.PULSE, 21), (wl.PULSE, 10), (wl.GBSINE, 16), (wl.GBSINE, 8)],
                         ids=["n63", "n30", "n64", "n32"])
def test_factor_rows(lib, model, k_max):
    print("[case] factor_rows", model, k_max, flush=True)
    P = wl.N_PARAMS[model]
    K = np.concatenate([np.arange(k_max + 1), [k_max, k_max, 1]])
    off = wl.counts_to_offsets(K)
    blocks = wl.spd_blocks(K * P, seed=31 + k_max)
    n = k_max * P
    # the last pivot not positive; a NaN in the last row; a NaN above the
    # diagonal, which is not read
    blocks[k_max + 1][n - 1, n - 1] *= -1.0
    blocks[k_max + 2][n - 1, 0] = np.nan
    blocks[k_max][0, n - 1] = np.nan
    fo, Fp = wl.pack_blocks(blocks)
    ridge = 10.0 ** np.random.default_rng(7).uniform(-3, 0, P)
    d = torch.zeros(64, dtype=torch.float64, device="cuda")
    prob = lib.Problem(model, d, 0.0, 1.0 / 63, 1.0, k_max, len(K), int(off[-1]))
    W = lib.metric_factor(prob, pm.to_dev(off), pm.to_dev(fo), pm.to_dev(Fp), ridge)
    with pytest.raises(lib.SmcxError, match="positive definite"):
        prob.device_status()
    W = W.cpu().numpy()
    for i, k in enumerate(K):
        m = int(k) * P
        got = W[fo[i]:fo[i + 1]].reshape(m, m)
        if m == 0:
            continue
        A = np.tril(blocks[i]) + np.tril(blocks[i], -1).T + np.diag(np.tile(ridge, int(k)))
        # definite unless an entry is NaN or a diagonal one not positive (the
        # ridge can outweigh a small negative one)
        if np.isnan(A).any() or np.any(np.diag(A) <= 0):
            assert i > k_max and np.all(np.isnan(got))
            continue
        D = np.sqrt(np.diag(A))
        ref = np.linalg.inv(np.linalg.cholesky(A / np.outer(D, D)))
        err = np.abs(got * D - ref)
        assert np.all(err <= 1e-10 * np.abs(ref).max(axis=1, keepdims=True)), (i, err.max())
        assert np.array_equal(np.triu(got, 1), np.zeros((m, m)))
    # in place, and for selected particles only
    mask = (np.arange(len(K)) % 2).astype(np.uint8)
    F = pm.to_dev(Fp)
    lib.metric_factor(prob, pm.to_dev(off), pm.to_dev(fo), F, ridge, out=F, mask=pm.to_dev(mask))
    F = F.cpu().numpy()
    for i in range(len(K)):
        want = W if mask[i] else Fp
        assert np.array_equal(F[fo[i]:fo[i + 1]], want[fo[i]:fo[i + 1]], equal_nan=True)
