"""Birth/death in chunks of five to eight tiles: few particles (a wave per tile) and
many (a wave per particle) bitwise the same; nine tiles, where few take the plain form too."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,T,S,chunk", [("pulse_batch", (1 << 18) + 9, 0, 0), ("pulse_batch", 8192, 16, 8192),
                                           ("pulse_batch", 9001, 16, 5120), ("pulse_batch", 9300, 16, 9216),
                                           ("pulse_batch", 4000, 8, 3584), ("gb_grad", 14001, 16, 7168),
                                           ("gb_grad", 4097, 8, 4096)])
def test_long_chunks(lib, cfg, T, S, chunk):
    print("[case] delta_long_chunks", cfg, T, S, chunk, flush=True)
    n = 20
    N = 26 * torch.cuda.get_device_properties(0).multi_processor_count  # past the rule at one chunk
    w = wl.make_config(cfg, N=n, k_lo=0, k_hi=4, T=T, beta="uniform", rj=True)
    nch = -(-T // (chunk or 4096))
    rep = -(-N // (n * nch)) + 1
    off = np.concatenate([[0], np.cumsum(np.tile(w.K, rep))]).astype(np.int64)
    di = w.extra["death_idx"].copy()
    di[::5] = -1
    d = pm.to_dev(pm.data_of(w))
    res = []
    for o, r in ((w.offsets, 1), (off, rep)):
        prob = lib.Problem(w.model, d, w.t_start, w.dt, w.sigma, w.k_max, len(o) - 1, int(o[-1]))
        if chunk:
            prob.set_tiling(lib.KIND_DELTA, S, chunk, 1)
        else:
            assert prob.get_tiling(lib.KIND_DELTA)[1] > 4096
        o, t, b, tb, dj = (pm.to_dev(x) for x in (
            o, np.tile(w.theta, (r, 1)), np.tile(w.beta, r), np.tile(w.extra["theta_birth"], (r, 1)), np.tile(di, r)))
        out = [*lib.delta_logl_birth_death(prob, o, t, b, tb, dj),
               lib.delta_logl_birth_death(prob, o, t, b, tb, None)[0],
               lib.delta_logl_birth_death(prob, o, t, b, None, dj)[1]]
        torch.cuda.synchronize()
        prob.device_status()
        res.append([x.cpu().numpy() for x in out])
    for a, b in zip(*res):
        for q in (0, rep // 2, rep - 1):
            assert np.array_equal(b[q * n:(q + 1) * n], a)
