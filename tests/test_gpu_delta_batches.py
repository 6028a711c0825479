"""Birth/death of pulses on handles made for hundreds of components: where particles mostly
have few, constants are kept batch by batch, and a particle of many has the bits of a
call in which all have many. Batch edges, empty particles, both lane tilings, few
items and many, a bridge split, no birth and no death."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu

K_EDGES = np.array([0, 1, 3, 126, 127, 128, 129, 253, 254, 255, 300])


@pytest.mark.parametrize("T,S,split,rest", [(1, 0, 0, 60), (1025, 0, 0, 60), (1025, 8, 300, 60), (4096, 0, 0, 4000),
                                            (9001, 0, 4000, 60), ((1 << 18) + 77, 0, 0, 60)])
def test_batches(lib, T, S, split, rest):
    print("[case] delta_batches", T, S, split, rest, flush=True)
    n, k_max, rng = len(K_EDGES), 300, np.random.default_rng(40)
    w = wl.make_config("pulse_batch", N=n + 1, k_lo=k_max, k_hi=k_max, T=max(T, 2), beta="uniform", seed=41)
    th = np.concatenate([w.theta[w.offsets[i]:w.offsets[i] + k] for i, k in enumerate(K_EDGES)])
    many = w.theta[w.offsets[n]:w.offsets[n + 1]]
    d = pm.to_dev(pm.data_of(w)[:T])
    death = np.array([0 if k == 1 else k // 2 + k // 3 - 1 if k else -1 for k in K_EDGES], dtype=np.int32)
    res = []
    for extra in (np.ones(rest, dtype=np.int64), np.full(n, k_max)):  # few rows a particle, many
        K = np.concatenate([K_EDGES, extra])
        N = len(K)
        assert (K.sum() <= 63 * N) == (extra[0] == 1)
        theta = np.concatenate([th] + [many[:k] for k in extra])
        off = np.concatenate([[0], np.cumsum(K)]).astype(np.int64)
        beta = np.concatenate([w.beta[:n], np.ones(N - n)])
        tb = np.concatenate([wl.draw_components(w.model, n, np.random.default_rng(42)),
                             wl.draw_components(w.model, N - n, rng)])
        di = np.concatenate([death, np.zeros(N - n, dtype=np.int32)])
        prob = lib.Problem(w.model, d, w.t_start, w.dt, w.sigma, k_max, N, len(theta))
        if S:
            prob.set_tiling(lib.KIND_DELTA, S, 1024, 1)
        prob.set_bridge_split(split)
        o, t, b, x, j = (pm.to_dev(v) for v in (off, theta, beta, tb, di))
        out = [*lib.delta_logl_birth_death(prob, o, t, b, x, j), lib.delta_logl_birth_death(prob, o, t, b, x, None)[0],
               lib.delta_logl_birth_death(prob, o, t, b, None, j)[1]]
        torch.cuda.synchronize()
        prob.device_status()
        res.append([v.cpu().numpy()[:n] for v in out])
    for u, v in zip(*res):
        assert np.array_equal(u, v)
