"""Frequency-domain calls of few particles (four waves each) and of many (a wave
each): bitwise the same, for source counts around the rounds of four, bands of
one and two sizes, a bridge between two records, masked particles."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wide,bridge", [(0, False), (0, True), (200, False), (256, True)])
def test_split(lib, orc, wide, bridge):
    print("[case] gblisa_split", wide, bridge, flush=True)
    K = np.array([0, 1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 16, 17, 33, 1, 0])
    n, k_max = len(K), 33
    big = wl.make_gblisa(N=n, k_lo=k_max, k_hi=k_max, n_inj=4, beta="uniform", noise=True, seed=901)
    theta = np.concatenate([big.theta[big.offsets[i]:big.offsets[i] + K[i]] for i in range(n)])
    d = big.noise + orc.gblisa_spectrum(big.inj, big.T_obs, big.k0, big.B)
    if wide:
        d = np.pad(d, ((0, 0), (0, wide - big.B)))
    rng = np.random.default_rng(902)
    tb, mask = wl.draw_gblisa(n, rng), (np.arange(n) % 3 != 1).astype(np.uint8)
    di = np.array([rng.integers(-1, k) if k else -1 for k in K], dtype=np.int32)
    p, g = rng.normal(size=theta.shape), rng.normal(size=theta.shape)
    rep = 4 * torch.cuda.get_device_properties(0).multi_processor_count // n + 2  # past the rule
    res = []
    for r in (1, rep):
        off = np.concatenate([[0], np.cumsum(np.tile(K, r))]).astype(np.int64)
        prob, part = (lib.Problem.frequency_domain(wl.GBLISA, pm.to_dev(x), big.k0, big.T_obs, s, k_max,
                                                   n * r, int(off[-1]))
                      for x, s in ((d, big.S), (0.7 * d, 1.3 * big.S)))
        if bridge:
            prob.set_bridge_partner(part)
        o, t, b, m, bt, dj, mom, gr = (pm.to_dev(x) for x in (
            off, np.tile(theta, (r, 1)), np.tile(big.beta, r), np.tile(mask, r), np.tile(tb, (r, 1)),
            np.tile(di, r), np.tile(p, (r, 1)), np.tile(g, (r, 1))))
        out = [lib.logl_batch(prob, o, t, b), *lib.logl_grad_batch(prob, o, t, b),
               *lib.logl_grad_batch(prob, o, t, b, logl=torch.zeros_like(b), grad=torch.zeros_like(t), mask=m),
               *lib.delta_logl_birth_death(prob, o, t, b, bt, dj),
               *lib.leapfrog(prob, o, b, 1e-21, t, mom, gr)]
        torch.cuda.synchronize()
        prob.device_status()
        res.append([x.cpu().numpy() for x in out])
    for a, b in zip(*res):
        k = len(a)
        for q in (0, rep // 2, rep - 1):
            assert np.array_equal(b[q * k:(q + 1) * k], a)
