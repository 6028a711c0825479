"""Few work items take a workgroup each, a wave per tile; many take a wave each.
A particle's results are bitwise the same: two, three and four tiles, ragged
ends, several chunks, pulses that leave tiles empty, every call with a
likelihood pass, masked and invalid particles."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,T,tiling", [("pulse_batch", 2049, None), ("pulse_batch", 4096, None),
                                          ("pulse_batch", 6145, None), ("pulse_batch", 16384, None),
                                          ("pulse_batch", 700, (8, 1024)), ("pulse_batch", 8200, (64, 8192)),
                                          ("gb_grad", 1025, None), ("gb_grad", 4095, None),
                                          ("gb_grad", 9000, None)])
def test_tile_waves(lib, cfg, T, tiling):
    print("[case] tile_waves", cfg, T, tiling, flush=True)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 60
    N = 70 * n_cu  # past the rule at one wave per item and tile
    w = wl.make_config(cfg, N=n, k_lo=0, k_hi=4, T=T, beta="uniform")
    rep = N // n + 1
    K = np.tile(w.K, rep)
    off = np.concatenate([[0], np.cumsum(K)]).astype(np.int64)
    th, beta = np.tile(w.theta, (rep, 1)), np.tile(w.beta, rep)
    mask = np.tile(np.arange(n) % 3 != 0, rep).astype(np.uint8)
    rng = np.random.default_rng(3)
    p, g = rng.normal(size=(w.M, w.P)), rng.normal(size=(w.M, w.P))
    d = pm.to_dev(pm.data_of(w))
    res = []
    for o, t, b, m, r in ((w.offsets, w.theta, w.beta, mask[:n], 1), (off, th, beta, mask, rep)):
        prob = lib.Problem(w.model, d, w.t_start, w.dt, w.sigma, w.k_max, len(b), t.shape[0])
        if tiling:
            for kind in (lib.KIND_LOGL, lib.KIND_GRAD):
                prob.set_tiling(kind, tiling[0], tiling[1], 1)
        o, t, b, m = (pm.to_dev(x) for x in (o, t, b, m))
        out = [lib.logl_batch(prob, o, t, b), *lib.logl_grad_batch(prob, o, t, b)]
        out += lib.logl_grad_batch(prob, o, t, b, logl=torch.zeros_like(b), grad=torch.zeros_like(t), mask=m)
        out += lib.leapfrog(prob, o, b, 1e-5, t, pm.to_dev(np.tile(p, (r, 1))), pm.to_dev(np.tile(g, (r, 1))))
        out.append(lib.reweight_extend(prob, T // 3, T, o, t, 1.0)[0])
        torch.cuda.synchronize()
        try:  # the random momenta drive some sinusoids out of range: flagged in both
            prob.device_status()
            status = ""
        except lib.SmcxError as e:
            status = str(e)
        res.append((status, [x.cpu().numpy() for x in out]))
    assert res[0][0] == res[1][0] and (cfg == "gb_grad" or res[0][0] == "")
    for a, b in zip(res[0][1], res[1][1]):
        k = len(b) // rep
        assert len(a) == k
        for q in (0, rep // 2, rep - 1):
            assert np.array_equal(b[q * k:(q + 1) * k], a, equal_nan=True)


def test_invalid_particle_among_few(lib):
    print("[case] tile_waves invalid", flush=True)
    w = wl.make_config("pulse_batch", N=40, k_lo=3, k_hi=3, T=4096)
    prob = lib.Problem(w.model, pm.to_dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, 3, 40, w.M)
    off, th = pm.to_dev(w.offsets), pm.to_dev(w.theta)
    l0, g0 = (x.cpu().numpy() for x in lib.logl_grad_batch(prob, off, th))
    bad = w.offsets.copy()
    bad[8] += 1  # particle 7 has four rows (k_max is three), particle 8 two
    l, g = (x.cpu().numpy() for x in lib.logl_grad_batch(prob, pm.to_dev(bad), th))
    with pytest.raises(lib.SmcxError, match="k_max"):
        prob.device_status()
    assert np.isnan(l[7]) and np.array_equal(np.delete(l, [7, 8]), np.delete(l0, [7, 8]))
    assert np.all(np.isnan(g[21:25])) and np.array_equal(g[27:], g0[27:]) and np.array_equal(g[:21], g0[:21])
