"""The default birth/death chunks of pulses: never longer than 8192 samples, however long
the record (few particles have no other waves to spread over), and the results
against the oracle over many of them."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 4096, 4097, 8192, 1 << 18, (1 << 19) + 1, 1 << 20, 1 << 22])
def test_default_chunk_is_bounded(lib, T):
    print("[case] delta_chunks", T, flush=True)
    d = torch.zeros(T, dtype=torch.float64, device="cuda")
    prob = lib.Problem(wl.PULSE, d, 0.0, 1.0 / max(T - 1, 1), 1.0, 2, 1, 2)
    S, chunk, _ = prob.get_tiling(lib.KIND_DELTA)
    assert chunk <= 8192 and chunk % (64 * S) == 0
    if T <= 4096:
        assert chunk >= T


@pytest.mark.parametrize("T", [(1 << 20) + 5])
def test_many_chunks(lib, orc, T):
    print("[case] delta_many_chunks", T, flush=True)
    w = wl.make_config("pulse_batch", N=3, k_lo=1, k_hi=3, T=T, beta="uniform", seed=23)
    rng = np.random.default_rng(24)
    tb, di = wl.draw_components(w.model, w.N, rng), np.zeros(w.N, dtype=np.int32)
    d, dev = pm.data_of(w), pm.to_dev
    prob = lib.Problem(w.model, dev(d), w.t_start, w.dt, w.sigma, w.k_max, w.N, w.M)
    db, dd = lib.delta_logl_birth_death(prob, dev(w.offsets), dev(w.theta), dev(w.beta), dev(tb), dev(di))
    torch.cuda.synchronize()
    prob.device_status()
    rb, rd = orc.delta_logl_birth_death(w.model, d, w.t_start, w.dt, w.sigma, w.offsets, w.theta, w.beta, tb, di)
    sb = pm.delta_scale(w.model, w, list(tb), w.beta, w.sigma, rb)
    sd = pm.delta_scale(w.model, w, [w.theta[o] for o in w.offsets[:-1]], w.beta, w.sigma, rd)
    assert np.all(np.abs(db.cpu().numpy() - rb) <= 1e-6 * sb)
    assert np.all(np.abs(dd.cpu().numpy() - rd) <= 1e-6 * sd)
