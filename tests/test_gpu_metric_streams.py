"""Time-domain metric calls use none of the handle's workspace: on streams of their
own, beside likelihood and resampling calls and beside each other, they and
those give what they give alone."""
import numpy as np
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu
ROUNDS = 6


def _population(seed, N, k_hi, T):
    w = wl.make_config("pulse_batch", N=N, k_lo=0, k_hi=k_hi, T=T, beta="uniform", seed=seed)
    return w, [pm.to_dev(x) for x in (w.offsets, w.theta, w.beta)]


@pytest.mark.parametrize("k_hi,T", [(7, 2048), (20, 700), (5, 9000)])
def test_calls_side_by_side(lib, k_hi, T):
    print("[case] metric_streams", k_hi, T, flush=True)
    big, b = _population(1, 5000, k_hi, T)
    small, s = _population(2, 4100, k_hi, T)
    few, f = _population(3, 700, k_hi, T)
    prob = lib.Problem(big.model, pm.to_dev(pm.data_of(big)), big.t_start, big.dt, big.sigma, k_hi,
                       big.N, big.M)
    W = pm.to_dev(np.random.default_rng(4).dirichlet(np.ones(big.N)))
    fo = lib.metric_offsets(prob, b[0])
    size = int(fo[-1])
    jobs = {  # one stream each
        "metric": lambda: lib.gauss_newton_metric(prob, *b, f_offsets=fo, out=torch.empty(
            size, dtype=torch.float64, device="cuda"))[1],
        "blocks": lambda: lib.gauss_newton_metric_blocks(prob, *s),
        "grad": lambda: torch.cat([x.flatten() for x in lib.logl_grad_batch(prob, *f)]),
        "resample": lambda: lib.resample_systematic(prob, b[0], b[1], W, 0.25)[1],
    }
    alone = {k: j().clone() for k, j in jobs.items()}
    torch.cuda.synchronize()
    streams = {k: torch.cuda.Stream() for k in jobs}
    got = {k: [] for k in jobs}
    for _ in range(ROUNDS):
        for k, j in jobs.items():
            with torch.cuda.stream(streams[k]):
                got[k].append(j())
    torch.cuda.synchronize()
    prob.device_status()
    for k in jobs:
        for x in got[k]:
            assert torch.equal(x, alone[k]), k
