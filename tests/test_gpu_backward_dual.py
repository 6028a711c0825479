"""LogLGrad's backward on dual numbers (forward mode over the backward pass): the
incoming gradient's tangent goes through the same products as its value."""
import pytest
import torch
from torch.autograd import forward_ad as fw

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_backward_of_dual_numbers(lib):
    print("[case] backward_dual", flush=True)
    N = 19
    w = wl.make_config("pulse_small", N=N, k_lo=0, k_hi=5, T=300, seed=12)
    off, be, th = pm.to_dev(w.offsets), pm.to_dev(w.beta), pm.to_dev(w.theta)
    prob = lib.Problem(w.model, pm.to_dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, w.k_max, N, w.M)
    _, grad = lib.logl_grad_batch(prob, off, th, be)
    K = off[1:] - off[:-1]
    rows = lambda v: grad * torch.repeat_interleave(v, K)[:, None]  # noqa: E731
    gen = torch.Generator(device="cuda").manual_seed(5)
    v, t = (torch.randn(N, dtype=torch.float64, device="cuda", generator=gen) for _ in range(2))
    leaf = th.clone().requires_grad_(True)
    with fw.dual_level():
        logl = lib.LogLGrad.apply(leaf, off, be, prob)
        back, = torch.autograd.grad(logl, leaf, fw.make_dual(v, t))
        value, tangent = fw.unpack_dual(back)
    assert torch.equal(value, rows(v))
    assert tangent is not None and torch.equal(tangent, rows(t))
