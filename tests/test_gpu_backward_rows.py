"""LogLGrad's backward: one kernel for plain tensors, torch operations where the
backward itself is recorded or batched. Both are one product per value: equal
bits."""
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,k_lo,k_hi", [(1, 1, 1), (16, 0, 5), (17, 6, 6), (700, 0, 24)])
def test_backward_rows(lib, N, k_lo, k_hi):
    print("[case] backward_rows", N, k_lo, k_hi, flush=True)
    w = wl.make_config("pulse_small", N=N, k_lo=k_lo, k_hi=k_hi, T=300, seed=11)
    off, be, th0 = pm.to_dev(w.offsets), pm.to_dev(w.beta), pm.to_dev(w.theta)
    prob = lib.Problem(w.model, pm.to_dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, w.k_max, N, w.M)
    _, grad = lib.logl_grad_batch(prob, off, th0, be)
    K = off[1:] - off[:-1]

    def back(g_of, **kw):
        th = th0.clone().requires_grad_(True)
        logl = lib.LogLGrad.apply(th, off, be, prob)
        return torch.autograd.grad(logl, th, g_of, **kw)[0]

    wide = torch.randn(2 * N, dtype=torch.float64, device="cuda")
    one = torch.ones((), dtype=torch.float64, device="cuda").expand(N)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), lambda t: t.cuda()):
        hooked = back(wide[:N])
    for g, got in ((wide[:N], back(wide[:N])), (wide[1::2], back(wide[1::2])), (one, back(one)),
                   (wide[:N], hooked), (wide.neg()[N:], back(wide.neg()[N:]))):
        assert torch.equal(got, grad * torch.repeat_interleave(g.contiguous(), K)[:, None])
    # recorded and batched backwards
    g = wide[:N].clone().requires_grad_(True)
    rec = back(g, create_graph=True)
    assert torch.equal(rec, back(wide[:N]))
    gg, = torch.autograd.grad(rec.sum(), g)
    ref = torch.zeros(N, dtype=torch.float64, device="cuda").index_add_(
        0, torch.repeat_interleave(torch.arange(N, device="cuda"), K), grad.sum(1))
    assert torch.allclose(gg, ref, rtol=1e-12, atol=1e-12 * float(grad.abs().max()))
    both = back(torch.stack([wide[:N], wide[N:]]), is_grads_batched=True)
    assert torch.equal(both[0], back(wide[:N])) and torch.equal(both[1], back(wide[N:]))
