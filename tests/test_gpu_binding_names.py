"""The binding's calls and LogLGrad's backward where torch lacks the short ways that
they take in its private names: the public ones give the same."""
import pytest
import torch

import parity as pm
from paper_2609_17674_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_has_storage", "_functorch",
                                     "_len_torch_dispatch_stack"])
def test_without_a_private_name(lib, monkeypatch, missing):
    print("[case] binding_names", missing, flush=True)
    N = 12
    w = wl.make_config("pulse_small", N=N, k_lo=1, k_hi=4, T=200, seed=14)
    off, be, th = pm.to_dev(w.offsets), pm.to_dev(w.beta), pm.to_dev(w.theta)
    prob = lib.Problem(w.model, pm.to_dev(pm.data_of(w)), w.t_start, w.dt, w.sigma, w.k_max, N, w.M)

    def both():
        leaf = th.clone().requires_grad_(True)
        logl = lib.LogLGrad.apply(leaf, off, be, prob)
        return logl.detach(), torch.autograd.grad(logl.sum(), leaf)[0]

    ref = both()

    class Without:  # torch._C but for one name
        def __getattr__(self, name):
            if name == missing:
                raise AttributeError(name)
            return getattr(torch._C, name)

    class Torch:
        _C = Without()

        def __getattr__(self, name):
            return getattr(torch, name)

    monkeypatch.setattr(lib, "torch", Torch())
    got = both()
    with torch.cuda.stream(torch.cuda.Stream()):
        side = both()
        torch.cuda.current_stream().synchronize()
    for a, b in zip(ref + ref, got + side):
        assert torch.equal(a, b)
