"""The native calls of the Python binding: whose products a differentiable operation
runs, what a graph keeps alive, errors in a backward pass, other threads and streams."""
import gc
import threading
import weakref

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

RMAX = 8.0


@pytest.fixture()
def fitting():
    """(torch, fit, a library, theta, counts, var, K)"""
    import torch
    from paper_2106_09122_amd import fit, psflib
    d = synth.config_inputs(1)
    lib = psflib.Library(torch.from_numpy(d["cube"]).cuda(), d["radii"], d["N"], d["S"])
    th = torch.tensor(synth.DISK_START, dtype=torch.float64, device="cuda")
    rng = np.random.default_rng(3)
    counts = torch.from_numpy(rng.random(lib.M) * 100.0).cuda()
    var = torch.from_numpy(1.0 + rng.random(lib.M)).cuda()
    yield torch, fit, lib, th, counts, var, 1e9
    lib.close()


class _Own:
    """A library object with products of its own."""

    def __init__(self, lib):
        self.lib, self.N, self.S, self.ncols, self.M, self.device = lib, lib.N, lib.S, lib.ncols, lib.M, lib.device
        self.calls = []

    def apply(self, scene):
        self.calls.append(("apply", threading.get_ident(), scene.requires_grad))
        return self.lib.apply(scene)

    def apply_adjoint(self, g):
        self.calls.append(("adjoint", threading.get_ident(), g.requires_grad))
        return self.lib.apply_adjoint(g)


def test_loss_and_grad_of_other_objects(fitting):
    """The chain runs directly, each product once on the calling thread, in every
    grad mode: the loss and gradient of the library itself, bitwise."""
    torch, fit, lib, th, counts, var, K = fitting
    L, g = fit.loss_and_grad(lib, th, counts, var, K, RMAX)
    me = threading.get_ident()
    for mode in (torch.enable_grad, torch.no_grad, torch.inference_mode):
        own = _Own(lib)
        with mode():
            L1, g1 = fit.loss_and_grad(own, th, counts, var, K, RMAX)
        assert own.calls == [("apply", me, False), ("adjoint", me, False)]
        assert torch.equal(L1, L) and torch.equal(g1, g)
        assert L1.shape == L.shape and not L1.requires_grad and not g1.requires_grad
