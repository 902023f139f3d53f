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


def _step(fit, lib, th, counts, var, K):
    t = th.clone().requires_grad_(True)
    L = fit.chi2(fit.simulate(lib, fit.render_disk(t, lib.N, lib.S, RMAX)), counts, var, K)
    L.backward()
    return L.detach(), t.grad


@pytest.mark.parametrize("where", ["instance", "class", "subclass"])
def test_replaced_products_are_called(fitting, monkeypatch, where):
    from paper_2106_09122_amd import psflib
    torch, fit, lib, th, counts, var, K = fitting
    want = _step(fit, lib, th, counts, var, K)
    calls = []

    def counted(name):
        plain = getattr(psflib.Library, name)

        def call(*a):
            calls.append(name)
            return plain(*((lib,) + a if where == "instance" else a))
        return call

    own = {name: counted(name) for name in ("apply", "apply_adjoint")}
    if where == "subclass":
        monkeypatch.setattr(lib, "__class__", type("Counted", (psflib.Library,), own))
    else:
        for name, f in own.items():
            monkeypatch.setattr(lib if where == "instance" else psflib.Library, name, f)
    L, g = _step(fit, lib, th, counts, var, K)
    assert calls == ["apply", "apply_adjoint"]
    assert torch.equal(L, want[0]) and torch.equal(g, want[1])
    L, g = fit.loss_and_grad(lib, th, counts, var, K, RMAX)
    assert calls == ["apply", "apply_adjoint"] * 2
    monkeypatch.undo()
    lib.apply(torch.zeros(lib.ncols, device="cuda"))
    assert len(calls) == 4


def test_adjoint_replaced_after_the_forward_pass(fitting, monkeypatch):
    """A backward pass looks the adjoint up when it runs; what it raises comes out."""
    torch, fit, lib, th, counts, var, K = fitting
    Z = torch.rand(lib.ncols, device="cuda", requires_grad=True)
    plain = lib.apply_adjoint
    calls = []

    def counted(g):
        calls.append(g.shape)
        return plain(g)

    S = fit.simulate(lib, Z)
    monkeypatch.setattr(lib, "apply_adjoint", counted)
    S.sum().backward()
    assert len(calls) == 1 and torch.equal(Z.grad, plain(torch.ones(lib.M, device="cuda")))

    def refuses(g):
        raise ValueError("not today")

    S = fit.simulate(lib, Z)
    monkeypatch.setattr(lib, "apply_adjoint", refuses)
    with pytest.raises(ValueError, match="not today"):
        S.sum().backward()


def test_arguments_that_are_not_tensors(fitting):
    torch, fit, lib, th, counts, var, K = fitting
    S = lib.apply(torch.zeros(lib.ncols, device="cuda"))
    for c, v in ((counts.cpu().numpy(), var), (None, var), (counts, var.cpu().numpy()), (counts, 1.0)):
        with pytest.raises(ValueError, match="must be a float64 tensor"):
            fit.chi2(S, c, v, K)
    with pytest.raises(ValueError, match="must be a float64 tensor"):
        fit.loss_and_grad(lib, th, counts, var.cpu().numpy(), K, RMAX)
    with pytest.raises(AttributeError):
        fit.simulate(lib, np.zeros(lib.ncols, np.float32))
    with pytest.raises(AttributeError):
        fit.loss_and_grad(lib, np.zeros(5), counts, var, K, RMAX)


def test_more_parameters_than_the_disk_has(fitting):
    """The disk is drawn from the first five of a longer vector; a shorter one is
    refused (tests/test_binding_errors.py)."""
    torch, fit, lib, th, counts, var, K = fitting
    longer = torch.cat([th, torch.ones(1, dtype=torch.float64, device="cuda")])
    assert torch.equal(fit.render_disk(longer, lib.N, lib.S, RMAX), fit.render_disk(th, lib.N, lib.S, RMAX))


def test_graph_keeps_the_library(fitting):
    torch, fit, lib, th, counts, var, K = fitting
    from paper_2106_09122_amd import psflib
    d = synth.config_inputs(1)
    Z = torch.rand(lib.ncols, device="cuda", requires_grad=True)
    want = lib.apply_adjoint(torch.ones(lib.M, device="cuda"))
    other = psflib.Library(torch.from_numpy(d["cube"]).cuda(), d["radii"], d["N"], d["S"])
    S = fit.simulate(other, Z)
    del other
    gc.collect()
    junk = [torch.full((lib.nbytes // 4,), 7.0, device="cuda") for _ in range(4)]  # would take freed memory
    S.sum().backward()
    assert torch.equal(Z.grad, want)
    del junk


def test_library_that_holds_a_graph_is_freed(fitting):
    """An image of its own kept on the library: a cycle that ends with the last
    outside reference."""
    torch, fit, lib, th, counts, var, K = fitting
    from paper_2106_09122_amd import psflib
    d = synth.config_inputs(1)
    Z = torch.rand(lib.ncols, device="cuda", requires_grad=True)
    gc.collect()
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    other = psflib.Library(torch.from_numpy(d["cube"]).cuda(), d["radii"], d["N"], d["S"])
    other.last = fit.simulate(other, Z)
    gone = weakref.ref(other)
    del other
    gc.collect()
    assert gone() is None
    assert torch.cuda.memory_allocated() == before


def test_library_closed_between_the_passes(fitting):
    torch, fit, lib, th, counts, var, K = fitting
    from paper_2106_09122_amd import psflib
    Z = torch.rand(lib.ncols, device="cuda", requires_grad=True)
    S = fit.simulate(lib, Z)
    lib.close()
    with pytest.raises(psflib.PsflibError) as e:
        S.sum().backward()
    assert e.value.status == psflib.ERR_INVALID_ARG
    with pytest.raises(psflib.PsflibError):
        lib.apply(Z.detach())


def test_backward_on_another_thread_and_stream(fitting):
    torch, fit, lib, th, counts, var, K = fitting
    want = _step(fit, lib, th, counts, var, K)
    t = th.clone().requires_grad_(True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        L = fit.chi2(fit.simulate(lib, fit.render_disk(t, lib.N, lib.S, RMAX)), counts, var, K)
    raised = []

    def run():
        try:
            L.backward()
        except BaseException as e:  # noqa: BLE001  (handed to the test)
            raised.append(e)

    th2 = threading.Thread(target=run)
    th2.start()
    th2.join()
    assert not raised
    torch.cuda.synchronize()
    assert torch.equal(L.detach(), want[0]) and torch.equal(t.grad, want[1])
