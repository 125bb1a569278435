"""Backward calls whose saved inputs come back from elsewhere: autograd may hand a backward call equal tensors at other addresses
(saved-tensor hooks that copy, recomputed checkpoints, data that have been set) or other tensors, and no sweeps of the forward
call are then taken over."""
import pytest
import torch
from torch.utils.checkpoint import checkpoint

from paper_2509_10613_amd import autograd as ska
from paper_2509_10613_amd import binding as sk

pytestmark = pytest.mark.gpu

LL = sk.SK_FLAG_LEAD_LAG


def paths(seed, n, L, d, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return ((torch.randn(n, L, d, generator=g, device="cuda", dtype=torch.float64) / (d * L) ** 0.5).cumsum(1)).to(dtype)


def _pair(x, y, lam, flags):
    return ska.sig_kernel(x, y, lam, lam, flags)


def _gram(x, y, lam, flags):
    return ska.sig_kernel_gram(x, y, lam, lam, flags)


def _one_set(x, y, lam, flags):
    return ska.sig_kernel_gram(x, None, lam, lam, flags)


CLASSES = {_pair: lambda x, y, lam, flags: ska._PairKernel.apply(x, y, lam, lam, flags),
           _gram: lambda x, y, lam, flags: ska._GramKernel.apply(x, y, lam, lam, flags),
           _one_set: lambda x, y, lam, flags: ska._GramKernelSym.apply(x, lam, lam, flags)}

# (wrapper, paths on either side, points, order, flags): few pairs keep both sweeps, the others the forward one (float: none)
CALLS = {
    "pairs": (_pair, 6, 6, 30, 1, 0),
    "pairs, lead-lag": (_pair, 4, 4, 30, 0, LL | 1),
    "pairs, bands": (_pair, 2, 2, 400, 0, 0),
    "many pairs": (_pair, 300, 300, 70, 1, 0),
    "gram": (_gram, 5, 7, 30, 1, 0),
    "gram, lead-lag": (_gram, 40, 40, 60, 1, LL),
    "gram of one set": (_one_set, 6, 6, 30, 1, 0),
}
HELD = []


def _copying():
    # (what the backward call gets lies elsewhere: the saved tensor itself is held)
    return torch.autograd.graph.saved_tensors_hooks(lambda t: HELD.append(t) or t, lambda t: t.clone())


@pytest.mark.parametrize("way", ["copies", "host", "checkpoint", "set"])
@pytest.mark.parametrize("native", [True, False], ids=["native", "classes"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", list(CALLS))
def test_gradients_do_not_depend_on_where_saved_inputs_lie(name, dtype, native, way):
    wrapper, n, m, L, lam, flags = CALLS[name]
    call = wrapper if native else CLASSES[wrapper]
    x, y = paths(11, n, L, 3, dtype).requires_grad_(), paths(12, m, L - 4, 3, dtype).requires_grad_()
    wanted = (x,) if name == "gram of one set" else (x, y)

    saved = []

    def loss(a, b):
        saved[:] = a * 1.0, b * 1.0                     # (the saved inputs are the products)
        k = call(*saved, lam, flags)
        return (k * torch.linspace(0.5, 1.5, k.numel(), device="cuda", dtype=dtype).reshape(k.shape)).sum()
    ref = torch.autograd.grad(loss(x, y), wanted)
    if way == "checkpoint":
        out = checkpoint(loss, x, y, use_reentrant=False)
    elif way == "set":
        out = loss(x, y)
        for t in saved:
            HELD.append(t.data)
            t.data = t.data.clone()
    else:
        with _copying() if way == "copies" else torch.autograd.graph.save_on_cpu():
            out = loss(x, y)
    saved.clear()
    block = [torch.full_like(t, 9.0) for t in (x, x, y, y)]     # (memory that the saved inputs may have lain in)
    for again in (True, False):
        got = torch.autograd.grad(out, wanted, retain_graph=again and way != "checkpoint")
        tol = 1e-12 if dtype == torch.float64 else 1e-5
        for g, r in zip(got, ref):
            assert float((g - r).abs().max()) <= tol * max(1.0, float(r.abs().max()))
        if way == "checkpoint":
            break
    HELD.clear()
    del block


@pytest.mark.parametrize("native", [True, False], ids=["native", "classes"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("name", list(CALLS))
def test_hooks_may_give_back_other_paths(name, dtype, native):
    # half of what was saved, in the same memory: gradients are those at the paths that came back, and no workspace is held for them
    wrapper, n, m, L, lam, flags = CALLS[name]
    call = wrapper if native else CLASSES[wrapper]
    x, y = paths(11, n, L, 3, dtype).requires_grad_(), paths(12, m, L - 4, 3, dtype).requires_grad_()
    wanted = (x,) if name == "gram of one set" else (x, y)
    halves = [(t.detach() * 0.5).requires_grad_() for t in (x, y)]
    ref = torch.autograd.grad(call(*halves, lam, flags).sum(), halves[:len(wanted)])
    call(x.detach(), y.detach(), lam, flags)
    saved = x * 1.0, y * 1.0
    before = torch.cuda.memory_allocated()
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.detach(), lambda t: t.mul_(0.5)):
        k = call(*saved, lam, flags)
    assert torch.cuda.memory_allocated() - before <= k.numel() * k.element_size() + 1024
    got = torch.autograd.grad(k.sum(), wanted)
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    for g, r in zip(got, ref):
        assert float((g - r).abs().max()) <= tol * max(1.0, float(r.abs().max()))


# what a hook may give back that is no place for a kernel to read the forward call's numbers from
UNFIT = {"host": lambda t: t.cpu(), "strides": lambda t: t.transpose(0, -1).contiguous().transpose(0, -1), "type": lambda t: t.float(),
         "points": lambda t: t[..., :-1].contiguous()}


def _signature(x, y, lam, flags):
    return ska.signature(x, 3)


@pytest.mark.parametrize("unfit", list(UNFIT))
@pytest.mark.parametrize("call", [_pair, _gram, _one_set, _signature])
def test_saved_tensors_that_come_back_unfit_are_refused(call, unfit):
    x, y = paths(13, 6, 30, 3, torch.float64).requires_grad_(), paths(14, 6, 30, 3, torch.float64)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, UNFIT[unfit]):
        out = call(x, y, 1, 0)
    with pytest.raises(ValueError):
        out.sum().backward()
    assert x.grad is None


@pytest.mark.parametrize("call", [_pair, _gram, _one_set, _signature])
def test_upstream_gradients_that_do_not_fit_are_refused(call):
    x, y = paths(13, 6, 30, 3, torch.float64).requires_grad_(), paths(14, 6, 30, 3, torch.float64)
    out = call(x, y, 1, 0)
    for g in (torch.ones_like(out).cpu(), torch.ones_like(out).float(), torch.ones_like(out)[:-1]):
        with pytest.raises(ValueError):
            out.grad_fn(g)


def test_what_the_library_refuses_is_its_own_exception():
    # 2000 channels have signatures but no gradients
    x = paths(15, 2, 4, 2000, torch.float64).requires_grad_()
    for out in (ska.signature(x, 1), ska._Signature.apply(x, 1, 0)):
        with pytest.raises(sk.SigKernelError, match="1024 channels"):
            out.sum().backward()
