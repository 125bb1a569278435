"""Workspaces that autograd's forward calls hold on to for their backward calls: how many bytes all live graphs may hold
together, when they are given back, and calls that go on without one."""
import gc

import numpy as np
import pytest
import torch

from paper_2509_10613_amd import _native
from paper_2509_10613_amd import autograd as ska
from paper_2509_10613_amd import binding as sk


@pytest.fixture
def small_limits(monkeypatch):
    gc.collect()
    monkeypatch.setattr(ska, "_KEEP_LIMIT", 1 << 16)
    monkeypatch.setattr(ska, "_large_held", {})
    return monkeypatch


def test_bytes_held_by_all_live_workspaces(small_limits):
    small_limits.setattr(ska, "_KEEP_LARGE", 5 << 16)
    a = ska._keep_workspace(2 << 16, "cpu")
    b = ska._keep_workspace(2 << 16, "cpu")
    assert a.numel() == 2 << 16 and b is not None and ska._large_held == {"cpu": 4 << 16}
    assert ska._keep_workspace(2 << 16, "cpu") is None
    assert ska._keep_workspace(10, "cpu").numel() == 256 and ska._keep_workspace(1 << 16, "cpu") is not None
    del a
    assert ska._large_held == {"cpu": 2 << 16}
    c = ska._keep_workspace(3 << 16, "cpu")
    assert c is not None
    del b, c
    assert ska._large_held == {"cpu": 0}


def test_no_room_for_a_workspace(small_limits):
    def full(*args, **kwargs):
        raise torch.OutOfMemoryError("no room")
    small_limits.setattr(torch, "empty", full)
    assert ska._keep_workspace(1 << 10, "cpu") is None
    assert ska._keep_workspace(1 << 20, "cpu") is None and ska._large_held == {"cpu": 0}


@pytest.mark.parametrize("gram,symmetric,N,M,L,d,lam,flags,dt,form", [
    (False, False, 8, 0, 120, 3, 1, 0, sk.SK_F64, "sweeps"), (False, False, 64, 0, 101, 4, 0, 9, sk.SK_F32, "sweeps"),
    (False, False, 300, 0, 70, 3, 1, 0, sk.SK_F64, "forward"), (False, False, 300, 0, 70, 3, 1, 0, sk.SK_F32, None),
    (True, False, 5, 7, 30, 3, 1, 0, sk.SK_F64, "sweeps"), (True, True, 6, 6, 30, 3, 1, 0, sk.SK_F32, "sweeps"),
    (True, False, 40, 40, 60, 3, 1, 8, sk.SK_F64, "forward"),
    (True, False, 92, 92, 128, 3, 1, 0, sk.SK_F64, "forward"), (True, True, 92, 92, 64, 4, 0, 0, sk.SK_F64, None),    # four pairs a wave: none
    (False, False, 0, 0, 30, 3, 1, 0, sk.SK_F64, None), (False, False, 8, 0, 1, 3, 1, 0, sk.SK_F64, None),
])
def test_what_forward_calls_keep(gram, symmetric, N, M, L, d, lam, flags, dt, form):
    nbytes, *bits = _native.kept_form(gram, symmetric, N, M, L, L, d, lam, lam, flags, dt)
    if form is None:
        assert nbytes == 0
        return
    keep, have = {"sweeps": (sk.SK_FLAG_KEEP_SWEEPS, sk.SK_FLAG_HAVE_SWEEPS), "forward": (sk.SK_FLAG_KEEP_FORWARD, sk.SK_FLAG_HAVE_FORWARD)}[form]
    assert bits == [keep, have]
    assert nbytes == sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM if gram else sk.SK_OP_FWD, N, M, L, L, d, lam, lam, flags | keep, dt) > 0
    assert nbytes == sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM_BWD if gram else sk.SK_OP_BWD, N, M, L, L, d, lam, lam, flags | have, dt)


def _pairs(B=8, L=120, d=3):
    rng = np.random.default_rng(95)
    inc = rng.normal(0.0, (2.0 / (d * L)) ** 0.5, (2, B, L, d))
    x, y = (torch.tensor(np.cumsum(v, axis=1), device="cuda", requires_grad=True) for v in inc)
    need = sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, B, 0, L, L, d, 1, 1, sk.SK_FLAG_KEEP_SWEEPS, sk.SK_F64)
    assert sk.keeps_sweeps(B, L, L, d, 1, 1, 0, sk.SK_F64) and need > 1 << 16
    assert _native.kept_form(False, False, B, 0, L, L, d, 1, 1, 0, sk.SK_F64) == (need, sk.SK_FLAG_KEEP_SWEEPS, sk.SK_FLAG_HAVE_SWEEPS)
    return x, y, need


def _close(got, ref):
    return all(float((g - r).abs().max()) <= 1e-11 * float(r.abs().max()) for g, r in zip(got, ref))


@pytest.mark.gpu
def test_live_graphs_share_the_bytes_and_give_them_back(small_limits):
    x, y, need = _pairs()
    ref = torch.autograd.grad(ska.sig_kernel(x, y, 1, 1).sum(), (x, y))
    key = str(x.device)
    small_limits.setattr(ska, "_KEEP_LARGE", 2 * need)
    assert ska._large_held.get(key, 0) == 0
    losses = [ska.sig_kernel(x, y, 1, 1).sum() for _ in range(4)]            # two keep their sweep, two do not
    assert ska._large_held[key] == 2 * need
    assert [n.grad_fn.next_functions[0][0].ws is not None for n in losses] == [True, True, False, False]
    for n, loss in enumerate(losses):
        assert _close(torch.autograd.grad(loss, (x, y), retain_graph=True), ref)
        assert ska._large_held[key] == max(0, 1 - n) * need                  # given back though the graph lives
        assert _close(torch.autograd.grad(loss, (x, y)), ref)                # ... which sweeps forward again
    assert ska._large_held[key] == 0
    loss = ska.sig_kernel(x, y, 1, 1).sum()
    assert ska._large_held[key] == need
    del loss                                                                 # a graph that is dropped
    assert ska._large_held[key] == 0


@pytest.mark.gpu
def test_calls_go_on_where_a_workspace_does_not_fit(small_limits):
    x, y, need = _pairs()
    X = torch.cat([x.detach(), y.detach()]).requires_grad_()
    calls = [lambda: ska.sig_kernel(x, y, 1, 1).sum(), lambda: ska.sig_kernel_gram(x, y, 1, 1, sk.SK_FLAG_LEAD_LAG).sum(),
             lambda: ska.sig_kernel_gram(X, None, 1, 1).sum()]
    wanted = [(x, y), (x, y), (X,)]
    small_limits.setattr(ska, "_KEEP_LIMIT", 1 << 30)
    refs = [torch.autograd.grad(c(), w) for c, w in zip(calls, wanted)]
    empty = torch.empty

    def full(*args, **kwargs):
        if kwargs.get("dtype") == torch.uint8:
            raise torch.OutOfMemoryError("no room")
        return empty(*args, **kwargs)
    for c, w, ref in zip(calls, wanted, refs):
        small_limits.setattr(ska, "_KEEP_LIMIT", 256)
        small_limits.setattr(ska, "_KEEP_LARGE", 0)
        assert _close(torch.autograd.grad(c(), w), ref)                      # nothing is kept; the calls' own workspaces are there now
        small_limits.setattr(ska, "_KEEP_LIMIT", 1 << 30)
        small_limits.setattr(torch, "empty", full)
        try:
            loss = c()
        finally:
            small_limits.setattr(torch, "empty", empty)
        assert _close(torch.autograd.grad(loss, w), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("B,L,call", [(250, 256, lambda x, y: ska.sig_kernel(x, y, 1, 1)),
                                      (15, 200, lambda x, y: ska.sig_kernel_gram(x, y, 1, 1, sk.SK_FLAG_LEAD_LAG)),
                                      (48, 100, lambda x, y: ska.sig_kernel_gram(x + y, None, 1, 1))], ids=["pairs", "gram", "gram of one set"])
def test_native_calls_go_on_where_a_workspace_does_not_fit(B, L, call):
    # the allocator's own limit during the forward call: below what that call would keep, above what it needs
    gc.collect()
    sk._ws_cache.clear()
    torch.cuda.empty_cache()
    x, y, _ = _pairs(B, L, 3)
    before = torch.cuda.memory_allocated()
    k = call(x, y)
    held = torch.cuda.memory_allocated() - before
    assert held > 64 << 20
    ref = torch.autograd.grad(k.sum(), (x, y))
    del k
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    print("kept %d, allocated %d, reserved %d" % (held, torch.cuda.memory_allocated(), torch.cuda.memory_reserved()), flush=True)
    room = torch.cuda.memory_reserved() + held // 4 * 3
    torch.cuda.set_per_process_memory_fraction(room / torch.cuda.get_device_properties(0).total_memory)
    try:
        before = torch.cuda.memory_allocated()
        k = call(x, y)
        assert k.grad_fn.name().startswith("SigKernel") and torch.cuda.memory_allocated() - before < 32 << 20
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert _close(torch.autograd.grad(k.sum(), (x, y)), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("call", [lambda x, y: ska.sig_kernel(x, y, 1, 1), lambda x, y: ska.sig_kernel_gram(x, y, 1, 1)], ids=["pairs", "gram"])
def test_small_workspaces_of_all_live_graphs_have_a_bound_too(monkeypatch, call):
    gc.collect()
    x, y, _ = _pairs(12, 100, 3)
    ref = torch.autograd.grad(call(x, y).sum(), (x, y))

    def held(n):
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        ks = [call(x, y) for _ in range(n)]
        return ks, (torch.cuda.memory_allocated() - before)
    ks, one = held(1)
    assert one > 1 << 20
    del ks
    monkeypatch.setattr(ska, "_KEEP_ALL", 3 * one)
    for _ in range(2):                            # what a graph held is given back with it
        ks, all_of_them = held(9)
        assert 2 * one <= all_of_them <= 3 * one + (1 << 16)
        for k in ks:
            assert _close(torch.autograd.grad(k.sum(), (x, y), retain_graph=True), ref)
        torch.autograd.grad(ks[0].sum(), (x, y))  # ... or with the backward call that uses it up
        more, rest = held(2)
        assert one // 2 <= rest <= one + (1 << 16)
        del ks, more, k
