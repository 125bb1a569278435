"""Workspaces that autograd's forward calls hold on to for their backward calls: how many bytes all live graphs may hold
together, when they are given back, and calls that go on without one."""
import gc

import numpy as np
import pytest
import torch

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


def _pairs(B=8, L=120, d=3):
    rng = np.random.default_rng(95)
    inc = rng.normal(0.0, (2.0 / (d * L)) ** 0.5, (2, B, L, d))
    x, y = (torch.tensor(np.cumsum(v, axis=1), device="cuda", requires_grad=True) for v in inc)
    need = sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, B, 0, L, L, d, 1, 1, sk.SK_FLAG_KEEP_FORWARD, sk.SK_F64)
    assert sk.keeps_forward(B, L, L, d, 1, 1, 0, sk.SK_F64) and need > 1 << 16
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
