"""The kernels for any channel count (sk_wide.hip) against the oracle: one and several strips, one wave per pair and several
waves in a pipeline (more strips than waves among them), rows above the grid, channel counts around the tiles of the
matrix cores, refinement inside and above the blocks, the lead-lag forms, the time channel, float arrays, K(X, X), and
increments so large that the inverse recurrence of the other kernels would drift."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_10613_amd import autograd as ska
from paper_2509_10613_amd import binding as sk
from paper_2509_10613_amd import workloads
from tests.test_gpu_parity import check_grads, check_values, dev, host, rounded

pytestmark = pytest.mark.gpu

LL = sk.SK_FLAG_LEAD_LAG


def paths(seed, n, L, d, scale):
    return np.cumsum(np.random.default_rng(seed).normal(0.0, scale / (d * L) ** 0.5, (n, L, d)), axis=1)


def check(X, Y, W, gram, lam1, lam2, flags, dtype):
    sym = Y is None
    x = dev(X, dtype)
    y = x if sym else dev(Y, dtype)
    Xr = rounded(X, dtype)
    Yr = Xr if sym else rounded(Y, dtype)
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    op = sk.SK_OP_GRAM_BWD if gram else sk.SK_OP_BWD
    desc = sk.sigkernel_describe(op, len(X), len(Yr) if gram else 0, X.shape[1], Yr.shape[1], X.shape[2], lam1, lam2, flags, sdt)
    print(desc, flush=True)
    assert "kernel=wide_bwd_kernel" in desc, desc
    if gram:
        Kf = sk.sigkernel_gram(x, y, None, lam1, lam2, flags)
        K, gX, gY = sk.sigkernel_gram(x, y, dev(W, dtype), lam1, lam2, flags)
        Kr, gXr, gYr = oracle.gram(Xr, Xr if sym else Yr, rounded(W, dtype), lam1, lam2, flags)
    else:
        Kf = sk.sigkernel_fwd(x, y, lam1, lam2, flags)
        K, gX, gY = sk.sigkernel_bwd(x, y, dev(W, dtype), lam1, lam2, flags)
        Kr, gXr, gYr = oracle.bwd(Xr, Yr, rounded(W, dtype), lam1, lam2, flags)
    torch.cuda.synchronize()
    check_values(host(Kf), Kr, dtype, "K (forward only)")
    check_values(host(K), Kr, dtype, "K")
    check_grads(host(gX), gXr, dtype, "grad_X")
    if not sym:
        check_grads(host(gY), gYr, dtype, "grad_Y")
    return desc


@pytest.mark.parametrize("B,L1,L2,d,lam1,lam2,flags,dtype,waves", [
    (5, 20, 17, 17, 0, 0, 0, torch.float64, 1),        # one strip, part of it above the grid
    (4, 65, 64, 20, 0, 0, 1, torch.float64, 1),        # a full strip
    (3, 66, 2, 33, 0, 0, 0, torch.float64, 2),         # two strips, one column; channels beyond two tiles
    (3, 140, 150, 18, 0, 0, 1, torch.float32, 3),
    (2, 300, 70, 19, 1, 1, 0, torch.float64, 5),
    (2, 610, 40, 12, 0, 0, 1, torch.float64, 8),       # ten strips, eight waves: a second round; twelve channels
    (3, 90, 130, 16, 2, 2, 0, torch.float64, 2),       # blocks of 4 x 4 cells
    (2, 40, 30, 20, 3, 3, 1, torch.float64, 2),        # refinement above the blocks
    (2, 50, 30, 20, 0, 2, 0, torch.float64, 1),        # unequal orders
    (2, 30, 50, 20, 2, 1, 1, torch.float64, 1),
    (3, 70, 40, 18, 0, 0, LL | 1, torch.float64, 2),   # lead-lag inside the blocks
    (3, 70, 40, 18, 1, 1, LL, torch.float64, 2),
    (2, 40, 30, 18, 2, 2, LL | 1, torch.float64, 2),   # above the blocks
    (2, 30, 40, 18, 0, 1, LL | 1, torch.float64, 1),
    (2200, 70, 9, 17, 0, 0, 0, torch.float64, 1),      # one wave per pair, two strips, several pairs per wave
    (1, 2, 2, 40, 0, 0, 0, torch.float64, 1),          # a single cell
])
def test_pairs(B, L1, L2, d, lam1, lam2, flags, dtype, waves):
    X, Y = paths(1500 + L1, B, L1, d, 1.0), paths(1600 + L2, B, L2, d, 1.0)
    desc = check(X, Y, workloads.upstream_weights(91, (B,)), False, lam1, lam2, flags, dtype)
    assert " threads=%d " % (64 * waves) in desc, desc


@pytest.mark.parametrize("N,M,L1,L2,d,lam,flags,dtype", [
    (20, 31, 30, 20, 20, 0, 1, torch.float64),
    (50, 60, 12, 40, 17, 1, 0, torch.float32),
    (13, 0, 70, 70, 24, 0, 0, torch.float64),           # K(X, X)
    (70, 0, 12, 12, 18, 2, 1, torch.float32),
    (9, 0, 20, 20, 18, 1, LL, torch.float64),
    (6, 11, 150, 230, 10, 0, 0, torch.float64),         # nine to sixteen channels, y increments too long for LDS
])
def test_gram(N, M, L1, L2, d, lam, flags, dtype):
    X = paths(1700 + N, N, L1, d, 1.0)
    Y = paths(1800 + M, M, L2, d, 1.0) if M else None
    check(X, Y, workloads.upstream_weights(92, (N, M or N)), True, lam, lam, flags, dtype)


def test_large_increments():
    # products of increments of several units: B(p) of Eq. (1) may vanish, and nothing divides by it here
    X, Y = paths(1901, 4, 80, 20, 1.0), paths(1902, 4, 70, 20, 1.0)
    X[:, 10:12] += 3.0 / 20 ** 0.5
    Y[:, 20:23] -= 2.5 / 20 ** 0.5
    check(X, Y, workloads.upstream_weights(93, (4,)), False, 0, 0, 0, torch.float64)


def test_small_scratch_entry_point_still_takes_what_it_took():
    # sigkernel_bwd_static holds 64 MiB; where the wide kernels need more, it takes the kernels that need less
    B, L, d = 40, 400, 20
    X, Y = paths(1903, B, L, d, 1.0), paths(1904, B, L, d, 1.0)
    x, y, g = dev(X), dev(Y), dev(workloads.upstream_weights(94, (B,)))
    assert sk.sigkernel_workspace_bytes(sk.SK_OP_BWD, B, 0, L, L, d, 0, 0, 0, sk.SK_F64) > sk.SK_STATIC_SCRATCH_BYTES
    k, gx, gy = sk.sigkernel_bwd(x, y, g)
    k1, gx1, gy1 = torch.empty_like(k), torch.empty_like(gx), torch.empty_like(gy)
    sk.sigkernel_bwd_static(x, y, g, gx1, gy1, k1)
    torch.cuda.synchronize()
    check_values(host(k1), host(k), torch.float64, "k")
    check_grads(host(gx1), host(gx), torch.float64, "grad_x")
    check_grads(host(gy1), host(gy), torch.float64, "grad_y")


def sizes(op, n, m, L1, L2, d, lam, flags, sdt):
    shape = (op, n, m, L1, L2, d, lam, lam, flags, sdt)
    return sk.sigkernel_workspace_least_bytes(*shape), sk.sigkernel_workspace_bytes(*shape)


@pytest.mark.parametrize("n,m,L1,L2,d,lam,flags,dtype", [
    (300, None, 70, 40, 18, 1, 0, torch.float64),      # pairs: a wave or several per pair, by the workgroups there is room for
    (40, None, 520, 30, 17, 0, 1, torch.float64),      # nine strips
    (3, None, 300, 280, 20, 0, 0, torch.float64),      # the channel loops, where there is room for no wide workgroup
    (2, None, 90, 90, 18, 0, LL, torch.float32),
    (30, 41, 70, 66, 20, 0, 0, torch.float64),
    (25, 0, 70, 70, 17, 1, 1, torch.float32),          # K(X, X)
    (7, 9, 150, 230, 12, 0, 0, torch.float64),         # backward: y side too long for LDS
])
def test_workspaces_between_the_least_and_the_best(n, m, L1, L2, d, lam, flags, dtype):
    gram, sym = m is not None, m == 0
    X, Y = paths(2001, n, L1, d, 1.0), paths(2002, m or n, L2, d, 1.0)
    W = workloads.upstream_weights(98, (n, m or n) if gram else (n,))
    x = dev(X, dtype)
    y = x if sym else dev(Y, dtype)
    Xr = rounded(X, dtype)
    Yr = Xr if sym else rounded(Y, dtype)
    w, sdt = dev(W, dtype), sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    ref = (oracle.gram if gram else oracle.bwd)(Xr, Yr, rounded(W, dtype), lam, lam, flags)
    for back in (False, True):
        op = (sk.SK_OP_GRAM_BWD if back else sk.SK_OP_GRAM) if gram else (sk.SK_OP_BWD if back else sk.SK_OP_FWD)
        least, best = sizes(op, n, (m or n) if gram else 0, L1, L2, d, lam, flags, sdt)
        assert 0 < least <= best and (best > least or d <= 16)
        for size in sorted({least, least + 256, least + (best - least) // 3 // 256 * 256, best - 256 if best > least else best, best}):
            print("%s %d of %d" % ("backward" if back else "forward", size, best), flush=True)
            ws = torch.full((size,), 0xa5, dtype=torch.uint8, device="cuda")
            if not back:
                k = sk.sigkernel_gram(x, y, None, lam, lam, flags, ws=ws) if gram else sk.sigkernel_fwd(x, y, lam, lam, flags, ws=ws)
                check_values(host(k), ref[0], dtype, "K")
                continue
            k, gx, gy = sk.sigkernel_gram(x, y, w, lam, lam, flags, ws=ws) if gram else sk.sigkernel_bwd(x, y, w, lam, lam, flags, ws=ws)
            check_values(host(k), ref[0], dtype, "K")
            check_grads(host(gx), ref[1], dtype, "grad_X")
            if not sym:
                check_grads(host(gy), ref[2], dtype, "grad_Y")
        if sym:      # (needs less than the query says, which is K(X, Y)'s)
            continue
        with pytest.raises(sk.SigKernelError, match="workspace"):
            small = torch.empty(least - 256, dtype=torch.uint8, device="cuda")
            if gram:
                sk.sigkernel_gram(x, y, w if back else None, lam, lam, flags, ws=small)
            elif back:
                sk.sigkernel_bwd(x, y, w, lam, lam, flags, ws=small)
            else:
                sk.sigkernel_fwd(x, y, lam, lam, flags, ws=small)


def test_mmd_in_the_least_workspace():
    X, Y = dev(paths(2003, 12, 60, 18, 1.0)), dev(paths(2004, 9, 50, 18, 1.0))
    ref = sk.sigkernel_mmd2(X, Y)
    shape = (12, 9, 60, 50, 18, 0, 0, 0, sk.SK_F64)
    for want in (True, False):
        least = sk.load().sigkernel_mmd2_workspace_least_bytes(*shape, int(want))
        assert least < sk.load().sigkernel_mmd2_workspace_bytes(*shape, int(want))
        got = sk.sigkernel_mmd2(X, Y, want_x=want, want_y=want, ws=torch.full((least,), 0xa5, dtype=torch.uint8, device="cuda"))
        for g, r in zip(got, ref):
            assert g is None or float((g - r).abs().max()) <= 1e-12 * float(r.abs().max())
        with pytest.raises(sk.SigKernelError, match="workspace"):
            sk.sigkernel_mmd2(X, Y, want_x=want, want_y=want, ws=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("what", ["pairs", "gram", "mmd"])
@pytest.mark.parametrize("through", ["wrappers", "classes", "binding"])
def test_calls_go_on_where_the_device_has_no_room(through, what):
    # 1 GiB of memory for calls that are fastest with more (the allocator's own limit; nothing else is refused)
    n, L, d = {"pairs": (200, 600, 17), "gram": (40, 300, 20), "mmd": (40, 300, 20)}[what]
    x, y = (dev(paths(s, n, L, d, 1.0)).requires_grad_() for s in (2005, 2006))
    call = {"pairs": {"wrappers": lambda: ska.sig_kernel(x, y), "classes": lambda: ska._PairKernel.apply(x, y, 0, 0, 0)},
            "gram": {"wrappers": lambda: ska.sig_kernel_gram(x, y), "classes": lambda: ska._GramKernel.apply(x, y, 0, 0, 0)},
            "mmd": {"wrappers": lambda: ska.sig_mmd2(x, y), "classes": lambda: ska._Mmd2.apply(x, y, 0, 0, 0)}}[what]

    def step():
        if through != "binding":
            k = call[through]()
            return (k.detach(), *torch.autograd.grad(k.sum(), (x, y)))
        a, b = x.detach(), y.detach()
        if what == "mmd":
            return sk.sigkernel_mmd2(a, b)
        k = sk.sigkernel_gram(a, b) if what == "gram" else sk.sigkernel_fwd(a, b)
        return (k, *((sk.sigkernel_gram if what == "gram" else sk.sigkernel_bwd)(a, b, torch.ones_like(k))[1:]))
    ref = step()
    op = sk.SK_OP_BWD if what == "pairs" else sk.SK_OP_GRAM_BWD
    need = sizes(op, n, 0 if what == "pairs" else n, L, L, d, 0, 0, sk.SK_F64)
    assert need[0] < 1 << 30 < need[1]
    total = torch.cuda.get_device_properties(0).total_memory
    sk._ws_cache.clear()
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (1 << 30)) / total)
    try:
        got = step()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        sk._ws_cache.clear()
    for g, r in zip(got, ref):
        assert float((g - r).abs().max()) <= 1e-11 * float(r.abs().max())
