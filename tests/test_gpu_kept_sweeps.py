"""Forward and adjoint sweeps side by side, and the launch of independent tasks that takes both over (sk_split_*.hip): against the
oracle, by the shapes at which strips, tasks, groups of tasks and windows begin and end; the signature of what is kept."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_10613_amd import binding as sk
from paper_2509_10613_amd import workloads
from tests.test_gpu_parity import check_grads, check_values, dev, host, rounded

pytestmark = pytest.mark.gpu

LL = sk.SK_FLAG_LEAD_LAG
KEEP, HAVE = sk.SK_FLAG_KEEP_SWEEPS, sk.SK_FLAG_HAVE_SWEEPS


def paths(seed, n, L, d):
    return np.cumsum(np.random.default_rng(seed).normal(0.0, 1.0 / (d * L) ** 0.5, (n, L, d)), axis=1)


def need(op, n, m, L1, L2, d, lam1, lam2, flags, dtype):
    return sk.sigkernel_workspace_bytes(op, n, m, L1, L2, d, lam1, lam2, flags, sk.SK_F64 if dtype == torch.float64 else sk.SK_F32)


def run(X, Y, W, lam1, lam2, flags, dtype, gram):
    sym = Y is None
    x = dev(X, dtype)
    y = x if sym else dev(Y, dtype)
    Xr = rounded(X, dtype)
    Yr = Xr if sym else rounded(Y, dtype)
    n, L1, d = X.shape
    m, L2 = y.shape[0], y.shape[1]
    w = dev(W, dtype)
    op = (sk.SK_OP_GRAM, sk.SK_OP_GRAM_BWD) if gram else (sk.SK_OP_FWD, sk.SK_OP_BWD)
    mm = m if gram else 0
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    assert sk.keeps_sweeps(n, L1, L2, d, lam1, lam2, flags, sdt, gram_M=m if gram else None)
    desc = sk.sigkernel_describe(op[1], n, mm, L1, L2, d, lam1, lam2, flags | HAVE, sdt)
    print(desc, flush=True)
    size = need(op[0], n, mm, L1, L2, d, lam1, lam2, flags | KEEP, dtype)
    assert size == need(op[1], n, mm, L1, L2, d, lam1, lam2, flags | HAVE, dtype)
    ws = torch.full((size,), 0xa5, dtype=torch.uint8, device="cuda")        # nothing is read before it is written

    def forward(f):
        return sk.sigkernel_gram(x, y, None, lam1, lam2, f, ws=ws) if gram else sk.sigkernel_fwd(x, y, lam1, lam2, f, ws=ws)

    def backward(f, xx=x, **kw):
        if gram:
            return sk.sigkernel_gram(xx, xx if sym else y, w, lam1, lam2, f, ws=ws)
        return sk.sigkernel_bwd(xx, y, w, lam1, lam2, f, ws=ws, **kw)
    ref = oracle.gram(Xr, Yr, rounded(W, dtype), lam1, lam2, flags) if gram else oracle.bwd(Xr, Yr, rounded(W, dtype), lam1, lam2, flags)
    kf = forward(flags | KEEP)
    for _ in range(2):                                                      # what is kept may be taken over again
        k, gx, gy = backward(flags | HAVE)
        torch.cuda.synchronize()
        check_values(host(kf), ref[0], dtype, "k")
        check_values(host(k), ref[0], dtype, "k of the backward call")
        check_grads(host(gx), ref[1], dtype, "grad_x")
        if not sym:
            check_grads(host(gy), ref[2], dtype, "grad_y")
    if not gram:
        _, gx1, none = backward(flags | HAVE, want_y=False)
        assert none is None and float((gx1 - gx).abs().max()) <= 1e-12 * max(1.0, float(gx.abs().max()))
    # other paths, and a call of another kind on the workspace: NaN, never numbers
    other = x.clone()
    assert bool(torch.isnan(backward(flags | HAVE, other)[1]).all())
    plain = need(op[1], n, mm, L1, L2, d, lam1, lam2, flags, dtype)
    if plain <= size:
        backward(flags)
        assert bool(torch.isnan(backward(flags | HAVE)[1]).all())
    return desc


@pytest.mark.parametrize("B,L1,L2,d,lam1,lam2,flags,dtype", [
    (3, 33, 9, 3, 0, 0, 0, torch.float64),          # one strip, mostly above the grid; a single group of short tasks
    (4, 65, 66, 2, 0, 0, 1, torch.float64),         # a full strip
    (2, 66, 64, 5, 0, 0, 0, torch.float32),
    (3, 129, 200, 4, 0, 0, 0, torch.float64),       # two full strips
    (2, 130, 130, 8, 0, 0, 1, torch.float64),       # two block rows per lane
    (2, 257, 300, 5, 1, 1, 1, torch.float64),       # two strips of two block rows per lane
    (2, 300, 700, 3, 0, 0, 0, torch.float64),       # three strips, several groups of tasks
    (2, 510, 60, 3, 0, 0, 0, torch.float64),        # four strips
    (2, 100, 90, 16, 0, 0, 0, torch.float64),       # sixteen channels
    (2, 90, 250, 12, 1, 1, 1, torch.float64),
    (3, 40, 50, 8, 2, 2, 0, torch.float64),         # blocks of 4 x 4 cells
    (2, 30, 25, 6, 3, 3, 1, torch.float64),         # refinement above the blocks
    (2, 20, 40, 3, 1, 3, 0, torch.float64),         # unequal orders
    (2, 40, 20, 3, 2, 0, 1, torch.float64),
    (3, 60, 70, 4, 0, 0, LL | 1, torch.float32),    # lead-lag inside the blocks
    (3, 40, 40, 4, 1, 1, LL, torch.float64),
    (2, 24, 30, 4, 2, 2, LL | 1, torch.float64),    # above the blocks
    (2, 20, 30, 5, 0, 1, LL, torch.float64),
    (200, 40, 30, 3, 0, 0, 0, torch.float64),
    (3, 900, 700, 3, 0, 0, 1, torch.float64),       # bands
    (2, 600, 1100, 8, 1, 1, 0, torch.float32),
    (2, 530, 400, 5, 2, 2, 1, torch.float64),
    (2, 330, 300, 3, 1, 1, LL | 1, torch.float64),
    (2, 300, 260, 3, 2, 2, LL, torch.float64),
    (1, 2, 2, 2, 0, 0, 0, torch.float64),           # a single cell
])
def test_pairs(B, L1, L2, d, lam1, lam2, flags, dtype):
    run(paths(2100 + L1, B, L1, d), paths(2200 + L2, B, L2, d), workloads.upstream_weights(95, (B,)), lam1, lam2, flags, dtype, False)


@pytest.mark.parametrize("N,M,L1,L2,d,lam,flags,dtype", [
    (5, 7, 50, 70, 3, 1, 1, torch.float64),
    (4, 0, 90, 90, 5, 0, 0, torch.float64),          # K(X, X)
    (3, 4, 30, 40, 4, 1, LL, torch.float32),
    (2, 2, 800, 700, 3, 0, 0, torch.float64),        # bands
])
def test_gram(N, M, L1, L2, d, lam, flags, dtype):
    run(paths(2300 + N, N, L1, d), paths(2400 + M, M, L2, d) if M else None, workloads.upstream_weights(96, (N, M or N)), lam, lam, flags,
        dtype, True)


def test_large_increments_and_upstream_gradients():
    # no inverse recurrence: increments of order one stay exact.  An upstream gradient of NaN or zero reaches its pair only.
    X, Y = paths(2501, 3, 150, 3), paths(2502, 3, 140, 3)
    X[:, 1:4] += 1.3
    Y[:, 2:6] -= 1.1
    run(X, Y, workloads.upstream_weights(97, (3,)), 0, 0, 0, torch.float64, False)
    x, y = dev(X), dev(Y)
    ws = torch.empty(need(sk.SK_OP_FWD, 3, 0, 150, 140, 3, 0, 0, KEEP, torch.float64), dtype=torch.uint8, device="cuda")
    sk.sigkernel_fwd(x, y, 0, 0, KEEP, ws=ws)
    _, gx, gy = sk.sigkernel_bwd(x, y, dev(np.array([1.0, np.nan, 0.0])), 0, 0, HAVE, ws=ws)
    assert bool(torch.isnan(gx[1]).all()) and bool(torch.isnan(gy[1]).all())
    assert bool((gx[2] == 0).all()) and bool(torch.isfinite(gx[0]).all()) and bool((gx[0] != 0).any())


def test_a_wait_that_runs_out_gives_nan():
    X, Y = paths(2503, 2, 700, 3), paths(2504, 2, 650, 3)
    x, y, w = dev(X), dev(Y), dev(np.ones(2))
    f = sk.SK_FLAG_SHORT_WAITS
    ws = torch.empty(need(sk.SK_OP_FWD, 2, 0, 700, 650, 3, 0, 0, f | KEEP, torch.float64), dtype=torch.uint8, device="cuda")
    kf = sk.sigkernel_fwd(x, y, 0, 0, f | KEEP, ws=ws)
    k, gx, gy = sk.sigkernel_bwd(x, y, w, 0, 0, HAVE, ws=ws)
    torch.cuda.synchronize()
    # (with a single poll the sweeps may still have been in time)
    kr, gxr, gyr = oracle.bwd(X, Y, np.ones(2), 0, 0, 0)
    if bool(torch.isnan(gx).any()):
        assert bool(torch.isnan(gx).all()) and bool(torch.isnan(gy).all()) and bool(torch.isnan(k).all())
    else:
        check_values(host(kf), kr, torch.float64, "k")
        check_grads(host(gx), gxr, torch.float64, "grad_x")
    # the workspace serves the next call
    sk.sigkernel_fwd(x, y, 0, 0, KEEP, ws=ws)
    k, gx, gy = sk.sigkernel_bwd(x, y, w, 0, 0, HAVE, ws=ws)
    check_values(host(k), kr, torch.float64, "k")
    check_grads(host(gx), gxr, torch.float64, "grad_x")
    check_grads(host(gy), gyr, torch.float64, "grad_y")
