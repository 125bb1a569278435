"""The backward sweep of Gram matrices with four path pairs per wavefront (sk_four.hip) against the oracle: one and
several bands, rows above the grid, rows of the Gram matrix that are no multiple of four, refinement inside and above the
blocks, the time channel, float arrays, K(X, X), and pairs that drift and are taken out of their quad."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_10613_amd import binding as sk
from paper_2509_10613_amd import workloads
from tests.test_gpu_parity import check_grads, check_rows, check_values, dev, host, rounded

pytestmark = pytest.mark.gpu


def paths(seed, n, L, d, var):
    rng = np.random.default_rng(seed)
    return np.cumsum(rng.normal(0.0, var ** 0.5, (n, L, d)), axis=1)


# (Sixteen lanes with four block rows each, two from eight channels on and for blocks of 4 x 4 cells, are a band.)
@pytest.mark.parametrize("nx,ny,L1,L2,d,lam1,lam2,flags,sym,dtype", [
    (70, 66, 65, 64, 3, 0, 0, 0, False, torch.float64),      # one band, every row of every lane inside the grid
    (65, 72, 66, 12, 2, 0, 0, 1, False, torch.float64),      # 65 block rows: a second band for one of them
    (70, 68, 129, 5, 3, 0, 0, 1, False, torch.float32),      # two full bands, fewer columns than lanes
    (67, 66, 130, 40, 3, 1, 1, 0, False, torch.float64),     # three bands of 2 x 2 cells
    (65, 66, 70, 30, 8, 1, 1, 1, False, torch.float64),      # three bands of two rows per lane
    (130, 35, 20, 40, 5, 2, 2, 1, False, torch.float64),     # blocks of 4 x 4 cells
    (90, 54, 9, 10, 4, 3, 3, 0, False, torch.float64),       # refinement above the blocks
    (80, 61, 24, 20, 6, 0, 2, 1, False, torch.float64),      # unequal orders
    (93, 0, 33, 33, 3, 1, 1, 1, True, torch.float64),        # K(X, X): rows of the triangle
    (91, 0, 70, 70, 4, 0, 0, 0, True, torch.float32),
    (70, 0, 18, 18, 2, 0, 1, 0, True, torch.float64),        # K(X, X) with unequal orders: every pair
    (90, 50, 35, 30, 12, 0, 0, 1, False, torch.float64),     # twelve channels, two bands
    (70, 40, 20, 34, 14, 2, 2, 0, False, torch.float64),     # sixteen channels, blocks of 4 x 4 cells
    (4600, 1, 6, 20, 2, 0, 0, 0, False, torch.float64),      # fewer rows than lanes, one y path
])
def test_four_pairs_per_wave(nx, ny, L1, L2, d, lam1, lam2, flags, sym, dtype):
    X = paths(1300 + nx + d, nx, L1, d, 1.0 / (d * L1))
    Y = X if sym else paths(1400 + ny, ny, L2, d, 1.0 / (d * L2))
    ny = nx if sym else ny
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    desc = sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, L1, Y.shape[1], d, lam1, lam2, flags, sdt)
    assert (" symmetric_mode=four " in desc) if sym else desc.startswith("mode=four "), desc
    W = workloads.upstream_weights(88, (nx, ny))
    x = dev(X, dtype)
    K, gX, gY = sk.sigkernel_gram(x, x if sym else dev(Y, dtype), dev(W, dtype), lam1, lam2, flags)
    torch.cuda.synchronize()
    Xr = rounded(X, dtype)
    Kr, gXr, gYr = oracle.gram(Xr, Xr if sym else rounded(Y, dtype), rounded(W, dtype), lam1, lam2, flags)
    check_values(host(K), Kr, dtype, "K")
    check_grads(host(gX), gXr, dtype, "grad_X")
    if not sym:
        check_grads(host(gY), gYr, dtype, "grad_Y")


def run_with_counters(X, Y, W, lam, flags, dtype):
    """K, gradients, the pairs that drifted, and how often a wavefront asked the launch's counter for a quad."""
    sym = Y is None
    nx, L1, d = X.shape
    ny, L2 = (nx, L1) if sym else Y.shape[:2]
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    desc = sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, L1, L2, d, lam, lam, flags, sdt)
    assert (" symmetric_mode=four " in desc) if sym else desc.startswith("mode=four "), desc
    grid = int(desc.split(" symmetric_grid=" if sym else " grid=")[1].split()[0])
    quads = sum((m + 4) // 4 for m in range(nx)) if sym else ny * ((nx + 3) // 4)
    assert grid < quads, desc                       # wavefronts go on with further quads
    ws = torch.empty(sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM_BWD, nx, ny, L1, L2, d, lam, lam, flags, sdt),
                     dtype=torch.uint8, device="cuda")
    x = dev(X, dtype)
    out = sk.sigkernel_gram(x, x if sym else dev(Y, dtype), dev(W, dtype), lam, lam, flags, ws=ws)
    torch.cuda.synchronize()
    at = int(desc.split("drifted_pairs_counter_at=", 1)[1].split()[0])
    return out, int(ws[at:at + 4].view(torch.int32)[0]), int(ws[at - 4:at].view(torch.int32)[0])


@pytest.mark.parametrize("nx,ny,L1,L2,d,lam,flags,counted,dtype", [
    (300, 0, 60, 60, 3, 1, 0, True, torch.float64),          # K(X, X), one band: the triangle's rows, the launch's counter
    (300, 0, 70, 70, 3, 0, 1, True, torch.float64),          # ... several bands, the time channel
    (260, 130, 70, 64, 11, 0, 1, True, torch.float64),       # twelve channels, three bands
    (260, 250, 24, 20, 5, 2, 1, True, torch.float32),        # blocks of 4 x 4 cells
    (131, 90, 20, 24, 2, 0, 0, False, torch.float64),        # short: equal shares only; a last quad of three pairs
])
def test_wavefronts_with_several_quads(nx, ny, L1, L2, d, lam, flags, counted, dtype):
    X = paths(1700 + nx + d, nx, L1, d, 1.0 / (d * L1))
    Y = paths(1701 + ny, ny, L2, d, 1.0 / (d * L2)) if ny else None
    W = workloads.upstream_weights(92, (nx, ny or nx))
    (K, gX, gY), drifted, asked = run_with_counters(X, Y, W, lam, flags, dtype)
    assert drifted == 0 and (asked > 0) == counted
    Xr = rounded(X, dtype)
    Kr, gXr, gYr = oracle.gram(Xr, Xr if Y is None else rounded(Y, dtype), rounded(W, dtype), lam, lam, flags)
    check_values(host(K), Kr, dtype, "K")
    check_rows(host(gX), gXr, dtype, "grad_X")
    if ny:
        check_rows(host(gY), gYr, dtype, "grad_Y")


@pytest.mark.parametrize("nx,ny,L1,L2,d,lam,flags", [(260, 140, 40, 36, 3, 1, 1), (300, 0, 50, 50, 3, 1, 0),
                                                     (260, 0, 70, 70, 4, 0, 1), (250, 130, 40, 30, 12, 0, 0)])
def test_pairs_that_drift_leave_their_quads_and_the_wavefronts_go_on(nx, ny, L1, L2, d, lam, flags):
    X = paths(1710 + nx + d, nx, L1, d, 1.0 / (d * L1))
    Y = paths(1711 + ny, ny, L2, d, 1.0 / (d * L2)) if ny else None
    rng = np.random.default_rng(1712)
    wild = 0
    for P, rows in ((X, (7, 100, 201)), (Y, (3, 60))):
        if P is not None:
            for r in rows:
                P[r, 1:] = np.cumsum(rng.choice([-1.0, 1.0], size=(P.shape[1] - 1, d)) * (1.6 / d ** 0.5), axis=0)
            wild += len(rows)
    W = workloads.upstream_weights(93, (nx, ny or nx))
    (K, gX, gY), drifted, _ = run_with_counters(X, Y, W, lam, flags, torch.float64)
    assert 3 <= drifted <= wild * max(nx, ny) * (1 if ny else 2)
    Kr, gXr, gYr = oracle.gram(X, X if Y is None else Y, W, lam, lam, flags)
    check_values(host(K), Kr, torch.float64, "K")
    check_rows(host(gX), gXr, torch.float64, "grad_X")
    if ny:
        check_rows(host(gY), gYr, torch.float64, "grad_Y")


@pytest.mark.parametrize("L,d,lam,squared", [(100, 5, 1, 20.0), (100, 3, 1, 10.0), (60, 5, 0, 10.0), (40, 3, 2, 20.0),
                                             (60, 8, 1, 20.0), (40, 12, 1, 20.0), (30, 16, 0, 10.0)])
def test_four_pairs_per_wave_on_larger_increments(L, d, lam, squared):
    # The inverse recurrence holds on paths on which the one-pair kernels' does (they list 0, 0, 513 and 8 pairs of the first
    # four, with gradients within 7e-14, 2e-13, 4e-12 and 7e-13 of their largest entry; of the last three, with two block rows
    # per lane, 0, 0 and about 100, within 4e-14, 2e-14 and 2e-12).  Bounds: one pair in 500, and what
    # the drift guard lets pass of forward values (3e-12).
    nx, ny = 96, 48
    X, Y = paths(1600 + L + d, nx, L, d, squared / (d * (L - 1))), paths(1601 + L + d, ny, L, d, squared / (d * (L - 1)))
    W = workloads.upstream_weights(90, (nx, ny))
    desc = sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, L, L, d, lam, lam, 0, sk.SK_F64)
    assert "pairs_per_wave=4" in desc, desc
    ws = torch.empty(sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM_BWD, nx, ny, L, L, d, lam, lam, 0, sk.SK_F64),
                     dtype=torch.uint8, device="cuda")
    K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), lam, lam, 0, ws=ws)
    torch.cuda.synchronize()
    at = int(desc.split("drifted_pairs_counter_at=", 1)[1].split()[0])
    assert int(ws[at:at + 4].view(torch.int32)[0]) <= nx * ny // 500
    _, gXr, gYr = oracle.gram(X, Y, W, lam, lam, 0, dtype=np.longdouble)
    for got, ref in ((host(gX), np.asarray(gXr, np.float64)), (host(gY), np.asarray(gYr, np.float64))):
        err = np.max(np.abs(got - ref), axis=(1, 2)) / np.max(np.abs(ref), axis=(1, 2))
        assert np.max(err) <= 3e-12, np.max(err)


@pytest.mark.parametrize("L1,L2,d,lam", [(40, 40, 3, 1), (150, 30, 4, 0)])
def test_four_pairs_per_wave_with_pairs_that_drift(L1, L2, d, lam):
    # one path of either side with increments of order one: its pairs leave their quads, the others stay
    nx, ny = 72, 66
    X, Y = paths(1500, nx, L1, d, 1.0 / (d * L1)), paths(1501, ny, L2, d, 1.0 / (d * L2))
    rng = np.random.default_rng(1502)
    X[7, 1:] = np.cumsum(rng.choice([-1.0, 1.0], size=(L1 - 1, d)) * (1.6 / d ** 0.5), axis=0)
    Y[3, 1:] = np.cumsum(rng.choice([-1.0, 1.0], size=(L2 - 1, d)) * (1.6 / d ** 0.5), axis=0)
    W = workloads.upstream_weights(89, (nx, ny))
    need = sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM_BWD, nx, ny, L1, L2, d, lam, lam, 0, sk.SK_F64)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    desc = sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, L1, L2, d, lam, lam, 0, sk.SK_F64)
    assert "pairs_per_wave=4" in desc, desc
    K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), lam, lam, 0, ws=ws)
    torch.cuda.synchronize()
    at = int(desc.split("drifted_pairs_counter_at=", 1)[1].split()[0])
    n = int(ws[at:at + 4].view(torch.int32)[0])
    assert 0 < n <= nx + ny - 1
    Kr, gXr, gYr = oracle.gram(X, Y, W, lam, lam, 0)
    check_values(host(K), Kr, torch.float64, "K")
    check_rows(host(gX), gXr, torch.float64, "grad_X")
    check_rows(host(gY), gYr, torch.float64, "grad_Y")


@pytest.mark.parametrize("L1,L2,d,lam,flags", [(40, 40, 3, 1, 0), (150, 30, 4, 0, 0), (70, 24, 11, 0, 1)])
def test_quads_whose_pairs_all_drift_and_the_quads_after_them(L1, L2, d, lam, flags):
    # four neighbouring x paths with increments of order one: one quad of every Gram row has no pair left, and the wavefronts
    # go on with further quads
    nx, ny = 132, 72
    X, Y = paths(1510, nx, L1, d, 1.0 / (d * L1)), paths(1511, ny, L2, d, 1.0 / (d * L2))
    rng = np.random.default_rng(1512)
    X[4:8, 1:] = np.cumsum(rng.choice([-1.0, 1.0], size=(4, L1 - 1, d)) * ((12.0 if lam else 6.0) / d ** 0.5), axis=1)
    W = workloads.upstream_weights(91, (nx, ny))
    desc = sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, L1, L2, d, lam, lam, flags, sk.SK_F64)
    assert "pairs_per_wave=4" in desc and int(desc.split(" grid=")[1].split()[0]) < ny * nx // 4, desc
    ws = torch.empty(sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM_BWD, nx, ny, L1, L2, d, lam, lam, flags, sk.SK_F64),
                     dtype=torch.uint8, device="cuda")
    K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), lam, lam, flags, ws=ws)
    torch.cuda.synchronize()
    at = int(desc.split("drifted_pairs_counter_at=", 1)[1].split()[0])
    assert int(ws[at:at + 4].view(torch.int32)[0]) == 4 * ny
    Kr, gXr, gYr = oracle.gram(X, Y, W, lam, lam, flags)
    check_values(host(K), Kr, torch.float64, "K")
    check_rows(host(gX), gXr, torch.float64, "grad_X")
    check_rows(host(gY), gYr, torch.float64, "grad_Y")
