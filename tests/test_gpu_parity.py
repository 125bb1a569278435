"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element, on the same
seeded inputs.  Tolerances (written here, used everywhere below):

  fp64: 1e-10, fp32: 1e-4, relative in the sense
    values    |gpu - ref| <= tol * max(1, |ref|)            per element
    gradients max|gpu - ref| <= tol * max(1, max|ref|)       per output tensor
  (gradient entries cross zero, so they are compared against the tensor's scale).
  fp32 runs are compared with the fp64 oracle evaluated on the fp32-rounded inputs.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_10613_amd import binding as sk
from paper_2509_10613_amd import workloads

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-10, torch.float32: 1e-4, "wild": 1e-9}


def dev(a, dtype=torch.float64):
    return torch.tensor(np.asarray(a), dtype=dtype, device="cuda")


def host(t):
    return t.detach().cpu().numpy().astype(np.float64)


def rounded(a, dtype):
    """The inputs as the GPU sees them (fp32 rounding applied), back in float64 for the oracle."""
    return host(dev(a, dtype))


def check_values(got, ref, dtype, what):
    tol = TOL[dtype]
    err = np.abs(got - ref) / np.maximum(1.0, np.abs(ref))
    print("%s: max scaled err %.3e (tol %.0e)" % (what, err.max() if err.size else 0.0, tol), flush=True)
    assert got.shape == ref.shape
    assert np.all(np.isfinite(got))
    assert (err.max() if err.size else 0.0) <= tol, what


def check_grads(got, ref, dtype, what):
    tol = TOL[dtype]
    scale = max(1.0, np.max(np.abs(ref))) if ref.size else 1.0
    err = (np.max(np.abs(got - ref)) if ref.size else 0.0) / scale
    print("%s: max err / scale %.3e (tol %.0e)" % (what, err, tol), flush=True)
    assert got.shape == ref.shape
    assert np.all(np.isfinite(got))
    assert err <= tol, what


def run_pairs(X, Y, lam1, lam2, flags, dtype, backward, seed=5, keep=False):
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    x, y = dev(X, dtype), dev(Y, dtype)
    k = sk.sigkernel_fwd(x, y, lam1, lam2, flags)
    torch.cuda.synchronize()
    kref = oracle.fwd(Xr, Yr, lam1, lam2, flags)
    check_values(host(k), kref, dtype, "k")
    if backward:
        gk = workloads.upstream_weights(seed, (X.shape[0],))
        gkr = rounded(gk, dtype)
        k2, gx, gy = sk.sigkernel_bwd(x, y, dev(gk, dtype), lam1, lam2, flags)
        torch.cuda.synchronize()
        kr, gxr, gyr = oracle.bwd(Xr, Yr, gkr, lam1, lam2, flags)
        check_values(host(k2), kr, dtype, "k (from bwd)")
        check_grads(host(gx), gxr, dtype, "grad_x")
        check_grads(host(gy), gyr, dtype, "grad_y")
        if keep:   # the step bench.py times: the forward call keeps its sweep for the backward call
            B, L1, d = X.shape
            sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
            need = sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, B, 0, L1, Y.shape[1], d, lam1, lam2,
                                                flags | sk.SK_FLAG_KEEP_FORWARD, sdt)
            ws = torch.empty(need, dtype=torch.uint8, device="cuda")
            k3 = sk.sigkernel_fwd(x, y, lam1, lam2, flags | sk.SK_FLAG_KEEP_FORWARD, ws=ws)
            k4, gx, gy = sk.sigkernel_bwd(x, y, dev(gk, dtype), lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
            torch.cuda.synchronize()
            check_values(host(k3), kr, dtype, "k (kept sweep)")
            check_values(host(k4), kr, dtype, "k (from bwd after a kept sweep)")
            check_grads(host(gx), gxr, dtype, "grad_x (kept sweep)")
            check_grads(host(gy), gyr, dtype, "grad_y (kept sweep)")


def rand_paths(seed, B, L, d, scale=0.3):
    rng = np.random.default_rng(seed)
    return np.cumsum(rng.normal(0, scale, size=(B, L, d)), axis=1)


# ------------------------------------------------------------------ the five configurations
def test_c1_forward_fp64():
    w, X, Y = workloads.make("c1")
    run_pairs(X, Y, w.lam, w.lam, w.flags, torch.float64, backward=False)


def test_c2_forward_backward_fp64_full_size():
    w, X, Y = workloads.make("c2")
    assert sk.keeps_forward(w.n_x, w.L, w.L, w.d, w.lam, w.lam, w.flags, sk.SK_F64)
    run_pairs(X, Y, w.lam, w.lam, w.flags, torch.float64, backward=True, keep=True)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_c3_gram_reduced(dtype):
    w, X, Y = workloads.make("c3", n_x=20, n_y=12)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    W = workloads.upstream_weights(33, (20, 12))
    Wr = rounded(W, dtype)
    K = sk.sigkernel_gram(dev(X, dtype), dev(Y, dtype), None, w.lam, w.lam, w.flags)
    Kref, gXr, gYr = oracle.gram(Xr, Yr, Wr, w.lam, w.lam, w.flags)
    check_values(host(K), Kref, dtype, "K")
    K2, gX, gY = sk.sigkernel_gram(dev(X, dtype), dev(Y, dtype), dev(W, dtype), w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    check_values(host(K2), Kref, dtype, "K (from bwd)")
    check_grads(host(gX), gXr, dtype, "grad_X")
    check_grads(host(gY), gYr, dtype, "grad_Y")


def test_c4_long_sequences_two_pairs_full_length():
    w, X, Y = workloads.make("c4", n_x=2, n_y=2)
    run_pairs(X, Y, w.lam, w.lam, w.flags, torch.float64, backward=True, keep=True)


def test_c5_gram_reduced_and_symmetric():
    w, X, Y = workloads.make("c5", n_x=40, n_y=24)
    W = workloads.upstream_weights(55, (40, 24))
    x, y = dev(X), dev(Y)
    K, gX, gY = sk.sigkernel_gram(x, y, dev(W), w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    Kref, gXr, gYr = oracle.gram(X, Y, W, w.lam, w.lam, w.flags)
    check_values(host(K), Kref, torch.float64, "K")
    check_grads(host(gX), gXr, torch.float64, "grad_X")
    check_grads(host(gY), gYr, torch.float64, "grad_Y")
    # symmetric case K(X,X): same pointer for both arguments
    Ws = workloads.upstream_weights(56, (40, 40))
    Kxx, gXX, none = sk.sigkernel_gram(x, x, dev(Ws), w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    Kxr, gXXr, _ = oracle.gram(X, X, Ws, w.lam, w.lam, w.flags)
    assert none is None
    check_values(host(Kxx), Kxr, torch.float64, "K(X,X)")
    check_grads(host(gXX), gXXr, torch.float64, "grad_X total")
    assert torch.equal(Kxx, Kxx.T)      # k(x,y) = k(y,x) bit for bit


@pytest.mark.parametrize("name,nx,ny,dtype", [("c3", 64, 40, torch.float64), ("c3", 60, 44, torch.float32),
                                              ("c5", 80, 70, torch.float64)])
def test_gram_with_thousands_of_pairs(name, nx, ny, dtype):
    # enough pairs that every wave works through a run of them (the y path and its gradient accumulator stay
    # in LDS over the run), gradients included; then the symmetric case at the same size
    w, X, Y = workloads.make(name, n_x=nx, n_y=ny)
    mode = "mode=tile" if name == "c5" else "mode=solo"   # c5: contractions on the matrix cores
    assert mode in sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, w.L, w.L, w.d, w.lam, w.lam, w.flags, sk.SK_F64)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    W = workloads.upstream_weights(57, (nx, ny))
    K, gX, gY = sk.sigkernel_gram(dev(X, dtype), dev(Y, dtype), dev(W, dtype), w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    Kref, gXr, gYr = oracle.gram(Xr, Yr, rounded(W, dtype), w.lam, w.lam, w.flags)
    check_values(host(K), Kref, dtype, "K")
    check_grads(host(gX), gXr, dtype, "grad_X")
    check_grads(host(gY), gYr, dtype, "grad_Y")
    Kf = sk.sigkernel_gram(dev(X, dtype), dev(Y, dtype), None, w.lam, w.lam, w.flags)
    check_values(host(Kf), Kref, dtype, "K (forward only)")
    Ws = workloads.upstream_weights(58, (nx, nx))
    x = dev(X, dtype)
    Kxx, gXX, none = sk.sigkernel_gram(x, x, dev(Ws, dtype), w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    Kxr, gXXr, _ = oracle.gram(Xr, Xr, rounded(Ws, dtype), w.lam, w.lam, w.flags)
    assert none is None
    check_values(host(Kxx), Kxr, dtype, "K(X,X)")
    check_grads(host(gXX), gXXr, dtype, "grad_X total")
    assert torch.equal(Kxx, Kxx.T)


@pytest.mark.parametrize("L1,L2,d,flags,dtype", [(64, 64, 16, 0, torch.float64), (40, 60, 16, 1, torch.float64),
                                                  (65, 34, 7, 1, torch.float64), (50, 65, 12, 0, torch.float32),
                                                  (34, 34, 8, 0, torch.float64)])
def test_tile_mode_shapes(L1, L2, d, flags, dtype):
    # tile kernels (increment Gram matrix of a pair in LDS, contractions by MFMA): unequal lengths, channel
    # counts that do not fill the operand registers, time augmentation, float callers, the largest grid (64 x 64)
    nx, ny = 37, 31   # more pairs than lock-step mode takes
    rng = np.random.default_rng(700 + L1 + d)
    X = np.cumsum(rng.normal(0.0, (1.0 / (d * L1)) ** 0.5, (nx, L1, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / (d * L2)) ** 0.5, (ny, L2, d)), axis=1)
    assert "mode=tile" in sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, L1, L2, d, 0, 0, flags, sk.SK_F64)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    W = workloads.upstream_weights(59, (nx, ny))
    K, gX, gY = sk.sigkernel_gram(dev(X, dtype), dev(Y, dtype), dev(W, dtype), 0, 0, flags)
    Kf = sk.sigkernel_gram(dev(X, dtype), dev(Y, dtype), None, 0, 0, flags)
    torch.cuda.synchronize()
    Kref, gXr, gYr = oracle.gram(Xr, Yr, rounded(W, dtype), 0, 0, flags)
    check_values(host(K), Kref, dtype, "K")
    check_values(host(Kf), Kref, dtype, "K (forward only)")
    check_grads(host(gX), gXr, dtype, "grad_X")
    check_grads(host(gY), gYr, dtype, "grad_Y")


@pytest.mark.parametrize("nx,ny,L1,L2,d,flags,sym,dtype", [(2003, 1, 64, 64, 16, 0, False, torch.float64),
                                                            (5, 300, 34, 65, 8, 1, False, torch.float64),
                                                            (301, 0, 64, 64, 16, 0, True, torch.float64),
                                                            (302, 0, 40, 40, 9, 1, True, torch.float64),
                                                            (330, 7, 50, 44, 12, 1, False, torch.float32),
                                                            (203, 0, 65, 65, 16, 0, True, torch.float32)])
def test_quad_mode_forward(nx, ny, L1, L2, d, flags, sym, dtype):
    # forward Gram calls on the tile kernels' shapes: four pairs of a Gram row per wave (16 lanes with four grid rows
    # each per pair).  Rows whose length is not a multiple of four (the last group repeats a pair and writes nothing
    # for it), a single row, many short rows, K(X, X), whose row m has the pairs n <= m only, float arrays, the
    # largest grid (64 x 64).
    rng = np.random.default_rng(900 + nx + d)
    X = np.cumsum(rng.normal(0.0, (1.0 / (d * L1)) ** 0.5, (nx, L1, d)), axis=1)
    Y = X if sym else np.cumsum(rng.normal(0.0, (1.0 / (d * L2)) ** 0.5, (ny, L2, d)), axis=1)
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    assert "mode=quad" in sk.sigkernel_describe(sk.SK_OP_GRAM, nx, Y.shape[0], L1, Y.shape[1], d, 0, 0, flags, sdt)
    x = dev(X, dtype)
    K = sk.sigkernel_gram(x, x if sym else dev(Y, dtype), None, 0, 0, flags)
    torch.cuda.synchronize()
    Xr = rounded(X, dtype)
    Kref = oracle.gram(Xr, Xr if sym else rounded(Y, dtype), None, 0, 0, flags)
    check_values(host(K), Kref, dtype, "K")
    if sym:
        assert torch.equal(K, K.T)


@pytest.mark.parametrize("nx,ny,L,d,lam,flags,build", [(300, 5, 128, 6, 1, 0, 1), (290, 6, 128, 5, 1, 1, 1),
                                                         (280, 7, 100, 8, 0, 0, 1), (270, 5, 65, 8, 2, 0, 1),
                                                         (300, 6, 64, 8, 1, 0, 2), (300, 5, 128, 3, 1, 0, 2),
                                                         (260, 6, 40, 16, 0, 8, 1), (260, 6, 30, 16, 0, 0, 1)])
def test_solo_backward_builds(nx, ny, L, d, lam, flags, build):
    # The solo backward kernels exist in a build for two waves per SIMD and one for a single wave (the whole register
    # file); the launcher takes the second where LDS leaves room for one workgroup per compute unit, and kernels with
    # many channels have no other.  Both builds against the oracle, the build named by the launch plan.
    rng = np.random.default_rng(1200 + L + d)
    X = np.cumsum(rng.normal(0.0, (1.0 / (d * L)) ** 0.5, (nx, L, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / (d * L)) ** 0.5, (ny, L, d)), axis=1)
    desc = sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, L, L, d, lam, lam, flags, sk.SK_F64)
    assert "mode=solo" in desc and ", %d> " % build in desc, desc
    W = workloads.upstream_weights(61, (nx, ny))
    K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), lam, lam, flags)
    torch.cuda.synchronize()
    Kref, gXr, gYr = oracle.gram(X, Y, W, lam, lam, flags)
    check_values(host(K), Kref, torch.float64, "K")
    check_grads(host(gX), gXr, torch.float64, "grad_X")
    check_grads(host(gY), gYr, torch.float64, "grad_Y")


def test_tile_mode_pair_batch():
    # a batch of pairs (not a Gram matrix) large enough to leave lock-step mode: every pair brings its own y path
    B, L, d = 1100, 48, 16
    rng = np.random.default_rng(77)
    X = np.cumsum(rng.normal(0.0, (1.0 / (d * L)) ** 0.5, (B, L, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / (d * L)) ** 0.5, (B, L, d)), axis=1)
    assert "mode=tile" in sk.sigkernel_describe(sk.SK_OP_BWD, B, 0, L, L, d, 0, 0, 0, sk.SK_F64)
    gk = workloads.upstream_weights(60, (B,))
    k, gx, gy = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), 0, 0, 0)
    kf = sk.sigkernel_fwd(dev(X), dev(Y), 0, 0, 0)
    torch.cuda.synchronize()
    kr, gxr, gyr = oracle.bwd(X, Y, gk, 0, 0, 0)
    check_values(host(k), kr, torch.float64, "k")
    check_values(host(kf), kr, torch.float64, "k (forward only)")
    check_grads(host(gx), gxr, torch.float64, "grad_x")
    check_grads(host(gy), gyr, torch.float64, "grad_y")


def test_short_paths_with_many_channels_stay_solo():
    # 16 channels but fewer than 33 cells per side, few x paths: the solo kernels (channel contraction on the vector units)
    nx, ny, L, d = 6, 700, 30, 16
    rng = np.random.default_rng(78)
    X = np.cumsum(rng.normal(0.0, (1.0 / (d * L)) ** 0.5, (nx, L, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / (d * L)) ** 0.5, (ny, L, d)), axis=1)
    assert "solo_bwd_kernel<0, 16, 1, 0, 0, 1>" in sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, nx, ny, L, L, d, 0, 0, 0, sk.SK_F64)
    W = workloads.upstream_weights(61, (nx, ny))
    K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), 0, 0, 0)
    torch.cuda.synchronize()
    Kref, gXr, gYr = oracle.gram(X, Y, W, 0, 0, 0)
    check_values(host(K), Kref, torch.float64, "K")
    check_grads(host(gX), gXr, torch.float64, "grad_X")
    check_grads(host(gY), gYr, torch.float64, "grad_Y")


@pytest.mark.parametrize("B,L1,L2,d,lam1,lam2,flags", [(4, 600, 600, 8, 2, 2, 0), (8, 700, 500, 5, 1, 1, 1),
                                                        (5, 400, 330, 3, 0, 0, 0), (2, 300, 900, 2, 2, 1, 0),
                                                        (6, 1000, 1000, 6, 0, 2, 1), (3, 321, 450, 4, 1, 0, 0)])
def test_band_mode_shapes(B, L1, L2, d, lam1, lam2, flags):
    # band kernels (few pairs of long paths: the strips of a pair spread over workgroups that run as one pipeline,
    # rows and progress counters crossing workgroups): two to four bands, a last band with fewer than four
    # strips, unequal lengths and dyadic orders (block columns shared by several refined columns), time
    # augmentation; forward alone and the two launches of the backward pass, twice in a row (the counters are
    # cleared by every call)
    rng = np.random.default_rng(800 + L1 + d)
    X = np.cumsum(rng.normal(0.0, (1.0 / L1) ** 0.5, (B, L1, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L2) ** 0.5, (B, L2, d)), axis=1)
    assert "mode=band" in sk.sigkernel_describe(sk.SK_OP_BWD, B, 0, L1, L2, d, lam1, lam2, flags, sk.SK_F64)
    gk = workloads.upstream_weights(62, (B,))
    kr, gxr, gyr = oracle.bwd(X, Y, gk, lam1, lam2, flags)
    for rep in range(2):
        kf = sk.sigkernel_fwd(dev(X), dev(Y), lam1, lam2, flags)
        k, gx, gy = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), lam1, lam2, flags)
        torch.cuda.synchronize()
        check_values(host(kf), kr, torch.float64, "k (forward only)")
        check_values(host(k), kr, torch.float64, "k")
        check_grads(host(gx), gxr, torch.float64, "grad_x")
        check_grads(host(gy), gyr, torch.float64, "grad_y")


def test_band_mode_wait_that_runs_out_gives_nan_and_ends():
    # SK_FLAG_SHORT_WAITS lets a band give up on the band above it after one poll: the kernels must still end, the
    # results must be NaN (never a number computed from rows that were not there), and the next call is clean
    B, L, d = 3, 600, 3
    rng = np.random.default_rng(91)
    X = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (B, L, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (B, L, d)), axis=1)
    assert "mode=band" in sk.sigkernel_describe(sk.SK_OP_BWD, B, 0, L, L, d, 1, 1, sk.SK_FLAG_SHORT_WAITS, sk.SK_F64)
    gk = workloads.upstream_weights(63, (B,))
    kf = sk.sigkernel_fwd(dev(X), dev(Y), 1, 1, sk.SK_FLAG_SHORT_WAITS)
    k, gx, gy = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), 1, 1, sk.SK_FLAG_SHORT_WAITS)
    torch.cuda.synchronize()
    assert np.all(np.isnan(host(kf))) and np.all(np.isnan(host(k)))
    assert np.all(np.isnan(host(gx))) and np.all(np.isnan(host(gy)))
    # the same with a kept forward sweep: the backward call sees how the forward call went
    need = sk.sigkernel_workspace_bytes(sk.SK_OP_BWD, B, 0, L, L, d, 1, 1, 0, sk.SK_F64)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    kf = sk.sigkernel_fwd(dev(X), dev(Y), 1, 1, sk.SK_FLAG_SHORT_WAITS | sk.SK_FLAG_KEEP_FORWARD, ws=ws)
    k, gx, gy = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), 1, 1, sk.SK_FLAG_HAVE_FORWARD, ws=ws)
    torch.cuda.synchronize()
    assert np.all(np.isnan(host(kf))) and np.all(np.isnan(host(k)))
    assert np.all(np.isnan(host(gx))) and np.all(np.isnan(host(gy)))
    kr, gxr, gyr = oracle.bwd(X, Y, gk, 1, 1, 0)
    k, gx, gy = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), 1, 1, 0)
    torch.cuda.synchronize()
    check_values(host(k), kr, torch.float64, "k after a failed call")
    check_grads(host(gx), gxr, torch.float64, "grad_x after a failed call")
    check_grads(host(gy), gyr, torch.float64, "grad_y after a failed call")


@pytest.mark.parametrize("name,N,dtype", [("c3", 41, torch.float64), ("c5", 45, torch.float64), ("c5", 38, torch.float32)])
def test_symmetric_gram_solves_half_the_pairs(name, N, dtype):
    # K(X, X) in the solo / tile kernels: only the pairs n <= m are solved (odd and even N), both entries of K are
    # written, and the gradient is the total derivative for a weight matrix that is not symmetric
    w, X, _ = workloads.make(name, n_x=N, n_y=N)
    Xr = rounded(X, dtype)
    W = workloads.upstream_weights(68, (N, N))
    x = dev(X, dtype)
    K, gX, none = sk.sigkernel_gram(x, x, dev(W, dtype), w.lam, w.lam, w.flags)
    Kf = sk.sigkernel_gram(x, x, None, w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    Kr, gXr, _ = oracle.gram(Xr, Xr, rounded(W, dtype), w.lam, w.lam, w.flags)
    assert none is None
    check_values(host(K), Kr, dtype, "K(X,X)")
    check_values(host(Kf), Kr, dtype, "K(X,X) forward only")
    check_grads(host(gX), gXr, dtype, "grad_X total")
    assert torch.equal(K, K.T) and torch.equal(Kf, Kf.T)
    # the same through the general entry (a copy of X as Y): identical values, the two gradients add up
    y = dev(X, dtype).clone()
    K2, gX2, gY2 = sk.sigkernel_gram(x, y, dev(W, dtype), w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    assert torch.equal(K2, K)
    check_grads(host(gX2) + host(gY2), gXr, dtype, "grad_X + grad_Y of the general case")


# ------------------------------------------------------------------ lead-lag transform on the fly (Section 4)
LL = sk.SK_FLAG_LEAD_LAG


@pytest.mark.parametrize("B,L1,L2,d,lam1,lam2,flags,dtype", [
    (6, 40, 33, 2, 1, 1, LL, torch.float64),            # few pairs: lock-step
    (5, 20, 20, 3, 0, 2, LL | 1, torch.float64),        # with time augmentation of the transformed path
    (1300, 30, 25, 4, 0, 0, LL, torch.float64),         # many pairs: solo kernels
    (1300, 24, 31, 2, 1, 1, LL, torch.float32),         # ... and float callers
    (3, 260, 200, 3, 0, 0, LL, torch.float64),          # long paths: band kernels
])
def test_lead_lag_pairs(B, L1, L2, d, lam1, lam2, flags, dtype):
    rng = np.random.default_rng(900 + L1 + d)
    X = np.cumsum(rng.normal(0.0, (1.0 / L1) ** 0.5, (B, L1, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L2) ** 0.5, (B, L2, d)), axis=1)
    print(sk.sigkernel_describe(sk.SK_OP_BWD, B, 0, L1, L2, d, lam1, lam2, flags, sk.SK_F64), flush=True)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    gk = workloads.upstream_weights(64, (B,))
    kf = sk.sigkernel_fwd(dev(X, dtype), dev(Y, dtype), lam1, lam2, flags)
    k, gx, gy = sk.sigkernel_bwd(dev(X, dtype), dev(Y, dtype), dev(gk, dtype), lam1, lam2, flags)
    torch.cuda.synchronize()
    kr, gxr, gyr = oracle.bwd(Xr, Yr, rounded(gk, dtype), lam1, lam2, flags)
    check_values(host(kf), kr, dtype, "k (forward only)")
    check_values(host(k), kr, dtype, "k")
    check_grads(host(gx), gxr, dtype, "grad_x")
    check_grads(host(gy), gyr, dtype, "grad_y")


def test_lead_lag_gram():
    nx, ny, L, d = 21, 17, 36, 3
    rng = np.random.default_rng(95)
    X = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (nx, L, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (ny, L, d)), axis=1)
    W = workloads.upstream_weights(65, (nx, ny))
    K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), 1, 1, LL)
    x = dev(X)
    Ws = workloads.upstream_weights(66, (nx, nx))
    Kxx, gXX, none = sk.sigkernel_gram(x, x, dev(Ws), 1, 1, LL)
    torch.cuda.synchronize()
    Kr, gXr, gYr = oracle.gram(X, Y, W, 1, 1, LL)
    check_values(host(K), Kr, torch.float64, "K")
    check_grads(host(gX), gXr, torch.float64, "grad_X")
    check_grads(host(gY), gYr, torch.float64, "grad_Y")
    Kxr, gXXr, _ = oracle.gram(X, X, Ws, 1, 1, LL)
    assert none is None
    check_values(host(Kxx), Kxr, torch.float64, "K(X,X)")
    check_grads(host(gXX), gXXr, torch.float64, "grad_X total")


def lead_lag_form(op, B, M, L1, L2, d, lam1, lam2, flags):
    desc = sk.sigkernel_describe(op, B, M, L1, L2, d, lam1, lam2, flags, sk.SK_F64)
    return desc.split("lead_lag_form=", 1)[1].split(" ", 1)[0], desc


# The lead-lag form of the sweep: the grid of the original increments with one more level of refinement, whose diagonal
# quadrants carry p and whose other two carry the time constant alone.  The level lies inside the blocks for dyadic
# orders 0 and 1 (blocks of 2 x 2 and 4 x 4 cells) and above them from order 2 on; one or two block rows per lane;
# with and without the time channel (whose constant the off-diagonal quadrants keep); float callers.
@pytest.mark.parametrize("B,L1,L2,d,lam,flags,dtype", [
    (1300, 30, 25, 4, 0, LL, torch.float64),
    (1300, 100, 90, 3, 0, LL | 1, torch.float64),       # two block rows per lane
    (1300, 24, 31, 2, 1, LL, torch.float32),
    (1300, 40, 50, 5, 1, LL | 1, torch.float64),
    (1300, 20, 22, 3, 2, LL | 1, torch.float64),        # the level above the blocks
    (1100, 9, 12, 16, 3, LL, torch.float64),
    (1300, 2, 2, 3, 0, LL, torch.float64),              # one increment each: a single block
    (1300, 60, 3, 6, 1, LL | 1, torch.float64),
    (1300, 30, 25, 4, 0, LL | 1 | sk.SK_FLAG_BWD_REPLAY, torch.float64),   # the replaying backward, wave per pair
    (6, 90, 80, 2, 1, LL | sk.SK_FLAG_BWD_REPLAY, torch.float64),          # ... and cooperative
    (6, 50, 40, 3, 2, LL | 1 | sk.SK_FLAG_BWD_REPLAY, torch.float64),
])
def test_lead_lag_checkerboard_form_pairs(B, L1, L2, d, lam, flags, dtype):
    form, desc = lead_lag_form(sk.SK_OP_BWD, B, 0, L1, L2, d, lam, lam, flags)
    print(desc, flush=True)
    assert form == "checkerboard"
    rng = np.random.default_rng(910 + L1 + d)
    X = np.cumsum(rng.normal(0.0, (1.0 / L1) ** 0.5, (B, L1, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L2) ** 0.5, (B, L2, d)), axis=1)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    gk = workloads.upstream_weights(67, (B,))
    kf = sk.sigkernel_fwd(dev(X, dtype), dev(Y, dtype), lam, lam, flags)
    k, gx, gy = sk.sigkernel_bwd(dev(X, dtype), dev(Y, dtype), dev(gk, dtype), lam, lam, flags)
    torch.cuda.synchronize()
    kr, gxr, gyr = oracle.bwd(Xr, Yr, rounded(gk, dtype), lam, lam, flags)
    check_values(host(kf), kr, dtype, "k (forward only)")
    check_values(host(k), kr, dtype, "k")
    check_grads(host(gx), gxr, dtype, "grad_x")
    check_grads(host(gy), gyr, dtype, "grad_y")


@pytest.mark.parametrize("lam,flags", [(0, LL), (1, LL | 1), (2, LL)])
def test_lead_lag_checkerboard_form_gram(lam, flags):
    nx, ny, L, d = 40, 36, 28, 3
    assert lead_lag_form(sk.SK_OP_GRAM_BWD, nx, ny, L, L, d, lam, lam, flags)[0] == "checkerboard"
    rng = np.random.default_rng(96 + lam)
    X = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (nx, L, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (ny, L, d)), axis=1)
    W = workloads.upstream_weights(68, (nx, ny))
    Kf = sk.sigkernel_gram(dev(X), dev(Y), None, lam, lam, flags)
    K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), lam, lam, flags)
    x = dev(X)
    Ws = workloads.upstream_weights(69, (nx, nx))
    Kxx, gXX, none = sk.sigkernel_gram(x, x, dev(Ws), lam, lam, flags)   # the pairs n <= m only
    torch.cuda.synchronize()
    Kr, gXr, gYr = oracle.gram(X, Y, W, lam, lam, flags)
    check_values(host(Kf), Kr, torch.float64, "K (forward only)")
    check_values(host(K), Kr, torch.float64, "K")
    check_grads(host(gX), gXr, torch.float64, "grad_X")
    check_grads(host(gY), gYr, torch.float64, "grad_Y")
    Kxr, gXXr, _ = oracle.gram(X, X, Ws, lam, lam, flags)
    assert none is None
    check_values(host(Kxx), Kxr, torch.float64, "K(X,X)")
    check_grads(host(gXX), gXXr, torch.float64, "grad_X total")


@pytest.mark.parametrize("B,L1,L2,d,lam1,lam2,flags", [
    (1300, 20, 22, 3, 0, 2, LL | 1),      # solo; blocks of one cell below the lead-lag level
    (1300, 20, 22, 3, 2, 1, LL),
    (5, 40, 30, 2, 1, 3, LL | 1),         # lock-step
    (3, 150, 90, 4, 0, 1, LL),            # band
    (1100, 80, 20, 5, 3, 2, LL | 1),      # wave per pair
    (40, 60, 40, 20, 1, 0, LL),           # cooperative
])
def test_lead_lag_checkerboard_form_with_unequal_dyadic_orders(B, L1, L2, d, lam1, lam2, flags):
    desc = sk.sigkernel_describe(sk.SK_OP_BWD, B, 0, L1, L2, d, lam1, lam2, flags, sk.SK_F64)
    print(desc, flush=True)
    assert "lead_lag_form=checkerboard" in desc
    rng = np.random.default_rng(930 + L1 + d)
    X = np.cumsum(rng.normal(0.0, (1.0 / L1) ** 0.5, (B, L1, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L2) ** 0.5, (B, L2, d)), axis=1)
    gk = workloads.upstream_weights(76, (B,))
    kf = sk.sigkernel_fwd(dev(X), dev(Y), lam1, lam2, flags)
    k, gx, gy = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), lam1, lam2, flags)
    torch.cuda.synchronize()
    kr, gxr, gyr = oracle.bwd(X, Y, gk, lam1, lam2, flags)
    check_values(host(kf), kr, torch.float64, "k (forward only)")
    check_values(host(k), kr, torch.float64, "k")
    check_grads(host(gx), gxr, torch.float64, "grad_x")
    check_grads(host(gy), gyr, torch.float64, "grad_y")


@pytest.mark.parametrize("lam,flags", [(0, LL), (1, LL | 1), (2, LL | 1)])
def test_lead_lag_checkerboard_form_with_large_increments(lam, flags):
    # pairs whose inverse recurrence drifts are solved once more by the replay kernel, in its lead-lag form
    B, L1, L2, d = 1300, 14, 12, 3
    assert lead_lag_form(sk.SK_OP_BWD, B, 0, L1, L2, d, lam, lam, flags)[0] == "checkerboard"
    rng = np.random.default_rng(7300 + lam)
    dX = rng.normal(0.0, (1.0 / (d * L1)) ** 0.5, (B, L1, d))
    dY = rng.normal(0.0, (1.0 / (d * L2)) ** 0.5, (B, L2, d))
    big = 2.2 * 2 ** lam
    wild = np.arange(0, B, 13)
    dX[wild, 1::3, :] = rng.choice([-big, big], size=dX[wild, 1::3, :].shape) / d ** 0.5
    dY[wild, 1::3, :] = rng.choice([-big, big], size=dY[wild, 1::3, :].shape) / d ** 0.5
    X, Y = np.cumsum(dX, axis=1), np.cumsum(dY, axis=1)
    gk = workloads.upstream_weights(74, (B,))
    kr, gxr, gyr = oracle.bwd(X, Y, gk, lam, lam, flags)
    assert np.all(np.isfinite(kr))
    k, gx, gy, n = pairs_backward_with_ws(X, Y, gk, lam, lam, flags)
    print("lead-lag, order %d: %d of %d pairs solved once more; |k| up to %.3g" % (lam, n, B, np.abs(kr).max()), flush=True)
    assert 0 < n <= len(wild)
    check_values(host(k), kr, torch.float64, "k")
    check_rows(host(gx), gxr, torch.float64, "grad_x")
    check_rows(host(gy), gyr, torch.float64, "grad_y")


@pytest.mark.parametrize("B,L1,L2,d,lam,flags,dtype,mode", [
    (6, 40, 33, 2, 1, LL, torch.float64, "lock-step"),        # works on the caller's arrays
    (5, 70, 66, 3, 0, LL | 1, torch.float64, "lock-step"),
    (4, 30, 28, 5, 2, LL | 1, torch.float64, "lock-step"),    # the level above the blocks
    (6, 40, 33, 2, 1, LL | 1, torch.float32, "lock-step"),    # float callers: increments written out first
    (3, 260, 200, 3, 0, LL | 1, torch.float64, "band"),
    (2, 300, 280, 4, 1, LL | 1, torch.float64, "band"),
    (2, 200, 180, 2, 2, LL, torch.float64, "band"),
    (1100, 140, 20, 3, 0, LL | 1, torch.float64, "wave-per-pair"),
    (1100, 70, 20, 5, 1, LL, torch.float64, "wave-per-pair"),
    (1100, 40, 12, 5, 2, LL | 1, torch.float32, "wave-per-pair"),
    (600, 200, 40, 5, 0, LL | 1, torch.float64, "cooperative"),
    (600, 70, 20, 5, 1, LL, torch.float64, "cooperative"),
    (600, 40, 12, 5, 2, LL | 1, torch.float64, "cooperative"),
    (40, 200, 40, 20, 0, LL | 1, torch.float64, "wide"),            # more than 16 channels
    (40, 100, 40, 16, 1, LL, torch.float64, "wide"),
    (40, 100, 40, 16, 2, LL | 1, torch.float64, "wide"),
])
@pytest.mark.parametrize("big", [0.0, 2.2])
def test_lead_lag_checkerboard_form_few_pairs(B, L1, L2, d, lam, flags, dtype, mode, big):
    # the lock-step and band kernels; with increments of order one in a few places the inverse recurrence drifts and
    # the replay kernel takes over, in its lead-lag form (band mode: for every pair)
    if big and dtype == torch.float32:
        pytest.skip("kernel values of such paths are beyond the range of float")
    form, desc = lead_lag_form(sk.SK_OP_BWD, B, 0, L1, L2, d, lam, lam, flags)
    print(desc, flush=True)
    assert form == "checkerboard" and ("mode=" + mode) in desc
    rng = np.random.default_rng(920 + L1 + d)
    dX = rng.normal(0.0, (1.0 / (d * L1)) ** 0.5, (B, L1, d))
    dY = rng.normal(0.0, (1.0 / (d * L2)) ** 0.5, (B, L2, d))
    if big:
        dX[B // 2, 1:14:3, :] = rng.choice([-big, big], size=dX[B // 2, 1:14:3, :].shape) * 2 ** lam / d ** 0.5
        dY[B // 2, 1:14:3, :] = rng.choice([-big, big], size=dY[B // 2, 1:14:3, :].shape) * 2 ** lam / d ** 0.5
    X, Y = np.cumsum(dX, axis=1), np.cumsum(dY, axis=1)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    gk = workloads.upstream_weights(75, (B,))
    kr, gxr, gyr = oracle.bwd(Xr, Yr, rounded(gk, dtype), lam, lam, flags)
    assert np.all(np.isfinite(kr))
    kf = sk.sigkernel_fwd(dev(X, dtype), dev(Y, dtype), lam, lam, flags)
    k, gx, gy, n = pairs_backward_with_ws(X, Y, gk, lam, lam, flags, dtype)
    print("%d of %d pairs solved once more; |k| up to %.3g" % (n, B, np.abs(kr).max()), flush=True)
    if big and dtype == torch.float64:
        assert n != 0
    check_values(host(kf), kr, dtype, "k (forward only)")
    check_values(host(k), kr, dtype, "k")
    check_rows(host(gx), gxr, dtype, "grad_x")
    check_rows(host(gy), gyr, dtype, "grad_y")


# ------------------------------------------------------------------ seeded random shapes, every flag combination
def _random_cases(n, seed):
    rng = np.random.default_rng(seed)
    cases = []
    while len(cases) < n:
        gram = int(rng.integers(0, 3))                    # 0: pairs, 1: K(X, Y), 2: K(X, X)
        L1 = int(rng.choice([2, 3, 5, 9, 17, 33, 40, 64, 65, 70, 100, 129, 150, 200, 260, 300]))
        L2 = L1 if gram == 2 else int(rng.choice([2, 3, 6, 12, 31, 33, 50, 64, 66, 90, 128, 140, 257]))
        d = int(rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 17, 20]))
        lam1 = int(rng.integers(0, 4))
        lam2 = lam1 if rng.random() < 0.7 else int(rng.integers(0, 4))
        flags = int(rng.choice([0, 1, LL, LL | 1])) | (sk.SK_FLAG_BWD_REPLAY if rng.random() < 0.15 else 0)
        tile_like = rng.random() < 0.1                    # many pairs of at most 64 x 64 cells with 8 or 16 channels
        if tile_like:
            L1, L2, d = int(rng.integers(34, 66)), int(rng.integers(34, 66)), int(rng.choice([7, 8, 13, 16]))
            if gram == 2:
                L2 = L1
            lam1 = lam2 = 0
            flags &= 1
        ll = 2 if flags & LL else 1
        cells = ((L1 - 1) * ll << lam1) * ((L2 - 1) * ll << lam2)
        if cells > 3_000_000:
            continue
        if gram:
            nx = int(rng.choice([1, 2, 5, 12, 33, 40, 70]))
            ny = nx if gram == 2 else int(rng.choice([1, 3, 8, 20, 36, 64]))
            npairs = nx * ny
        else:
            nx = ny = npairs = int(rng.choice([1, 2, 3, 7, 40, 130, 300, 1100, 2600]))
        if tile_like and gram:
            nx = 40
            ny = nx if gram == 2 else 36
            npairs = nx * ny
        if npairs * cells > 60_000_000:
            continue
        dtype = torch.float32 if rng.random() < 0.2 else torch.float64
        keep = bool(rng.random() < 0.3)
        # a few paths with increments of order one: their pairs are solved once more by the replay kernel
        wild = bool(rng.random() < 0.25) and dtype == torch.float64 and min(L1, L2) >= 5
        cases.append((gram, nx, ny, L1, L2, d, lam1, lam2, flags, dtype, keep, wild, int(rng.integers(1, 1 << 30))))
    return cases


@pytest.mark.parametrize("chunk", range(8))
def test_random_shapes_against_the_oracle(chunk):
    # Shapes, dyadic orders, channel counts, flags, element types and call forms (pairs, K(X,Y), K(X,X); with and
    # without a kept forward sweep) drawn from a seeded generator: whatever launch plan they land in, the numbers are
    # the oracle's.
    check_random_cases(15, 4200 + chunk)


def ill_conditioned(k64, k80):
    """Whether the oracle's own rounding (double against x87 extended arithmetic) already takes a tenth of the
    tolerance: such inputs say nothing about the kernels."""
    k80 = np.asarray(k80, dtype=np.float64)
    return float(np.max(np.abs(k64 - k80) / np.maximum(1.0, np.abs(k80)))) > 1e-11


def check_random_cases(n, seed):
    for case in _random_cases(n, seed):
        gram, nx, ny, L1, L2, d, lam1, lam2, flags, dtype, keep, wild, seed = case
        sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
        # Gradients of paths with increments of order one are held to 1e-9: the default backward accepts a recovered
        # forward state within 1e-11 of the lane's largest value, and where the kernel values of such a pair cancel
        # along a row that has been seen to cost a decade (the replaying backward stays at 1e-12 there).
        gdt = "wild" if wild and not (flags & sk.SK_FLAG_BWD_REPLAY) else dtype
        op = sk.SK_OP_GRAM_BWD if gram else sk.SK_OP_BWD
        print(case, sk.sigkernel_describe(op, nx, ny if gram else 0, L1, L2, d, lam1, lam2, flags, sdt).split(" grid=")[0],
              flush=True)
        rng = np.random.default_rng(seed)
        dX = rng.normal(0.0, (1.0 / (d * L1)) ** 0.5, (nx, L1, d))
        dY = rng.normal(0.0, (1.0 / (d * L2)) ** 0.5, (ny, L2, d))
        if wild:
            big = 2.2 * 2 ** (0.25 * (lam1 + lam2)) / d ** 0.5
            wx, wy = rng.integers(0, nx, size=1 + nx // 16), rng.integers(0, ny, size=1 + ny // 16)
            dX[wx, 1:8:3, :] = rng.choice([-big, big], size=dX[wx, 1:8:3, :].shape)
            dY[wy, 1:8:3, :] = rng.choice([-big, big], size=dY[wy, 1:8:3, :].shape)
        X = np.cumsum(dX, axis=1)
        Y = X if gram == 2 else np.cumsum(dY, axis=1)
        Xr = rounded(X, dtype)
        Yr = Xr if gram == 2 else rounded(Y, dtype)
        x = dev(X, dtype)
        y = x if gram == 2 else dev(Y, dtype)
        of = flags & ~sk.SK_FLAG_BWD_REPLAY
        if gram:
            W = workloads.upstream_weights(seed % 1000, (nx, ny))
            Kr, gXr, gYr = oracle.gram(Xr, Yr, rounded(W, dtype), lam1, lam2, of)
            if not np.all(np.abs(Kr) < 1e30):
                continue                                  # beyond what the test's tolerances are meant for
            if wild and ill_conditioned(Kr, oracle.gram(Xr, Yr, None, lam1, lam2, of, dtype=np.longdouble)):
                continue
            if keep:
                need = sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM, nx, ny, L1, L2, d, lam1, lam2,
                                                    flags | sk.SK_FLAG_KEEP_FORWARD, sdt)
                ws = torch.empty(need, dtype=torch.uint8, device="cuda")
                Kf = sk.sigkernel_gram(x, y, None, lam1, lam2, flags | sk.SK_FLAG_KEEP_FORWARD, ws=ws)
                K, gX, gY = sk.sigkernel_gram(x, y, dev(W, dtype), lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
            else:
                Kf = sk.sigkernel_gram(x, y, None, lam1, lam2, flags)
                K, gX, gY = sk.sigkernel_gram(x, y, dev(W, dtype), lam1, lam2, flags)
            torch.cuda.synchronize()
            check_values(host(Kf), Kr, dtype, "K (forward call)")
            check_values(host(K), Kr, dtype, "K")
            check_rows(host(gX), gXr, gdt, "grad_X")
            if gram == 1:
                check_rows(host(gY), gYr, gdt, "grad_Y")
            else:
                assert gY is None
        else:
            gk = workloads.upstream_weights(seed % 1000, (nx,))
            kr, gxr, gyr = oracle.bwd(Xr, Yr, rounded(gk, dtype), lam1, lam2, of)
            if not np.all(np.abs(kr) < 1e30):
                continue
            if wild and ill_conditioned(kr, oracle.fwd(Xr, Yr, lam1, lam2, of, dtype=np.longdouble)):
                continue
            if keep:
                need = sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, nx, 0, L1, L2, d, lam1, lam2,
                                                    flags | sk.SK_FLAG_KEEP_FORWARD, sdt)
                ws = torch.empty(need, dtype=torch.uint8, device="cuda")
                kf = sk.sigkernel_fwd(x, y, lam1, lam2, flags | sk.SK_FLAG_KEEP_FORWARD, ws=ws)
                k, gx, gy = sk.sigkernel_bwd(x, y, dev(gk, dtype), lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
            else:
                kf = sk.sigkernel_fwd(x, y, lam1, lam2, flags)
                k, gx, gy = sk.sigkernel_bwd(x, y, dev(gk, dtype), lam1, lam2, flags)
            torch.cuda.synchronize()
            check_values(host(kf), kr, dtype, "k (forward call)")
            check_values(host(k), kr, dtype, "k")
            check_rows(host(gx), gxr, gdt, "grad_x")
            check_rows(host(gy), gyr, gdt, "grad_y")


# ------------------------------------------------------------------ autograd over the C ABI (Section 1)
def test_autograd_wrappers_give_the_oracle_gradients():
    from paper_2509_10613_amd import autograd as ska
    nx, ny, L, d = 9, 7, 24, 3
    rng = np.random.default_rng(96)
    X = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (nx, L, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (ny, L, d)), axis=1)
    x = dev(X).requires_grad_(True)
    y = dev(Y).requires_grad_(True)
    # a loss of the kind the abstract names: a (biased) squared maximum mean discrepancy between two sets of
    # paths; the reductions are the test's, the kernels and their gradients the library's
    loss = ska.sig_kernel_gram(x, None, 1, 1, 1).mean() - 2.0 * ska.sig_kernel_gram(x, y, 1, 1, 1).mean() + \
        ska.sig_kernel_gram(y, None, 1, 1, 1).mean()
    loss.backward()
    torch.cuda.synchronize()
    Kxx, gxx, _ = oracle.gram(X, X, np.full((nx, nx), 1.0 / (nx * nx)), 1, 1, 1)
    Kxy, gxy_x, gxy_y = oracle.gram(X, Y, np.full((nx, ny), -2.0 / (nx * ny)), 1, 1, 1)
    Kyy, gyy, _ = oracle.gram(Y, Y, np.full((ny, ny), 1.0 / (ny * ny)), 1, 1, 1)
    ref = Kxx.mean() - 2.0 * Kxy.mean() + Kyy.mean()
    assert abs(float(loss.detach()) - ref) <= 1e-10 * max(1.0, abs(ref))
    check_grads(host(x.grad), gxx + gxy_x, torch.float64, "d loss / dX")
    check_grads(host(y.grad), gyy + gxy_y, torch.float64, "d loss / dY")
    # pairs, one side without gradient
    xb = dev(X[:7]).requires_grad_(True)
    gk = workloads.upstream_weights(67, (7,))
    k = ska.sig_kernel(xb, dev(Y), 0, 1, 0)
    (k * dev(gk)).sum().backward()
    torch.cuda.synchronize()
    kr, gxr, _ = oracle.bwd(X[:7], Y, gk, 0, 1, 0)
    check_values(host(k), kr, torch.float64, "k")
    check_grads(host(xb.grad), gxr, torch.float64, "d/dx through autograd")
    # two graphs alive at once (a forward call that keeps its sweep keeps it in a workspace of its own), and a graph
    # that is walked twice
    from paper_2509_10613_amd import binding
    assert binding.keeps_forward(7, L, L, d, 1, 1, 1, binding.SK_F64)
    xa = dev(X[:7]).requires_grad_(True)
    xc = dev(X[2:9]).requires_grad_(True)
    k1 = ska.sig_kernel(xa, dev(Y), 1, 1, 1)
    k2 = ska.sig_kernel(xc, dev(Y), 1, 1, 1)
    (k1 * dev(gk)).sum().backward(retain_graph=True)
    first = xa.grad.clone()
    (k2 * dev(gk)).sum().backward()
    xa.grad = None
    (k1 * dev(gk)).sum().backward()
    torch.cuda.synchronize()
    assert torch.equal(xa.grad, first)
    check_grads(host(xa.grad), oracle.bwd(X[:7], Y, gk, 1, 1, 1)[1], torch.float64, "d/dx, first graph")
    check_grads(host(xc.grad), oracle.bwd(X[2:9], Y, gk, 1, 1, 1)[1], torch.float64, "d/dx, second graph")
    # Gram matrices large enough for the solo kernels: the wrappers keep the forward sweep there too
    nx, ny = 40, 36
    X = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (nx, L, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / L) ** 0.5, (ny, L, d)), axis=1)
    assert binding.keeps_forward(nx, L, L, d, 1, 1, 1, binding.SK_F64, gram_M=ny)
    x = dev(X).requires_grad_(True)
    y = dev(Y).requires_grad_(True)
    Wxy = workloads.upstream_weights(68, (nx, ny))
    Wxx = workloads.upstream_weights(69, (nx, nx))
    loss = (ska.sig_kernel_gram(x, y, 1, 1, 1) * dev(Wxy)).sum() + (ska.sig_kernel_gram(x, None, 1, 1, 1) * dev(Wxx)).sum()
    loss.backward()
    torch.cuda.synchronize()
    Kxy, gx1, gy1 = oracle.gram(X, Y, Wxy, 1, 1, 1)
    Kxx, gx2, _ = oracle.gram(X, X, Wxx, 1, 1, 1)     # the total derivative of K(X, X)
    ref = (Kxy * Wxy).sum() + (Kxx * Wxx).sum()
    assert abs(float(loss.detach()) - ref) <= 1e-10 * max(1.0, abs(ref))
    check_grads(host(x.grad), gx1 + gx2, torch.float64, "d loss / dX, kept sweeps")
    check_grads(host(y.grad), gy1, torch.float64, "d loss / dY, kept sweeps")


@pytest.mark.parametrize("N,M,L1,L2,d,lam,flags,dtype", [(9, 7, 24, 30, 3, 1, 1, torch.float64),
                                                         (40, 44, 64, 64, 16, 0, 0, torch.float64),
                                                         (33, 20, 40, 40, 3, 1, 0, torch.float32)])
def test_mmd2_entry_point(N, M, L1, L2, d, lam, flags, dtype):
    # sigkernel_mmd2: three Gram computations (the two symmetric ones solve half their pairs), constant upstream
    # weights generated on the device, one reduction; value and gradients against the oracle's definition
    from paper_2509_10613_amd import autograd as ska
    rng = np.random.default_rng(97 + N)
    X = np.cumsum(rng.normal(0.0, (1.0 / (d * L1)) ** 0.5, (N, L1, d)), axis=1)
    Y = np.cumsum(rng.normal(0.02, (1.5 / (d * L2)) ** 0.5, (M, L2, d)), axis=1)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    loss, gX, gY = sk.sigkernel_mmd2(dev(X, dtype), dev(Y, dtype), lam, lam, flags)
    loss_only, none_x, none_y = sk.sigkernel_mmd2(dev(X, dtype), dev(Y, dtype), lam, lam, flags, want_x=False, want_y=False)
    torch.cuda.synchronize()
    ref, gXr, gYr = oracle.mmd2(Xr, Yr, lam, lam, flags)
    tol = TOL[dtype]
    assert none_x is None and none_y is None
    # the loss is a difference of means of kernel values of order one: its error is measured against those
    assert abs(float(loss[0]) - ref) <= tol and abs(float(loss_only[0]) - ref) <= tol
    gscale = max(np.max(np.abs(gXr)), np.max(np.abs(gYr)))
    assert np.all(np.isfinite(host(gX))) and np.all(np.isfinite(host(gY)))
    assert np.max(np.abs(host(gX) - gXr)) <= tol * max(1.0, gscale)
    assert np.max(np.abs(host(gY) - gYr)) <= tol * max(1.0, gscale)
    # through autograd, one side only
    x = dev(X, dtype).requires_grad_(True)
    (3.0 * ska.sig_mmd2(x, dev(Y, dtype), lam, lam, flags)).backward()
    torch.cuda.synchronize()
    assert np.max(np.abs(host(x.grad) - 3.0 * gXr)) <= 3.0 * tol * max(1.0, gscale)


# ------------------------------------------------------------------ full-size runs: the launches bench.py times
def check_rows(got, ref, dtype, what):
    """Gradients of several paths, each path against its own scale (stricter than one scale per tensor)."""
    for i in range(ref.shape[0]):
        check_grads(got[i], ref[i], dtype, "%s [%d]" % (what, i))


def translation_residual(g):
    """A kernel does not change when a path is translated, so the gradients of a path's points sum to zero per
    channel; returns the largest such sum relative to the largest gradient entry."""
    return float(np.max(np.abs(g.sum(axis=1))) / max(1.0, np.max(np.abs(g))))


def test_c4_full_size_all_pairs():
    # all 32 pairs: 256 band workgroups, one per compute unit, the strips of a pair handed from workgroup to workgroup
    # through global rows and progress counters - the launch bench.py times.  Values of every pair against the oracle;
    # gradients of the first, a middle and the last pair (workgroups 0.., and the last of the grid) against the oracle,
    # of every pair against translation invariance; the one-call backward and the kept-sweep pair of calls.
    w, X, Y = workloads.make("c4")
    B = w.n_x
    desc = sk.sigkernel_describe(sk.SK_OP_BWD, B, 0, w.L, w.L, w.d, w.lam, w.lam, w.flags, sk.SK_F64)
    assert "mode=band" in desc and "grid=256" in desc
    x, y = dev(X), dev(Y)
    gk = workloads.upstream_weights(41, (B,))
    kf = sk.sigkernel_fwd(x, y, w.lam, w.lam, w.flags)
    k1, gx1, gy1 = sk.sigkernel_bwd(x, y, dev(gk), w.lam, w.lam, w.flags)
    need = sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, B, 0, w.L, w.L, w.d, w.lam, w.lam,
                                        w.flags | sk.SK_FLAG_KEEP_FORWARD, sk.SK_F64)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    k2 = sk.sigkernel_fwd(x, y, w.lam, w.lam, w.flags | sk.SK_FLAG_KEEP_FORWARD, ws=ws)
    k3, gx2, gy2 = sk.sigkernel_bwd(x, y, dev(gk), w.lam, w.lam, w.flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
    torch.cuda.synchronize()
    print("c4: GPU calls done", flush=True)
    kref = oracle.fwd(X, Y, w.lam, w.lam, w.flags)
    for name, k in (("forward call", kf), ("one-call backward", k1), ("kept sweep", k2), ("backward after kept sweep", k3)):
        check_values(host(k), kref, torch.float64, "k, all pairs, " + name)
    sample = [0, B // 2 - 1, B - 1]
    kr, gxr, gyr = oracle.bwd(X[sample], Y[sample], gk[sample], w.lam, w.lam, w.flags)
    for name, gx, gy in (("one call", gx1, gy1), ("kept sweep", gx2, gy2)):
        gx, gy = host(gx), host(gy)
        check_rows(gx[sample], gxr, torch.float64, "grad_x, " + name)
        check_rows(gy[sample], gyr, torch.float64, "grad_y, " + name)
        assert np.all(np.isfinite(gx)) and np.all(np.isfinite(gy))
        assert translation_residual(gx) <= 1e-10 and translation_residual(gy) <= 1e-10


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_c3_full_size_gram_forward_and_backward(dtype):
    # the whole 256 x 256 Gram matrix and both gradients against the oracle (4.2e9 cells: seconds on the host), for
    # the forward call, the one-call backward, and the pair of calls of a training step that keeps the forward sweep
    w, X, Y = workloads.make("c3")
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    W = workloads.upstream_weights(35, (w.n_x, w.n_y))
    Wr = rounded(W, dtype)
    x, y, wd = dev(X, dtype), dev(Y, dtype), dev(W, dtype)
    Kf = sk.sigkernel_gram(x, y, None, w.lam, w.lam, w.flags)
    K1, gX1, gY1 = sk.sigkernel_gram(x, y, wd, w.lam, w.lam, w.flags)
    KEEP, HAVE = sk.SK_FLAG_KEEP_FORWARD, sk.SK_FLAG_HAVE_FORWARD
    need = max(sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM, w.n_x, w.n_y, w.L, w.L, w.d, w.lam, w.lam, w.flags | KEEP, sdt),
               sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM_BWD, w.n_x, w.n_y, w.L, w.L, w.d, w.lam, w.lam, w.flags | HAVE, sdt))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    K2 = sk.sigkernel_gram(x, y, None, w.lam, w.lam, w.flags | KEEP, ws=ws)
    K3, gX2, gY2 = sk.sigkernel_gram(x, y, wd, w.lam, w.lam, w.flags | HAVE, ws=ws)
    torch.cuda.synchronize()
    print("c3: GPU calls done", flush=True)
    Kref, gXr, gYr = oracle.gram(Xr, Yr, Wr, w.lam, w.lam, w.flags)
    for name, K in (("forward call", Kf), ("one-call backward", K1), ("kept sweep", K2), ("backward after kept sweep", K3)):
        check_values(host(K), Kref, dtype, "K, " + name)
    for name, gX, gY in (("one call", gX1, gY1), ("kept sweep", gX2, gY2)):
        check_rows(host(gX), gXr, dtype, "grad_X, " + name)
        check_rows(host(gY), gYr, dtype, "grad_Y, " + name)


def test_c5_full_size_gram_sampled_rows_and_columns():
    # 1024 x 1024 pairs, K(X, Y) and K(X, X), forward and backward as bench.py times them.  Against the oracle: sampled
    # rows of K and grad_X (one oracle row of 1024 pairs each), sampled columns of K and grad_Y, sampled entries and
    # rows of the total derivative of the symmetric case; on everything: finite, translation invariance, symmetry.
    w, X, Y = workloads.make("c5")
    N, M = w.n_x, w.n_y
    W = workloads.upstream_weights(51, (N, M))
    Ws = workloads.upstream_weights(52, (N, N))
    x, y = dev(X), dev(Y)
    Kf = sk.sigkernel_gram(x, y, None, w.lam, w.lam, w.flags)
    K, gX, gY = sk.sigkernel_gram(x, y, dev(W), w.lam, w.lam, w.flags)
    Kxxf = sk.sigkernel_gram(x, x, None, w.lam, w.lam, w.flags)
    Kxx, gXX, _ = sk.sigkernel_gram(x, x, dev(Ws), w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    print("c5: GPU calls done", flush=True)
    assert torch.equal(Kf, K) and torch.equal(Kxxf, Kxx) and torch.equal(Kxx, Kxx.T)
    K, gX, gY, Kxx, gXX = host(K), host(gX), host(gY), host(Kxx), host(gXX)
    for t in (K, gX, gY, Kxx, gXX):
        assert np.all(np.isfinite(t))
    for g in (gX, gY, gXX):
        assert translation_residual(g) <= 1e-10
    rng = np.random.default_rng(12)
    rows = [0, N - 1] + [int(v) for v in rng.integers(1, N - 1, 3)]
    cols = [0, M - 1] + [int(v) for v in rng.integers(1, M - 1, 3)]
    for n in rows:
        Kr, gXr, _ = oracle.gram(X[n:n + 1], Y, W[n:n + 1], w.lam, w.lam, w.flags)
        check_values(K[n], Kr[0], torch.float64, "K row %d" % n)
        check_grads(gX[n], gXr[0], torch.float64, "grad_X row %d" % n)
    for m in cols:
        Kr, _, gYr = oracle.gram(X, Y[m:m + 1], W[:, m:m + 1], w.lam, w.lam, w.flags)
        check_values(K[:, m], Kr[:, 0], torch.float64, "K column %d" % m)
        check_grads(gY[m], gYr[0], torch.float64, "grad_Y row %d" % m)
    # K(X, X): rows of K and of the total derivative (path n appears as the first argument in row n of K and as the
    # second argument in column n)
    for n in rows[:4]:
        Kr, g1, _ = oracle.gram(X[n:n + 1], X, Ws[n:n + 1], w.lam, w.lam, w.flags)
        _, _, g2 = oracle.gram(X, X[n:n + 1], Ws[:, n:n + 1], w.lam, w.lam, w.flags)
        check_values(Kxx[n], Kr[0], torch.float64, "K(X,X) row %d" % n)
        check_grads(gXX[n], g1[0] + g2[0], torch.float64, "total derivative of K(X,X), row %d" % n)
    assert np.all(np.diag(Kxx) > 0.0)


def test_symmetric_gram_with_unequal_dyadic_orders():
    # k with orders (l1, l2) of (y, x) equals k with orders (l2, l1) of (x, y), not k with (l1, l2): for unequal orders
    # K(X, X) is not a symmetric matrix and every pair has to be solved (four pairs per wave, shared increment buffer)
    N, L, d, lam1, lam2 = 300, 20, 3, 0, 1
    assert " symmetric_mode=four " in sk.sigkernel_describe(sk.SK_OP_GRAM_BWD, N, N, L, L, d, lam1, lam2, 0, sk.SK_F64)
    X = rand_paths(8700, N, L, d, 0.25)
    W = workloads.upstream_weights(87, (N, N))
    x = dev(X)
    Kf = sk.sigkernel_gram(x, x, None, lam1, lam2, 0)
    K, gX, none = sk.sigkernel_gram(x, x, dev(W), lam1, lam2, 0)
    torch.cuda.synchronize()
    Kr, gXr, _ = oracle.gram(X, X, W, lam1, lam2, 0)
    assert none is None
    assert np.max(np.abs(Kr - Kr.T)) > 1e-6        # what the test is about
    check_values(host(Kf), Kr, torch.float64, "K(X,X), orders (0,1), forward only")
    check_values(host(K), Kr, torch.float64, "K(X,X), orders (0,1)")
    check_grads(host(gX), gXr, torch.float64, "total derivative, orders (0,1)")
    # and through the squared MMD, whose symmetric blocks use one order each: (l1, l1) and (l2, l2)
    Y = rand_paths(8701, 40, L, d, 0.25)
    loss, gX2, gY2 = sk.sigkernel_mmd2(dev(X[:50]), dev(Y), lam1, lam2, 0)
    torch.cuda.synchronize()
    ref, gXr2, gYr2 = oracle.mmd2(X[:50], Y, lam1, lam2, 0)
    assert abs(float(loss[0]) - ref) <= 1e-10
    check_grads(host(gX2), gXr2, torch.float64, "mmd2 grad_X, orders (0,1)")
    check_grads(host(gY2), gYr2, torch.float64, "mmd2 grad_Y, orders (0,1)")


# ------------------------------------------------------------------ shapes, orders, channels, edges
@pytest.mark.parametrize("L1,L2,d,lam1,lam2,flags", [
    (2, 2, 1, 0, 0, 0),        # a single cell
    (2, 9, 3, 0, 0, 1),
    (33, 17, 2, 0, 0, 0),
    (66, 70, 4, 0, 0, 1),      # two strips, ragged second strip
    (130, 40, 3, 0, 0, 0),     # three strips
    (20, 35, 5, 1, 1, 0),
    (70, 30, 6, 1, 1, 1),      # 69 coarse rows at block order 1: ragged
    (12, 50, 8, 2, 2, 0),
    (40, 9, 7, 2, 2, 1),       # d = 7 runs in the 8-channel kernel
    (9, 11, 2, 3, 3, 0),       # order above the block order: residual shift on both sides
    (10, 21, 3, 2, 0, 0),      # unequal orders
    (21, 10, 3, 0, 3, 1),
    (15, 14, 16, 1, 2, 0),
    (11, 13, 11, 0, 0, 0),     # d = 11 runs in the 16-channel kernel
    (9, 12, 20, 1, 1, 1),      # d = 20: runtime channel loop
    (14, 7, 37, 0, 1, 0),
    (300, 50, 3, 0, 0, 0),     # small batches of long paths: three, four and two strips of 128 block rows
    (500, 40, 2, 0, 0, 1),
    (140, 20, 3, 2, 2, 0),
    (100, 300, 4, 1, 1, 1),    # many more columns than rows
])
def test_shapes_orders_channels_fp64(L1, L2, d, lam1, lam2, flags):
    B = 5
    X = rand_paths(1000 + L1 * 31 + d, B, L1, d, 0.25)
    Y = rand_paths(2000 + L2 * 17 + d, B, L2, d, 0.25)
    run_pairs(X, Y, lam1, lam2, flags, torch.float64, backward=True)


@pytest.mark.parametrize("L1,L2,d,lam", [(40, 33, 3, 0), (70, 66, 5, 1), (30, 20, 2, 2), (20, 12, 24, 1)])
def test_shapes_fp32(L1, L2, d, lam):
    B = 6
    X = rand_paths(3000 + L1, B, L1, d, 0.2)
    Y = rand_paths(4000 + L2, B, L2, d, 0.2)
    run_pairs(X, Y, lam, lam, 0, torch.float32, backward=True)


@pytest.mark.parametrize("B,L1,L2,d,lam1,lam2,flags,dtype", [
    (5, 66, 70, 4, 0, 0, 1, torch.float64),      # two strips, ragged second strip
    (5, 20, 35, 5, 1, 1, 0, torch.float64),      # one strip
    (3, 100, 300, 4, 1, 1, 1, torch.float64),    # two block rows per lane, many more columns than rows
    (4, 12, 50, 8, 2, 2, 0, torch.float64),
    (2, 40, 9, 7, 2, 2, 1, torch.float64),
    (5, 9, 12, 20, 1, 1, 1, torch.float64),      # run-time channel loop: no split form, the flags change nothing
    (6, 40, 33, 3, 0, 0, 0, torch.float32),      # float paths: likewise
    (5000, 6, 5, 2, 1, 1, 0, torch.float64),     # many pairs: solo kernels, checkpoints and bottom row per pair
    (3000, 40, 33, 3, 0, 0, 1, torch.float32),
    (5, 20, 18, 3, 1, 1, sk.SK_FLAG_LEAD_LAG, torch.float64),
    (5, 400, 330, 3, 0, 0, 0, torch.float64),    # band kernels: the two launches of the backward call, one per call
    (8, 700, 500, 5, 1, 1, 1, torch.float64),
    (3, 321, 450, 4, 1, 0, 0, torch.float32),
    (3, 260, 200, 3, 0, 0, sk.SK_FLAG_LEAD_LAG, torch.float64),
])
def test_forward_sweep_kept_for_the_backward_call(B, L1, L2, d, lam1, lam2, flags, dtype):
    """sigkernel_fwd with SK_FLAG_KEEP_FORWARD followed by sigkernel_bwd with SK_FLAG_HAVE_FORWARD on the same
    workspace: the same arithmetic as the backward call alone, so the same bits (band kernels: their gradient sums
    meet in global atomics, in any order); and both against the oracle."""
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    desc = sk.sigkernel_describe(sk.SK_OP_BWD, B, 0, L1, L2, d, lam1, lam2, flags, sdt)
    band = "mode=band" in desc or "mode=solo" in desc      # modes whose gradient sums meet in atomics
    assert ("mode=band" in desc) == (min(L1, L2) >= 200) and ("mode=solo" in desc) == (B >= 700)

    def same(a, b):
        if not band:
            return torch.equal(a, b)
        return float((a - b).abs().max()) <= TOL[dtype] * max(1.0, float(b.abs().max()))
    X = rand_paths(8100 + L1, B, L1, d, 0.25)
    Y = rand_paths(8200 + L2, B, L2, d, 0.25)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    x, y = dev(X, dtype), dev(Y, dtype)
    gk = dev(np.random.default_rng(83).normal(size=B), dtype)
    k0, gx0, gy0 = sk.sigkernel_bwd(x, y, gk, lam1, lam2, flags)
    need = sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, B, 0, L1, L2, d, lam1, lam2, flags | sk.SK_FLAG_KEEP_FORWARD,
                                        sk.SK_F64 if dtype == torch.float64 else sk.SK_F32)
    assert need >= sk.sigkernel_workspace_bytes(sk.SK_OP_BWD, B, 0, L1, L2, d, lam1, lam2, flags,
                                                sk.SK_F64 if dtype == torch.float64 else sk.SK_F32)
    ws = sk.workspace(need, x.device)
    for rep in range(2):                         # the second pass finds the workspace as the first one left it
        k1 = sk.sigkernel_fwd(x, y, lam1, lam2, flags | sk.SK_FLAG_KEEP_FORWARD, ws=ws)
        k2, gx1, gy1 = sk.sigkernel_bwd(x, y, gk, lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(k1, k0) and torch.equal(k2, k0)
        assert same(gx1, gx0) and same(gy1, gy0)
    kref, gxr, gyr = oracle.bwd(Xr, Yr, host(gk), lam1, lam2, flags)
    check_values(host(k1), kref, dtype, "k of the kept sweep")
    check_grads(host(gx1), gxr, dtype, "grad_x after a kept sweep")
    check_grads(host(gy1), gyr, dtype, "grad_y after a kept sweep")
    # only one gradient wanted
    _, gx2, _ = sk.sigkernel_bwd(x, y, gk, lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws, want_y=False)
    assert same(gx2, gx0)
    # a workspace that holds another call's sweep, or none: NaN gradients, never numbers (where the flags do anything)
    if sk.keeps_forward(B, L1, L2, d, lam1, lam2, flags, sdt):
        x2 = x.clone()
        _, gx3, gy3 = sk.sigkernel_bwd(x2, y, gk, lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
        assert torch.all(torch.isnan(gx3)) and torch.all(torch.isnan(gy3))
        _, gx3, gy3 = sk.sigkernel_bwd(x, y, gk, lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)   # still there
        assert same(gx3, gx0) and same(gy3, gy0)
        blank = torch.zeros(need, dtype=torch.uint8, device="cuda")
        _, gx3, gy3 = sk.sigkernel_bwd(x, y, gk, lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=blank)
        assert torch.all(torch.isnan(gx3)) and torch.all(torch.isnan(gy3))
        # a backward call that sweeps forward itself uses the same memory: the kept sweep is gone afterwards (where
        # that call lays the workspace out in the same way: not the solo kernels)
        if "mode=solo" not in desc:
            sk.sigkernel_fwd(x, y, lam1, lam2, flags | sk.SK_FLAG_KEEP_FORWARD, ws=ws)
            sk.sigkernel_bwd(x2, y, gk, lam1, lam2, flags, ws=ws)
            _, gx3, gy3 = sk.sigkernel_bwd(x, y, gk, lam1, lam2, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
            assert torch.all(torch.isnan(gx3)) and torch.all(torch.isnan(gy3))
        _, gx3, gy3 = sk.sigkernel_bwd(x, y, gk, lam1, lam2, flags, ws=ws)
        assert same(gx3, gx0) and same(gy3, gy0)
    # the kept sweep needs the backward call's workspace: the forward call's own is refused where it is smaller
    small = sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, B, 0, L1, L2, d, lam1, lam2, flags, sdt)
    if small < need:
        with pytest.raises(sk.SigKernelError):
            sk.sigkernel_fwd(x, y, lam1, lam2, flags | sk.SK_FLAG_KEEP_FORWARD,
                             ws=torch.empty(small, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("N,M,L,d,lam,flags,dtype,sym", [(40, 30, 128, 3, 1, 0, torch.float64, False),   # c3's shape
                                                          (36, 36, 40, 5, 1, 1, torch.float64, True),
                                                          (60, 50, 30, 2, 0, 0, torch.float32, False)])
def test_forward_sweep_of_a_gram_matrix_kept_for_its_backward_call(N, M, L, d, lam, flags, dtype, sym):
    """sigkernel_gram with SK_FLAG_KEEP_FORWARD, then sigkernel_gram with grad_K and SK_FLAG_HAVE_FORWARD on the same
    workspace (solo kernels: checkpoints and bottom row per pair), against the call that sweeps forward itself and
    against the oracle."""
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    X = rand_paths(8500 + N, N, L, d, 0.2)
    Y = X if sym else rand_paths(8600 + M, M, L, d, 0.2)
    Xr, Yr = rounded(X, dtype), rounded(Y, dtype)
    x = dev(X, dtype)
    y = x if sym else dev(Y, dtype)
    assert sk.keeps_forward(N, L, L, d, lam, lam, flags, sdt, gram_M=M)
    W = workloads.upstream_weights(86, (N, M))
    w = dev(W, dtype)
    K0, gX0, gY0 = sk.sigkernel_gram(x, y, w, lam, lam, flags)
    need = sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM, N, M, L, L, d, lam, lam, flags | sk.SK_FLAG_KEEP_FORWARD, sdt)
    assert need == sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM_BWD, N, M, L, L, d, lam, lam,
                                                flags | sk.SK_FLAG_HAVE_FORWARD, sdt)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    tol = TOL[dtype]
    for rep in range(2):
        K1 = sk.sigkernel_gram(x, y, None, lam, lam, flags | sk.SK_FLAG_KEEP_FORWARD, ws=ws)
        K2, gX, gY = sk.sigkernel_gram(x, y, w, lam, lam, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(K1, K0) and torch.equal(K2, K0)
        assert float((gX - gX0).abs().max()) <= tol * max(1.0, float(gX0.abs().max()))
        if not sym:
            assert float((gY - gY0).abs().max()) <= tol * max(1.0, float(gY0.abs().max()))
    Kr, gXr, gYr = oracle.gram(Xr, Yr, rounded(W, dtype), lam, lam, flags)
    check_values(host(K1), Kr, dtype, "K of the kept sweep")
    check_grads(host(gX), gXr + (gYr if sym else 0.0), dtype, "grad_X after a kept sweep")
    if not sym:
        check_grads(host(gY), gYr, dtype, "grad_Y after a kept sweep")
    # another call's sweep in the workspace: NaN, not numbers
    x2 = x.clone()
    _, gX3, _ = sk.sigkernel_gram(x2, x2 if sym else y, w, lam, lam, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
    assert torch.all(torch.isnan(gX3))
    _, gX3, _ = sk.sigkernel_gram(x, y, w, lam, lam, flags | sk.SK_FLAG_HAVE_FORWARD, ws=ws)
    assert float((gX3 - gX0).abs().max()) <= tol * max(1.0, float(gX0.abs().max()))


def test_kept_forward_sweep_degenerate_shapes():
    # no increments on one side, an empty batch: the flags change nothing
    KEEP, HAVE = sk.SK_FLAG_KEEP_FORWARD, sk.SK_FLAG_HAVE_FORWARD
    x = dev(rand_paths(1, 3, 1, 2))
    y = dev(rand_paths(2, 3, 6, 2))
    assert torch.all(sk.sigkernel_fwd(x, y, 0, 0, KEEP) == 1.0)
    k, gx, gy = sk.sigkernel_bwd(x, y, torch.ones(3, dtype=torch.float64, device="cuda"), 0, 0, HAVE)
    assert torch.all(k == 1.0) and torch.all(gx == 0.0) and torch.all(gy == 0.0)
    e = torch.empty((0, 4, 2), dtype=torch.float64, device="cuda")
    assert sk.sigkernel_fwd(e, e, 1, 1, KEEP).shape == (0,)
    k, gx, gy = sk.sigkernel_bwd(e, e, torch.empty(0, dtype=torch.float64, device="cuda"), 1, 1, HAVE)
    assert k.shape == (0,) and gx.shape == (0, 4, 2)
    # a single cell
    X, Y = rand_paths(3, 2, 2, 1, 0.5), rand_paths(4, 2, 2, 1, 0.5)
    ws = torch.empty(sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, 2, 0, 2, 2, 1, 0, 0, KEEP, sk.SK_F64), dtype=torch.uint8,
                     device="cuda")
    gk = dev(np.array([0.5, -2.0]))
    xd, yd = dev(X), dev(Y)
    k1 = sk.sigkernel_fwd(xd, yd, 0, 0, KEEP, ws=ws)
    k2, gx, gy = sk.sigkernel_bwd(xd, yd, gk, 0, 0, HAVE, ws=ws)
    torch.cuda.synchronize()
    kr, gxr, gyr = oracle.bwd(X, Y, host(gk), 0, 0, 0)
    check_values(host(k1), kr, torch.float64, "k")
    check_values(host(k2), kr, torch.float64, "k_out")
    check_grads(host(gx), gxr, torch.float64, "grad_x")
    check_grads(host(gy), gyr, torch.float64, "grad_y")


@pytest.mark.parametrize("B,L,d,lam,flags", [(6, 70, 5, 1, 1),        # lock-step, kept forward sweep
                                             (3000, 12, 3, 1, 0)])     # solo: preparation, sweep, finalisation
def test_calls_can_be_captured_in_a_hip_graph(B, L, d, lam, flags):
    """The entry points only enqueue kernels on the caller's stream (no allocation, no synchronisation, no memset), so a
    training step can be captured once and replayed: every replay, with eager work in between, gives the eager bits
    (many pairs: the gradient sums meet in global atomics, so those are compared to the tolerance)."""
    X, Y = rand_paths(8300 + B, B, L, d, 0.25), rand_paths(8400 + B, B, L, d, 0.25)
    x, y = dev(X), dev(Y)
    gk = dev(np.random.default_rng(85).normal(size=B))
    assert sk.keeps_forward(B, L, L, d, lam, lam, flags, sk.SK_F64)
    keeps = B == 6            # the lock-step kernels: every sum in a fixed order
    KEEP, HAVE = sk.SK_FLAG_KEEP_FORWARD, sk.SK_FLAG_HAVE_FORWARD
    need = max(sk.sigkernel_workspace_bytes(sk.SK_OP_FWD, B, 0, L, L, d, lam, lam, flags | KEEP, sk.SK_F64),
               sk.sigkernel_workspace_bytes(sk.SK_OP_BWD, B, 0, L, L, d, lam, lam, flags, sk.SK_F64))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    k = torch.empty(B, dtype=torch.float64, device="cuda")
    k2 = torch.empty_like(k)
    gx, gy = torch.empty_like(x), torch.empty_like(y)

    def step():
        sk.sigkernel_fwd(x, y, lam, lam, flags | KEEP, k=k, ws=ws)
        sk.sigkernel_bwd(x, y, gk, lam, lam, flags | HAVE, grad_x=gx, grad_y=gy, k_out=k2, ws=ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        for _ in range(2):
            step()            # first launches set kernel attributes: not inside a capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    ref = (k.clone(), k2.clone(), gx.clone(), gy.clone())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        for t in (k, k2, gx, gy):
            t.fill_(float(rep))                                     # eager work between the replays
        other = sk.sigkernel_fwd(y, x, lam, lam, flags)             # ... and an eager call of the library
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(k, ref[0]) and torch.equal(k2, ref[1]) and torch.equal(other, ref[0])
        if keeps:
            assert torch.equal(gx, ref[2]) and torch.equal(gy, ref[3])
        else:
            check_grads(host(gx), host(ref[2]), torch.float64, "grad_x of replay %d" % rep)
            check_grads(host(gy), host(ref[3]), torch.float64, "grad_y of replay %d" % rep)
    kr, gxr, gyr = oracle.bwd(X, Y, host(gk), lam, lam, flags)
    check_values(host(k), kr, torch.float64, "k from the graph")
    check_grads(host(gx), gxr, torch.float64, "grad_x from the graph")


def test_event_timing_tags():
    # the benchmark's timing hook: launches are recorded under the tag that was current, and read per tag
    X, Y = rand_paths(8800, 6, 40, 3, 0.2), rand_paths(8801, 6, 40, 3, 0.2)
    x, y = dev(X), dev(Y)
    gk = dev(np.ones(6))
    sk.sigkernel_event_timing_read()           # drop whatever earlier tests left
    sk.sigkernel_event_timing(1)
    sk.sigkernel_fwd(x, y, 1, 1)
    sk.sigkernel_event_timing(2)
    sk.sigkernel_fwd(x, y, 1, 1)
    sk.sigkernel_bwd(x, y, gk, 1, 1)
    sk.sigkernel_event_timing(0)
    sk.sigkernel_fwd(x, y, 1, 1)               # not recorded
    f_ms, nf, b_ms, nb = sk.sigkernel_event_timing_read(2)
    assert (nf, nb) == (1, 1) and f_ms > 0.0 and b_ms > 0.0
    f_ms, nf, b_ms, nb = sk.sigkernel_event_timing_read()      # the rest: tag 1
    assert (nf, nb) == (1, 0) and f_ms > 0.0
    assert sk.sigkernel_event_timing_read() == (0.0, 0, 0.0, 0)


def test_more_pairs_than_wave_slots():
    # every wave slot handles several pairs in turn, so its scratch rows and checkpoints are reused
    X = rand_paths(71, 5000, 6, 2, 0.3)
    Y = rand_paths(72, 5000, 5, 2, 0.3)
    run_pairs(X, Y, 1, 1, 0, torch.float64, backward=True)


def test_degenerate_inputs():
    x = dev(rand_paths(1, 3, 1, 2))
    y = dev(rand_paths(2, 3, 6, 2))
    assert torch.all(sk.sigkernel_fwd(x, y) == 1.0)                       # L1 = 1: no increments
    k, gx, gy = sk.sigkernel_bwd(x, y, torch.ones(3, dtype=torch.float64, device="cuda"))
    assert torch.all(k == 1.0) and torch.all(gx == 0.0) and torch.all(gy == 0.0)
    e = torch.empty((0, 4, 2), dtype=torch.float64, device="cuda")
    assert sk.sigkernel_fwd(e, e).shape == (0,)                            # empty batch
    z = torch.zeros((4, 9, 3), dtype=torch.float64, device="cuda")
    assert torch.all(sk.sigkernel_fwd(z, dev(rand_paths(3, 4, 7, 3)), 1, 1) == 1.0)   # zero path: k = 1 exactly
    with pytest.raises(sk.SigKernelError):
        small = torch.empty(256, dtype=torch.uint8, device="cuda")
        sk.sigkernel_fwd(dev(rand_paths(4, 2, 5, 2)), dev(rand_paths(5, 2, 5, 2)), ws=small)


def test_symmetry_and_batch_independence():
    X = rand_paths(81, 7, 45, 3, 0.3)
    Y = rand_paths(82, 7, 45, 3, 0.3)
    x, y = dev(X), dev(Y)
    kxy = sk.sigkernel_fwd(x, y, 1, 1)
    kyx = sk.sigkernel_fwd(y, x, 1, 1)
    assert torch.equal(kxy, kyx)
    assert torch.equal(sk.sigkernel_fwd(x, y, 2, 1), sk.sigkernel_fwd(y, x, 1, 2))
    one = sk.sigkernel_fwd(x[3:4].contiguous(), y[3:4].contiguous(), 1, 1)
    assert one[0] == kxy[3]
    K = sk.sigkernel_gram(x, y, None, 1, 1)
    for n, m in [(0, 0), (2, 5), (6, 1)]:
        assert K[n, m] == sk.sigkernel_fwd(x[n:n + 1].contiguous(), y[m:m + 1].contiguous(), 1, 1)[0]


def test_repeated_calls_kernel_values_bitwise_gradients_to_rounding():
    # Kernel values are computed by one wave in a fixed order: the same bits every time.  Gradient sums are collected
    # with floating-point atomics whose order of arrival varies from launch to launch: equal up to rounding (1e-13 of
    # the tensor's scale), which is what the library states about them.
    for name, nx, ny in (("c3", 40, 36), ("c5", 48, 40)):
        w, X, Y = workloads.make(name, n_x=nx, n_y=ny)
        W = dev(workloads.upstream_weights(77, (nx, ny)))
        x, y = dev(X), dev(Y)
        runs = [sk.sigkernel_gram(x, y, W, w.lam, w.lam, w.flags) for _ in range(3)]
        torch.cuda.synchronize()
        for K, gX, gY in runs[1:]:
            assert torch.equal(K, runs[0][0])
            for g, g0 in ((gX, runs[0][1]), (gY, runs[0][2])):
                assert float((g - g0).abs().max() / g0.abs().max().clamp(min=1.0)) <= 1e-13
    w, X, Y = workloads.make("c2", n_x=16, n_y=16)
    gk = dev(workloads.upstream_weights(78, (16,)))
    runs = [sk.sigkernel_bwd(dev(X), dev(Y), gk, w.lam, w.lam, w.flags) for _ in range(3)]
    torch.cuda.synchronize()
    for k, gx, gy in runs[1:]:
        assert torch.equal(k, runs[0][0])
        for g, g0 in ((gx, runs[0][1]), (gy, runs[0][2])):
            assert float((g - g0).abs().max() / g0.abs().max().clamp(min=1.0)) <= 1e-13


def test_only_one_gradient_requested():
    X = rand_paths(91, 4, 20, 3)
    Y = rand_paths(92, 4, 25, 3)
    gk = np.ones(4)
    _, gxr, gyr = oracle.bwd(X, Y, gk, 1, 1, 0)
    _, gx, none = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), 1, 1, 0, want_y=False)
    assert none is None
    check_grads(host(gx), gxr, torch.float64, "grad_x only")
    _, none, gy = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), 1, 1, 0, want_x=False)
    assert none is None
    check_grads(host(gy), gyr, torch.float64, "grad_y only")


# ------------------------------------------------------------------ the two backward variants
@pytest.mark.parametrize("L1,L2,d,lam,B", [(70, 66, 5, 1, 6), (130, 40, 3, 0, 5), (200, 180, 8, 2, 3), (33, 65, 20, 1, 4)])
def test_backward_replay_variant(L1, L2, d, lam, B):
    # SK_FLAG_BWD_REPLAY: forward segments are replayed instead of inverting Eq. (1)
    X = rand_paths(5000 + L1, B, L1, d, 0.2)
    Y = rand_paths(6000 + L2, B, L2, d, 0.2)
    gk = workloads.upstream_weights(11, (B,))
    kr, gxr, gyr = oracle.bwd(X, Y, gk, lam, lam, 0)
    k, gx, gy = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), lam, lam, sk.SK_FLAG_BWD_REPLAY)
    torch.cuda.synchronize()
    check_values(host(k), kr, torch.float64, "k (replay)")
    check_grads(host(gx), gxr, torch.float64, "grad_x (replay)")
    check_grads(host(gy), gyr, torch.float64, "grad_y (replay)")


def test_backward_replay_variant_many_pairs():
    w, X, Y = workloads.make("c3", n_x=40, n_y=40)     # 1600 pairs: one wave per pair
    W = workloads.upstream_weights(34, (40, 40))
    Kref, gXr, gYr = oracle.gram(X, Y, W, w.lam, w.lam, w.flags)
    K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), w.lam, w.lam, w.flags | sk.SK_FLAG_BWD_REPLAY)
    torch.cuda.synchronize()
    check_values(host(K), Kref, torch.float64, "K (replay)")
    check_grads(host(gX), gXr, torch.float64, "grad_X (replay)")
    check_grads(host(gY), gYr, torch.float64, "grad_Y (replay)")
    K2, gX2, gY2 = sk.sigkernel_gram(dev(X), dev(Y), dev(W), w.lam, w.lam, w.flags)
    torch.cuda.synchronize()
    check_grads(host(gX2), gXr, torch.float64, "grad_X (default)")
    check_grads(host(gY2), gYr, torch.float64, "grad_Y (default)")


def drifted_pairs(op, B_or_N, M, L1, L2, d, lam1, lam2, flags, dtype, ws):
    """How many pairs the reverse sweep of the last call on `ws` handed to the replay kernel (the library's launch
    description says where in the workspace it counts them); -1: the launch mode does not count per pair."""
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    desc = sk.sigkernel_describe(op, B_or_N, M, L1, L2, d, lam1, lam2, flags, sdt)
    at = int(desc.split("drifted_pairs_counter_at=", 1)[1].split()[0])
    torch.cuda.synchronize()
    n = int(ws[at:at + 4].view(torch.int32)[0])
    mode = desc.split("mode=", 1)[1].split()[0]
    return n if mode in ("lock-step", "solo", "tile", "four") else -1


def pairs_backward_with_ws(X, Y, gk, lam1, lam2, flags, dtype=torch.float64):
    B, L1, d = X.shape
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    ws = torch.empty(sk.sigkernel_workspace_bytes(sk.SK_OP_BWD, B, 0, L1, Y.shape[1], d, lam1, lam2, flags, sdt),
                     dtype=torch.uint8, device="cuda")
    k, gx, gy = sk.sigkernel_bwd(dev(X, dtype), dev(Y, dtype), dev(gk, dtype), lam1, lam2, flags, ws=ws)
    torch.cuda.synchronize()
    return k, gx, gy, drifted_pairs(sk.SK_OP_BWD, B, 0, L1, Y.shape[1], d, lam1, lam2, flags, dtype, ws)


@pytest.mark.parametrize("scale", [0.5, 1.5, 4.0])
def test_default_backward_is_exact_for_large_increments(scale):
    # Large increments make the inverse of Eq. (1) ill-conditioned (and B(p) = 0 at p = sqrt(12)).  The default backward
    # notices (its drift check), leaves such pairs out, and solves them once more by replaying forward segments: the
    # gradients are the oracle's whatever the input (Section 3.4: exact gradients of the scheme).
    B, L, d = 4, 150, 3
    X = rand_paths(7001, B, L, d, 0.1) * scale
    Y = rand_paths(7002, B, L, d, 0.1) * scale
    gk = np.ones(B)
    kr, gxr, gyr = oracle.bwd(X, Y, gk, 1, 1, 0)
    k, gx, gy, n = pairs_backward_with_ws(X, Y, gk, 1, 1, 0)
    print("scale %g: %d of %d pairs solved once more" % (scale, n, B), flush=True)
    check_values(host(k), kr, torch.float64, "k")
    check_rows(host(gx), gxr, torch.float64, "grad_x (scale %g)" % scale)
    check_rows(host(gy), gyr, torch.float64, "grad_y (scale %g)" % scale)
    assert (n == 0) if scale == 0.5 else (n >= 0)
    if scale == 4.0:
        assert n > 0          # the case the second launch exists for
    k2, gx2, gy2 = sk.sigkernel_bwd(dev(X), dev(Y), dev(gk), 1, 1, sk.SK_FLAG_BWD_REPLAY)
    torch.cuda.synchronize()
    check_rows(host(gx2), gxr, torch.float64, "grad_x (replay, scale %g)" % scale)
    check_rows(host(gy2), gyr, torch.float64, "grad_y (replay, scale %g)" % scale)


@pytest.mark.parametrize("B,L1,L2,d,lam,mode", [(5, 70, 66, 3, 1, "lock-step"),      # fused: works on the caller's arrays
                                                  (6, 150, 140, 5, 0, "lock-step"),    # two strips
                                                  (2600, 14, 12, 3, 1, "solo"),
                                                  (1300, 40, 44, 16, 0, "tile"),
                                                  (3, 400, 330, 3, 0, "band"),
                                                  (1100, 140, 20, 3, 0, "wave-per-pair"),
                                                  (300, 140, 20, 3, 0, "cooperative"),
                                                  (40, 200, 40, 20, 0, "wide")])
@pytest.mark.parametrize("where", ["first columns", "last rows", "one pair"])
def test_large_increments_in_every_launch_mode(B, L1, L2, d, lam, mode, where):
    # Increments of order one in a few places of otherwise benign paths: in the first columns (the stretch left of the
    # first checkpoint, which is compared with the boundary value), in the last rows, or in one pair of the batch only
    # (then the other pairs must come through the fast path: the count says so).  Every launch mode.
    assert ("mode=" + mode) in sk.sigkernel_describe(sk.SK_OP_BWD, B, 0, L1, L2, d, lam, lam, 0, sk.SK_F64)
    rng = np.random.default_rng(7100 + L1 + d)
    dX = rng.normal(0.0, (1.0 / (d * L1)) ** 0.5, (B, L1, d))
    dY = rng.normal(0.0, (1.0 / (d * L2)) ** 0.5, (B, L2, d))
    big = 2.2
    if where == "first columns":
        dY[:, 1:4, :] = rng.choice([-big, big], size=(B, 3, d)) / d ** 0.5
        dX[:, 1::7, :] = rng.choice([-big, big], size=dX[:, 1::7, :].shape) / d ** 0.5
    elif where == "last rows":
        dX[:, -3:, :] = rng.choice([-big, big], size=(B, 3, d)) / d ** 0.5
        dY[:, 2::5, :] = rng.choice([-big, big], size=dY[:, 2::5, :].shape) / d ** 0.5
    else:
        dX[B // 2, 1::3, :] = rng.choice([-big, big], size=dX[B // 2, 1::3, :].shape) / d ** 0.5
        dY[B // 2, 1::3, :] = rng.choice([-big, big], size=dY[B // 2, 1::3, :].shape) / d ** 0.5
    X, Y = np.cumsum(dX, axis=1), np.cumsum(dY, axis=1)
    gk = workloads.upstream_weights(71, (B,))
    kr, gxr, gyr = oracle.bwd(X, Y, gk, lam, lam, 0)
    assert np.all(np.isfinite(kr))
    k, gx, gy, n = pairs_backward_with_ws(X, Y, gk, lam, lam, 0)
    print("%s, %s: %d of %d pairs solved once more; |k| up to %.3g" % (mode, where, n, B, np.abs(kr).max()), flush=True)
    check_values(host(k), kr, torch.float64, "k")
    check_rows(host(gx), gxr, torch.float64, "grad_x")
    check_rows(host(gy), gyr, torch.float64, "grad_y")
    if n >= 0 and where == "one pair":
        assert n <= 1


def test_gram_with_one_wild_path_among_benign_ones():
    # c3's shape cut down (solo kernels) and c5's (tile kernels): one path of X has increments of order one.  Only the
    # pairs of its row are solved once more; K, grad_X and grad_Y are the oracle's; then the symmetric case.
    for name, nx, ny in (("c3", 40, 36), ("c5", 48, 40)):
        w, X, Y = workloads.make(name, n_x=nx, n_y=ny)
        rng = np.random.default_rng(72)
        dXw = rng.choice([-1.0, 1.0], size=(w.L - 1, w.d)) * (2.0 / w.d ** 0.5)
        X[7, 1:, :] = np.cumsum(dXw, axis=0)
        Y[3, 1:, :] = np.cumsum(dXw[::-1] * 0.8, axis=0)
        W = workloads.upstream_weights(73, (nx, ny))
        need = sk.sigkernel_workspace_bytes(sk.SK_OP_GRAM_BWD, nx, ny, w.L, w.L, w.d, w.lam, w.lam, w.flags, sk.SK_F64)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        K, gX, gY = sk.sigkernel_gram(dev(X), dev(Y), dev(W), w.lam, w.lam, w.flags, ws=ws)
        n = drifted_pairs(sk.SK_OP_GRAM_BWD, nx, ny, w.L, w.L, w.d, w.lam, w.lam, w.flags, torch.float64, ws)
        Kr, gXr, gYr = oracle.gram(X, Y, W, w.lam, w.lam, w.flags)
        print("%s: %d of %d pairs solved once more; |K| up to %.3g" % (name, n, nx * ny, np.abs(Kr).max()), flush=True)
        assert 0 < n <= nx + ny - 1
        check_values(host(K), Kr, torch.float64, "K")
        check_rows(host(gX), gXr, torch.float64, "grad_X")
        check_rows(host(gY), gYr, torch.float64, "grad_Y")
        x = dev(X)
        Ws = workloads.upstream_weights(74, (nx, nx))
        Kxx, gXX, _ = sk.sigkernel_gram(x, x, dev(Ws), w.lam, w.lam, w.flags, ws=ws)
        n = drifted_pairs(sk.SK_OP_GRAM_BWD, nx, nx, w.L, w.L, w.d, w.lam, w.lam, w.flags, torch.float64, ws)
        Kxr, gXXr, _ = oracle.gram(X, X, Ws, w.lam, w.lam, w.flags)
        assert 0 < n <= 2 * nx - 1
        check_values(host(Kxx), Kxr, torch.float64, "K(X,X)")
        check_rows(host(gXX), gXXr, torch.float64, "total derivative of K(X,X)")
