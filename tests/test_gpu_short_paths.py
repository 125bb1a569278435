"""The signature kernels that hold several paths in a wavefront read the points themselves and write the caller's type:
chunks of points, waves and pieces that do not come out even, signatures that do and do not fit the LDS buffer.

Tolerance: an entry of level k is a sum of products of k increments, formed in at most n steps of k + 1 roundings each, so
its error is at most (n + 1)(N + 2) 2^-53 times what the absolute increments give, V^k / k! with V their sum over the path;
float results are rounded once more.
"""
import math

import numpy as np
import pytest
import torch

from oracle import signature as osig
from paper_2509_10613_amd import binding as sk

pytestmark = pytest.mark.gpu

T, LL = sk.SK_FLAG_TIME_AUG, sk.SK_FLAG_LEAD_LAG
WHOLE = sk.SK_SIG_PIECES(0)


# (B, L, d, N, flags): two paths per wave hold 511 // d points of a path at a time; 5 * 1024 + 3 paths are six to a wave
@pytest.mark.parametrize("B,L,d,N,flags", [
    (3, 254, 2, 2, WHOLE), (3, 255, 2, 2, WHOLE), (3, 256, 2, 2, WHOLE), (5, 300, 3, 2, WHOLE | T), (1, 513, 1, 3, WHOLE | LL),
    (2, 3, 1, 1, 0), (1, 1, 2, 3, 0), (3, 1, 2, 3, T | LL), (4, 2, 3, 2, LL), (3, 60, 2, 2, WHOLE | LL | T),
    (5 * 1024 + 3, 9, 2, 3, 0), (5 * 1024 + 3, 12, 2, 4, T), (3000, 7, 3, 2, LL | T), (2 * 1024, 6, 2, 6, 0),
    (3, 41, 2, 3, sk.SK_SIG_PIECES(3)), (2, 9, 2, 2, sk.SK_SIG_PIECES(4) | T), (3, 11, 2, 2, sk.SK_SIG_PIECES(3) | LL | T),
    (700, 10, 9, 3, sk.SK_SIG_DEPTH(2)), (9, 8, 4, 3, T), (5, 6, 15, 1, T | LL), (40, 70, 20, 1, WHOLE | T),
])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_several_paths_per_wave(B, L, d, N, flags, dtype):
    rng = np.random.default_rng(17 * B + L + d)
    x = torch.tensor(np.cumsum(rng.normal(0, 0.3, size=(B, L, d)), axis=1), dtype=dtype)
    desc = sk.signature_describe(B, L, d, N, flags, sk.SK_F64 if dtype == torch.float64 else sk.SK_F32)
    print(desc, flush=True)
    assert ", true, " in desc and "paths_per_wave=1 " not in desc
    got = sk.signature_fwd(x.cuda(), N, flags).cpu().double().numpy()
    xd = x.double().numpy()
    some = np.unique(np.concatenate([np.arange(min(B, 40)), np.arange(max(0, B - 40), B)]))    # (the oracle is slow)
    ref = osig.signature(xd[some], N, flags & (T | LL))
    one = sk.signature_fwd(x.cuda(), N, flags | sk.SK_SIG_ONE_PATH_PER_WAVE).cpu().double().numpy()
    D = d * (2 if flags & LL else 1) + (1 if flags & T else 0)
    V = np.abs(np.diff(xd, axis=1)).sum((1, 2)) * (2 if flags & LL else 1) + (1 if flags & T else 0)
    n = (L - 1) * (2 if flags & LL else 1)
    scale = np.concatenate([np.repeat((V ** k / math.factorial(k))[:, None], D ** k, axis=1) for k in range(N + 1)], axis=1)
    bound = (n + 1) * (N + 2) * 2.0 ** -53 * scale
    if dtype == torch.float32:
        bound = bound + 2.0 ** -24 * np.abs(got) * (1 + 2.0 ** -20) + 2.0 ** -150
    assert np.all(np.abs(got[some] - ref) <= 2 * bound[some])       # (the oracle's own roundings)
    assert np.all(np.abs(got - one) <= 2 * bound)


# (a piece of ten segments in eight has at most two, and the last ones none)
@pytest.mark.parametrize("P,flags", [(0, 0), (1, T), (3, 0), (3, T), (3, LL), (4, LL | T)])
@pytest.mark.parametrize("d,N", [(2, 2), (3, 1), (5, 2), (20, 1)])
def test_a_path_that_ends_in_infinity_has_moved_that_far(P, flags, d, N):
    # level 1 is where a path ends less where it starts; pieces that reach past the end don't move there
    rng = np.random.default_rng(P + d)
    x = np.cumsum(rng.normal(0, 0.3, size=(4, 11, d)), axis=1)
    x[1, -1, 0], x[2, -1, d - 1] = np.inf, -np.inf
    f = flags | sk.SK_SIG_PIECES(P)
    desc = sk.signature_describe(4, 11, d, N, f, sk.SK_F64)
    print(desc, flush=True)
    assert "pieces_per_path=%d " % 2 ** P in desc and (d >= 5 and flags & LL or ", true, " in desc and "paths_per_wave=1 " not in desc)
    got = sk.signature_fwd(torch.tensor(x).cuda(), N, f).cpu().numpy()
    move = x[:, -1] - x[:, 0]
    move = np.concatenate([move] + [move] * bool(flags & LL) + [np.ones((4, 1))] * bool(flags & T), axis=1)
    assert np.allclose(got[:, 1:1 + move.shape[1]], move, rtol=0, atol=1e-12) and np.isfinite(got[[0, 3]]).all()
