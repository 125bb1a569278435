"""Signatures of paths cut into pieces, and their gradients: every level count with a kernel of its own, sums short enough
for one lane and for eight, batches that do not fill a wavefront, pieces past the end of the path.

Tolerance: an entry of level k is a sum of products of k increments, formed in at most n + P steps of k + 1 roundings each, so
its error is at most (n + P)(N + 2) 2^-53 times what the absolute increments give, at most exp(V) with V their sum over the
path; for the gradient twice as many steps, times the largest upstream value and the number of entries it sums over.
"""
import math

import numpy as np
import pytest
import torch

from oracle import signature as osig
from paper_2509_10613_amd import binding as sk

pytestmark = pytest.mark.gpu

T, LL = sk.SK_FLAG_TIME_AUG, sk.SK_FLAG_LEAD_LAG


# (paths, points, channels, levels, flags, log2 of the pieces)
@pytest.mark.parametrize("B,L,d,N,flags,q", [
    (3, 40, 20, 1, 0, 2), (5, 40, 3, 2, 0, 3), (2, 30, 7, 3, 0, 2), (2, 21, 4, 4, LL, 2), (2, 33, 3, 5, T, 3), (2, 17, 2, 6, 0, 1),
    (1, 17, 3, 7, 0, 2), (3, 9, 2, 8, 0, 2), (1, 9, 2, 9, T, 1), (1, 9, 2, 10, 0, 2), (1, 7, 2, 11, 0, 1), (1, 6, 2, 12, 0, 1),
    (1, 5, 2, 13, 0, 1), (2, 70, 1, 3, 0, 4), (4, 5, 2, 3, 0, 4), (3, 2, 3, 3, LL | T, 3), (17, 65, 2, 2, 0, 5),
])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_pieces(B, L, d, N, flags, q, dtype):
    rng = np.random.default_rng(31 * L + d + N)
    x = torch.tensor(np.cumsum(rng.normal(0, 0.6 / math.sqrt(L * d), size=(B, L, d)), axis=1), dtype=dtype)
    n = sk.signature_length(d, N, flags)
    up = torch.tensor(rng.normal(size=(B, n)), dtype=dtype)
    flag = flags | sk.SK_SIG_PIECES(q)
    print(sk.signature_bwd_describe(B, L, d, N, flag, sk.SK_F64), flush=True)
    got = sk.signature_fwd(x.cuda(), N, flag).cpu().double().numpy()
    grad = sk.signature_bwd(x.cuda(), up.cuda(), N, flag).cpu().double().numpy()
    ref = osig.signature(x.double().numpy(), N, flags)
    gref = osig.signature_backward(x.double().numpy(), up.double().numpy(), N, flags)
    V = float(np.abs(np.diff(x.double().numpy(), axis=1)).sum((1, 2)).max()) * (2 if flags & LL else 1) + (1 if flags & T else 0)
    eps = ((L - 1) * (2 if flags & LL else 1) + 2 ** q) * (N + 2) * 2.0 ** -53 * math.exp(V)
    scale = 2 * eps * float(up.abs().max()) * sum(V ** k / math.factorial(k) * (d * (2 if flags & LL else 1) + 1) for k in range(N))
    out = 2.0 ** -23 if dtype == torch.float32 else 0.0
    assert np.all(np.abs(got - ref) <= 2 * eps + out * np.abs(ref))       # (twice: the oracle's own roundings)
    assert np.all(np.abs(grad - gref) <= 2 * scale + out * np.abs(gref))
