"""Backward kernel of truncated signatures with the sum over words on the matrix cores (sg_horner_bwd_matrix.hip): every
channel count, one and two words per lane, path lengths around the sixteen segments it takes at a time, against the oracle
(check: 1e-10 of the gradient's largest entry) and, where that would take long, against the other kernel."""
import numpy as np
import pytest
import torch

from paper_2509_10613_amd import binding as sk
from tests.test_gpu_signature_bwd import check, dev, host, paths

pytestmark = pytest.mark.gpu


def matrix_kernel(B, L, d, N, flags=0):
    return sk.signature_bwd_describe(B, L, d, N, flags, sk.SK_F64).split("kernel=")[1]


@pytest.mark.parametrize("L", [17, 18, 32, 34])          # 16, 17, 31 and 33 segments
@pytest.mark.parametrize("D,N", [(5, 3), (8, 3), (6, 4), (9, 3), (16, 3), (5, 5), (11, 4)])
def test_path_lengths_against_the_oracle(D, N, L):
    assert matrix_kernel(2, L, D, N).startswith("horner_bwd_matrix_kernel<%d, %d, 1>" % (D, N - 2))
    check(paths(40 + D + L, 2, L, D, 0.15), N)


@pytest.mark.parametrize("flags,d,N,dtype", [(sk.SK_FLAG_TIME_AUG, 6, 3, torch.float32), (sk.SK_FLAG_LEAD_LAG, 3, 4, torch.float64),
                                             (sk.SK_FLAG_LEAD_LAG | sk.SK_FLAG_TIME_AUG, 4, 3, torch.float64)])
def test_transformed_paths(flags, d, N, dtype):
    assert matrix_kernel(3, 21, d, N, flags).startswith("horner_bwd_matrix_kernel")
    check(paths(60 + d, 3, 21, d, 0.15), N, flags, dtype)


def test_pieces():
    for q in (1, 2):
        assert matrix_kernel(2, 70, 6, 4, sk.SK_SIG_PIECES(q)).startswith("horner_bwd_matrix_kernel")
        check(paths(71, 2, 70, 6, 0.1), 4, sk.SK_SIG_PIECES(q))


@pytest.mark.parametrize("D", range(5, 17))
@pytest.mark.parametrize("N", [3, 4, 5])
def test_two_words_per_lane_against_the_other_kernel(D, N):
    # the least batch with two words per lane; a difference of rounding only: both kernels are held to 1e-10 of the oracle
    lanes = {1: 8 if D <= 8 else 16, 2: 4 if D <= 8 else 8}
    waves = lambda s: -(-D ** (N - 2) // (64 // lanes[s]))  # noqa: E731
    B = 1024 // waves(1) + 1
    if (D < 11 or N > 4) and B * waves(2) > 2048:
        B = 2048 // waves(2)
    L = 19
    words = 2 if B * waves(1) > 1024 else 1
    if not matrix_kernel(B, L, D, N).startswith("horner_bwd_matrix_kernel<%d, %d, %d>" % (D, N - 2, words)):
        pytest.fail(matrix_kernel(B, L, D, N))
    x = dev(paths(80 + D, B, L, D, 0.15))
    g = torch.randn(B, sk.signature_length(D, N, 0), dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(D))
    got = host(sk.signature_bwd(x, g, N, 0))
    ref = host(sk.signature_bwd(x, g, N, sk.SK_SIG_ONE_PATH_PER_WAVE))
    assert np.all(np.isfinite(got)) and np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))
