"""Forward sweep of Gram matrices with four path pairs per wavefront (sk_quad.hip): five to eight block rows per lane,
at the fewest and the most grid rows of each, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_10613_amd import binding as sk
from tests.test_gpu_parity import check_values, dev, host, rounded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mb,rows", [(65, 5), (80, 5), (81, 6), (96, 6), (97, 7), (112, 7), (113, 8), (128, 8)])
@pytest.mark.parametrize("d,lam,flags,dtype", [(8, 0, 0, torch.float64), (8, 1, 1, torch.float32), (3, 1, 0, torch.float64),
                                               (7, 1, 0, torch.float64)])
def test_quad_rows(mb, rows, d, lam, flags, dtype):
    if flags & sk.SK_FLAG_TIME_AUG:
        d -= 1
    nx, ny, L1, L2 = 403, 3, mb + 1, 9 + mb // 40
    rng = np.random.default_rng(1500 + mb + d)
    X = np.cumsum(rng.normal(0.0, (1.0 / (d * L1)) ** 0.5, (nx, L1, d)), axis=1)
    Y = np.cumsum(rng.normal(0.0, (1.0 / (d * L2)) ** 0.5, (ny, L2, d)), axis=1)
    sdt = sk.SK_F64 if dtype == torch.float64 else sk.SK_F32
    desc = sk.sigkernel_describe(sk.SK_OP_GRAM, nx, ny, L1, L2, d, lam, lam, flags, sdt)
    assert "mode=quad" in desc and " rows_per_lane=%d " % rows in desc, desc
    K = sk.sigkernel_gram(dev(X, dtype), dev(Y, dtype), None, lam, lam, flags)
    torch.cuda.synchronize()
    check_values(host(K), oracle.gram(rounded(X, dtype), rounded(Y, dtype), None, lam, lam, flags), dtype, "K")
