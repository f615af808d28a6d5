"""A coordinate whose basis column is zero is not updated, whatever the residual: also where the
residual is past the float32 range and its inner products are not finite.  Values left alone are
left alone bit for bit, so no tolerance."""

import numpy as np
import pytest

import paper_1802_08938_amd as did
from tests._gpu import announce, require_gpu, run_gpu

pytestmark = pytest.mark.gpu

BIG = 1e30  # B C is 10^60: float32 residuals overflow


@pytest.mark.parametrize("M,N,K", [(40, 70, 2), (70, 130, 17), (64, 16_500, 6), (60, 16_400, 49)])
@pytest.mark.parametrize("refresh", [1, 2])
def test_zero_columns_keep_their_coordinates(M, N, K, refresh):
    torch = require_gpu()
    zero = {1, K - 1}
    rng = np.random.default_rng(M + N + K)
    X = rng.random((M, N)).astype(np.float32)
    B, C = BIG * rng.random((M, K)), BIG * rng.random((K, N))
    B[:, sorted(zero)] = 0.0
    o = did.did_default_opts()
    o.refresh_every = refresh
    announce(f"zero columns of B M={M} N={N} K={K} refresh_every={refresh}")
    out = run_gpu(torch, X, K, iters=(1,), opts=o, B0=B, C0=C)
    for k in zero:
        np.testing.assert_array_equal(out[1][1][k], out["init"][1][k])
