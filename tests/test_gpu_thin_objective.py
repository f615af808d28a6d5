"""The thin path's objective: its own pass (did_objective, and the C half of DBCD) sums one
partial per block, an iteration sums f among its other partials.  Both are float64 sums of the
same M N nonnegative terms in different orders, each off by less than (terms added in a row) *
2^-53 relative: at most 1200 columns a thread of 16 rows, 4 waves and 1280 blocks here, so 1e-11."""

import numpy as np
import pytest

import paper_1802_08938_amd as did
from tests._gpu import announce, device_x, require_gpu
from workloads import to_f32_colmajor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (5, 3, 3), (5, 65_537, 3), (5, 300_000, 3),  # one block, 257 blocks, a full launch
    (2, 513, 1), (8, 257, 4), (8, 200_000, 4),
    (8, 511, 8), (8, 100_000, 5),
    (16, 300, 4), (9, 70_000, 2),
])
@pytest.mark.parametrize("algorithm", [did.DID_ALG_DID, did.DID_ALG_DBCD])
def test_objective_is_the_recorded_one(M, N, K, algorithm):
    torch = require_gpu()
    rng = np.random.default_rng(M * 1000 + K)
    X = to_f32_colmajor(rng.random((M, K)) @ rng.random((K, N)) + 0.01 * rng.random((M, N)))
    o = did.did_default_opts()
    o.algorithm = algorithm
    announce(f"thin objective M={M} N={N} K={K} algorithm={algorithm}")
    Xd = device_x(torch, X)
    h = did.did_init_ex(Xd, M, N, K, 7, o)
    try:
        f = []
        for _ in range(3):
            f.append(did.did_objective(h))
            did.did_iterate(h, 1)
        B, C = np.empty((K, M), np.float32), np.empty((N, K), np.float32)
        did.did_factors(h, B, C)
        np.testing.assert_allclose(did.did_history(h), f, rtol=1e-11)
        exact = 0.5 * np.sum((X.astype(np.float64) - B.astype(np.float64).T @ C.astype(np.float64).T) ** 2)
        # (X - B C formed in float64 in both: cancellation of 12 bits or less at these residuals)
        np.testing.assert_allclose(did.did_objective(h), exact, rtol=1e-9)
    finally:
        did.did_free(h)
