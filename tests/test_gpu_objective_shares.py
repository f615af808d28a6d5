"""did_objective on wide, short X, where its pass takes the rows whole while an iteration's column
pass takes them in shares: both sum the same float32 tile sums in float64, in different orders
(fewer than 10^5 of them, all nonnegative, so within 10^5 * 2^-53 of each other)."""

import numpy as np
import pytest

import paper_1802_08938_amd as did
from tests._gpu import announce, device_x, require_gpu
from workloads import to_f32_colmajor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["given", "tiled", "bf16"])
@pytest.mark.parametrize("M,N,K,col_waves", [
    (260, 65_440, 3, 0),  # 9 chunks in two shares, 512 column blocks, the last of one tile
    (330, 66_000, 4, 8),  # 8 waves per block: 258 column blocks
    (300, 65_400, 4, 0),  # 511 column blocks
])
def test_objective_is_the_recorded_one(M, N, K, col_waves, storage):
    torch = require_gpu()
    rng = np.random.default_rng(M + N)
    X = to_f32_colmajor(rng.random((M, K), dtype=np.float32) @ rng.random((K, N), dtype=np.float32))
    o = did.did_default_opts()
    o.x_tiled, o.x_dtype = int(storage == "tiled"), did.DID_BF16 if storage == "bf16" else did.DID_F32
    o.col_waves = col_waves
    announce(f"objective shares {storage} M={M} N={N} K={K} col_waves={col_waves}")
    Xd = device_x(torch, X)
    h = did.did_init_ex(Xd, M, N, K, 3, o)
    try:
        f = []
        for _ in range(2):
            f.append(did.did_objective(h))
            did.did_iterate(h, 1)
        np.testing.assert_allclose(did.did_history(h), f, rtol=2e-11)
    finally:
        did.did_free(h)
