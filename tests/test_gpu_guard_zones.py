"""Guard zones stand behind every buffer that a kernel writes: H and the partials of W and V, which
share one buffer without them, have a zone each, exactly at their ends, and the results do not
depend on it."""

import numpy as np
import pytest

import paper_1802_08938_amd as did
from tests._gpu import announce, device_x, read_factors, require_gpu
from workloads import serving_x, to_f32_colmajor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,tiled,refresh,zones", [
    # flag, X, B, C, Bq, Bsc, G, Gpart, V, W, H, W and V partials, Cq, Csc, ranges, f partials,
    # history, objective, counter
    (300, 2000, 10, 0, 1, 20),
    (130, 777, 40, 1, 1, 20),
    (2049, 70, 64, 0, 1, 20),     # row shares of the column pass
    (97, 1234, 33, 0, 4, 23),     # and the residual, delta B, delta C
    (5, 4000, 3, 0, 1, 14),       # thin: one buffer of block partials
])
def test_zone_behind_each_buffer(monkeypatch, M, N, K, tiled, refresh, zones):
    torch = require_gpu()
    announce(f"guard zones {M}x{N} K={K} tiled={tiled} refresh={refresh}")
    X = device_x(torch, to_f32_colmajor(serving_x(M, N, K, seed=M + N + K)))
    o = did.did_default_opts()
    o.x_tiled, o.refresh_every = tiled, refresh
    got = []
    for guard in ("0", "1"):
        monkeypatch.setenv("DID_DEBUG_GUARD_ZONES", guard)
        h = did.did_init_ex(X, M, N, K, 11, o)
        try:
            did.did_iterate(h, 1)
            did.did_iterate(h, 3)
            did.did_sync(h)
            assert did.did_debug_check_guards(h) == (0, zones if guard == "1" else 0)
            got.append(read_factors(h, M, N, K))
        finally:
            did.did_free(h)
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
