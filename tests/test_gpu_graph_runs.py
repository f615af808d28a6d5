"""Longer runs replay a graph of several iterations: every count around a run's length, alone
and after earlier calls, gives the iterates and objectives of single launches bit for bit (the
same kernels on the same values, so no tolerance)."""

import numpy as np
import pytest

import paper_1802_08938_amd as did
from tests._gpu import announce, device_x, read_factors, require_gpu
from workloads import serving_x, to_f32_colmajor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("calls", [
    (16,),             # the first count that replays the longer graph from the start
    (15, 4, 3),        # the single graph, then one run of four, then a short call
    (19, 1, 6, 2),     # a remainder of three, single launches between, a remainder of two
    (40, 5),
])
def test_runs_equal_single_launches(calls):
    torch = require_gpu()
    M, N, K = 210, 1500, 19
    X32 = to_f32_colmajor(serving_x(M, N, K, seed=5))
    announce(f"graph runs {calls}")
    X = device_x(torch, X32)
    he, hg = did.did_init(X, M, N, K, 7), did.did_init(X, M, N, K, 7)
    try:
        for n in calls:
            for _ in range(n):
                did.did_iterate(he, 1)
            did.did_iterate(hg, n)
            fe, fg = did.did_objective(he), did.did_objective(hg)  # eager work between the replays
            a, b = read_factors(he, M, N, K), read_factors(hg, M, N, K)
            np.testing.assert_array_equal(a[0], b[0])
            np.testing.assert_array_equal(a[1], b[1])
            assert fe == fg
        np.testing.assert_array_equal(np.array(did.did_history(he)), np.array(did.did_history(hg)))
        assert did.did_iterations(hg) == sum(calls)
    finally:
        did.did_free(he)
        did.did_free(hg)
