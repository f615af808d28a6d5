"""Dispatch cells of the sweep and the W-order packing by values: the 64-columns-per-wave sweep
(N > 16384) at every count of 16-coordinate blocks, a wave whose second tile does not exist, and
the grouped kernels with both sweep forms and more than one tile per packing wave in one group.

The bars are check_factors' (1e-5 normwise, 1e-4 per line): the chains run in float64, so only
the float32 products in H and W contribute, as on every other shape."""

import numpy as np
import pytest

import oracle
import paper_1802_08938_amd as did
from tests._gpu import announce, check_factors, device_x, read_factors, require_gpu, run_gpu
from workloads import as_oracle_input, serving_x, to_f32_colmajor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (40, 16_385, 12),  # one 16-block; 513 tiles, the last a single column
    (45, 16_401, 16),  # ... filled; 17 columns in the last tile
    (50, 16_401, 24),  # two 16-blocks
    (70, 16_449, 32),  # ... filled; 515 tiles, a last block of two tiles and a column
    (60, 16_401, 40),  # three
    (64, 16_401, 49),  # four: a wave's second tile does not exist
    (70, 16_417, 63),  # ... and neither do its last columns (514 tiles, one in the last)
])
@pytest.mark.parametrize("refresh", [1, 2])
def test_wide_sweep_at_each_block_count(M, N, K, refresh):
    torch = require_gpu()
    X32 = to_f32_colmajor(serving_x(M, N, K, seed=M + N + K))
    o = did.did_default_opts()
    o.refresh_every = refresh
    announce(f"wide sweep M={M} N={N} K={K} refresh_every={refresh}")
    out = run_gpu(torch, X32, K, iters=(1, 2), opts=o)
    B0, C0 = out["init"]
    X = as_oracle_input(X32)
    for t in (1, 2):
        Bo, Co, _ = oracle.did_run(X, B0, C0, t)
        assert np.all(out[t][0] >= 0.0) and np.all(out[t][1] >= 0.0)
        check_factors(out[t][0], Bo, out[t][1], Co, label=f"{M}x{N} K={K} refresh={refresh} t={t}")


@pytest.mark.parametrize("tiled", [0, 1])
def test_grouped_sweep_and_packing_equal_solo(tiled):
    """One batch over every sweep branch of both K classes; each member equal to its solo run
    bit for bit, and one iteration of each against the oracle."""
    torch = require_gpu()
    shapes = [
        (40, 16_401, 12), (50, 16_417, 24), (48, 16_385, 32),  # K <= 32, 64 columns per wave
        (36, 70_001, 20),                                      # and packing waves of two tiles
        (90, 1009, 11), (33, 16_384, 30),                      # 16 columns per wave, same group
        (60, 16_401, 40), (70, 16_417, 57), (66, 66_000, 48),  # K > 32
        (129, 777, 45), (80, 301, 64),
    ]
    o = did.did_default_opts()
    o.x_tiled = tiled
    X32 = [to_f32_colmajor(serving_x(M, N, K, seed=M + N + K)) for M, N, K in shapes]
    Xd = [device_x(torch, x) for x in X32]
    announce(f"grouped sweep cells, {len(shapes)} members, x_tiled={tiled}")
    solo, init = [], []
    for x, (M, N, K) in zip(Xd, shapes):
        h = did.did_init_ex(x, M, N, K, 7 + K, o)
        init.append(read_factors(h, M, N, K))
        did.did_iterate(h, 1)
        one = read_factors(h, M, N, K)
        did.did_iterate(h, 2)
        solo.append((one, read_factors(h, M, N, K)))
        did.did_free(h)
    hs = [did.did_init_ex(x, M, N, K, 7 + K, o) for x, (M, N, K) in zip(Xd, shapes)]
    b = did.did_batch_create()
    try:
        for step, n in enumerate((1, 2)):
            for h in hs:
                did.did_batch_add(b, h)
            did.did_batch_iterate(b, n)
            for i, (h, (M, N, K)) in enumerate(zip(hs, shapes)):
                did.did_batch_remove(b, h)
                got = read_factors(h, M, N, K)
                np.testing.assert_array_equal(got[0], solo[i][step][0])
                np.testing.assert_array_equal(got[1], solo[i][step][1])
    finally:
        did.did_batch_free(b)
        for h in hs:
            did.did_free(h)
    for i, (M, N, K) in enumerate(shapes):
        Bo, Co, _ = oracle.did_run(as_oracle_input(X32[i]), *init[i], 1)
        check_factors(solo[i][0][0], Bo, solo[i][0][1], Co, label=f"{M}x{N} K={K}")
