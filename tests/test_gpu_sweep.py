"""The coordinate sweep and the B update at the edges of their blocks: both forms of the
sweep (16 columns per wave up to N = 16384, 64 beyond), ragged last tiles and blocks, each
count of 16-coordinate blocks, against the FP64 oracle after one iteration.

The bars are check_factors' (1e-5 normwise, 1e-4 per line): the chains run in float64, so
only the float32 products in H and W contribute, as on every other shape."""

import numpy as np
import pytest

import oracle
import paper_1802_08938_amd as did
from tests._gpu import announce, check_factors, check_trajectory, require_gpu, run_gpu
from workloads import as_oracle_input, serving_x, to_f32_colmajor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (40, 65, 4),        # one step of four coordinates, a second block of one column
    (70, 257, 15),      # K just below one 16-block
    (129, 127, 17),     # K just above one, M and N one off a block
    (65, 16384, 5),     # the last N with 16 columns per wave
    (64, 16385, 33),    # the first with 64, its last tile a single column
    (66, 16433, 49),    # an odd number of tiles: a wave's second tile does not exist
    (80, 16640, 64),    # whole blocks, largest K
    (515, 90, 48),      # ragged blocks of rows of B, K at a whole number of 16-blocks
])
@pytest.mark.parametrize("refresh", [1, 2])
def test_sweep_and_b_update_block_edges(M, N, K, refresh):
    torch = require_gpu()
    X32 = to_f32_colmajor(serving_x(M, N, K, seed=M + N + K))
    o = did.did_default_opts()
    o.refresh_every = refresh
    announce(f"block edges M={M} N={N} K={K} refresh_every={refresh}")
    out = run_gpu(torch, X32, K, iters=(1, 2), opts=o)
    B0, C0 = out["init"]
    X = as_oracle_input(X32)
    for t in (1, 2):
        Bo, Co, _ = oracle.did_run(X, B0, C0, t)
        assert np.all(out[t][0] >= 0.0) and np.all(out[t][1] >= 0.0)
        check_factors(out[t][0], Bo, out[t][1], Co, label=f"{M}x{N} K={K} refresh={refresh} t={t}")


@pytest.mark.parametrize("M,N,K,cw", [
    (515, 90, 20, 4),     # 17 chunks over 4 shares
    (2049, 70, 64, 8),    # a last chunk of one row, 8 waves per block
    (4103, 33, 7, 4),     # many shares of a single column block, two tiles
    (1200, 1500, 33, 0),  # several column blocks and shares
])
def test_column_pass_row_shares(M, N, K, cw):
    """The column pass split over the rows of X: factors, history and objective against the
    oracle, and float32 X as given equal to the tiled form bit for bit (the same shares)."""
    torch = require_gpu()
    X32 = to_f32_colmajor(serving_x(M, N, K, seed=M + N + K))
    X = as_oracle_input(X32)
    announce(f"row shares M={M} N={N} K={K} col_waves={cw}")
    outs = []
    for tiled in (0, 1):
        o = did.did_default_opts()
        o.col_waves = cw
        o.x_tiled = tiled
        outs.append(run_gpu(torch, X32, K, iters=(1, 3), opts=o))
    out = outs[0]
    B0, C0 = out["init"]
    Bo, Co, _ = oracle.did_run(X, B0, C0, 1)
    check_factors(out[1][0], Bo, out[1][1], Co, label=f"{M}x{N} K={K}")
    _, _, fo = oracle.did_run(X, B0, C0, 3)
    check_trajectory(np.append(out["hist"], out["f"]), fo, label=f"{M}x{N} K={K}")
    for t in (1, 3):
        np.testing.assert_array_equal(outs[1][t][0], out[t][0])
        np.testing.assert_array_equal(outs[1][t][1], out[t][1])


@pytest.mark.parametrize("M,N,K", [
    (5, 65, 3),       # the 5 x 3 instance, one wave and one column over
    (5, 300_000, 3),  # more block partials than the finishing block has groups
    (2, 513, 1),      # 8 x 4, mostly padding
    (8, 257, 4),      # 8 x 4, no padding
    (8, 511, 8),      # 8 x 8: more slots than lanes
    (16, 300, 4),     # 16 x 4: more slots than lanes
    (9, 40_000, 2),   # 16 x 4 with padding
])
def test_thin_path_sums(M, N, K):
    """The thin path's block sums and finishing block: factors and objectives against the
    oracle, and the same bits from a second run."""
    torch = require_gpu()
    rng = np.random.default_rng(M * 100 + K)
    X32 = to_f32_colmajor(rng.random((M, K)) @ rng.random((K, N)) + 0.01 * rng.random((M, N)))
    X = as_oracle_input(X32)
    announce(f"thin sums M={M} N={N} K={K}")
    a, b = (run_gpu(torch, X32, K, iters=(1, 3)) for _ in range(2))
    B0, C0 = a["init"]
    Bo, Co, _ = oracle.did_run(X, B0, C0, 1)
    check_factors(a[1][0], Bo, a[1][1], Co, label=f"thin {M}x{N} K={K}")
    _, _, fo = oracle.did_run(X, B0, C0, 3)
    check_trajectory(np.append(a["hist"], a["f"]), fo, label=f"thin {M}x{N} K={K}")
    for t in (1, 3):
        np.testing.assert_array_equal(a[t][0], b[t][0])
        np.testing.assert_array_equal(a[t][1], b[t][1])
