"""The tile-order storage at ragged sizes: its two copies hold X (one iteration reads both, the
column pass one and the row pass the other), and the check of the entries reaches every edge.

Iterates against the FP64 oracle with check_factors' bars, as everywhere (the storage itself is
exact in float32; the bfloat16 form's oracle takes the rounded X)."""

import numpy as np
import pytest

import oracle
import paper_1802_08938_amd as did
from tests._gpu import announce, check_factors, device_x, require_gpu, run_gpu
from workloads import as_oracle_input, round_to_bf16, serving_x, to_f32_colmajor

pytestmark = pytest.mark.gpu

SHAPES = [
    (32, 32, 3),     # one whole tile
    (33, 31, 2),     # rows one past a tile, columns one short; rows no multiple of 4
    (36, 33, 5),     # both second tiles a few rows or one column wide
    (129, 65, 7),    # a block of four chunks and one more, a single last row and column
    (20, 2100, 4),   # more column tiles than rows of a tile
    (1100, 40, 9),   # several blocks for a column tile's chunks
]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("bf16", [False, True])
def test_tiled_copies_at_ragged_sizes(M, N, K, bf16):
    torch = require_gpu()
    X32 = to_f32_colmajor(serving_x(M, N, K, seed=M + N))
    o = did.did_default_opts()
    o.x_tiled = 1
    o.x_dtype = did.DID_BF16 if bf16 else did.DID_F32
    announce(f"tiled copies M={M} N={N} K={K} bf16={bf16}")
    out = run_gpu(torch, X32, K, iters=(1,), opts=o)
    B0, C0 = out["init"]
    X = round_to_bf16(X32) if bf16 else as_oracle_input(X32)
    Bo, Co, _ = oracle.did_run(X, B0, C0, 1)
    check_factors(out[1][0], Bo, out[1][1], Co, label=f"{M}x{N} bf16={bf16}")


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("bf16", [False, True])
def test_tiled_storage_refuses_bad_entries_at_the_edges(M, N, K, bf16):
    torch = require_gpu()
    o = did.did_default_opts()
    o.x_tiled = 1
    o.x_dtype = did.DID_BF16 if bf16 else did.DID_F32
    announce(f"refused entries M={M} N={N} bf16={bf16}")
    for (i, j), bad in zip([(0, 0), (M - 1, 0), (0, N - 1), (M - 1, N - 1), (M // 2, N // 2)],
                           [-1.0, np.nan, np.inf, -np.inf, -1e-30]):
        X32 = to_f32_colmajor(np.ones((M, N)))
        X32[i, j] = bad
        with pytest.raises(did.DidError) as err:
            did.did_init_ex(device_x(torch, X32), M, N, K, 1, o)
        assert err.value.code == did.DID_EINVAL and "finite and nonnegative" in str(err.value)
    X32 = to_f32_colmajor(np.zeros((M, N)))
    X32[M - 1, N - 1] = 3.0e38  # the largest values are accepted
    did.did_free(did.did_init_ex(device_x(torch, X32), M, N, K, 1, o))
