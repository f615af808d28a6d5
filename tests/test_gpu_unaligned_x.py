"""Borrowed column-major X whose columns start at any multiple of 4 bytes: the column pass's
16-byte loads at M no multiple of 4, and at a base no multiple of 16, against the FP64 oracle
(check_factors' bars, as everywhere)."""

import numpy as np
import pytest

import oracle
import paper_1802_08938_amd as did
from tests._gpu import announce, check_factors, read_factors, require_gpu
from workloads import as_oracle_input, serving_x, to_f32_colmajor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [32, 65, 66, 99, 100])  # whole chunks, and 1, 2, 3, 4 rows more
@pytest.mark.parametrize("offset", [0, 1, 2, 3])      # floats past a 16-byte boundary
def test_column_pass_reads_x_at_any_float(M, offset):
    torch = require_gpu()
    N, K = 161, 6
    X32 = to_f32_colmajor(serving_x(M, N, K, seed=M + offset))
    announce(f"X at offset {offset}, M={M}")
    room = torch.zeros(M * N + offset, device="cuda")
    room[offset:] = torch.from_numpy(np.ascontiguousarray(X32.T).reshape(-1)).to("cuda")
    X = room[offset:].view(N, M)
    torch.cuda.synchronize()
    o = did.did_default_opts()
    o.borrow_x = 1
    h = did.did_init_ex(X, M, N, K, 3, o)
    try:
        B0, C0 = read_factors(h, M, N, K)
        did.did_iterate(h, 1)
        B, C = read_factors(h, M, N, K)
    finally:
        did.did_free(h)
    Bo, Co, _ = oracle.did_run(as_oracle_input(X32), B0, C0, 1)
    check_factors(B, Bo, C, Co, label=f"M={M} offset={offset}")
