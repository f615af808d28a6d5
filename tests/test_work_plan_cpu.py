"""The scratch of the column pass's row shares and the row pass's column ranges: an instance
needs no more device memory than with unsplit column passes and ranges of at least 16 tiles
in buffers of their own, whatever its shape and options (so that budgets and arenas sized
for those still hold it).  Runs on the CPU: did_mem_estimate touches no device."""

import random

import pytest

import paper_1802_08938_amd as did


def _unsplit_bytes(M, N, K, n_blocks, row_blocks, refresh):
    KP = 32 if K <= 32 else 64
    NP, nch, T = KP * (KP + 1) // 2, -(-M // 32), -(-N // 32)
    Mpad = nch * 32
    target = row_blocks or min(4096, max(512, N // 256))
    want = max(1, min(-(-target // -(-nch // 4)), max(1, T // 16)))
    P = min(n_blocks, T) if n_blocks else 1
    S = max(1, -(-want // P))
    R = 0
    for p in range(P):
        n = T * (p + 1) // P - T * p // P
        R += min(S, n) if n > S else max(n, 1)
    bup, ks = -(-M // 64), KP // 16
    bq = nch * (2 * ks * 2 * 64 + 8) * 16
    cqe, cqw = (ks * 2 * 64 + 8) * 16, KP // 32 * 2 * 2 * 64 * 16
    t = 4 + M * K * 4 + K * N * 4 + bq + 2 * KP * 4 + KP * KP * 8 + bup * NP * 8 + KP * KP * 8 + KP * Mpad * 8
    t += min(T, 256) * NP * 8 + KP * N * 4 + T * (cqe + cqw) + 2 * KP * 4 + R * KP * Mpad * 4 + (R + 1) * 8
    t += -(-N // 128) * 8 + (1 << 16) * 8 + 8 + 8
    if refresh > 1:
        t += M * N * 4 + bq + T * cqe
    return t


@pytest.mark.parametrize("seed", range(4))
def test_splits_need_no_more_memory(seed):
    rng = random.Random(seed)
    for _ in range(300):
        M = max(17, int(round(2 ** rng.uniform(4.1, 14))))
        N = max(1, int(round(2 ** rng.uniform(0, 20))))
        K = rng.randint(1, min(64, M, N))
        o = did.did_default_opts()
        o.borrow_x = 1
        o.n_blocks = rng.choice([0, 0, 1, 4, 64])
        o.row_blocks = rng.choice([0, 0, 512, 8192])
        o.refresh_every = rng.choice([1, 1, 10])
        got = did.did_mem_estimate(M, N, K, o)
        assert got <= _unsplit_bytes(M, N, K, o.n_blocks, o.row_blocks, o.refresh_every), (M, N, K, o.n_blocks, o.row_blocks)
