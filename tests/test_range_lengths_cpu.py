"""The row pass's column ranges: W's float32 partials are summed over a range, so an instance
has at least ceil(row_blocks / slab groups) of them (ranges of 16 tiles where X is narrower),
never fewer for the sake of even launches.  Its scratch then holds at least that many partials
of W beside V's.  Runs on the CPU: did_mem_estimate touches no device."""

import random

import pytest

import paper_1802_08938_amd as did


def _least_bytes(M, N, K, n_blocks, row_blocks):
    """Device bytes with the fewest column ranges allowed and no room for anything else in the
    scratch of the partials (as given X, borrowed)."""
    KP = 32 if K <= 32 else 64
    NP, nch, T = KP * (KP + 1) // 2, -(-M // 32), -(-N // 32)
    Mpad, slab_groups = nch * 32, -(-nch // 4)
    want = -(-(row_blocks or min(4096, max(512, N // 256))) // slab_groups)
    want = max(1, min(want, max(1, T // 16)))
    P = min(n_blocks, T) if n_blocks else 1
    S = -(-want // P)
    R = sum(min(S, T * (p + 1) // P - T * p // P) for p in range(P))
    ks = KP // 16
    bq = nch * (2 * ks * 2 * 64 + 8) * 16
    cq = T * ((ks * 2 * 64 + 8) + KP // 32 * 2 * 2 * 64) * 16
    t = 4 + M * K * 4 + K * N * 4 + bq + 2 * KP * 4 + KP * KP * 8 + -(-M // 64) * NP * 8 + KP * KP * 8 + KP * Mpad * 8
    t += cq + 2 * KP * 4 + (R + 1) * 8 + -(-N // 128) * 8 + (1 << 16) * 8 + 8 + 8
    return t + R * K * Mpad * 4 + min(T, 256) * NP * 8


@pytest.mark.parametrize("M,N,K,n_blocks,row_blocks", [
    (33_000, 4000, 50, 0, 0),     # 258 slab groups: two ranges, not one
    (40_000, 1100, 10, 0, 0),     # 313 slab groups, X just wide enough for two
    (40_000, 16_000, 10, 0, 0),
    (5000, 7000, 50, 0, 0),       # 13 ranges of 40 slab groups
    (8000, 6000, 40, 0, 0),       # 9 of 63
    (5000, 4000, 64, 3, 511),     # an explicit target below two blocks per CU, three shards
    (1000, 9000, 33, 0, 700),
])
def test_ranges_of_tall_x(M, N, K, n_blocks, row_blocks):
    o = did.did_default_opts()
    o.borrow_x, o.n_blocks, o.row_blocks = 1, n_blocks, row_blocks
    assert did.did_mem_estimate(M, N, K, o) >= _least_bytes(M, N, K, n_blocks, row_blocks)


@pytest.mark.parametrize("seed", range(4))
def test_ranges_over_shapes(seed):
    rng = random.Random(seed)
    for _ in range(300):
        M = int(round(2 ** rng.uniform(4.1, 17)))
        N = int(round(2 ** rng.uniform(5, 20)))
        K = rng.randint(1, min(64, M, N))
        o = did.did_default_opts()
        o.borrow_x = 1
        o.n_blocks = rng.choice([0, 0, 1, 4, 64])
        o.row_blocks = rng.choice([0, 0, 300, 512, 700, 8192])
        if M <= 16 and K <= 8:  # the thin path
            continue
        got = did.did_mem_estimate(M, N, K, o)
        assert got >= _least_bytes(M, N, K, o.n_blocks, o.row_blocks), (M, N, K, o.n_blocks, o.row_blocks)
