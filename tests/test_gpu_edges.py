"""Edges of the sieve's bitmap, of its tiles and of the easy leaves' ranges:
every component of the decomposition against the oracle, exactly."""
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

SPAN = 983040  # integers of a segment of 2^18 bits (8 bits per 30 integers)


def check(pc, x, y, **kw):
    r = pc.decompose(x, y, **kw)
    o = O.decompose(x, y, 6, hard=O.HARD_SIEVE)
    got = (r.a, r.c, r.s1, r.s2_trivial, r.s2_easy, r.s2_hard, r.p2, r.n_easy, r.n_hard)
    want = (o.a, o.c, o.s1, o.s2t, o.s2e, o.s2h, o.p2, o.n_easy, o.n_hard)
    assert got == want, (x, y, kw)


@pytest.mark.parametrize("lo,hi", [(8, 64), (64, 125), (125, 180)])
def test_every_y_of_tiny_x(pc, lo, hi):
    # wheels of 1 to 6 primes (below 3 the sieve's bitmap does not apply)
    print("case: tiny", lo, hi, flush=True)
    for x in range(lo, hi):
        for y in range(O.icbrt(x), O.isqrt(x) + 1):
            check(pc, x, y)


@pytest.mark.parametrize("segments", [1, 2, 9])
@pytest.mark.parametrize("off", [-1, 0, 1, 29])
def test_range_ends_at_a_segment(pc, segments, off):
    z = segments * SPAN + off
    y = 10007
    print("case: z", z, flush=True)
    check(pc, z * y, y)
    check(pc, z * y + y - 1, y)


@pytest.mark.parametrize("tile_leaves", [1, 300, 5000])
@pytest.mark.parametrize("x,y", [(10**9, 1000), (10**11, 4641), (10**12 + 39, 31000)])
def test_tiles_of_few_columns(pc, x, y, tile_leaves):
    # down to one column per tile: each clears every earlier column on its own
    print("case: tiles", x, y, tile_leaves, flush=True)
    check(pc, x, y, tile_leaves=tile_leaves)


@pytest.mark.parametrize("x", [10**6 - 1, 10**8 + 7, 2**32, 10**10])
def test_easy_ranges_over_y(pc, x):
    # the common range of singles and groups and its ends move with y
    lo, hi = O.icbrt(x), O.isqrt(x)
    ys = sorted({lo, lo + 1, 2 * lo, 3 * lo + 1, (lo + hi) // 2, hi - 1, hi})
    print("case: easy", x, ys, flush=True)
    for y in ys:
        if lo <= y <= hi:
            check(pc, x, y)


@pytest.mark.parametrize("alpha,apart", [(4.0, True), (5.0, False), (0.0, False)])
def test_leaves_in_one_launch(pc, alpha, apart):
    # S1 and the easy leaves share a launch up to 512 segments unless times are asked for
    x = 10**14
    print("case: leaves in one launch", alpha, flush=True)
    r = pc.pi_count_ex(x, alpha=alpha)  # reads times: apart
    assert (r.segments > 512) == apart
    assert pc.pi_count(x, alpha) == r.pi == 3204941750802  # Table 1
