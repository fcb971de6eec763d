"""Wheels of 3 to 5 primes (y < 13) on every shape of the sieve.  Such a wheel
has a column to cross only where y + 1 is the next prime and z >= (y + 1)^2;
its crossing removes multiples over the whole segment, however small z is."""
import functools

import pytest

import oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [(32, 256), (32, 512), (64, 512), (64, 1024)]


@functools.lru_cache(maxsize=None)
def want(x, y):
    o = O.decompose(x, y, 6, hard=O.HARD_SIEVE)
    return (o.pi, o.a, o.c, o.s1, o.s2t, o.s2e, o.s2h, o.p2, o.n_easy, o.n_hard)


def check(pc, x, y, **kw):
    r = pc.decompose(x, y, **kw)
    got = (r.pi, r.a, r.c, r.s1, r.s2_trivial, r.s2_easy, r.s2_hard, r.p2, r.n_easy, r.n_hard)
    assert got == want(x, y), (x, y, kw)


@pytest.mark.parametrize("kib,wg", SHAPES)
@pytest.mark.parametrize("two_pass", [False, True])
@pytest.mark.parametrize("y,lo,hi", [(6, 294, 342), (10, 1210, 1330), (12, 2028, 2196)])
def test_the_one_column(pc, y, lo, hi, two_pass, kib, wg):
    print("case: one column", y, two_pass, kib, wg, flush=True)
    flags = pc.FLAG_TWO_PASS if two_pass else 0
    for x in range(lo, hi + 1):
        check(pc, x, y, segment_kib=kib, wg_size=wg, flags=flags)


@pytest.mark.parametrize("kib,wg", SHAPES)
def test_every_y(pc, kib, wg):
    print("case: every y", kib, wg, flush=True)
    for x in range(180, 343):
        for y in range(O.icbrt(x), O.isqrt(x) + 1):
            check(pc, x, y, segment_kib=kib, wg_size=wg)
