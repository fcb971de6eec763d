"""tile_leaves bounds a tile's work: it makes tiles smaller, never larger than
those that the launch's work calls for."""
import pytest

pytestmark = pytest.mark.gpu

OFF = 0xFFFFFFFF


@pytest.mark.parametrize("x", [10**9, 10**12, 10**15])
def test_a_large_bound_changes_nothing(pc, x):
    print("case: tile bound", x, flush=True)
    r = pc.pi_count_ex(x)
    for bound in (1 << 22, OFF - 1):
        b = pc.pi_count_ex(x, tile_leaves=bound)
        assert (b.pi, b.tiles) == (r.pi, r.tiles), bound
    small = pc.pi_count_ex(x, tile_leaves=1 << 12)
    assert small.pi == r.pi and small.tiles >= r.tiles
    off = pc.pi_count_ex(x, tile_leaves=OFF)
    assert (off.pi, off.tiles) == (r.pi, r.segments)


@pytest.mark.parametrize("n_small,large", [(40, []), (1500, []), (900, [10**12 + 39]),
                                           (200, [10**11, 10**13, 10**14])])
def test_rounds_of_whole_and_cut_queries(pc, n_small, large):
    # one-row queries below a workgroup's share of the round are not planned
    import random
    print("case: mixed round", n_small, large, flush=True)
    rng = random.Random(n_small)
    xs = [int(10 ** rng.uniform(6.1, 9.0)) for _ in range(n_small)] + large
    rng.shuffle(xs)
    got = list(pc.pi_count_batch(xs))
    assert got == [pc.pi_count(x) for x in xs]
    assert list(pc.pi_count_batch(xs, tile_leaves=1 << 12)) == got
