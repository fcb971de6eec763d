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
