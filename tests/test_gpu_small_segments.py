"""One-wavefront segments cut into column tiles, on their own and followed by
workgroup segments, against the oracle."""
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kib", [4, 8])
@pytest.mark.parametrize("tile_leaves", [0, 1, 300, 0xFFFFFFFF])
@pytest.mark.parametrize("x,y,span", [(10**9, 1000, 4), (10**9, 1000, 5000), (10**11, 4641, 60),
                                      (10**12 + 39, 31000, 30), (10**12, 10000, 1)])
def test_tiles_of_small_segments(pc, x, y, span, tile_leaves, kib):
    print("case: small segments", x, y, span, tile_leaves, kib, flush=True)
    o = O.decompose(x, y, 6, hard=O.HARD_SIEVE)
    for flags in (0, pc.FLAG_TWO_PASS):
        r = pc.decompose(x, y, small_span=span, small_kib=kib, tile_leaves=tile_leaves, flags=flags)
        assert r.small_segments > 0
        assert (r.pi, r.s2_hard, r.n_hard, r.p2) == (o.pi, o.s2h, o.n_hard, o.p2), flags
        if tile_leaves == 0xFFFFFFFF:
            assert r.tiles == r.segments
