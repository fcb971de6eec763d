"""Windows of the sieve whose leaves all fall into one wavefront's region (z
below a region's integers), many pieces of 64 of them, on every shape."""
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [dict(segment_kib=32, wg_size=256), dict(segment_kib=32, wg_size=512),
                                 dict(segment_kib=64, wg_size=512), dict(segment_kib=64, wg_size=1024),
                                 dict(small_span=1000, small_kib=4), dict(small_span=1000, small_kib=8)],
                         ids=lambda c: "-".join(str(v) for v in c.values()))
@pytest.mark.parametrize("x,y", [(10**6, 100), (10**7, 215), (5 * 10**7, 368), (10**9, 20000),
                                 (10**10, 100000)])
def test_leaves_of_one_region(pc, x, y, cfg):
    print("case: one region", x, y, cfg, flush=True)
    for flags in (0, pc.FLAG_TWO_PASS, pc.FLAG_NO_BATCH_LARGE):
        r = pc.decompose(x, y, flags=flags, tile_leaves=0xFFFFFFFF, **cfg)
        o = O.decompose(x, y, 6, hard=O.HARD_SIEVE)
        assert (r.pi, r.s2_hard, r.n_hard, r.p2) == (o.pi, o.s2h, o.n_hard, o.p2), flags
