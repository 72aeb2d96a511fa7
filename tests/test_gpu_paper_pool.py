"""The paper variant's pool at its documented size: 5/4 max_hits + 8 slots per
ray never run out with full 64-ray packets, since a packet stores at most
max_hits rows, (64 + 2) max_hits slots."""

import numpy as np
import pytest

from synthetic import scenes
from synthetic.cameras import look_at_camera, pinhole_rays

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kbuf,max_hits", [(0, 256), (16, 256), (16, 64)])
def test_documented_pool_suffices(kbuf, max_hits):
    """A translucent fog whose rays all reach max_hits, in full packets."""
    print("case paper pool", kbuf, max_hits, flush=True)
    import tests._gpu as G
    from paper_2501_19196_amd import renderer as R
    sc = scenes.random_scene(93, 8000, box=0.6, scale_lo=0.03, scale_hi=0.1)
    sc.opacity[:] = np.float32(0.02)
    o, d = pinhole_rays(look_at_camera((0, 0, -3), (0, 0, 0), (0, 1, 0), 64, 64, fov_y_deg=20))
    views, n = [(0, 64, 64)], o.shape[0]
    p = R.Params(max_hits=max_hits, hit_list=5 * max_hits // 4 + 8, flags=16, eps2=1e-3, kbuf=kbuf)
    _, state, status, (bvh, g, rays) = G.render(sc, o, d, p, views=views)
    assert status == 0
    lists = R.hit_lists(rays, p, state, cap=max_hits)
    assert (lists["count"] == max_hits).all()
    np.testing.assert_array_equal(lists["stored"], lists["count"])
    # rows and slots of the packets, from the counting variant
    q = R.Params(**{**p.__dict__, "flags": p.flags | 8})
    _, _, status, (bvh2, _, _) = G.render(sc, o, d, q, views=views, g=g)
    c = R.read_counters(bvh2)
    print(c, flush=True)
    assert status == 0
    assert c["packets"] == n // 64
    assert c["list_rows"] <= max_hits * c["packets"]
    assert c["list_slots"] <= (64 + 2) * max_hits * c["packets"]
    # the variant's lists are those of the plain render here (no ray stops at eps1)
    p0 = R.Params(max_hits=max_hits, hit_list=4 * max_hits, kbuf=kbuf)
    _, st0, _, _ = G.render(sc, o, d, p0, views=views, bvh=bvh, g=g)
    l0 = R.hit_lists(rays, p0, st0, cap=max_hits)
    np.testing.assert_array_equal(l0["stored"], l0["count"])
    np.testing.assert_array_equal(l0["ids"], lists["ids"])
