"""The packet size of small launches, read from the header of the stored-list
pool: 16 rays where rays are traced through the BVH, 64 for brute force (whose
packets each test every Gaussian, so smaller ones only repeat the work) and for
the paper variant."""

import numpy as np
import pytest
import torch

from synthetic import scenes
from synthetic.cameras import look_at_camera, pinhole_rays

pytestmark = pytest.mark.gpu


def _log2_packet(state, n):
    a = lambda x: (x + 255) // 256 * 256
    pool = a(a(a(16 * n) + 16 * n) + 16 * n)
    return int(state.view(torch.uint8)[pool + 12:pool + 16].view(torch.int32).item())


@pytest.mark.parametrize("flags,log2", [(0, 4), (1, 6), (16, 6)])
def test_packet_size_of_a_small_launch(flags, log2):
    print("case packet size", flags, flush=True)
    import tests._gpu as G
    from paper_2501_19196_amd import renderer as R
    sc = scenes.scene_config1(n=400)
    o, d = pinhole_rays(look_at_camera((0, 0, -3), (0, 0, 0), (0, 1, 0), 40, 24))
    views, n = [(0, 40, 24)], o.shape[0]
    ref, _, _, (bvh, g, rays) = G.render(sc, o, d, R.Params(), views=views)
    p = R.Params(hit_list=256, max_hits=128, flags=flags)
    out, st, status, _ = G.render(sc, o, d, p, views=views, bvh=bvh, g=g)
    assert status == 0
    np.testing.assert_array_equal(out, ref)
    assert _log2_packet(st, n) == log2
    lists = R.hit_lists(rays, p, st, cap=128)
    np.testing.assert_array_equal(lists["stored"], lists["count"])
    grad = torch.ones(n, 3, device="cuda")
    a = R.render_bwd(bvh, g, rays, p, grad, st)
    p0 = R.Params(max_hits=128)
    _, st0, _, _ = G.render(sc, o, d, p0, views=views, bvh=bvh, g=g)
    b = R.render_bwd(bvh, g, rays, p0, grad, st0)
    if flags != 16:  # the same contributions summed in another order
        for x, y in zip(a, b):
            assert float((x - y).double().norm()) <= 1e-4 * float(y.double().norm())
