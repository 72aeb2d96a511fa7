"""The frontier forward against the depth-first walk (a call that bounds the
traversal stack takes the walk) and brute force: the same hits in the same
order, so images, final transmittances and stored lists agree bit for bit.
The cases sit where the frontier kernel decides something: the packet size
(launches of 98304 rays and one more; 4-ray packets where the Gaussians far
outnumber the rays), rays of one packet along several axes, bundles too wide
for it, slopes of exactly 0, a camera inside the scene, depth limits, buffers
that overflow (so rays are traced in rounds), and leaf pools that do."""

import numpy as np
import pytest
import torch

from synthetic import scenes
from synthetic.cameras import look_at_camera, pinhole_rays

pytestmark = pytest.mark.gpu


def _g():
    import tests._gpu as G
    from paper_2501_19196_amd import renderer as R
    return G, R


def _same(sc, o, d, views=None, t_max=None, kbufs=(0, 16, 32), max_hits=512, lists=True, **kw):
    G, R = _g()
    cap = 256 if lists else 0
    ref, st0, s0, (bvh, g, rays) = G.render(sc, o, d, R.Params(stack_depth=64, hit_list=cap, max_hits=max_hits, **kw),
                                            views=views, t_max=t_max)
    assert s0 == 0
    n = o.shape[0]
    c0 = G.colour_state(st0, n)
    sel = np.unique(np.linspace(0, n - 1, 400).astype(np.int64))
    l0 = R.hit_lists(rays, R.Params(stack_depth=64, hit_list=cap, max_hits=max_hits, **kw), st0, cap=256, select=sel) \
        if lists else None
    for kbuf in kbufs:
        p = R.Params(kbuf=kbuf, hit_list=cap, max_hits=max_hits, **kw)
        out, st, s, _ = G.render(sc, o, d, p, views=views, t_max=t_max, bvh=bvh, g=g)
        assert s == 0
        np.testing.assert_array_equal(out, ref, err_msg=f"kbuf {kbuf}")
        np.testing.assert_array_equal(G.colour_state(st, n), c0, err_msg=f"kbuf {kbuf}")
        if lists:
            l1 = R.hit_lists(rays, p, st, cap=256, select=sel)
            full = (l0["stored"] == l0["count"]) & (l1["stored"] == l1["count"])
            np.testing.assert_array_equal(l1["count"], l0["count"])
            np.testing.assert_array_equal(l1["ids"][full], l0["ids"][full])
    return ref


def _camera(w, h, eye=(0, 0, -3), at=(0, 0, 0), up=(0, 1, 0)):
    return pinhole_rays(look_at_camera(eye, at, up, w, h))


@pytest.mark.parametrize("n,w,h", [(1, 9, 7), (2, 9, 7), (3, 33, 17), (64, 65, 63), (2000, 251, 187)])
def test_small_scenes_with_a_centre_column(n, w, h):
    """Odd widths: the centre column's slope is exactly 0."""
    print("case small", n, w, h, flush=True)
    o, d = _camera(w, h)
    _same(scenes.random_scene(90 + n, n), o, d, views=[(0, w, h)])


@pytest.mark.parametrize("n,w,h", [(20000, 384, 256), (20000, 331, 297), (2048, 331, 297), (2049, 331, 297), (98306, 331, 297), (98307, 331, 297)])
def test_packet_size_boundary(n, w, h):
    """98304 rays take 16-ray packets, 98307 rays 64-ray ones unless there are as many Gaussians,
    and up to 2048 Gaussians are walked there."""
    print("case packet size", n, w, h, flush=True)
    o, d = _camera(w, h, eye=(0, 0, -4))
    _same(scenes.scene_config2(seed=91, n=n), o, d, views=[(0, w, h)], kbufs=(0,))


def test_four_ray_packets_without_lists():
    print("case 4-ray packets", flush=True)
    o, d = _camera(63, 41, eye=(0, -7, 3.5), at=(0, 0, 0.5), up=(0, 0, 1))
    _same(scenes.scene_config4(seed=92, n=60000), o, d, views=[(0, 63, 41)], lists=False)


def test_overflowing_buffers_and_pools():
    """Large overlapping Gaussians: more hits pend than a buffer holds, and more leaves than the pool."""
    print("case overflow", flush=True)
    sc = scenes.random_scene(93, 30000, box=0.6, scale_lo=0.05, scale_hi=0.2)
    sc.opacity[:] = np.float32(0.02)
    o, d = _camera(64, 48)
    _same(sc, o, d, views=[(0, 64, 48)], max_hits=0)


def test_camera_inside_and_limits():
    print("case inside", flush=True)
    sc = scenes.scene_config4(seed=94, n=30000)
    o, d = _camera(120, 90, eye=(0.5, 0.3, 0.9), at=(2, 1, 1), up=(0, 0, 1))
    _same(sc, o, d, views=[(0, 120, 90)])
    rng = np.random.default_rng(94)
    t_max = np.float32(rng.uniform(0.0, 3.0, size=o.shape[0]))
    t_max[::7] = -np.inf
    t_max[::11] = np.inf
    _same(sc, o, d, views=[(0, 120, 90)], t_max=t_max, t_min=0.25)


def test_incoherent_rays_in_one_packet():
    """Random origins and directions (not unit): several axes per packet, and bundles left to the walk."""
    print("case incoherent", flush=True)
    rng = np.random.default_rng(95)
    sc = scenes.random_scene(95, 3000)
    o = np.float32(rng.uniform(-2, 2, size=(1000, 3)))
    d = np.float32(rng.normal(size=(1000, 3)) * rng.uniform(0.1, 5.0, size=(1000, 1)))
    d[::50] = np.float32([0, 0, 2])
    d[1::50] = np.float32([0, -3, 0])
    ref = _same(sc, o, d)
    # two groups in every packet, one of them with depth limits
    o3, d3 = _camera(64, 32)
    d3[1::2] = np.float32([[1, 0.2, 0.1]]) + 0.05 * np.float32(rng.normal(size=(d3[1::2].shape)))
    t3 = np.where(np.arange(len(o3)) % 4 == 1, 2.0, np.inf).astype(np.float32)
    _same(sc, o3 * np.float32([1, 1, 0.3]), d3, views=[(0, 64, 32)], t_max=t3)
    G, R = _g()
    out, _, _, _ = G.render(sc, o, d, R.Params(flags=1))
    np.testing.assert_array_equal(out, ref)
    big = scenes.scene_config4(seed=96, n=100000)
    o2, d2 = _camera(640, 480, eye=(0, -7, 3.5), at=(0, 0, 0.5), up=(0, 0, 1))
    sel = rng.permutation(o2.shape[0])[:512]
    _same(big, o2[sel], d2[sel], kbufs=(0,))


def test_grazing_flats():
    """Edge-on flat Gaussians, whose entry distance rounds the most."""
    print("case grazing", flush=True)
    sc = scenes.random_scene(97, 4000, box=0.8, flat_frac=1.0, scale_lo=0.05, scale_hi=0.2)
    o, d = _camera(96, 80, eye=(0.0, 0.02, -3.0))
    _same(sc, o, d, views=[(0, 96, 80)])
