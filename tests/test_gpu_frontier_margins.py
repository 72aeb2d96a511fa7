"""The margins of the frontier forward's bounds, against the depth-first walk (a
call that bounds the traversal stack): a camera at the coordinate origin and a
scene far from it, where only the scene's size says how much the ray test
rounds, and rays that are not finite next to rays that are."""

import numpy as np
import pytest

from synthetic import scenes
from synthetic.cameras import look_at_camera, pinhole_rays

pytestmark = pytest.mark.gpu


def _g():
    import tests._gpu as G
    from paper_2501_19196_amd import renderer as R
    return G, R


def _edge_on(seed, n, dist):
    """Flat Gaussians whose plane holds the z axis up to a hundredth, met by it anywhere inside or near the rim."""
    rng = np.random.default_rng(seed)
    sc = scenes.random_scene(seed, n)
    ph, tilt, psi = rng.uniform(0, 2 * np.pi, n), 0.01 * rng.normal(size=n), rng.uniform(0, 2 * np.pi, n)
    nrm = np.stack([np.cos(ph) * np.cos(tilt), np.sin(ph) * np.cos(tilt), np.sin(tilt)], 1)
    a = np.stack([-np.cos(ph) * np.sin(tilt), -np.sin(ph) * np.sin(tilt), np.cos(tilt)], 1)
    b = np.cross(nrm, a)
    e1 = np.cos(psi)[:, None] * a + np.sin(psi)[:, None] * b
    R = np.stack([nrm, e1, np.cross(nrm, e1)], 2)  # columns: the body axes
    s = np.stack([np.full(n, 1e-5), 0.01 * np.exp(rng.uniform(0, 1, n)), 0.01 * np.exp(rng.uniform(0, 1, n))], 1)
    off = rng.normal(size=(n, 3))
    off *= (np.sqrt(11.3449) * rng.uniform(0, 1.3, n) / np.linalg.norm(off, axis=1))[:, None]
    mean = np.einsum("nij,nj->ni", R, off * s)
    mean[:, 2] += dist * rng.uniform(0.5, 1.5, n)
    w = 0.5 * np.sqrt(np.maximum(1e-12, 1 + R[:, 0, 0] + R[:, 1, 1] + R[:, 2, 2]))
    q = np.stack([w, (R[:, 2, 1] - R[:, 1, 2]) / (4 * w), (R[:, 0, 2] - R[:, 2, 0]) / (4 * w),
                  (R[:, 1, 0] - R[:, 0, 1]) / (4 * w)], 1)
    for name, v in (("mean", mean), ("scale", s), ("quat", q / np.linalg.norm(q, axis=1, keepdims=True))):
        getattr(sc, name)[:] = np.float32(v)
    sc.opacity[:] = np.float32(3e-4)
    return sc


@pytest.mark.parametrize("direction", [(0, 0, 1), (1e-9, 0, 1), (0, 0, -1)])
def test_axis_ray_from_the_origin_meets_every_flat(direction):
    """One ray through 8000 flats 5 to 15 thousand units away: the hits are the walk's, in number and effect."""
    print("case axis ray", direction, flush=True)
    G, R = _g()
    sc = _edge_on(11, 8000, 1e4)
    if direction[2] < 0:
        sc.mean[:, 2] *= -1
        sc.quat[:, 3] *= -1  # mirrored in z: the rotation's y and x parts turn round
        sc.quat[:, 0] *= -1
    o, d = np.zeros((1, 3), np.float32), np.float32([direction])
    kw = dict(max_hits=0, eps1=0.0)
    for lists in (0, 64):
        ref, s0, st0, (bvh, g, rays) = G.render(sc, o, d, R.Params(stack_depth=64, hit_list=lists, **kw))
        out, s1, st1, _ = G.render(sc, o, d, R.Params(hit_list=lists, **kw), bvh=bvh, g=g)
        assert st0 == 0 and st1 == 0
        if lists:
            a = R.hit_lists(rays, R.Params(hit_list=lists, **kw), s1, cap=8)["count"]
            b = R.hit_lists(rays, R.Params(hit_list=lists, **kw), s0, cap=8)["count"]
            print("hits", int(a[0]), int(b[0]), flush=True)
            assert b[0] > 4000
            np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(out, ref)
        np.testing.assert_array_equal(G.colour_state(s1, 1), G.colour_state(s0, 1))


def test_rays_that_are_not_finite_leave_the_others_alone():
    print("case non-finite rays", flush=True)
    G, R = _g()
    sc = scenes.random_scene(12, 3000)
    o, d = pinhole_rays(look_at_camera((0, 0, -3), (0, 0, 0), (0, 1, 0), 32, 32))
    o, d = o.copy(), d.copy()
    inf, nan = np.float32(np.inf), np.float32(np.nan)
    o[5, 0], o[40, 2], o[77, 1] = inf, -inf, nan
    d[100, 0], d[140, 2], d[180], d[220, 2] = nan, inf, 0.0, -inf
    ref, s0, st0, (bvh, g, _) = G.render(sc, o, d, R.Params(stack_depth=64))
    out, s1, st1, _ = G.render(sc, o, d, R.Params(), bvh=bvh, g=g)
    assert st0 == 0 and st1 == 0
    np.testing.assert_array_equal(out, ref)
    np.testing.assert_array_equal(G.colour_state(s1, 1024), G.colour_state(s0, 1024))
    good = np.ones(1024, bool)
    good[[5, 40, 77, 100, 140, 180, 220]] = False
    o2, d2 = pinhole_rays(look_at_camera((0, 0, -3), (0, 0, 0), (0, 1, 0), 32, 32))
    all_good, _, _, _ = G.render(sc, o2, d2, R.Params(), bvh=bvh, g=g)
    np.testing.assert_array_equal(out[good], all_good[good])
