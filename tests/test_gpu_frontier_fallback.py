"""What the frontier forward leaves to the walk: bundles that are too wide, leaves
tested in vain, rays of many rounds. They go on in the same packet, with the same
hits and no more of the list pool, and cost about what a walk does."""

import numpy as np
import pytest

from synthetic import scenes
from synthetic.cameras import look_at_camera, pinhole_rays

pytestmark = pytest.mark.gpu


def _g():
    import tests._gpu as G
    from paper_2501_19196_amd import renderer as R
    return G, R


def _same_lists(R, rays, pa, sa, pb, sb, cap):
    la, lb = R.hit_lists(rays, pa, sa, cap=cap), R.hit_lists(rays, pb, sb, cap=cap)
    np.testing.assert_array_equal(la["count"], lb["count"])
    np.testing.assert_array_equal(lb["stored"], lb["count"])
    np.testing.assert_array_equal(la["stored"], la["count"])
    np.testing.assert_array_equal(la["ids"], lb["ids"])


def test_a_group_left_to_the_walk_takes_no_second_pool():
    """Every packet holds eight rays of a camera and eight that span the scene along another axis: the second
    group is left to the walk after the first has stored its rows, and the pool is sized for one set of rows."""
    print("case two groups, lists", flush=True)
    G, R = _g()
    sc = scenes.scene_config4(seed=98, n=100000)
    o1, d1 = pinhole_rays(look_at_camera((0, -7, 3.5), (0, 0, 0.5), (0, 0, 1), 64, 32, fov_y_deg=25))
    rng = np.random.default_rng(98)
    n = o1.shape[0]
    o2 = np.float32(np.column_stack([np.full(n, -8.0), rng.uniform(-4, 4, n), rng.uniform(0, 3, n)]))
    d2 = np.float32(np.column_stack([np.ones(n), rng.uniform(-0.3, 0.3, (n, 2))]))
    o = np.concatenate([o1.reshape(-1, 8, 3), o2.reshape(-1, 8, 3)], axis=1).reshape(-1, 3)
    d = np.concatenate([d1.reshape(-1, 8, 3), d2.reshape(-1, 8, 3)], axis=1).reshape(-1, 3)
    pc = R.Params(hit_list=512, flags=8)
    _, _, s, (bvh, g, rays) = G.render(sc, o, d, pc)
    c = R.read_counters(bvh)
    per_ray = c["list_slots"] / (2 * n)
    print(c, "slots a ray", per_ray, flush=True)
    assert s == 0 and c["packets"] == 2 * n // 16
    # room for the rows, the last chunk of each packet (8 slots a ray) and what its chunks leave over
    p = R.Params(hit_list=int(np.ceil(1.15 * per_ray)) + 8)
    out, st, s, _ = G.render(sc, o, d, p, bvh=bvh, g=g)
    pw = R.Params(hit_list=512, stack_depth=64)
    ref, st0, s0, _ = G.render(sc, o, d, pw, bvh=bvh, g=g)
    assert s == 0 and s0 == 0
    np.testing.assert_array_equal(out, ref)
    _same_lists(R, rays, p, st, pw, st0, 512)


def _counts(R, G, sc, o, d, views, **kw):
    p = R.Params(**{**kw, "flags": 8})
    _, _, s, (bvh, _, _) = G.render(sc, o, d, p, views=views)
    assert s == 0
    return R.read_counters(bvh)


def test_wide_bundles_are_walked_early():
    """Parallel rays scattered over three units, sixteen a packet: the bundle holds a twentieth of the scene and
    few of its leaves meet a ray. The packets test about as many leaves as a walk does."""
    print("case wide bundles", flush=True)
    G, R = _g()
    sc = scenes.scene_config4(seed=98, n=30000)
    rng = np.random.default_rng(3)
    n = 1024
    c = np.repeat(rng.uniform(-2, 2, (n // 16, 2)), 16, 0)
    o = np.float32(np.column_stack([c + rng.uniform(-1.5, 1.5, (n, 2)), np.full(n, 6.0)]))
    d = np.float32(np.column_stack([rng.uniform(-0.02, 0.02, (n, 2)), -np.ones(n)]))
    a = _counts(R, G, sc, o, d, None, hit_list=128)
    b = _counts(R, G, sc, o, d, None, hit_list=128, stack_depth=64)
    print(a, b, flush=True)
    assert a["packets"] == b["packets"] == n // 16
    assert a["leaf_visits"] <= 2 * b["leaf_visits"]
    p, pw = R.Params(hit_list=128), R.Params(hit_list=128, stack_depth=64)
    out, st, s, (bvh, g, rays) = G.render(sc, o, d, p)
    ref, st0, s0, _ = G.render(sc, o, d, pw, bvh=bvh, g=g)
    assert s == 0 and s0 == 0
    np.testing.assert_array_equal(out, ref)
    _same_lists(R, rays, p, st, pw, st0, 128)


@pytest.mark.parametrize("w,h,wide", [(64, 64, False), (320, 320, True)])
def test_rays_of_many_rounds_go_on_in_the_walk(w, h, wide):
    """Large translucent Gaussians, 512 hits a ray: after the frontier's rounds (4 of a 64-ray packet, 8 of a
    16-ray one) the rays are walked from where they are, so there are that many rounds more than in a walk."""
    print("case many rounds", w, h, flush=True)
    G, R = _g()
    sc = scenes.random_scene(93, 3000, box=0.6, scale_lo=0.1, scale_hi=0.3)
    sc.opacity[:] = np.float32(0.02)
    o, d = pinhole_rays(look_at_camera((0, 0, -3), (0, 0, 0), (0, 1, 0), w, h, fov_y_deg=20))
    views = [(0, w, h)]
    a, b = _counts(R, G, sc, o, d, views), _counts(R, G, sc, o, d, views, stack_depth=64)
    print(a, b, flush=True)
    assert a["packets"] == b["packets"] == o.shape[0] // (64 if wide else 16)
    assert a["rounds"] > a["packets"] * (4 if wide else 8)  # the frontier's, then the walk's
    assert a["rounds"] <= b["rounds"] + a["packets"] * (4 if wide else 8)
    p, pw = R.Params(hit_list=768), R.Params(hit_list=768, stack_depth=64)
    out, st, s, (bvh, g, rays) = G.render(sc, o, d, p, views=views)
    ref, st0, s0, _ = G.render(sc, o, d, pw, views=views, bvh=bvh, g=g)
    assert s == 0 and s0 == 0
    np.testing.assert_array_equal(out, ref)
    sel = np.arange(0, o.shape[0], 97)
    la, lb = R.hit_lists(rays, p, st, cap=512, select=sel), R.hit_lists(rays, pw, st0, cap=512, select=sel)
    assert (lb["count"] == 512).mean() > 0.5
    for k in ("count", "stored", "ids"):
        np.testing.assert_array_equal(la[k], lb[k])


def test_secondary_sets_give_way_after_two_rounds():
    """A mirror floor and shadows seen in 96x96 pixels: the packets of reflected and shadow rays spread, and test
    about as many leaves in about as many rounds as a walk does, with its result."""
    print("case secondary sets", flush=True)
    G, R = _g()
    import torch
    sc = scenes.scene_config4(seed=98, n=500000)
    cam = look_at_camera((4.2, 4.2, 3), (0, 0, 0.5), (0, 0, 1), 96, 96)
    o, d = pinhole_rays(cam)
    quad = np.float32([[-3, -3, 0], [3, -3, 0], [3, 3, 0], [-3, 3, 0]])
    mesh = R.Mesh(G.dev(quad), G.dev(np.int32([[0, 1, 2], [0, 2, 3]])), G.dev(np.int32([1, 1])))
    mbvh, sh, g, rays = R.build_mesh_bvh(mesh), R.Shading(), G.gaussians(sc), G.rays_of(o, d, [(0, 96, 96)])
    got = []
    for depth in (0, 64):
        p = R.Params(hit_list=128, flags=8, stack_depth=depth)
        bvh = R.build_bvh(g, p)
        out, frame = R.render_mesh_fwd(bvh, mbvh, g, mesh, sh, rays, p)
        torch.cuda.synchronize()
        assert R.read_status(bvh) == 0
        lists = [R.mesh_hit_lists(rays, p, sh, frame, k, cap=512) for k in range(3)]
        got.append((out.cpu().numpy(), lists, R.read_counters(bvh)))
    (img, lists, c), (ref, ref_lists, cw) = got
    print(c, cw, flush=True)
    np.testing.assert_array_equal(img, ref)
    for a, b in zip(lists, ref_lists):
        np.testing.assert_array_equal(a["count"], b["count"])
        full = (a["stored"] == a["count"]) & (b["stored"] == b["count"])
        assert full.mean() > 0.9
        np.testing.assert_array_equal(a["ids"][full], b["ids"][full])
    assert c["packets"] == cw["packets"] == 3 * 24 * 24
    assert c["rounds"] <= cw["rounds"] + c["packets"]
    assert c["leaf_visits"] <= 1.25 * cw["leaf_visits"]


@pytest.mark.parametrize("w,h,views", [(96, 96, True), (97, 61, True), (1000, 1, False), (5, 3, True)])
def test_rows_of_small_packets_hold_four_steps(w, h, views):
    """A 16-ray packet ends a row after four steps (or a chunk), so its masks take few of its slots; the lists and
    the gradients are those of the traversal."""
    print("case four steps a row", w, h, flush=True)
    G, R = _g()
    sc = scenes.scene_config2(seed=99, n=20000)
    o, d = pinhole_rays(look_at_camera((0, 0, -4), (0, 0, 0), (0, 1, 0), w, h, fov_y_deg=35))
    vs = [(0, w, h)] if views else None
    p = R.Params(hit_list=512, flags=8)
    out, st, s, (bvh, g, rays) = G.render(sc, o, d, p, views=vs)
    c = R.read_counters(bvh)
    print(c, flush=True)
    assert s == 0
    assert c["list_slots"] == c["lane_composited"] + 2 * c["list_rows"]
    # a step has at least one hit; a row ends after four steps, or where a 128-slot chunk or the packet does
    assert c["list_rows"] <= c["lane_composited"] / 4 + c["list_slots"] / (128 - 16 - 2) + c["packets"]
    pw = R.Params(hit_list=512, stack_depth=64)
    ref, st0, s0, _ = G.render(sc, o, d, pw, views=vs, bvh=bvh, g=g)
    assert s0 == 0
    np.testing.assert_array_equal(out, ref)
    _same_lists(R, rays, p, st, pw, st0, 512)
    rng = np.random.default_rng(99)
    grad = G.dev(np.float32(rng.normal(size=(o.shape[0], 3))))
    a = R.render_bwd(bvh, g, rays, p, grad, st)
    p0 = R.Params()
    _, st1, _, _ = G.render(sc, o, d, p0, views=vs, bvh=bvh, g=g)
    b = R.render_bwd(bvh, g, rays, p0, grad, st1)
    for x, y in zip(a, b):  # sums of the same contributions in another order
        assert float((x - y).double().norm()) <= 1e-4 * float(y.double().norm())


def test_a_pool_of_the_mean_length_suffices_in_small_packets():
    """Mirror and shadow sets at 96x96, lists of 47 on average, a pool of 64 slots a ray: the lists are complete, as
    they are in 64-ray packets."""
    print("case pool reach", flush=True)
    G, R = _g()
    sc = scenes.scene_config4(seed=98, n=500000)
    o, d = pinhole_rays(look_at_camera((4.2, 4.2, 3), (0, 0, 0.5), (0, 0, 1), 96, 96))
    quad = np.float32([[-3, -3, 0], [3, -3, 0], [3, 3, 0], [-3, 3, 0]])
    mesh = R.Mesh(G.dev(quad), G.dev(np.int32([[0, 1, 2], [0, 2, 3]])), G.dev(np.int32([1, 1])))
    mbvh, sh, g, rays = R.build_mesh_bvh(mesh), R.Shading(), G.gaussians(sc), G.rays_of(o, d, [(0, 96, 96)])
    big = R.Params(hit_list=256)
    bvh = R.build_bvh(g, big)
    _, frame = R.render_mesh_fwd(bvh, mbvh, g, mesh, sh, rays, big)
    mean = sum(R.mesh_hit_lists(rays, big, sh, frame, k, cap=1)["count"].mean() for k in range(3)) / 3
    p = R.Params(hit_list=int(np.ceil(1.2 * mean)) + 4)
    print("mean list", mean, "slots", p.hit_list, flush=True)
    _, frame = R.render_mesh_fwd(bvh, mbvh, g, mesh, sh, rays, p)
    for k in range(3):
        lists = R.mesh_hit_lists(rays, p, sh, frame, k, cap=1)
        np.testing.assert_array_equal(lists["stored"], lists["count"])
