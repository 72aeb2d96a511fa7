"""rs_autotune times a kernel once: candidates that differ only in a knob which
their launch leaves aside carry the same time, so noise does not choose."""

import numpy as np
import pytest

from synthetic import scenes
from synthetic.cameras import look_at_camera, pinhole_rays

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,hit_list,stack_depth", [(400, 300, 64, 0), (400, 300, 0, 0), (96, 64, 64, 0), (400, 300, 64, 64)])
def test_twins_share_a_time_and_the_adjoint_reads_its_own_state(w, h, hit_list, stack_depth):
    print("case twins", w, h, hit_list, stack_depth, flush=True)
    import tests._gpu as G
    from paper_2501_19196_amd import renderer as R
    sc = scenes.scene_config2(seed=21, n=6000)
    o, d = pinhole_rays(look_at_camera((0, 0, -4), (0, 0, 0), (0, 1, 0), w, h))
    p = R.Params(hit_list=hit_list, stack_depth=stack_depth)
    _, st, status, (bvh, g, rays) = G.render(sc, o, d, p, views=[(0, w, h)])
    rng = np.random.default_rng(22)
    grad = G.dev(np.float32(rng.normal(size=(w * h, 3))))
    pf, pb, rows = R.autotune(bvh, g, rays, p, grad_rgb=grad, reps=2)
    assert status == 0 and len(rows) == 20
    small = w * h <= 98304
    keys = lambda k: k if stack_depth else 16 if k <= 16 else 24 if k <= 24 else 32
    for name, key in (("ms_fwd", lambda r: keys(r["kbuf"])), ("ms_bwd", lambda r: r["kbuf"])):
        times = {}
        for r in rows:
            assert r[name] > 0
            times.setdefault((key(r), r["persistent"], 0 if small else r["tile_width"]), set()).add(r[name])
        assert all(len(t) == 1 for t in times.values()), (name, times)
        assert len({t for s in times.values() for t in s}) > 1
    # the chosen shapes render and differentiate as the untuned ones do
    if hit_list:
        assert R.read_status(bvh) == 0
    ref = R.render_bwd(bvh, g, rays, p, grad, st)
    _, st2, _, _ = G.render(sc, o, d, pb, views=[(0, w, h)], bvh=bvh, g=g)
    for x, y in zip(R.render_bwd(bvh, g, rays, pb, grad, st2), ref):  # another order of the same sums
        assert float((x - y).double().norm()) <= 1e-4 * float(y.double().norm())
