"""Frames whose bin entries outgrow the buffers that earlier frames on the
context left: the entries are scattered again into grown buffers, which must
give what a fresh context gives, bit for bit.  Grids of one band of bin rows,
of two and of nine: no scatter may depend on what an earlier one left."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


def frame(r, sc, W, H, **kw):
    import torch
    import paper_2607_15951_amd as gs
    out = r.render(gs.scene_to_device(sc), scenes.default_camera(W, H), W, H, **kw)
    torch.cuda.synchronize()
    return {k: v.view(torch.int32).clone() for k, v in out.items()}, r.list_info()["num_pairs"]


@pytest.mark.parametrize("W,H,n", [
    (641, 487, 20011),
    (12288, 1088, 800),   # 864 bins
    (32768, 2064, 600),   # 4352 bins
])
def test_grown_frames_equal_a_fresh_context(W, H, n):
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    base = dict(scenes.make_scene("C1", n=n, seed=W, sh_degree=0))

    def scaled(d):
        return dict(base, log_scales=(base["log_scales"] + np.float32(d)).astype(np.float32))

    r = gs.Renderer(0)
    try:
        r.render(gs.scene_to_device(scenes.make_scene("C1", n=50, seed=1, sh_degree=0)),
                 scenes.default_camera(64, 64), 64, 64)   # little room for the next frame
        pairs = []
        for step, kw in ((0.0, {}), (1.5, {}), (1.5, {"reuse_lists": True}), (0.5, {}), (2.5, {})):
            got, k = frame(r, scaled(step), W, H, **kw)
            pairs.append(k)
            fresh = gs.Renderer(0)
            try:
                want, k0 = frame(fresh, scaled(step), W, H)
            finally:
                fresh.close()
            assert k == k0
            for key in want:
                assert torch.equal(got[key], want[key]), (step, kw, key)
        assert pairs[1] > 1.25 * pairs[0] and pairs[4] > 1.25 * pairs[1]
    finally:
        r.close()
