"""The depth order at the edges of the sort's shapes: one launch (up to 4096
keys a view, in steps of 1024), five launches (up to 98304 keys over all
views), two per pass up to 2.5M keys and three beyond, with the wide parts from
800000 on; packed rectangles and grids wider than 255 tiles; depths that are mostly distinct, in
a few values (stable ties), and of Gaussians behind the camera.  The order
must be the stable sort of the keys by depth, then index: the lists of one
large tile hold every visible Gaussian in that order."""
import numpy as np
import pytest

import scenes

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


def order_of(lists, t):
    off = lists["tile_offsets"].cpu().numpy().view(np.uint32)
    return lists["values"].cpu().numpy().view(np.uint32)[off[t]:off[t + 1]]


@pytest.mark.parametrize("views,n,width,items", [
    (1, 1, 32, 8), (1, 1023, 32, 8), (1, 1025, 32, 4), (2, 2049, 32, 8), (1, 4096, 4112, 8), (3, 4097, 32, 16),
    (1, 20000, 4112, 8), (1, 98304, 32, 8), (1, 98305, 32, 8), (3, 40000, 32, 4), (1, 600001, 32, 4),
    (1, 600001, 32, 8), (1, 600001, 32, 16), (2, 400001, 32, 8), (1, 2500000, 32, 8), (1, 2500001, 32, 8),
    (1, 2500001, 32, 4),
])
def test_depth_order(views, n, width, items):
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    rng = np.random.default_rng(n + views)
    sc = dict(scenes.make_scene("C1", n=n, seed=3, sh_degree=0))
    means = np.zeros((3, n), np.float32)
    means[2] = rng.uniform(-1.0, 9.0, n)                     # some behind the camera or at it
    few = rng.random(n) < 0.5
    means[2, few] = rng.integers(1, 9, int(few.sum()))        # ties
    sc["means"] = means
    sc["log_scales"] = np.full_like(sc["log_scales"], -2.0)
    cam = dict(scenes.default_camera(width, 16), t=np.zeros(3, np.float32))
    r = gs.Renderer(0)
    try:
        r.set_tuning(sort_items=items)
        dev = gs.scene_to_device(sc, 0)
        if views == 1:
            r.render(dev, cam, width, 16)
        else:
            r.render_batched(dev, [cam] * views)
        torch.cuda.synchronize()
        lists = r.lists()
        keys = r.projection()["depth_key"].cpu().numpy().view(np.uint32)
        touched = r.projection()["tiles_touched"].cpu().numpy().view(np.uint32)
        torch.cuda.synchronize()
    finally:
        r.close()
    tiles = (width + 15) // 16
    mid = tiles // 2
    assert n < 1000 or (touched > 0).mean() > 0.5
    for v in range(views):
        # every Gaussian lies on the optical axis: the middle tile lists all that are on screen
        ids = np.arange(v * n, (v + 1) * n)[touched[v * n:(v + 1) * n] > 0]
        want = ids[np.argsort(keys[ids], kind="stable")]
        assert np.array_equal(order_of(lists, v * tiles + mid), want.astype(np.uint32))
