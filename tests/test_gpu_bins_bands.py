"""Grids of more than 768 bins are cut into bands of bin rows.  Views of one
band, of two and of nine in one batch give what they give alone, with
rectangles of a tile up to the whole image (which lie in every band); and the
bin scatter of such a grid takes a small part of its frame: by one wave a
chunk with its cursors in the count table it took ten times the blend."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


def test_views_of_several_bands_in_one_batch():
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    sc = dict(scenes.make_scene("C1", n=3000, seed=12, sh_degree=0))
    rng = np.random.default_rng(12)
    sc["log_scales"] = (sc["log_scales"] + rng.uniform(-2.0, 3.5, 3000)).astype(np.float32)
    dev = gs.scene_to_device(sc)
    cams = [scenes.default_camera(W, H) for W, H in ((640, 480), (6144, 2064), (32768, 2064), (1040, 12304))]
    r = gs.Renderer(0)
    try:
        outs = r.render_batched(dev, cams)
        torch.cuda.synchronize()
        for cam, out in zip(cams, outs):
            one = gs.Renderer(0)
            try:
                want = one.render(dev, cam, cam["width"], cam["height"])
                torch.cuda.synchronize()
                for k in want:
                    assert torch.equal(out[k].view(torch.int32), want[k].view(torch.int32)), (cam["width"], k)
            finally:
                one.close()
    finally:
        r.close()


@pytest.mark.parametrize("W,H,n,grow", [(9216, 9216, 300_000, -2.0), (16384, 8192, 100_000, -1.0)])
def test_scatter_of_a_large_grid_is_a_part_of_its_frame(W, H, n, grow):
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    sc = dict(scenes.make_scene("C3", n=n, seed=2, sh_degree=0))
    sc["log_scales"] = (sc["log_scales"] + np.float32(grow)).astype(np.float32)
    dev, cam = gs.scene_to_device(sc), scenes.default_camera(W, H)
    r = gs.Renderer(0)
    try:
        r.set_profiling(True)
        best = None
        for _ in range(5):
            r.render(dev, cam, W, H)
            t = r.stage_times()
            best = t if best is None or t["bin_row_scatter"] < best["bin_row_scatter"] else best
        assert best["bin_row_scatter"] < best["blend"], best
    finally:
        r.close()
