"""The lists over bins of tiles that the blend picks its entries from: grids at
the edges of what each kernel of the binning takes (one tile, cut bins, more
than 255 tiles a side, where the sort carries no rectangles, more bins than
four waves' cursors fill the LDS with, more than fit one wave's), with
rectangles of about a tile up to most of the grid.  Sampled tiles against the
oracle: image, final T, n_contrib (which is a list position) and the per-tile
list.  The second frame on a context, whose bins' edge follows the first's
pairs per Gaussian, and a frame with a pair capacity give the same bits."""
import numpy as np
import pytest

import oracle
import scenes
from parity import IMAGE_TOL, check_projection, gpu_render

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]
TILE = 16


@pytest.mark.parametrize("W,H,n,grow", [
    (16, 16, 1, 0.0),          # one tile, one Gaussian
    (16, 16, 700, 0.0),        # several batches and rounds' remainders
    (129, 65, 63, 2.5),        # 9 x 5 tiles: bins cut on both sides; fewer than a wave's Gaussians
    (641, 487, 3000, 2.0),     # large rectangles: bin by bin
    (641, 487, 20011, -1.5),   # about a tile each: entry by entry
    (333, 197, 40000, 0.0),    # 13K counts: one scan launch
    (4097, 33, 1500, 1.0),     # 257 tiles wide: rectangles gathered
    (6144, 2040, 900, 1.0),    # 768 bins of 8x8 tiles: the long rounds
    (12288, 1088, 800, 1.0),   # 864 bins of 8x8 tiles: more than 768
    (32768, 2064, 600, 1.0),   # 4352 bins: cursors in the count table
])
def test_bins_against_oracle(W, H, n, grow):
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    sc = dict(scenes.make_scene("C1", n=n, seed=W + n, sh_degree=0))
    sc["log_scales"] = (sc["log_scales"] + np.float32(grow)).astype(np.float32)
    cam = scenes.default_camera(W, H)
    r = gs.Renderer(0)
    try:
        g = gpu_render(r, sc, cam)
        dev = gs.scene_to_device(sc, 0)
        first = r.render(dev, cam, W, H)   # the edge that the first frame's counts suggest
        torch.cuda.synchronize()
        first = {k: v.clone() for k, v in first.items()}
        for kw in (dict(), dict(pair_capacity=int(g["num_pairs"]) + 1)):
            again = r.render(dev, cam, W, H, **kw)
            torch.cuda.synchronize()
            for k, v in first.items():
                assert torch.equal(v, again[k]), (kw, k)
        assert np.array_equal(first["image"].cpu().numpy().astype(np.float64), g["image"])
        assert np.array_equal(first["n_contrib"].cpu().numpy(), g["n_contrib"])
    finally:
        r.close()
    proj = oracle.project(sc, cam)
    unsure = check_projection(g, proj, f"{W}x{H} n={n}")
    tx, ty = proj["tiles_x"], proj["tiles_y"]
    rng = np.random.default_rng(n)
    rect = proj["rect"].T.astype(np.int64)[proj["tiles_touched"] > 0]   # x0, y0, x1, y1
    mid = (rect[:, 1] + rect[:, 3]) // 2 * tx + (rect[:, 0] + rect[:, 2]) // 2
    tiles = np.unique(np.concatenate([
        [0, tx - 1, (ty - 1) * tx, ty * tx - 1], np.clip(mid[:40], 0, tx * ty - 1), rng.integers(0, tx * ty, 40)]))
    o = oracle.render_tiles(proj, tiles)
    amb = oracle.ambiguous_mask(o)
    entries = 0
    for t in tiles:
        want = oracle.tile_list(proj, int(t))
        got = g["values"][g["tile_offsets"][t]:g["tile_offsets"][t + 1]]
        entries += len(want)
        if np.isin(want, unsure).any() or np.isin(got, unsure).any():
            continue
        assert np.array_equal(got, want), t
        ys = slice((t // tx) * TILE, min((t // tx + 1) * TILE, H))
        xs = slice((t % tx) * TILE, min((t % tx + 1) * TILE, W))
        good = ~amb[ys, xs]
        assert np.array_equal(g["n_contrib"][ys, xs][good], o["n_contrib"][ys, xs][good]), t
        assert np.abs(g["final_T"][ys, xs] - o["final_T"][ys, xs])[good].max(initial=0.0) <= IMAGE_TOL, t
        d = np.abs(g["image"][:, ys, xs] - o["image"][:, ys, xs]).max(axis=0)
        assert d[good].max(initial=0.0) <= IMAGE_TOL, t
    assert entries > 0
