"""Grids of few tiles are blended by a kernel that composites eight entries at a
time with vector selects; the kernel that counts its work keeps the plain
loop.  Both must give the same bits: list lengths around the groups of eight
and the batches of 256, faint and opaque splats (early termination inside a
group), cut tiles, and colours that are infinite or NaN, which reach only the
pixels that composite their splat."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,n,logit,odd", [
    (16, 16, 1, -1.0, False), (16, 16, 3, -1.0, False), (17, 33, 4, 2.0, False), (40, 24, 5, -3.0, True),
    (24, 16, 8, -1.0, False), (24, 16, 9, 3.0, True),
    (40, 24, 257, -4.0, False), (40, 24, 600, 6.0, False), (40, 24, 600, -4.5, True), (200, 120, 5000, 0.0, True),
    (880, 880, 20000, 0.0, False),    # 3025 tiles
    (896, 896, 20000, 0.0, False),    # 3136: past the line
])
def test_few_tiles_same_bits(W, H, n, logit, odd):
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    rng = np.random.default_rng(n)
    sc = dict(scenes.make_scene("C1", n=n, seed=n, sh_degree=0))
    if n < 1000:
        sc["means"] = (sc["means"] * np.float32(0.1)).astype(np.float32)
        sc["log_scales"] = rng.uniform(-2.5, 0.0, sc["log_scales"].shape).astype(np.float32)
    sc["opacity_logits"] = (logit + rng.uniform(-1, 1, n)).astype(np.float32)
    if odd:
        sh = np.array(sc["sh"])
        sh[0, 0, ::3] = np.inf
        sh[0, 1, 1::5] = np.nan
        sc["sh"] = sh
    cam = scenes.default_camera(W, H)
    dev = gs.scene_to_device(sc, 0)
    r = gs.Renderer(0)
    try:
        got = []
        for work in (False, True, False):
            r.set_profiling(False, blend_work=work)
            out = r.render(dev, cam, W, H, background=(0.2, 0.4, 0.6))
            torch.cuda.synchronize()
            got.append({k: v.cpu().numpy().view(np.uint32).copy() for k, v in out.items()})
    finally:
        r.close()
    assert got[0]["n_contrib"].max() > 0
    for g in got[1:]:
        for k in got[0]:
            if odd and k == "image":   # NaN payloads may differ
                a, b = got[0][k].view(np.float32), g[k].view(np.float32)
                assert np.array_equal(np.isnan(a), np.isnan(b))
                assert np.array_equal(a[~np.isnan(a)], b[~np.isnan(b)])
            else:
                assert np.array_equal(got[0][k], g[k]), k
