"""How often the backward of the blend rounds, on splats whose gradients come
from one pixel each, so that every float operation on the way is known: the
opacity's gradient leaves the pixel as ga E (ga = dL/d(alpha), E the falloff),
and the centre's as gp (2 A' dx + B' dy) with one product and one fused step.
Equality, no tolerance."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu
F = np.float32
SIDE, TILES = 512, 32   # one splat in the middle of every tile


def frame(torch, gs, means, log_scales, quats, logits, seed):
    """Renders the splats and gives the red channel of each one's pixel (its
    tile's middle one) a gradient of 24 random bits, no other pixel any."""
    n = means.shape[1]
    assert n == TILES * TILES
    sc = {"sh_degree": 0, "attr_dtype": 0, "means": means, "log_scales": log_scales, "quats": quats,
          "opacity_logits": logits, "sh": np.zeros((1, 3, n), F)}   # colour 1/2
    cam = dict(scenes.default_camera(SIDE, SIDE), fx=F(1), fy=F(1), cx=F(0), cy=F(0))
    cam["R"], cam["t"] = np.eye(3, dtype=F), np.zeros(3, F)
    px, py = (8 + 16 * (np.arange(n) % TILES)), (8 + 16 * (np.arange(n) // TILES))
    G = np.random.default_rng(seed).uniform(0.5, 2.0, n).astype(F)
    grad = np.zeros((3, SIDE, SIDE), F)
    grad[0, py, px] = G
    r = gs.Renderer(0)
    try:
        dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() if isinstance(v, np.ndarray) else v
               for k, v in sc.items()}
        out = r.render(dev, cam, SIDE, SIDE)
        g = {k: v.cpu().numpy() for k, v in r.backward(dev, [torch.from_numpy(grad).cuda()]).items()}
        nc = out["n_contrib"].cpu().numpy()
    finally:
        r.close()
    assert nc[py, px].max() == 1   # no other splat reaches the pixel
    return G, g, nc[py, px] == 1


def places(dx=0.0, dy=0.0):
    n = TILES * TILES
    m = np.ones((3, n), F)
    m[0] = (8 + 16 * (np.arange(n) % TILES) + dx).astype(F)
    m[1] = (8 + 16 * (np.arange(n) // TILES) + dy).astype(F)
    return m


def test_opacity_gradient_is_rounded_once():
    """E = 1 and opacity 3/4: T and its reciprocal are powers of two, so that
    dL/d(opacity) = G / 2 exactly."""
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    n = TILES * TILES
    quats = np.zeros((4, n), F)
    quats[0] = 1
    logit = F(np.log(3.0))
    G, g, seen = frame(torch, gs, places(), np.full((3, n), -20.0, F), quats, np.full(n, logit, F), 1)
    assert seen.all()
    sig = 1.0 / (1.0 + np.exp(-np.float64(logit)))
    assert F(sig) == F(0.75)
    assert np.array_equal(g["opacity_logits"], (0.5 * G.astype(np.float64) * sig * (1 - sig)).astype(F))


def test_centre_gradient_is_one_fused_step():
    """Opacity 1/2, so that dL/dp is half the opacity's gradient exactly;
    flat splats turned about the optical axis, centres off the pixel."""
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    n = TILES * TILES
    rng = np.random.default_rng(2)
    th = rng.uniform(0.0, np.pi, n)
    quats = np.zeros((4, n), F)
    quats[0], quats[3] = np.cos(th / 2), np.sin(th / 2)
    ls = np.full((3, n), -20.0, F)
    ls[0], ls[1] = rng.uniform(-0.2, 0.15, n), -3.0
    means = places(rng.uniform(-1.2, 1.2, n), rng.uniform(-1.2, 1.2, n))
    G, g, seen = frame(torch, gs, means, ls, quats, np.zeros(n, F), 3)
    assert seen.sum() > n // 2
    # the conic, as the projection computes it (the splat lies in the plane z = 1)
    w, z = quats[0].astype(np.float64), quats[3].astype(np.float64)
    qn = np.sqrt(w * w + z * z)
    w, z = w / qn, z / qn
    c, s = 1 - 2 * z * z, 2 * w * z
    s0, s1 = np.exp(ls[0].astype(np.float64)), np.exp(ls[1].astype(np.float64))
    ca = (c * s0) ** 2 + (s * s1) ** 2 + 0.3
    cc = (s * s0) ** 2 + (c * s1) ** 2 + 0.3
    cb = c * s0 * s * s0 - s * s1 * c * s1
    det = ca * cc - cb * cb
    A, B, C = (cc / det).astype(F), (-cb / det).astype(F), (ca / det).astype(F)
    log2e, ln2 = F(1.4426950408889634), F(0.69314718055994531)
    A1, B1, C1 = F(-0.5) * log2e * A, -log2e * B, F(-0.5) * log2e * C
    wide = np.longdouble
    dx = (means[0].astype(np.float64) - (8 + 16 * (np.arange(n) % TILES))).astype(F)
    dy = (means[1].astype(np.float64) - (8 + 16 * (np.arange(n) // TILES))).astype(F)
    gp = F(0.5) * (F(4) * g["opacity_logits"])
    su = (wide(1) * (A1 + A1) * dx + B1 * dy).astype(F)          # fused: the product is not rounded
    sv = (wide(1) * B1 * dx + (C1 * dy + C1 * dy)).astype(F)
    ok = seen & (gp != 0)
    for k, slope in ((0, su), (1, sv)):
        want = (gp * slope) * ln2
        wrong = ok & (g["means"][k] != want)
        assert not wrong.any(), (k, int(wrong.sum()), int(ok.sum()), g["means"][k][wrong][:4], want[wrong][:4])
