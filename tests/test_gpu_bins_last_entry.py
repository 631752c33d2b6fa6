"""Lists that end a few entries below 2^32, the most that their 32-bit offsets
hold: 13256071 Gaussians in each of 324 bins of one tile.  All but the deepest
are too faint for any pixel, so every tile walks its list to the end, and the
image, final T and the deepest one's gradients are those of it alone."""
import pytest

import scenes

pytestmark = pytest.mark.gpu
W = H = 288   # 18 x 18 tiles; the first frame's bins are single tiles


def covering(n, torch):
    dev = {"sh_degree": 0, "attr_dtype": 0}
    dev["means"] = torch.zeros((3, n), device="cuda")
    dev["means"][2] = torch.linspace(2.0, 3.0, n, device="cuda")
    dev["log_scales"] = torch.full((3, n), 0.5, device="cuda")
    dev["quats"] = torch.zeros((4, n), device="cuda")
    dev["quats"][0] = 1.0
    dev["opacity_logits"] = torch.full((n,), -9.0, device="cuda")
    dev["sh"] = torch.full((1, 3, n), 0.25, device="cuda")
    dev["means"][2, -1] = 4.0
    dev["opacity_logits"][-1] = 0.5
    dev["sh"][0, :, -1] = torch.tensor([0.9, 0.2, -0.4], device="cuda")
    return dev


def test_lists_that_end_below_2_32():
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    tiles = (W // 16) * (H // 16)
    n = (2 ** 32 - 1) // tiles
    cam = dict(scenes.default_camera(W, H))
    cam["t"] = cam["t"] * 0
    grad = [torch.ones((3, H, W), device="cuda")]
    alone = covering(1, torch)
    alone["means"][2, 0] = 4.0
    ref = gs.Renderer(0)
    r = gs.Renderer(0)
    try:
        want = {k: v.clone() for k, v in ref.render(alone, cam, W, H).items()}
        assert ref.list_info()["num_pairs"] == tiles and int(want["n_contrib"].min()) == 1
        g_want = ref.backward(alone, grad)
        dev = covering(n, torch)
        out = r.render(dev, cam, W, H)
        torch.cuda.synchronize()
        assert r.list_info()["num_pairs"] == tiles * n
        assert torch.equal(out["image"], want["image"]) and torch.equal(out["final_T"], want["final_T"])
        assert torch.equal(out["n_contrib"], want["n_contrib"] * n)
        g = r.backward(dev, grad)
        torch.cuda.synchronize()
        for k, w in g_want.items():
            # one term per tile, added in any order: 324 roundings of 2^-24
            assert torch.allclose(g[k][..., -1], w[..., 0], rtol=5e-5, atol=1e-5 * float(w.abs().max())), k
            assert float(g[k][..., :-1].abs().max()) == 0.0, k
    finally:
        r.close()
        ref.close()
