"""Renders with a pair capacity read nothing back that they wait for, so a
program may queue them one behind another, and may capture one after a single
warm-up has sized the workspace.  The counters of the first, which choose the
bins of later ones, come back meanwhile: neither their arrival nor their
absence may show in the results, fail a render or end a capture."""
import pytest

import scenes

pytestmark = pytest.mark.gpu


def small_splats(n, seed):
    sc = dict(scenes.make_scene("C2", n=n, seed=seed, sh_degree=0))
    sc["log_scales"] = sc["log_scales"] * 0 - 5.5   # a few pixels: finer bins than the image size suggests
    return sc


def test_queued_frames_before_the_counters_are_back():
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    sc = small_splats(50_000, 3)
    dev, cam = gs.scene_to_device(sc), scenes.default_camera(640, 480)
    r = gs.Renderer(0)
    ref = gs.Renderer(0)
    try:
        want = ref.render(dev, cam, 640, 480)
        cap = 2 * int(ref.list_info()["num_pairs"]) + 1000
        x = torch.rand((8192, 8192), device="cuda")
        torch.cuda.synchronize()
        for _ in range(10):
            x = x @ x   # tens of milliseconds that the renders wait behind
            x = x / x.abs().max()
        outs = [r.render(dev, cam, 640, 480, pair_capacity=cap) for _ in range(4)]
        torch.cuda.synchronize()
        outs.append(r.render(dev, cam, 640, 480, pair_capacity=cap))
        torch.cuda.synchronize()
        for k, out in enumerate(outs):
            for name in want:
                assert torch.equal(out[name].view(torch.int32), want[name].view(torch.int32)), (k, name)
    finally:
        r.close()
        ref.close()


@pytest.mark.parametrize("items", [4, 8])
def test_capture_after_one_warm_up(items):
    """Four views of 300000 splats whose bins are to be finer than the first
    frame takes them, with a count table several times as large."""
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    dev = gs.scene_to_device(small_splats(300_000, 4))
    cams = [scenes.look_at_camera([0.3 * v - 0.5, 0.1 * v, -2.6], 640, 480) for v in range(4)]
    r = gs.Renderer(0)
    ref = gs.Renderer(0)
    try:
        want = [{k: t.clone() for k, t in o.items()} for o in ref.render_batched(dev, cams)]
        cap = 2 * int(ref.list_info()["num_pairs"]) + 1000
        r.set_tuning(bin_row_items=items)
        warm = r.render_batched(dev, cams, pair_capacity=cap)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            outs = r.render_batched(dev, cams, pair_capacity=cap)
        for rep in range(4):
            graph.replay()
            torch.cuda.synchronize()
            for o, w in zip(outs, want):
                for name in w:
                    assert torch.equal(o[name].view(torch.int32), w[name].view(torch.int32)), (rep, name)
                    o[name].zero_()
            # eager work between the replays, whose bins follow the counters
            again = r.render_batched(dev, cams, pair_capacity=cap)
            torch.cuda.synchronize()
            for o, w in zip(again, want):
                assert torch.equal(o["n_contrib"], w["n_contrib"]), rep
        assert len(warm) == 4
    finally:
        r.close()
        ref.close()
