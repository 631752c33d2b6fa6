"""Kept lists (GS_RENDER_REUSE_LISTS) and the layout of their offset table,
which depends on the tuning's bin_row_items and on the bins: a frame that
could keep its predecessor's lists must not read them by another layout.
Every pair of bin_row_items, the autotuner with the flag, and a captured
render replayed after an eager one of other bins; all bit for bit the plain
render's."""
import ctypes as C

import numpy as np
import pytest

import scenes
from test_gpu_list_reuse import plain, same, snapshot

pytestmark = pytest.mark.gpu
W, H = 3840, 2160   # 510 bins of 8x8 tiles: 60000 Gaussians in 59, 118 or 235 chunks by bin_row_items


@pytest.fixture(scope="module")
def case():
    pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    dev = gs.scene_to_device(scenes.make_scene("C3", n=60_000, seed=5, sh_degree=0))
    cam = scenes.default_camera(W, H)
    return dev, cam, plain(dev, cam, W, H)


@pytest.mark.parametrize("first", [4, 8, 16])
@pytest.mark.parametrize("capacity", [False, True])
def test_tuning_between_kept_frames(case, first, capacity):
    import paper_2607_15951_amd as gs
    dev, cam, want = case
    cap = len(want["values"]) + 1000 if capacity else 0
    r = gs.Renderer(0)
    try:
        r.set_tuning(bin_row_items=first)
        for _ in range(2):
            r.render(dev, cam, W, H, pair_capacity=cap)
        for items in (16, 8, 4, 16, 4, 8, 8):
            before = r.tuning()["bin_row_items"]
            r.set_tuning(bin_row_items=items)
            got = snapshot(r, r.render(dev, cam, W, H, pair_capacity=cap, reuse_lists=True))
            same(got, want, f"bin_row_items {before} -> {items}")
            assert r.list_reuse() == {"reused": before == items, "changed": 0}
            got = snapshot(r, r.render(dev, cam, W, H, pair_capacity=cap, reuse_lists=True))
            same(got, want, f"kept at {items}")
            assert r.list_reuse() == {"reused": True, "changed": 0}
    finally:
        r.close()


def test_a_smaller_shape_that_is_no_other_layout():
    """100000 Gaussians over 60 bins: bin_row_items 4 and 8 are one shape, but 4
    asks for a larger table, which must not lose the kept lists."""
    import paper_2607_15951_amd as gs
    dev, cam = gs.scene_to_device(scenes.make_scene("C3", n=100_000, seed=6, sh_degree=0)), scenes.default_camera(1280, 720)
    want = plain(dev, cam, 1280, 720)
    r = gs.Renderer(0)
    try:
        for _ in range(2):
            r.render(dev, cam, 1280, 720)
        for items in (4, 8, 4):
            r.set_tuning(bin_row_items=items)
            same(snapshot(r, r.render(dev, cam, 1280, 720, reuse_lists=True)), want, f"bin_row_items {items}")
            assert r.list_reuse()["changed"] == 0
    finally:
        r.close()


def test_autotune_with_the_flag(case):
    import torch
    import paper_2607_15951_amd as gs
    dev, cam, want = case
    r = gs.Renderer(0)
    try:
        out = r.render(dev, cam, W, H)
        views, outs = r._views([cam], [out], dev["means"].device)
        g, opts, t = gs.make_gaussians(dev), gs.make_opts(flags=gs.RENDER_REUSE_LISTS), gs.gs_tuning()
        st = r._L.gs_autotune(r._ctx, C.byref(g), views, 1, C.byref(opts), 1,
                              C.c_void_p(torch.cuda.current_stream().cuda_stream), C.byref(t), None)
        r._check(st)
        same(snapshot(r, out), want, "autotune's last frame")
        same(snapshot(r, r.render(dev, cam, W, H, reuse_lists=True)), want, "after autotune")
    finally:
        r.close()


def test_more_views_than_one_launch_sets_up():
    """17 views: their table takes launches of its own."""
    import torch
    import paper_2607_15951_amd as gs
    dev = gs.scene_to_device(scenes.make_scene("C2", n=20_000, seed=9, sh_degree=0))
    cams = [scenes.look_at_camera([0.2 * v - 1.5, 0.1, -2.6], 192, 112) for v in range(17)]
    r = gs.Renderer(0)
    try:
        want = [{k: v.clone() for k, v in o.items()} for o in r.render_batched(dev, cams)]
        for items in (8, 16, 16, 4):
            before = r.tuning()["bin_row_items"]
            r.set_tuning(bin_row_items=items)
            outs = r.render_batched(dev, cams, reuse_lists=True)
            torch.cuda.synchronize()
            assert r.list_reuse()["changed"] == 0
            assert r.list_reuse()["reused"] or before != items
            for o, w in zip(outs, want):
                for k in w:
                    assert torch.equal(o[k].view(torch.int32), w[k].view(torch.int32)), (items, k)
    finally:
        r.close()


def test_captured_kept_lists_replayed_after_another_layout():
    """A caller's own capture with the flag, replayed after eager frames of the
    same views whose tuning (hence layout) is another one."""
    import torch
    import paper_2607_15951_amd as gs
    dev, cam = gs.scene_to_device(scenes.make_scene("C3", n=60_000, seed=5, sh_degree=0)), scenes.default_camera(W, H)
    want = plain(dev, cam, W, H)
    cap = len(want["values"]) + 1000
    r = gs.Renderer(0)
    try:
        r.set_tuning(bin_row_items=4)   # the layout with the most chunks sizes the table
        for _ in range(2):
            r.render(dev, cam, W, H, pair_capacity=cap)
            torch.cuda.synchronize()
        r.set_tuning(bin_row_items=16)
        r.render(dev, cam, W, H, pair_capacity=cap)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            out = r.render(dev, cam, W, H, pair_capacity=cap, reuse_lists=True)
        for rep in range(4):
            if rep != 1:
                r.set_tuning(bin_row_items=(4, 8)[rep % 2])
                other = r.render(dev, cam, W, H, pair_capacity=cap)
                torch.cuda.synchronize()
                assert np.array_equal(other["n_contrib"].cpu().numpy(), want["nc"])
            for v in out.values():
                v.zero_()
            graph.replay()
            torch.cuda.synchronize()
            for k, w in (("image", "image"), ("final_T", "T"), ("n_contrib", "nc")):
                assert np.array_equal(out[k].cpu().numpy().view(np.uint32), want[w].view(np.uint32)), (rep, k)
    finally:
        r.close()
