"""The width of the depth sort (gs_tuning.sort_items): a width that a caller
sets is the one the sort takes, whatever the number of keys; a context that
was never given one chooses by that number.  On the host by the words of
counts that a sort needs cleared, which grow with its blocks; on the GPU every
choice gives the same order."""
import ctypes as C

import numpy as np
import pytest

import paper_2607_15951_amd as gs
import scenes


def clear_words(n, items):
    f = gs.load_library()._ZN4gsmi22depth_sort_clear_wordsElii   # gsmi::depth_sort_clear_words
    f.argtypes, f.restype = [C.c_int64, C.c_int, C.c_int], C.c_size_t
    return f(n, 1, items)


@pytest.mark.parametrize("n", [200_000, 799_999, 800_000, 1_000_000, 2_500_000])
def test_a_set_width_is_taken(n):
    def groups(items):   # 32 blocks of 256 threads each
        return -(-(-(-n // (256 * items))) // 32)
    for items in (4, 8, 16):
        assert clear_words(n, items) == 256 * groups(items)
    assert clear_words(n, 0) == 256 * groups(16 if n >= 800_000 else 8)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [799_999, 800_000, 2_500_001])
def test_every_width_gives_the_same_order(n):
    torch = pytest.importorskip("torch")
    sc = dict(scenes.make_scene("C1", n=n, seed=4, sh_degree=0))
    sc["log_scales"] = np.full_like(sc["log_scales"], -5.0)
    cam = scenes.default_camera(64, 48)
    dev = gs.scene_to_device(sc, 0)
    got = []
    for items in (None, 4, 8, 16):
        r = gs.Renderer(0)
        try:
            assert r.tuning()["sort_items"] == 8
            if items:
                r.set_tuning(sort_items=items)
                assert r.tuning()["sort_items"] == items
            r.render(dev, cam, 64, 48)
            got.append(r.lists(keys=True))
            torch.cuda.synchronize()
        finally:
            r.close()
    keys = got[0]["keys"].cpu().numpy().view(np.uint64)
    assert len(keys) > n / 2 and np.all(keys[1:] >= keys[:-1])
    for g in got[1:]:
        for k in ("tile_offsets", "values", "keys"):
            assert torch.equal(g[k], got[0][k]), k
