"""A backward captured by itself and replayed after eager renders of the same
views: it must follow the bins of the render that ran before the replay, which
change with the counters of earlier frames and with the tuning.  Gradients as
an eager backward's to the rounding of float atomics."""
import numpy as np
import pytest

import scenes
from test_gpu_capacity_frames import small_splats

pytestmark = pytest.mark.gpu


def test_replayed_backward_follows_the_last_render():
    torch = pytest.importorskip("torch")
    import paper_2607_15951_amd as gs
    dev = gs.scene_to_device(small_splats(60_000, 8))
    cams = [scenes.default_camera(640, 480), scenes.look_at_camera([0.4, 0.2, -2.5], 333, 197)]
    gen = torch.Generator(device="cuda").manual_seed(5)
    grads = [torch.rand((3, c["height"], c["width"]), device="cuda", generator=gen) - 0.5 for c in cams]
    outs = [{"image": torch.empty((3, c["height"], c["width"]), device="cuda"),
             "final_T": torch.empty((c["height"], c["width"]), device="cuda"),
             "n_contrib": torch.empty((c["height"], c["width"]), dtype=torch.int32, device="cuda")} for c in cams]
    ref = gs.Renderer(0)
    r = gs.Renderer(0)
    try:
        ref.render_batched(dev, cams)
        cap = 2 * int(ref.list_info()["num_pairs"]) + 1000
        want = {k: v.cpu().numpy().astype(np.float64) for k, v in ref.backward(dev, grads).items()}
        r.set_tuning(bin_row_items=4)   # its shape sizes the table
        r.render_batched(dev, cams, pair_capacity=cap, outs=outs)
        r.backward(dev, grads)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            got = r.backward(dev, grads)
        for rep, items in enumerate((4, 4, 16, 8)):
            r.set_tuning(bin_row_items=items)
            r.render_batched(dev, cams, pair_capacity=cap, outs=outs)   # from the second on by learned bins
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for k, w in want.items():
                if k == "quats":   # spheres: no rotation gradient, only its rounding
                    assert np.abs(got[k].cpu().numpy()).max() < 1e-12
                    continue
                d = got[k].cpu().numpy().astype(np.float64) - w
                assert np.linalg.norm(d) < 1e-5 * np.linalg.norm(w), (rep, k)
    finally:
        r.close()
        ref.close()
