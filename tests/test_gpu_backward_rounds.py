"""Gradients of tiles whose lists end at the edges of the backward's batches of
128 entries, of its rounds over 1024 entries of a bin, and of the ring of 2048
picked ones: one less, as many and one more, with splats faint enough that
every pixel walks the whole list.  The tolerances are those of the other
gradient tests: a composited entry is met with 2u relative error in the
transmittance and in what lies behind it (u = 2^-24), 2.5e-4 of a group's
largest gradient if all 2100 errors had one sign; they do not, and their walk
adds about sqrt(2100) 2u, 6e-6."""
import numpy as np
import pytest

import scenes
from test_gpu_backward import renderer, small_case  # noqa: F401  (fixture)

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


@pytest.mark.parametrize("n", [127, 128, 129, 383, 385, 1023, 1024, 1025, 2047, 2049, 2100])
def test_backward_list_lengths(renderer, n):  # noqa: F811
    sc = dict(scenes.make_scene("C1", n=n, seed=90 + n, sh_degree=0))
    # every splat covers the whole image of four tiles, two of them cut
    sc["means"] = (sc["means"] * np.float32(0.02)).astype(np.float32)
    rng = np.random.default_rng(n)
    sc["log_scales"] = rng.uniform(0.2, 0.6, sc["log_scales"].shape).astype(np.float32)
    # alphas just above 1/255 near the centres
    sc["opacity_logits"] = rng.uniform(-5.45, -5.25, sc["opacity_logits"].shape).astype(np.float32)
    got, want = small_case(renderer, sc, scenes.default_camera(24, 19), f"list of {n}", bg=(0.3, 0.1, 0.6), seed=n)
    # the deepest splat is reached (some pixel composites it)
    depth = sc["means"][2]
    deepest = np.argsort(depth, kind="stable")[-max(3, n // 50):]
    assert np.abs(want["opacity_logits"][deepest]).max() > 0
    assert np.abs(got["opacity_logits"][deepest]).max() > 0
