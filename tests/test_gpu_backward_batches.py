"""Gradients of tiles whose lists end at the edges of the backward's batches of
256 entries: lists of one entry, of one batch less one, full and one more, of
several batches, with faint splats (every pixel walks the whole list) and with
opaque ones (alpha clamps, pixels stop early).  The tolerances are those of
the other gradient tests: 2u relative error per composited entry in the
transmittance and in what lies behind an entry (u = 2^-24), so at most 7e-5 of
a group's largest gradient at 600 entries."""
import numpy as np
import pytest

import scenes
from test_gpu_backward import renderer, small_case  # noqa: F401  (fixture)

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("oracle_lib")]


@pytest.mark.parametrize("n,logit", [(1, -2.0), (64, -3.0), (255, -4.0), (256, -4.0), (257, -4.0), (600, -4.5),
                                     (257, 8.0)])
def test_backward_list_lengths(renderer, n, logit):  # noqa: F811
    sc = dict(scenes.make_scene("C1", n=n, seed=60 + n, sh_degree=0))
    # every splat covers the whole image of four tiles, two of them cut
    sc["means"] = (sc["means"] * np.float32(0.05)).astype(np.float32)
    rng = np.random.default_rng(n)
    sc["log_scales"] = rng.uniform(-0.5, 0.2, sc["log_scales"].shape).astype(np.float32)
    sc["opacity_logits"] = (logit + rng.uniform(-0.5, 0.5, sc["opacity_logits"].shape)).astype(np.float32)
    small_case(renderer, sc, scenes.default_camera(24, 19), f"list of {n}, logit {logit}", bg=(0.3, 0.1, 0.6),
               seed=n)
