"""GPU compositing branches against the FP64 oracle: clamped splats among plain ones."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from parity_util import settings  # noqa: E402
from test_gpu_parity import R, fwd_bwd_parity, say  # noqa: E402, F401


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("every", [1, 40, 400])
def test_clamped_splats_among_plain_ones(R, tile, every):
    # the backward takes a stage of 64 entries with a shorter alpha where no splat of it can be
    # clamped (opacity below alpha_max): stages with all, some and hardly any clamped splats
    w = scenes.make_cfg1()
    g = w.gaussians.subset(np.arange(w.gaussians.n))
    g.opacities = g.opacities.copy()
    g.opacities[::every] = 0.999
    c = w.cameras[0]
    say("clamped", tile, every)
    rep, grep = fwd_bwd_parity(R, g, [c, c.crop(13, 7, 37, 29)], settings(tile=tile, bg=(0.2, 0.1, 0.4)))
    say(rep, grep)
