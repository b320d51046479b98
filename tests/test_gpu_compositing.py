"""GPU compositing branches against the FP64 oracle: clamped splats among plain ones."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from parity_util import settings, to_dev  # noqa: E402
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


@pytest.mark.parametrize("w,h", [(8, 8), (2048, 16), (512, 512), (520, 512), (1024, 600)])
def test_backward_work_items_over_many_tiles(R, w, h):
    # 1, 512, 4,096, 4,160 and 9,600 tiles of 8: up to 4,096 a slice of the queue counts
    # the items in front of it itself, of more the slices are added up first; eager (twice over one saved state) and captured (replayed) backwards
    # must agree up to the order of the float atomics
    g = scenes.make_cfg1().gaussians
    f = float(max(w, h))
    cam = scenes.Camera(w, h, f, f, w / 2.0, h / 2.0, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))
    rng = np.random.default_rng(w + h)
    target = (torch.from_numpy(rng.random((3, h, w), dtype=np.float32)).cuda(), None)
    s = settings(tile=8)
    params = to_dev(g)
    say("items", w, h)
    images, saved = R.forward(*params, [cam], s)
    loss, gc, gd = R.loss_l1(saved, images, [target], 0.1)
    first = R.backward(saved, gc)
    second = R.backward(saved, gc)
    graph = R.Graph(*params, [cam], [target], s)
    replays = []
    for _ in range(3):
        graph.launch()
        torch.cuda.synchronize()
        replays.append({k: v.clone() for k, v in graph.grads.items()})
    for other in [second] + replays:
        for k in first:
            scale = float(first[k].abs().max())
            # float sums of the same terms in another order: 1e-5 of the group's largest value
            assert float((first[k] - other[k]).abs().max()) <= 1e-5 * scale + 1e-20, (k, scale)


@pytest.mark.parametrize("w,h", [(512, 512), (520, 512), (1024, 600)])
def test_work_items_of_small_tiles_cover_every_entry(R, w, h):
    # the gradients over 4,096, 4,160 and 9,600 tiles of 8 (beyond 4,096 the items are placed by sums of
    # slices) equal those over a quarter of the tiles of 16, where every block counts for itself: the
    # same pixels take the same splats, summed in another order
    g = scenes.make_cfg1().gaussians
    f = float(max(w, h))
    cam = scenes.Camera(w, h, f, f, w / 2.0, h / 2.0, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))
    gc = torch.from_numpy(np.random.default_rng(w + h).standard_normal((3, h, w)).astype(np.float32)).cuda()
    params = to_dev(g)
    say("items of 8 and 16", w, h)
    grads, images = [], []
    for tile in (8, 16):
        im, saved = R.forward(*params, [cam], settings(tile=tile))
        images.append(im[0])
        grads.append(R.backward(saved, [gc]))
    for a, b in zip(*images):
        assert torch.equal(a, b)
    for k in grads[0]:
        # sums of up to 10^5 terms of either sign in another order, through the projection's chain rule: 1e-4
        # of the group's largest value (an item left out or taken twice changes whole splats)
        scale = float(grads[0][k].abs().max())
        assert float((grads[0][k] - grads[1][k]).abs().max()) <= 1e-4 * scale, k
