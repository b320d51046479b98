"""GPU binning against the oracle's sorted keys: more tile columns and rows than one window of
bins, more pairs in a round than one listing holds, chunks that span several small views."""
import threading

import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from parity_util import check_keys, oracle_for, settings, to_dev  # noqa: E402
from test_gpu_parity import R, run_fwd, say  # noqa: E402, F401


def _keys(R, g, cams, s):
    _, _, saved = run_fwd(R, g, cams, s)
    check_keys(saved.debug_export(), oracle_for(g, cams, s))
    return saved.info()


@pytest.mark.parametrize("exact", [False, True])
@pytest.mark.parametrize("w,h,scale", [(2100, 40, 1.0), (40, 2100, 1.0), (2049, 2057, 1.0), (2048, 512, 12.0)])
def test_many_columns_and_rows(R, w, h, scale, exact):
    # tiles of 8: 263 and 257 bins are past one window of 256, 256 fill it; splats 12 times wider
    # give rounds of 256 items more than 4,096 pairs
    base = scenes.make_cfg1().gaussians
    g = base.subset(np.arange(0, base.n, 2))
    g.scales = (g.scales * scale).astype(np.float32)
    f = float(max(w, h))
    cam = scenes.Camera(w, h, f, f, w / 2.0, h / 2.0, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))
    say("bins", w, h, scale, exact)
    info = _keys(R, g, [cam], settings(tile=8, exact_tiles=exact))
    assert info["num_keys"] > (100 * g.n if scale > 1 else g.n)


@pytest.mark.parametrize("n", [1, 5, 255, 257, 2000])
def test_chunks_spanning_views(R, n):
    # sixteen views of uneven sizes: a chunk of 256 depth-sorted records holds records of several
    # views (n small), or the last of one and the first of the next
    g = scenes.make_cfg1().gaussians.subset(np.arange(n))
    c = scenes.make_cfg1().cameras[0]
    cams = [c.crop(3 * k, 2 * k, 128 - 5 * k, 96 - 3 * k) for k in range(16)]
    say("views", n)
    _keys(R, g, cams, settings(tile=8, exact_tiles=n % 2 == 1))


@pytest.mark.parametrize("views,n", [(1, 1), (3, 1365 * 256), (16, 65536), (16, 65537), (3, 1366 * 256), (16, 200000)])
def test_block_sums_of_many_gaussians(R, views, n):
    # block sums of 256 records each: 1, 4,095 and 4,096 are scanned by one block, 4,112, 4,098 and
    # 12,512 by tiles of 256; captured steps leave up to 4,096 to the compaction.  Splats of a
    # twentieth of the size: hundreds of thousands of records whose tile lists stay short
    base = scenes.make_cfg1().gaussians
    rng = np.random.default_rng(n)
    g = base.subset(rng.integers(0, base.n, n))
    g.means = (g.means + rng.normal(0, 0.05, g.means.shape)).astype(np.float32)
    g.scales = (g.scales * 0.05).astype(np.float32)
    c = scenes.make_cfg1().cameras[0]
    cams = [c.crop(k, 2 * k, 64 - 2 * k, 48 - k) for k in range(views)]
    say("block sums", views, n)
    s = settings(tile=16)
    _keys(R, g, cams, s)
    params = to_dev(g)
    images, _ = R.forward(*params, cams, s)
    target = [(torch.zeros_like(im[0]), None) for im in images]
    graph = R.Graph(*params, cams, target, s)
    for _ in range(3):
        graph.launch()
        graph.sync()   # raises where a capacity overflowed
        for a, b in zip(graph.images, images):
            assert torch.equal(a[0], b[0])


def test_more_pairs_than_keys_can_number(R):
    # 1,048,577 splats over all 258 x 258 tiles: 7e10 pairs.  65,536 records of them alone have more
    # than 2^32; the forward says so whether one block adds up the block sums or (as here) many do
    n = 4096 * 256 + 1
    params = [torch.zeros((n, 3)), torch.full((n, 3), 100.0), torch.zeros((n, 4)), torch.full((n,), 0.5),
              torch.zeros((n, 1, 3))]
    params[0][:, 2] = 2.0
    params[2][:, 0] = 1.0
    cam = scenes.Camera(2064, 2064, 1000.0, 1000.0, 1032.0, 1032.0, np.eye(3, dtype=np.float32),
                        np.zeros(3, np.float32))
    say("pairs")
    for m in (n - 1, n):
        with pytest.raises(Exception, match="2\\^32"):
            R.forward(*[p[:m].cuda() for p in params], [cam], settings(tile=8))


class _Pieces:
    """A caller's allocator that refuses blocks above `limit` bytes."""

    def __init__(self, limit):
        self.limit, self.held, self.asked = limit, {}, []

    def alloc(self, nbytes, stream):
        self.asked.append(nbytes)
        if nbytes > self.limit:
            return 0
        t = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
        p = (t.data_ptr() + 255) // 256 * 256
        self.held[p] = t
        return p

    def free(self, ptr, stream):
        torch.cuda.synchronize()
        del self.held[ptr]


@pytest.mark.parametrize("limit,separate", [(1 << 40, False), (1000000, True), (8 << 10, None)])
def test_allocator_that_refuses_one_large_block(R, limit, separate):
    # the arrays of a forward (the largest takes 983,040 bytes) come as one block, or where that
    # is refused one by one; where an
    # array is refused too the call fails and gives everything back
    g = scenes.make_cfg1().gaussians.subset(np.arange(400))
    cam = scenes.make_cfg1().cameras[0].crop(0, 0, 64, 48)
    params, s = to_dev(g), settings(tile=16)
    images, saved = R.forward(*params, [cam], s)
    grads = R.backward(saved, [torch.ones_like(images[0][0])])
    pieces = _Pieces(limit)
    ctx = R.Context(torch.cuda.current_device(), torch.cuda.current_stream().cuda_stream, pieces)
    say("allocator", limit)
    with R.using(ctx):
        if separate is None:
            with pytest.raises(Exception, match="ENOMEM"):
                R.forward(*params, [cam], s)
            assert not pieces.held
            return
        images2, saved2 = R.forward(*params, [cam], s)
        grads2 = R.backward(saved2, [torch.ones_like(images[0][0])])
    assert (max(pieces.asked) > limit) == separate
    for a, b in zip(images[0], images2[0]):
        assert torch.equal(a, b)
    for k in grads:
        assert float((grads[k] - grads2[k]).abs().max()) <= 1e-5 * float(grads[k].abs().max()) + 1e-20
    saved2.free()


class _Budget(_Pieces):
    """A caller's allocator that holds at most `limit` bytes at a time."""

    def __init__(self, limit):
        super().__init__(limit)
        self.now, self.peak, self.size = 0, 0, {}

    def alloc(self, nbytes, stream):
        if self.now + nbytes > self.limit:
            return 0
        p = _Pieces.alloc(self, nbytes, stream)
        self.size[p] = nbytes
        self.now += nbytes
        self.peak = max(self.peak, self.now)
        return p

    def free(self, ptr, stream):
        _Pieces.free(self, ptr, stream)
        self.now -= self.size.pop(ptr)


def test_allocator_without_room_for_the_larger_plan(R):
    # 10.3M pairs over 256 columns: 10.3M tile counts (41 MB), of which a third do where the memory for
    # all is refused: the same images and keys
    base = scenes.make_cfg1().gaussians
    g = base.subset(np.arange(0, base.n, 2))
    g.scales = (g.scales * 60).astype(np.float32)
    f = 2048.0
    cam = scenes.Camera(2048, 512, f, f, 1024.0, 256.0, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))
    params, s = to_dev(g), settings(tile=8)
    results, peak = [], 1 << 40
    for spare in (0, 8 << 20):
        budget = _Budget(peak - spare)
        ctx = R.Context(torch.cuda.current_device(), torch.cuda.current_stream().cuda_stream, budget)
        say("budget", budget.limit)
        with R.using(ctx):
            images, saved = R.forward(*params, [cam], s)
            info, dbg = saved.info(), saved.debug_export()
            saved.free()
        peak = budget.peak
        results.append((images[0], dbg))
    assert 9 << 20 < info["num_keys"] < 12 << 20
    for a, b in zip(results[0][0], results[1][0]):
        assert torch.equal(a, b)
    for k in ("keys", "values", "ranges"):
        np.testing.assert_array_equal(results[0][1][k], results[1][1][k])


def test_states_taken_and_given_back_in_any_order(R):
    # forwards of changing sizes on one context, their states freed in another order (some by a second
    # thread, some by their owners going away), blocks going round between them: every state that is
    # alive keeps its own memory
    base = scenes.make_cfg1()
    rng = np.random.default_rng(11)
    ctx = R.Context(torch.cuda.current_device(), torch.cuda.current_stream().cuda_stream)
    cases = []
    for n in (40, 400, 900, 1500, 2000):
        g = base.gaussians.subset(np.arange(n))
        cam = base.cameras[0].crop(0, 0, 48 + n // 25, 40 + n // 40)
        params = to_dev(g)
        images, saved = R.forward(*params, [cam], settings(tile=16))
        gc = torch.from_numpy(rng.standard_normal(images[0][0].shape).astype(np.float32)).cuda()
        cases.append((params, cam, gc, images[0][0].clone(), R.backward(saved, [gc])))
    say("states")
    alive = []
    with R.using(ctx):
        for _ in range(120):
            if len(alive) < 6 and rng.random() < 0.6:
                c = cases[rng.integers(len(cases))]
                images, saved = R.forward(*c[0], [c[1]], settings(tile=16))
                assert torch.equal(images[0][0], c[3])
                alive.append((c, saved))
            elif alive:
                (params, cam, gc, image, want), saved = alive.pop(rng.integers(len(alive)))
                grads = R.backward(saved, [gc])
                for k in want:  # (the same terms, summed in another order)
                    assert float((grads[k] - want[k]).abs().max()) <= 1e-5 * float(want[k].abs().max()) + 1e-20, k
                how = rng.integers(3)
                if how == 0:
                    saved.free()
                elif how == 1:
                    th = threading.Thread(target=saved.free)
                    th.start()
                    th.join()
                del saved
    torch.cuda.synchronize()


def test_work_hint_while_another_stream_writes_it(R):
    # a context whose stream is changed without waiting: the second forward reads the work hint of the
    # tile grid while the first one's compositing, on the other stream, writes it.  Whatever order of
    # the tiles comes of it, every tile is composited once
    g = scenes.make_cfg2(n=60000).gaussians
    base = scenes.make_cfg2(n=16).cameras[0]
    s = settings(tile=8)
    params = to_dev(g)
    cams = [scenes.Camera(640, 480, f, f, 320.0, 240.0, base.R, base.t) for f in (150.0, 600.0)]
    wanted = [R.forward(*params, [c], s)[0][0] for c in cams]
    streams = [torch.cuda.Stream() for _ in cams]
    ctx = R.Context(torch.cuda.current_device(), streams[0].cuda_stream)
    torch.cuda.synchronize()
    say("two streams")
    for _ in range(10):
        kept = []
        with R.using(ctx):
            for k in (0, 1):
                ctx.lib.gsr_ctx_set_stream(ctx.h, streams[k].cuda_stream)
                kept.append(R.forward(*params, [cams[k]], s))
        torch.cuda.synchronize()
        for (images, saved), want in zip(kept, wanted):
            for a, b in zip(images[0], want):
                assert torch.equal(a, b)
            saved.free()
        torch.cuda.synchronize()


@pytest.mark.parametrize("views,n", [(1, 2), (1, 4096), (5, 4096), (1, 4097), (2, 16384), (1, 16385), (3, 20000),
                                     (1, 458752), (2, 458753), (1, 917504), (2, 917505)])
def test_depth_sort_sizes(R, views, n):
    # sorted by one block a view up to 4,096 and 16,384 keys; by tiles of 2,048 or 4,096 keys whose
    # histograms each block adds up, up to 224 tiles (458,752, 917,504 keys) a view; row-scanned beyond.  Depths of
    # few values, all near the same: ties keep the record order
    base = scenes.make_cfg1().gaussians
    rng = np.random.default_rng(n + views)
    g = base.subset(rng.integers(0, base.n, n))
    g.means = g.means.copy()
    g.means[:, :2] *= 0.05
    g.means[:, 2] = (2.0 + rng.integers(0, 700, n) * 2.0 ** -12).astype(np.float32)
    g.scales = (g.scales * 0.02).astype(np.float32)
    f = 60.0
    cams = [scenes.Camera(64 - 8 * k, 48, f, f, 32.0 - 8 * k, 24.0, np.eye(3, dtype=np.float32),
                          np.zeros(3, np.float32)) for k in range(views)]
    say("depth sort", views, n)
    _keys(R, g, cams, settings(tile=16))
