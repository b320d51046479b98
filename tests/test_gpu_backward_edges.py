"""GPU backward at the edges of binary32: needles whose rounded conic is not positive definite, pixels
close to a splat's centre, NaN gradients."""
import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from parity_util import oracle_for, settings, to_dev  # noqa: E402
from test_gpu_parity import R, run_fwd, say  # noqa: E402, F401

F32 = np.float32
I3, Z3 = np.eye(3, dtype=F32), np.zeros(3, F32)
Y00 = 0.5 / np.sqrt(np.pi)

# (low-pass, window at 640x480 with f = 320, needles: mean, scales, quaternion): long thin splats whose
# det = a c - b^2 cancels in binary32, so that exp(-q/2) exceeds 1 at pixels of the window
NEEDLES = {
    "default": (0.3, (576, 367), [((-0.1347728, -0.29704165, 0.4189062), (2.9465544, 3.560347e-05, 3.560347e-05),
                                   (-0.01368332, 0.41084337, -0.93534404, -0.5304637))]),
    "small": (0.01, (339, 55), [((-0.18990733, 0.3012675, 0.4147552), (2.9164885, 7.627780e-05, 7.627780e-05),
                                 (0.55986929, -1.23856509, -0.88682085, -1.34563553))]),
    "none": (0.0, (576, 214), [((-1.1865001, 0.5636072, 1.2031643), (1.1536512, 5.416020e-05, 5.416020e-05),
                                (0.39329809, 1.06880009, 0.20485803, -1.25134671))]),
}
OPACITY = 0.9895


def needle_scene(kind, count=60, seed=3):
    """(Gaussians, camera, low-pass): the needles over and under ordinary splats of the window."""
    lowpass, (x0, y0), needles = NEEDLES[kind]
    w, h = 64, 48
    cam = scenes.Camera(640, 480, 320.0, 320.0, 320.0, 240.0, I3, Z3).crop(x0, y0, w, h)
    rng = np.random.default_rng(seed)
    z = needles[0][0][2] * rng.uniform(0.5, 2.0, count)
    u, v = rng.uniform(0, w, count), rng.uniform(0, h, count)
    means = np.stack([(u - cam.cx) / cam.fx * z, (v - cam.cy) / cam.fy * z, z], 1)
    g = scenes.random_gaussians(rng, means, 0)
    g.scales = (z[:, None] / 320.0 * rng.uniform(3.0, 12.0, (count, 3))).astype(F32)
    g.opacities = rng.uniform(0.1, 0.6, count).astype(F32)
    n = len(needles)
    arrays = [np.concatenate([np.asarray(a, F32).reshape(n, *b.shape[1:]), b]) for a, b in zip(
        ([x[0] for x in needles], [x[1] for x in needles], [x[2] for x in needles], [OPACITY] * n,
         rng.uniform(-0.5, 0.5, (n, 1, 3))), g.arrays())]
    return scenes.Gaussians(*[np.ascontiguousarray(a, F32) for a in arrays], 0), cam, lowpass


def replay(g, cam, s, mu, conic, depth, rect, g_color, g_alpha, clamp=True):
    """dL/d(opacities, sh) in 64 bits for the splat values that the kernels compute in binary32: q' by
    the same operations (binary64 products and one rounding stand for each fused multiply-add), then
    the rules and the compositing recurrence.  Also the smallest relative distance of a
    splat value from the skip and clamp thresholds, and the pixels where a value is clamped.
    clamp=False: the clamp left out (what the gradients must not be)."""
    k = F32(-0.72134752044448170368)
    h, w, t = cam.height, cam.width, s.tile
    py, px = (a.reshape(-1).astype(F32) for a in np.mgrid[0:h, 0:w])
    order = [i for i in np.argsort(depth, kind="stable") if rect[i, 0] <= rect[i, 1]]
    G, take = [], []
    for i in order:
        ap, bp, cp = k * conic[i, 0], (F32(2) * k) * conic[i, 1], k * conic[i, 2]
        dx, dy = px - mu[i, 0], py - mu[i, 1]
        inner = (np.float64(ap) * dx + (bp * dy)).astype(F32)
        q = (np.float64(1) * inner * dx + ((cp * dy) * dy)).astype(F32)
        G.append(np.exp2(q.astype(np.float64)))
        tx, ty = px // t, py // t
        take.append((tx >= rect[i, 0]) & (tx <= rect[i, 1]) & (ty >= rect[i, 2]) & (ty <= rect[i, 3]))
    G, take = torch.tensor(np.array(G)), torch.tensor(np.array(take))
    o = torch.tensor(g.opacities[order].astype(np.float64), requires_grad=True)
    sh = torch.tensor(g.sh[order, 0].astype(np.float64), requires_grad=True)
    a = o[:, None] * G
    amin, amax = float(F32(s.alpha_min)), float(F32(s.alpha_max))
    margin = min(float((a.detach()[take] / x - 1).abs().min()) for x in (amin, amax))
    act = take & (a >= amin)
    clamped = act & (a > amax)
    a = torch.where(act, a, torch.zeros_like(a))
    if clamp:
        a = torch.where(clamped, torch.full_like(a, amax), a)
    T = torch.cumprod(torch.cat([torch.ones_like(a[:1]), 1 - a[:-1]]), 0)
    assert not clamp or float((T * (1 - a)).detach().min()) > s.T_min  # no pixel stops
    wgt = a * T
    col = torch.clamp(0.5 + Y00 * sh, min=0)
    colour = (wgt[:, None, :] * col[:, :, None]).sum(0)
    alpha = 1 - T[-1] * (1 - a[-1])
    ((colour * torch.tensor(g_color.reshape(3, -1).astype(np.float64))).sum()
     + (alpha * torch.tensor(g_alpha.reshape(-1).astype(np.float64))).sum()).backward()
    do, dsh = np.zeros(g.n), np.zeros((g.n, 3))
    do[order], dsh[order] = o.grad.numpy(), sh.grad.numpy()
    return dict(opacities=do, sh=dsh), margin, int(clamped.any(0).sum())


def close(got, ref):
    """1e-3 of the value or of a hundredth of the group's largest.  Recovering T costs at most 64
    reciprocals of 1e-7 each in a stage (6e-6 of the value); the colour behind a splat is off by
    6e-8 of the image over T and counts T times, some 1e-7 a pixel where 1e-5 of sums over
    tens of pixels is allowed; exp2 and the products behind it add 1e-6."""
    return np.abs(got - ref) <= 1e-3 * np.maximum(np.abs(ref), 1e-2 * np.abs(ref).max())


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("kind", sorted(NEEDLES))
def test_needles_past_the_clamp(R, kind, tile):
    # the forward clamps o exp(-q/2) > alpha_max; the backward has to divide by the same 1 - alpha, and
    # gives the clamped pixels no gradient of the opacity
    g, cam, lowpass = needle_scene(kind)
    s = settings(tile=tile, lowpass=lowpass, guard=100.0, T_min=1e-9)
    say("needles", kind, tile)
    _, images, saved = run_fwd(R, g, [cam], s)
    d = saved.debug_export()
    rng = np.random.default_rng(17)
    gc = rng.standard_normal((3, cam.height, cam.width)).astype(F32)
    ga = rng.standard_normal((cam.height, cam.width)).astype(F32)
    ref, margin, clamped = replay(g, cam, s, d["mu"], d["conic"], d["depth"], d["rect"], gc, ga)
    assert margin > 1e-6 and clamped >= 3  # (decisions clear of the rounding of exp2)
    grads = R.backward(saved, [torch.from_numpy(gc).cuda()], None, [torch.from_numpy(ga).cuda()])
    for k, v in grads.items():
        assert torch.isfinite(v).all(), k
    for k in ref:
        got = grads[k].cpu().numpy().astype(np.float64).reshape(ref[k].shape)
        ok = close(got, ref[k])
        assert ok.all(), (k, got[~ok][:4], ref[k][~ok][:4])


@pytest.mark.parametrize("tile", [8, 16, 32])
def test_second_pixel_close_to_the_centre(R, tile):
    # one pixel a splat has a gradient: the lower one of a lane's two (tiles of 16 and 32), its centre a
    # 256th of a pixel below the splat's.  dL/d(conic C) is then u dy^2 with dy^2 = 1.5e-5, which is
    # lost (6e-8 of u) if it is formed from the upper pixel's offset
    w = h = 128
    f, z, d = 2000.0, 2.0, 2.0 ** -8
    cam = scenes.Camera(w, h, f, f, w / 2.0, h / 2.0, I3, Z3)
    x, y = (a.reshape(-1) for a in np.meshgrid(np.arange(9, w, 16), np.arange(9, h, 16)))
    n = len(x)
    means = np.stack([(x - w / 2.0) * z / f, (y - d - h / 2.0) * z / f, np.full(n, z)], 1)
    g = scenes.random_gaussians(np.random.default_rng(5), means, 0)
    g.scales = (z / f * np.linspace(0.5, 1.5, n)[:, None] * np.ones((1, 3))).astype(F32)
    g.quats = np.tile([1, 0, 0, 0], (n, 1)).astype(F32)
    g.opacities = np.linspace(0.3, 0.8, n).astype(F32)
    s = settings(tile=tile)
    say("moments", tile)
    _, images, saved = run_fwd(R, g, [cam], s)
    gc = np.zeros((3, h, w), F32)
    gc[:, y, x] = 1.0
    grads = R.backward(saved, [torch.from_numpy(gc).cuda()])
    orc = oracle_for(g, [cam], s)
    orc.forward()
    ref = orc.backward([gc.astype(np.float64)], None, None)["scales"][:, 1]
    got = grads["scales"].cpu().numpy().astype(np.float64)[:, 1]
    # some forty roundings of 6e-8 between the pixel and the scale
    np.testing.assert_allclose(got, ref, rtol=2e-5)


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("output", ["alpha", "colour", "depth"])
def test_nan_gradient_stays_with_its_pixel(R, tile, output):
    # two splats of one wavefront that share no pixel: a NaN in an output's gradient at a pixel of the
    # first leaves the shape, opacity and place of the second as they are without it
    f, z = 100.0, 2.0
    cam = scenes.Camera(tile, tile, f, f, tile / 2.0, tile / 2.0, I3, Z3)
    px = np.array([[1.0, 3.0], [min(tile, 16) - 2.0, 4.0]])
    means = np.concatenate([(px - tile / 2.0) * z / f, np.full((2, 1), z)], 1)
    g = scenes.random_gaussians(np.random.default_rng(6), means, 0)
    g.scales = np.full((2, 3), 0.5 * z / f, F32)
    g.opacities = np.full(2, 0.7, F32)
    _, images, saved = run_fwd(R, g, [cam], settings(tile=tile, lowpass=0.1))
    d = saved.debug_export()
    assert d["n_used"].max() == 1  # no pixel takes both
    rng = np.random.default_rng(7)
    out = [rng.standard_normal(k).astype(F32) for k in ((3, tile, tile), (tile, tile), (tile, tile))]
    say("nan", tile, output)

    def run():
        c, e, a = (torch.from_numpy(v.copy()).cuda() for v in out)
        return R.backward(saved, [c], [e], [a])

    clean = run()
    out[("colour", "depth", "alpha").index(output)][..., 3, 1] = np.nan
    bad = run()
    # (the sums of colour and depth gradients take the pixel's gradient times a weight of zero, and the
    # depth's goes on into the means)
    for k in ("scales", "quats", "opacities") + (("means",) if output != "depth" else ()):
        assert torch.isnan(bad[k][0]).any(), k
        assert torch.equal(bad[k][1], clean[k][1]), k  # (one sum a value: no order to differ in)
