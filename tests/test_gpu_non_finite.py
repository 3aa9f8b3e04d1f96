"""Values that are not finite stay where they belong, in every form of the
compositing (waves per tile, slabs per wave): an upstream gradient of a pixel
reaches the Gaussians that composite on that pixel, an infinite colour the
pixels its Gaussian composites on, and a Gaussian at infinity no pixel.  The footprints come from
the projection formula in FP64; everything outside them is bit for bit what it is
with a finite value in that place."""
import numpy as np
import pytest

from paper_2607_14481_amd import gsr
from paper_2607_14481_amd import scenes as S
from paper_2607_14481_amd.rasterizer import GaussianRasterizer

from ._util import params_to_device, poses_to_device

pytestmark = pytest.mark.gpu

# (width, height, tile height): one to four waves a tile, one to eight slabs a wave
FORMS = [(96, 80, 4), (96, 80, 8), (96, 80, 16), (96, 80, 32), (1280, 720, 16), (1920, 1080, 8), (1920, 1080, 16),
         (1920, 1080, 32), (2560, 1440, 32), (2752, 1568, 16), (3072, 1728, 32)]


def _scene(w, h, n=240):
    """Faint round Gaussians within 30 pixels of the image's centre, and their alphas [n, 100, 100] there."""
    rng = np.random.default_rng(w + h)
    f, z = 300.0, rng.uniform(2.0, 3.0, n)
    px = rng.uniform(-30, 30, (n, 2))
    means = np.c_[px[:, 0] * z / f, px[:, 1] * z / f, z].astype(np.float32)
    log_scales = np.repeat(np.log(rng.uniform(0.5, 4.0, n) * z / f), 3).reshape(n, 3).astype(np.float32)
    opac = rng.uniform(0.05, 0.3, n).astype(np.float32)
    quats = np.tile(np.float32([1, 0, 0, 0]), (n, 1))
    sc = S.Scene(means, log_scales, quats, opac, rng.uniform(-0.4, 0.4, (n, 1, 3)).astype(np.float32), 0)
    cam = S.Camera(w, h, f, f, 0.5 * w, 0.5 * h, np.eye(4, dtype=np.float32))
    m, s2 = means.astype(np.float64), np.exp(2 * log_scales[:, 0].astype(np.float64))
    x, y = m[:, 0] / m[:, 2], m[:, 1] / m[:, 2]
    k = s2 * (f / m[:, 2]) ** 2
    a, b, c = k * (1 + x * x) + 0.3, k * x * y, k * (1 + y * y) + 0.3
    ys, xs = np.mgrid[-50:50, -50:50] + 0.5
    dx, dy = xs[None] - f * x[:, None, None], ys[None] - f * y[:, None, None]
    a, b, c = (t[:, None, None] for t in (a, b, c))
    alpha = opac[:, None, None] * np.exp(-0.5 * (c * dx * dx - 2 * b * dx * dy + a * dy * dy) / (a * c - b * b))
    assert np.exp(np.log1p(-alpha).sum(0)).min() > 1e-3  # no pixel stops early
    return sc, cam, alpha


def _same(got, ref, rows, what):
    for name, x, y in zip(("means", "log_scales", "quats", "opacities", "sh"), got, ref):
        x, y = x.cpu().numpy()[rows], y.cpu().numpy()[rows]
        assert np.isfinite(x).all(), (what, name)
        np.testing.assert_array_equal(x, y, err_msg=f"{what}: {name}")


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("w,h,tile_h", FORMS)
def test_upstream_of_one_pixel(w, h, tile_h, value):
    import torch
    sc, cam, alpha = _scene(w, h)
    at = alpha[:, 53, 46]  # pixel (w / 2 - 4, h / 2 + 3)
    assert (np.abs(255 * at - 1) > 1e-4).all()
    on = at >= 1 / 255
    assert 5 < on.sum() < len(on) / 2
    rast = GaussianRasterizer([cam], 0, tile_h=tile_h)
    params, w2c = params_to_device(sc), poses_to_device([cam])
    rgb, ws = rast.forward(params, w2c)
    up = torch.rand(3, h, w, generator=torch.Generator("cuda").manual_seed(1), device="cuda") - 0.5
    grads = []
    for x in (value, 0.0):
        up[:, h // 2 + 3, w // 2 - 4] = x
        g, _, _ = rast.backward(ws, params, w2c, (0.0, 0.0, 0.0), rgb, up.reshape(-1))
        grads.append([t.clone() for t in g])
    _same(*grads, ~on, "not on the pixel")
    assert not torch.isfinite(grads[0][4].cpu()[torch.tensor(on)]).all(dim=-1).any()


@pytest.mark.parametrize("w,h,tile_h", FORMS)
def test_gaussian_at_infinity(w, h, tile_h):
    """A mean at infinity in front of the camera has no centre on the image and
    composites nowhere: the image, the other Gaussians' gradients and its own of
    the shape and the opacity (zero) are those without it."""
    import torch
    sc, cam, _ = _scene(w, h)
    params, w2c = params_to_device(sc), poses_to_device([cam])
    last = torch.arange(len(sc.means), device="cuda") == len(sc.means) - 1
    target = torch.rand(3 * h * w, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    out = []
    for far in (True, False):
        p = [t.clone() for t in params]
        if far:
            p[0][last] = torch.tensor([0.0, 0.0, np.inf], device="cuda")
        else:
            p[3][last] = 0.0  # culled
        rast = GaussianRasterizer([cam], 0, tile_h=tile_h)
        rgb, ws = rast.forward(p, w2c)
        grads, _, _ = rast.backward(ws, p, w2c, (0.0, 0.0, 0.0), rgb, target - 0.5)
        step = rast.step_l1(p, w2c, (0.0, 0.0, 0.0), target)
        out.append(([rgb, step[0]], grads, step[2]))
    for x, y in zip(out[0][0], out[1][0]):
        np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())
    for k in (1, 2):
        _same(out[0][k], out[1][k], ~last.cpu().numpy(), "the others")
        for g in out[0][k][1:4]:
            assert (g[last] == 0).all()


@pytest.mark.parametrize("w,h,tile_h", FORMS)
def test_infinite_colour(w, h, tile_h):
    """One Gaussian with an infinite red: the pixels outside its footprint and the
    gradients of the Gaussians that share none of its pixels are those with a
    finite red."""
    import torch
    sc, cam, alpha = _scene(w, h)
    near = np.abs(255 * alpha - 1) < 1e-4
    on = alpha >= 1 / 255
    shares = ((on | near)[:, None] & (on | near)[None]).any((2, 3))
    j = int(np.argmin(shares.sum(1) + 1000.0 * (on.sum((1, 2)) < 20)))
    assert not near[j].any() and (~shares[j]).sum() > 20
    outside = np.ones((h, w), bool)
    a, b = min(50, h // 2), min(50, w // 2)  # (the alphas' window is 100 x 100, the image may be smaller)
    outside[h // 2 - a:h // 2 + a, w // 2 - b:w // 2 + b] = ~on[j][50 - a:50 + a, 50 - b:50 + b]
    params, w2c = params_to_device(sc), poses_to_device([cam])
    target = torch.rand(3 * h * w, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    up = torch.rand(3 * h * w, generator=torch.Generator("cuda").manual_seed(2), device="cuda") - 0.5
    out = []
    for red in (np.inf, 0.2):
        p = [t.clone() for t in params]
        p[4][j, 0, 0] = red
        rast = GaussianRasterizer([cam], 0, tile_h=tile_h)
        rgb, ws = rast.forward(p, w2c)
        grads, _, _ = rast.backward(ws, p, w2c, (0.0, 0.0, 0.0), rgb, up)
        records = gsr.export_state(ws, p, 0, [cam], cfg=rast.cfg)["records"]
        assert np.isinf(records[j, 6]) == (red == np.inf) and np.isfinite(records[:, 7:9]).all()
        step = rast.step_l1(p, w2c, (0.0, 0.0, 0.0), target)
        out.append(([rgb, step[0]], grads, step[2]))
    for x, y in zip(out[0][0], out[1][0]):
        x, y = (t.cpu().numpy().reshape(3, h, w) for t in (x, y))
        np.testing.assert_array_equal(x[:, outside], y[:, outside])
        assert np.isinf(x[0, ~outside]).all() and np.isfinite(x[1:]).all()
    for k in (1, 2):
        _same(out[0][k], out[1][k], ~shares[j], "the others")
