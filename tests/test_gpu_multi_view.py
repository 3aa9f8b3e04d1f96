"""Projection of several views in one call, forward and backward, at the edges
of its work split: groups of 64 Gaussians, passes of 256 visible items, several
groups per workgroup, spherical-harmonics rows staged once for several views.
The images and gradients of one call over all views are those of one call per
view, added up.

Tolerances: a view's image is composited from the same records, so it may
differ by rounding of the colours only (a few 2^-24).  A gradient is a sum, in
another order, of at most 32 views' parts and of the tiles' parts in them:
relative to the norm 32 * 2^-24 = 2e-6, and cancellation between the parts may
cost one digit and a half."""
import numpy as np
import pytest

from paper_2607_14481_amd import scenes as S
from paper_2607_14481_amd.rasterizer import GaussianRasterizer

from ._util import log, params_to_device, poses_to_device, rel_err

pytestmark = pytest.mark.gpu

IMAGE_TOL, GRAD_TOL = 2e-6, 6e-5


def _scene(n, deg):
    rng = np.random.Generator(np.random.PCG64(50 + n + deg))
    means = np.stack([rng.uniform(-2, 2, n), rng.uniform(-2, 2, n), rng.uniform(3.0, 6.0, n)], 1)
    quats = rng.standard_normal((n, 4))
    quats /= np.linalg.norm(quats, axis=1, keepdims=True)
    small = -3.0 if n < 5000 else -4.5
    return S.Scene(means.astype(np.float32), rng.normal(small, 0.4, (n, 3)).astype(np.float32),
                   quats.astype(np.float32), rng.uniform(0.05, 0.9, n).astype(np.float32),
                   rng.uniform(-0.4, 0.4, (n, (deg + 1) ** 2, 3)).astype(np.float32), deg)


def _cameras(views):
    cams = []
    for v in range(views):
        a = 0.25 * (v / max(views - 1, 1) - 0.5)
        pose = np.eye(4, dtype=np.float32)
        pose[:3, :3] = [[np.cos(a), 0, np.sin(a)], [0, 1, 0], [-np.sin(a), 0, np.cos(a)]]
        pose[2, 3] = -40.0 if views > 2 and v == 1 else 0.1 * v  # one view sees nothing
        w, h = 40 + 8 * (v % 3), 33 + 5 * (v % 4)
        cams.append(S.Camera(w, h, 0.9 * w, 0.9 * w, 0.5 * w, 0.5 * h, pose))
    return cams


def _run(sc, params, cams, upstream):
    import torch
    rast = GaussianRasterizer(cams, sc.sh_degree)
    w2c = poses_to_device(cams)
    rgb, ws = rast.forward(params, w2c, (0.1, 0.2, 0.3))
    grads, g_w2c, twist = rast.backward(ws, params, w2c, (0.1, 0.2, 0.3), rgb, upstream)
    torch.cuda.synchronize()
    return [t.cpu().numpy().astype(np.float64) for t in (rgb, *grads, g_w2c, twist)]


@pytest.mark.parametrize("n,views,deg", [
    (1, 3, 3), (63, 3, 0), (64, 2, 1), (65, 4, 2), (257, 7, 3), (1000, 32, 1), (700, 32, 2), (129, 3, 1),
    (33_000, 32, 0), (33_000, 32, 1), (33_000, 32, 2), (33_000, 32, 3), (140_000, 3, 3), (140_000, 8, 2)])
def test_views_add_up(n, views, deg):
    import torch
    sc, cams = _scene(n, deg), _cameras(views)
    params = params_to_device(sc)
    sizes = [3 * c.width * c.height for c in cams]
    up = torch.tensor(np.random.Generator(np.random.PCG64(3)).uniform(-1, 1, sum(sizes)).astype(np.float32),
                      device="cuda")
    log(f"{n} Gaussians, {views} views, degree {deg}")
    got = _run(sc, params, cams, up)
    ref, at = None, 0
    for v, c in enumerate(cams):
        one = _run(sc, params, [c], up[at:at + sizes[v]].contiguous())
        assert np.abs(got[0][at:at + sizes[v]] - one[0]).max() <= IMAGE_TOL
        if np.any(one[6]):
            assert rel_err(got[6][v], one[6][0]) <= GRAD_TOL
            assert rel_err(got[7][v], one[7][0]) <= GRAD_TOL
        else:
            assert not np.any(got[6][v]) and not np.any(got[7][v])
        ref = one[1:6] if ref is None else [a + b for a, b in zip(ref, one[1:6])]
        at += sizes[v]
    for a, b, name in zip(got[1:6], ref, ("means", "log_scales", "quats", "opacities", "sh")):
        if n > 1:
            log(f"  {name}: {rel_err(a, b):.2e}")
        assert rel_err(a, b) <= GRAD_TOL, name
