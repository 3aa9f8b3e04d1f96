"""Compositing with several waves per tile: on both sides of each line of the
rule that picks how many (by the tile count of the call), and at list lengths
around the batches a tile's list is walked in (groups of 4 records, sub-batches
of 64, batches of 64 per wave), the image and every gradient are the FP64
oracle's, and the one-call step is bitwise the two passes."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2607_14481_amd import scenes as S

from ._util import compare_grads, compare_view, gpu_render, log, params_to_device, poses_to_device

pytestmark = pytest.mark.gpu


def _check(scene, cam, tile_h, label):
    import torch
    from paper_2607_14481_amd.rasterizer import GaussianRasterizer
    up = S.random_upstream(17, (cam.height, cam.width, 3))
    bg = (0.1, 0.2, 0.3)
    ref = O.render(scene, cam, bg=bg, dL_dimg=up)
    out = gpu_render(scene, [cam], bg=bg, upstream=[up], tile_h=tile_h)
    compare_view(out["imgs"][0], ref, label)
    compare_grads(out, ref, label)
    rast = GaussianRasterizer([cam], scene.sh_degree, tile_h=tile_h)
    params, w2c = params_to_device(scene), poses_to_device([cam])
    target = torch.full((3 * cam.width * cam.height,), 0.35, device="cuda")
    rgb, ws = rast.forward(params, w2c, bg)
    grads, g_w2c, twist = rast.backward_l1(ws, params, w2c, bg, rgb, target)
    rgb1, _, grads1, g_w2c1, twist1 = rast.step_l1(params, w2c, bg, target)
    for a, b in zip([rgb, *grads, g_w2c, twist], [rgb1, *grads1, g_w2c1, twist1]):
        assert torch.equal(a, b), label


@pytest.mark.parametrize("tile_h,tiles_x,tiles_y", [
    (8, 64, 50), (8, 97, 33), (16, 64, 50), (16, 97, 33), (16, 75, 60), (16, 82, 55),
    (32, 64, 50), (32, 97, 33), (32, 75, 60), (32, 82, 55), (32, 120, 75), (32, 107, 85)])
def test_tile_count_lines(tile_h, tiles_x, tiles_y):
    w, h = 16 * tiles_x - 5, tile_h * tiles_y - 3
    log(f"wave split: {tiles_x * tiles_y} tiles of 16x{tile_h} ({w}x{h})")
    wl = S.small_view(seed=21, n=600, width=w, height=h, sh_degree=1, log_scale_mean=-2.5)
    _check(wl.scene, wl.cameras[0], tile_h, f"{tiles_x * tiles_y} tiles 16x{tile_h}")


@pytest.mark.parametrize("height", [13, 976])  # one row of tiles, or 4,575 tiles (one wave each)
@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 64, 65, 255, 256, 257, 321])
def test_list_lengths(n, height):
    width = 1200 if height > 100 else 14
    rng = np.random.Generator(np.random.PCG64(100 + n))
    wl = S.small_view(seed=31, n=n, width=width, height=height, sh_degree=0)
    sc = wl.scene
    # every Gaussian reaches the first tile, faint enough that the list is used to its end
    cam = S.Camera(width, height, 16.0, 16.0, 7.0, 6.0, np.eye(4, dtype=np.float32))
    means = np.stack([rng.uniform(-0.6, 0.6, n), rng.uniform(-0.6, 0.6, n), rng.uniform(2.0, 3.0, n)], 1)
    scene = S.Scene(means.astype(np.float32), np.full((n, 3), -2.0, np.float32) + sc.log_scales * 0.1, sc.quats,
                    rng.uniform(0.008, 0.025, n).astype(np.float32), sc.sh, 0)
    log(f"list of {n} records, image {width}x{height}")
    _check(scene, cam, 16, f"list {n} h{height}")


@pytest.mark.parametrize("tile_h", [16, 32])
@pytest.mark.parametrize("tiles_x,tiles_y", [(200, 200), (201, 200)])
def test_forward_tile_count_line(tile_h, tiles_x, tiles_y):
    """40,000 tiles and more: the forward takes fewer waves a tile, the same image to the bit (the one-call
    step, whose waves the rule leaves alone, against it, and the work it counts)."""
    import torch
    from paper_2607_14481_amd import gsr
    from paper_2607_14481_amd.rasterizer import GaussianRasterizer
    w, h = 16 * tiles_x - 5, tile_h * tiles_y - 3
    wl = S.small_view(seed=23, n=3000, width=w, height=h, sh_degree=0, log_scale_mean=-2.0)
    cam = wl.cameras[0]
    params, w2c = params_to_device(wl.scene), poses_to_device([cam])
    target = torch.full((3 * w * h,), 0.35, device="cuda")
    rast = GaussianRasterizer([cam], 0, tile_h=tile_h)
    rgb, ws = rast.forward(params, w2c)
    grads, _, twist = rast.backward_l1(ws, params, w2c, (0.0, 0.0, 0.0), rgb, target)
    step = rast.step_l1(params, w2c, (0.0, 0.0, 0.0), target)
    for a, b in zip([rgb, *grads, twist], [step[0], *step[2], step[4]]):
        assert torch.equal(a, b)
    other = GaussianRasterizer([cam], 0, tile_h=8)
    rast.stats = other.stats = True
    counts = [gsr.query_stats(r.forward(params, w2c)[1])["contributors"] for r in (rast, other)]
    log(f"{tiles_x * tiles_y} tiles of 16x{tile_h}: {counts} contributors")
    assert counts[0] > 0 and abs(counts[0] - counts[1]) <= 1e-5 * counts[1]
