"""The pairs' counting sort by tile at its edges: bands of tile rows (one, two,
three and more bands than the image has rows, and images whose tile counters
need several bands), views of different sizes with one that sees nothing, item
counts around the groups dealt to the workgroups, boxes of one tile and of the
whole image.  Whole numbers, so the pair list and the ranges must equal the
oracle's exactly."""
import numpy as np
import pytest

from paper_2607_14481_amd import gsr
from paper_2607_14481_amd import scenes as S
from paper_2607_14481_amd.rasterizer import GaussianRasterizer

from ._util import log, oracle_bin_from_gpu_state, params_to_device, poses_to_device

pytestmark = pytest.mark.gpu


def _scene(n, seed, reach, every):
    rng = np.random.Generator(np.random.PCG64(seed))
    means = np.stack([rng.uniform(-reach, reach, n), rng.uniform(-reach, reach, n), rng.uniform(2.0, 9.0, n)], 1)
    log_scales = rng.uniform(-5.0, -2.5, (n, 3))
    log_scales[::every] = 1.5  # boxes of most of the image
    quats = rng.standard_normal((n, 4))
    quats /= np.linalg.norm(quats, axis=1, keepdims=True)
    return S.Scene(means.astype(np.float32), log_scales.astype(np.float32), quats.astype(np.float32),
                   rng.uniform(0.1, 0.9, n).astype(np.float32), rng.uniform(-0.3, 0.3, (n, 1, 3)).astype(np.float32), 0)


def _camera(width, height, away=False):
    pose = np.eye(4, dtype=np.float32)
    if away:
        pose[2, 3] = -50.0  # everything behind the camera
    f = 0.5 * max(width, height)
    return S.Camera(width, height, f, f, 0.5 * width, 0.5 * height, pose)


def _check(n, cams, tile_h, capacity, label, reach=2.0, every=37):
    import torch
    sc = _scene(n, 7 + n, reach, every)
    rast = GaussianRasterizer(cams, 0, tile_h=tile_h, sync=True)
    params, w2c = params_to_device(sc), poses_to_device(cams)
    _, ws = rast.forward(params, w2c, (0.0, 0.0, 0.0), ws=rast.workspace(n, capacity))
    torch.cuda.synchronize()
    st = gsr.export_state(ws, params, 0, cams, rast.cfg)
    tiles, items, ranges = oracle_bin_from_gpu_state(st, cams, n, tile_h)
    log(f"{label}: {st['M']} pairs")
    assert st["M"] == len(tiles)
    np.testing.assert_array_equal(st["pair_tiles"].astype(np.uint64), tiles)
    np.testing.assert_array_equal(st["pair_items"].astype(np.uint64), items)
    gr = st["ranges"].astype(np.int64)
    nonempty = ranges[:, 1] > ranges[:, 0]
    np.testing.assert_array_equal(gr[nonempty], ranges[nonempty])
    assert np.all(gr[~nonempty, 0] == gr[~nonempty, 1])
    # each record's last word: the item's first pair in (item, tile) order
    seen = st["tile_counts"] > 0
    first = np.cumsum(st["tile_counts"].astype(np.int64)) - st["tile_counts"]
    np.testing.assert_array_equal(st["records"][seen, 11].view(np.uint32), first[seen])


@pytest.mark.parametrize("capacity", [60_000, 2_600_000, 2_600_001, 6_000_000, 40_000_000])
@pytest.mark.parametrize("width,height,tile_h", [(333, 210, 16), (250, 131, 8), (5, 3, 32)])
def test_bands(capacity, width, height, tile_h):
    _check(700, [_camera(width, height)], tile_h, capacity, f"{width}x{height}/{tile_h} capacity {capacity}")


@pytest.mark.parametrize("n", [1, 15, 16, 17, 1000, 4097])
def test_views(n):
    cams = [_camera(200, 120), _camera(90, 40, away=True), _camera(64, 300), _camera(16, 16), _camera(31, 17, away=True)]
    _check(n, cams, 16, 16_000_000 if n < 100 else 2_000_000, f"{n} items, 5 views")


@pytest.mark.parametrize("n", [60, 20_000])
def test_many_tiles(n):
    # 256 x 300 tiles of 16x8: counters for 76,800 tiles exceed one workgroup's LDS
    _check(n, [_camera(4096, 2400), _camera(40, 24)], 8, 9_000_000 if n > 100 else 600_000, f"{n} items, 76,800 tiles",
           reach=3.0, every=37 if n < 100 else 2000)


@pytest.mark.parametrize("n,width,height,tile_h,capacity", [
    (8192, 120, 150, 4, 32 * 32768), (8192, 120, 150, 4, 32 * 32768 + 1),  # 38 rows of tiles: bands of two
    (8193, 120, 150, 4, 32 * 32768), (1, 17, 4, 4, 32768), (300, 17, 4, 4, 32769),
    (1023, 2000, 40, 8, 5 * 32768), (1025, 2000, 40, 8, 5 * 32768 + 1), (9000, 64, 64, 16, 70_000)])
def test_one_launch_lines(n, width, height, tile_h, capacity):
    _check(n, [_camera(width, height)], tile_h, capacity, f"{n} items, {width}x{height}/{tile_h}, capacity {capacity}",
           every=400)


@pytest.mark.parametrize("tiles_x,tiles_y", [(32, 32), (25, 41), (64, 32), (61, 34), (64, 33), (96, 32), (81, 38)])
def test_thread_runs(tiles_x, tiles_y):
    """Bands of 1,024, 2,048 and 3,072 tiles and one or a few more: a thread's run is of one or three."""
    _check(9000, [_camera(16 * tiles_x, 16 * tiles_y - 5)], 16, 900_000, f"{tiles_x * tiles_y} tiles", every=900)
