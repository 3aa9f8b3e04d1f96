"""Edges of two kernels' work split: the Adam step's row forms and its groups of
64 listed Gaussians (bitwise the dense step's rows), against the FP64 update oracle with the tolerances of the update
tests; the cut's four nodes per thread, over forests whose siblings lie
anywhere, where the cut is the FP64 reference's exactly."""
from types import SimpleNamespace

import numpy as np
import pytest

from oracle import update as U
from paper_2607_14481_amd import gsr
from paper_2607_14481_amd import scenes as S

from .test_gpu_hierarchy import _check
from .test_gpu_update import LRS, _acfg, _compare, _dev, _host, _random_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 200])
def test_adam_groups(n, deg):
    import torch
    rng = np.random.default_rng(100 * n + deg)
    p, shapes = _random_state(rng, n, deg)
    zero = {k: np.zeros(s, np.float32) for k, s in shapes.items()}
    P, M, V = _dev(p), _dev(zero), _dev(zero)
    g = {k: rng.standard_normal(s).astype(np.float32) for k, s in shapes.items()}
    gsr.adam_step(P, _dev(g), M, V, deg, 1, _acfg(gsr))
    torch.cuda.synchronize()
    refP, refM, refV = U.adam(p, g, zero, zero, 1, LRS, 0.9, 0.999, 1e-8)
    _compare(_host(P), refP, "params")
    _compare(_host(M), refM, "exp_avg")
    _compare(_host(V), refV, "exp_avg_sq", rtol=1e-4, atol=1e-9)


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [32_767, 32_768, 32_831])  # the flat walk; listed rows, whole and ragged last groups
def test_sparse_adam_is_the_dense_step_on_the_seen(n, deg):
    import torch
    from paper_2607_14481_amd.rasterizer import GaussianRasterizer
    from ._util import params_to_device, poses_to_device
    wl = S.small_view(seed=n + deg, n=n, width=96, height=72, sh_degree=deg, xy_half=5.0, log_scale_mean=-4.0)
    rast = GaussianRasterizer(wl.cameras, deg)
    params = params_to_device(wl.scene)
    _, ws = rast.forward(params, poses_to_device(wl.cameras))
    st = gsr.export_state(ws, params, deg, wl.cameras, rast.cfg)
    seen = torch.tensor(st["tile_counts"].astype(np.int64) > 0, device="cuda")
    assert 0 < int(seen.sum()) < n
    g = [torch.randn_like(t) for t in params]
    both = []
    for sparse in (True, False):
        p, m, v = [t.clone() for t in params], [0.1 * t for t in g], [t * t for t in g]
        kw = dict(ws=ws, cams=wl.cameras, cfg=rast.cfg) if sparse else {}
        gsr.adam_step(p, g, m, v, deg, 2, _acfg(gsr, sparse=sparse), **kw)
        both.append((p, m, v))
    start = (params, [0.1 * t for t in g], [t * t for t in g])
    for a, b, c in zip(*both, start):
        for x, y, z in zip(a, b, c):
            assert torch.equal(x[seen], y[seen]) and torch.equal(x[~seen], z[~seen])


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 1023, 1025, 5002])
def test_cut_of_any_forest(n):
    rng = np.random.default_rng(n)
    means = np.c_[rng.uniform(0, 60, n), rng.uniform(-3, 3, n), rng.uniform(0, 3, n)]
    nodes = S._gaussian_body(rng, means, 0)
    # parents anywhere behind their children, runs of siblings and single nodes mixed; some roots
    up = np.minimum(np.arange(n) // rng.integers(1, 6, n) + n // 3 + 1, n)
    parent = np.where((up > np.arange(n)) & (up < n) & (rng.random(n) < 0.97), up, -1)
    h = SimpleNamespace(nodes=nodes, parent=parent, child_count=np.bincount(parent[parent >= 0], minlength=n))
    eye = np.array([-1.0, 0.0, 1.5])
    cam = S.pinhole(160, 120, S.look_at(eye, eye + [1.0, 0.0, 0.0]))
    for tau in (0.5, 8.0):
        _check(h, cam, f"forest of {n}, tau {tau}", tau)


@pytest.mark.parametrize("n", [8192 * 1024, 8192 * 1024 + 1])  # blocks of flags added up by each block, or scanned
def test_cut_of_many_nodes(n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    big = torch.rand(n, generator=g, device="cuda") < 0.4  # inner nodes far coarser than the threshold: they descend
    means = torch.zeros((n, 3), device="cuda")
    means[:, 2] = 10.0
    log_scales = torch.where(big, 3.0, -8.0)[:, None].repeat(1, 3).contiguous()
    nodes = [means, log_scales, torch.ones((n, 4), device="cuda"), torch.ones(n, device="cuda"),
             torch.zeros((n, 1, 3), device="cuda")]
    parent = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    cam = S.Camera(64, 48, 50.0, 50.0, 32.0, 24.0, np.eye(4, dtype=np.float32))
    cut = gsr.hierarchy_cut(nodes, 0, parent, big.to(torch.int32), cam, torch.eye(4, device="cuda"), 1.5)
    assert torch.equal(cut.to(torch.int64), torch.nonzero(~big)[:, 0])
