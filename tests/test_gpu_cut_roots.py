"""Roots of the level-of-detail cut are the nodes with a negative parent, -1 or
any other value: the cut of a forest whose roots are marked with several, in
every arrangement within the four nodes a thread takes, is the FP64 reference's
through each of the three entry points."""
import numpy as np
import pytest

from oracle import hierarchy_cut as HC
from paper_2607_14481_amd import gsr
from paper_2607_14481_amd import scenes as S

from ._util import params_to_device

pytestmark = pytest.mark.gpu

INT_MIN = -2 ** 31


@pytest.mark.parametrize("marks", [(-2,), (-1, -2), (-1, -2, -3, INT_MIN)])
@pytest.mark.parametrize("n", [1, 4, 6, 1021])
def test_any_negative_parent_is_a_root(n, marks):
    import torch
    rng = np.random.default_rng(n + len(marks))
    means = np.c_[rng.uniform(0, 60, n), rng.uniform(-3, 3, n), rng.uniform(0, 3, n)]
    nodes = S._gaussian_body(rng, means, 0)
    up = np.minimum(np.arange(n) // 3 + n // 3 + 1, n)
    inner = (up > np.arange(n)) & (up < n) & (rng.random(n) < 0.5) & (n > 6)
    parent = np.where(inner, up, rng.choice(marks, n))
    counts = np.bincount(parent[inner], minlength=n)
    eye = np.array([-1.0, 0.0, 1.5])
    cam = S.pinhole(160, 120, S.look_at(eye, eye + [1.0, 0.0, 0.0]))
    pose = np.asarray(cam.world_to_cam, np.float32)
    dev = params_to_device(nodes)
    par, cnt = (torch.tensor(a.astype(np.int32), device="cuda") for a in (parent, counts))
    w2c = torch.tensor(pose, device="cuda")
    out = torch.empty(n, dtype=torch.int32, device="cuda")
    size = torch.empty(1, dtype=torch.int64, device="cuda")
    scratch = torch.empty(gsr.lib().gsr_hierarchy_cut_scratch_bytes(n), dtype=torch.uint8, device="cuda")
    for tau in (0.5, 8.0):
        focal = max(cam.fx, cam.fy)
        assert not HC.ambiguous(nodes.means, nodes.log_scales, pose, focal, tau).any()
        ref = HC.cut(nodes.means, nodes.log_scales, parent, pose, focal, tau)
        got = gsr.hierarchy_cut(dev, 0, par, cnt, cam, w2c, tau)
        np.testing.assert_array_equal(got.cpu().numpy(), ref)
        gsr.hierarchy_cut_async(dev, 0, par, cnt, cam, w2c, tau, scratch, out, size)
        np.testing.assert_array_equal(out[:int(size)].cpu().numpy(), ref)
        k = gsr.hierarchy_cut_static(dev, 0, par, cnt, cam, w2c, tau, out)
        np.testing.assert_array_equal(out[:k].cpu().numpy(), ref)
