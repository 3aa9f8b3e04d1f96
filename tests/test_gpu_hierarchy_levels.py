"""Hierarchy build at the edges of its work split: chunks of 256 children (a
whole number of parents each), up to 64 parents in several chunks per workgroup,
ragged last parents, the smallest and largest branching, levels of one node,
every spherical-harmonics row form, children of one place and of equal scales.
Every node against the FP64 oracle's merge of the GPU's own children (the same
FP32 inputs), with the tolerances of the hierarchy tests: FP64 results rounded
to FP32 once, so a relative 1e-6 of the largest coordinate and 1e-5 of a
covariance."""
import numpy as np
import pytest

from paper_2607_14481_amd import gsr
from paper_2607_14481_amd import scenes as S

from .test_gpu_hierarchy import _compare_node
from ._util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_leaves,levels,branching,deg", [
    (1, 3, 2, 3), (2, 1, 2, 0), (5, 0, 8, 1), (63, 2, 64, 2), (64, 2, 64, 3), (65, 2, 64, 0), (255, 3, 2, 1),
    (257, 2, 3, 3), (2047, 2, 8, 0), (2049, 1, 8, 2), (40_001, 1, 5, 0), (300_007, 1, 2, 0), (280_000, 1, 8, 0),
    (1_100_003, 1, 8, 0), (70_000, 1, 64, 1)])
def test_every_level(n_leaves, levels, branching, deg):
    import torch
    from oracle import hierarchy_merge as M
    rng = np.random.default_rng(n_leaves + branching)
    means = np.c_[rng.uniform(0, 50, n_leaves), rng.uniform(-3, 3, n_leaves), rng.uniform(0, 3, n_leaves)]
    means[n_leaves // 2: n_leaves // 2 + 40] = means[n_leaves // 2]  # one place
    leaves = S._gaussian_body(rng, means, deg)
    arrays = [np.array(getattr(leaves, k), np.float32) for k in ("means", "log_scales", "quats", "opacities", "sh")]
    arrays[1][: n_leaves // 3] = -2.0  # spheres
    ls = gsr.hierarchy_layout(n_leaves, levels, branching)
    total = int(ls[-1])
    bufs = [torch.zeros((total,) + a.shape[1:], dtype=torch.float32, device="cuda") for a in arrays]
    for b, a in zip(bufs, arrays):
        b[:n_leaves] = torch.tensor(a, device="cuda")
    par = torch.full((total,), 77, dtype=torch.int32, device="cuda")
    cnt = torch.full((total,), 77, dtype=torch.int32, device="cuda")
    gsr.hierarchy_build(bufs, deg, n_leaves, levels, branching, parent=par, child_count=cnt)
    torch.cuda.synchronize()
    got = [b.cpu().numpy() for b in bufs]
    par, cnt = par.cpu().numpy(), cnt.cpu().numpy()
    for a, g in zip(arrays, got):
        np.testing.assert_array_equal(g[:n_leaves], a)
    for l in range(len(ls) - 1):
        idx = np.arange(int(ls[l]), int(ls[l + 1]))
        up = int(ls[l + 1]) + (idx - int(ls[l])) // branching if l + 2 < len(ls) else np.full(len(idx), -1)
        np.testing.assert_array_equal(par[idx], up)
        if l == 0:
            assert np.all(cnt[idx] == 0)
            continue
        below = int(ls[l] - ls[l - 1])
        first = (idx - int(ls[l])) * branching
        np.testing.assert_array_equal(cnt[idx], np.minimum(branching, below - first))
        pick = np.unique(np.r_[np.arange(min(len(idx), 130)), np.arange(max(0, len(idx) - 130), len(idx)),
                               rng.integers(0, len(idx), 60)])
        for j in pick:
            c = slice(int(ls[l - 1]) + j * branching, int(ls[l - 1]) + min((j + 1) * branching, below))
            ref = M.merge_group(*[g[c].astype(np.float64) for g in got])
            _compare_node([g[int(ls[l]) + j].astype(np.float64) for g in got], ref, f"level {l} node {j}")
    log(f"build {n_leaves} leaves, {levels} levels, branching {branching}, degree {deg}: {total} nodes")


@pytest.mark.parametrize("n_leaves,branching,deg", [
    (65_535, 2, 3), (65_533, 2, 3), (98_303, 3, 2), (98_301, 3, 2), (163_836, 5, 3), (524_287, 2, 0), (1_048_573, 4, 1),
    (1_835_003, 7, 2), (1_572_862, 6, 3)])
def test_levels_in_launches_apart(n_leaves, branching, deg):
    """Levels at and above the sizes from which the SH rows have a launch of their own
    (32,768 and 262,144 parents), and below."""
    test_every_level(n_leaves, 1, branching, deg)
