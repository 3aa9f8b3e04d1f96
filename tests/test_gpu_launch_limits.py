"""Levels of more parents than one launch takes: every parent is merged, up to the
last (city-scale hierarchies of hundreds of millions of leaves)."""
import pytest

from paper_2607_14481_amd import gsr

pytestmark = pytest.mark.gpu


def test_level_beyond_one_launch():
    """277.2 M leaves of degree 2 in pairs: 138.6 M parents, more than 2^32 threads with one
    for each of their 27 SH values and four for the geometry."""
    import torch
    n, degree, branching = 277_200_001, 2, 2
    total = int(gsr.hierarchy_layout(n, 1, branching)[-1])
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 4 * 40 * total + (4 << 30):
        pytest.skip("needs 70 GB of device memory")
    g = torch.Generator("cuda").manual_seed(3)
    nodes = [torch.empty((total, *s), device="cuda") for s in ((3,), (3,), (4,), (), (9, 3))]
    for t in nodes:
        t[:n].uniform_(0.1, 0.9, generator=g)
        t[n:] = -7.0
    parent, kids = (torch.full((total,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    gsr.hierarchy_build(nodes, degree, n, 1, branching, parent=parent, child_count=kids)
    assert not any((t[n:].reshape(total - n, -1)[:, -1] == -7.0).any() for t in nodes)
    assert int(parent[:n].min()) == n and int(parent[n - 1]) == total - 1 and (parent[n:] == -1).all()
    assert (kids[n:total - 1] == 2).all() and int(kids[total - 1]) == 1 and not kids[:n].any()
    for j in [*range(0, total - n - 1, 541_403), total - n - 2]:
        o, sh, mu = (nodes[k][2 * j:2 * j + 2].double() for k in (3, 4, 0))
        w = o / o.sum()
        torch.testing.assert_close(nodes[4][n + j].double(), (w[:, None, None] * sh).sum(0), rtol=1e-6, atol=1e-7)
        torch.testing.assert_close(nodes[0][n + j].double(), (w[:, None] * mu).sum(0), rtol=1e-6, atol=1e-7)
        torch.testing.assert_close(nodes[3][n + j].double(), 1 - (1 - o).prod(), rtol=1e-6, atol=1e-7)
    del nodes, parent, kids
    torch.cuda.empty_cache()
