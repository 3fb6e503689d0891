"""A tree of more than 2^25 leaves (of one point each), whose grids of one wave
per leaf have more than 2^31 work items: a lattice, whose neighbours and groups
are known."""
import pytest

pytestmark = pytest.mark.gpu

SIDE = 324  # 34 012 224 points


def test_more_leaves_than_2_25():
    import torch
    from paper_2604_05885_amd import api
    n = SIDE ** 3
    g = torch.arange(SIDE, dtype=torch.float32, device="cuda")
    p = torch.stack(torch.meshgrid(g, g, g, indexing="ij"), dim=-1).reshape(-1, 3).contiguous()
    i = torch.arange(n, dtype=torch.int32, device="cuda")
    with api.jz_build(p, api.default_opts(leaf_max=1, list_per_node=16.0)) as t:
        assert t.stats()["nodes"][0] == n > 2 ** 25
        assert torch.equal(t.fof(0.5), i)               # no links
        assert not bool(t.fof(1.0).any())               # one group
        idx, d2 = t.knn(2)
        assert torch.equal(idx[:, 0], i) and bool((d2[:, 0] == 0).all()) and bool((d2[:, 1] == 1).all())
        # the neighbour at distance 1 with the smallest index: one layer back, where there is one
        layer = SIDE * SIDE
        assert torch.equal(idx[layer:, 1], i[layer:] - layer)
    api.jz_release_cached()
