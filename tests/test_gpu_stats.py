"""The kNN statistics of trees whose leaves are shared by several waves: a
visited pair is one of the leaf list's, and counts once."""
import pytest

from paper_2604_05885_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf_max", [(1, 64), (64, 64), (65, 64), (1000, 64), (768, 1), (769, 1), (30000, 64)])
def test_visited_pairs(n, leaf_max):
    import torch
    from paper_2604_05885_amd import api
    for p in (inputs.uniform(n, 900 + n), inputs.clustered(n, max(1, n // 900), 901 + n)):
        with api.jz_build(torch.from_numpy(p).cuda(), api.default_opts(leaf_max=leaf_max)) as t:
            t.knn(min(n, 8))
            st = t.stats()
        assert st["nodes"][0] <= st["leaf_pairs_visited"] <= st["leaf_pairs"], st
