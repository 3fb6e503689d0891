"""GPU parity of the kNN node walk where its stream of source children changes
shape: parents with more children than a wave or than one LDS listing holds,
lists that need several listings, radii over many small nodes, and separate
point types. Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2604_05885_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jz():
    from paper_2604_05885_amd import api
    return api


def sets():
    yield "clustered", inputs.clustered(9000, 9, 71)
    yield "uniform", inputs.uniform(9000, 72)
    # one key for thousands of points: nodes are cut by position, a parent may
    # have hundreds of children
    p = inputs.uniform(5000, 73)
    p[:3000] = p[0]
    yield "identical", p


@pytest.mark.parametrize("leaf_max,coarsen,ngr,n_target,k", [
    (1, 64, 64, 1, 5), (1, 2, 1, 2, 9), (2, 64, 64, 20, 33), (5, 16, 3, 4, 17), (64, 64, 64, 1, 70),
    (3, 3, 64, 8, 256), (64, 2, 1, 1, 16)])
def test_walk_tree_shapes(jz, leaf_max, coarsen, ngr, n_target, k):
    import torch
    o = jz.default_opts(leaf_max=leaf_max, coarsen=coarsen, ngr=ngr, n_target=n_target)
    for name, p in sets():
        with jz.jz_build(torch.from_numpy(p).cuda(), o) as t:
            gi, gd = t.knn(k)
            gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
        wi, wd = oracle.knn_bf(p, k)
        assert np.array_equal(gi, wi), (name, leaf_max)
        assert np.array_equal(gd.view(np.uint32), wd.view(np.uint32)), (name, leaf_max)


@pytest.mark.parametrize("leaf_max,coarsen,k", [(1, 64, 6), (7, 4, 40), (64, 8, 16)])
def test_walk_point_types(jz, leaf_max, coarsen, k):
    """Sources and queries in different places: children that receive nothing,
    and radii that only far sources fill."""
    import torch
    s = inputs.clustered(4000, 4, 74)
    q = np.concatenate([inputs.uniform(2500, 75), s[:500]])
    o = jz.default_opts(leaf_max=leaf_max, coarsen=coarsen, n_target=4, ngr=5)
    with jz.jz_build_joint(torch.from_numpy(s).cuda(), torch.from_numpy(q).cuda(), o) as t:
        gi, gd = t.knn_query(k)
        gi, gd = gi.cpu().numpy(), gd.cpu().numpy()
    wi, wd = oracle.knn_cross_bf(s, q, k)
    assert np.array_equal(gi, wi) and np.array_equal(gd.view(np.uint32), wd.view(np.uint32))
