"""Trees with more super nodes than their dense pair lists have 32-bit offsets
for: the kNN call (all pairs) refuses, the FoF call (each pair once, so half as
many) still gives the oracle's groups."""
import numpy as np
import pytest

import oracle
from paper_2604_05885_amd import inputs

pytestmark = pytest.mark.gpu


def test_super_node_pairs_beyond_32_bits():
    import torch
    from paper_2604_05885_amd import api
    n = 50000  # super nodes of one leaf of one point: 2.5e9 pairs, half of them for FoF
    p = inputs.uniform(n, 77)
    b = inputs.linking_length(n, 0.4)
    opts = api.default_opts(leaf_max=1, ngr=1, n_target=2 ** 31 - 1)
    with api.jz_build(torch.from_numpy(p).cuda(), opts) as t:
        assert t.stats()["super_nodes"] == n and t.stats()["planes"] == 1
        with pytest.raises(api.JzError) as e:
            t.knn(4)
        assert e.value.status == api.JZ_E_CAPACITY and "super node" in str(e.value)
        label = t.fof(b).cpu().numpy()
    api.jz_release_cached()
    assert np.array_equal(label, oracle.fof_kd(p, b))
