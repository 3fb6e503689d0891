"""GPU parity of the catalogue where a wave's 1024 positions change from one
group to several, and where a group has just as many members as asked for."""
import numpy as np
import pytest

from paper_2604_05885_amd import inputs
from test_gpu_catalogue import check, jz  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1023,), (1024,), (1025,), (1, 1023, 1), (2048, 1, 1023),
                                   (5, 64, 1024, 3000, 1, 2), (63, 64, 65, 1000, 1, 1, 1, 900)])
def test_catalogue_group_sizes(jz, sizes):  # noqa: F811
    # groups of the given sizes: tight balls far apart, in shuffled input order
    rng = np.random.default_rng(sum(sizes))
    p = np.concatenate([inputs.uniform(m, 90 + i) * np.float32(2.0 ** -10) + np.float32(i)
                        for i, m in enumerate(sizes)]).astype(np.float32)
    rng.shuffle(p)
    vel = rng.normal(size=p.shape).astype(np.float32)
    for m in sorted({1, 2, max(sizes), max(sizes) + 1, min(sizes)}):
        g = check(jz, p, 0.01, m, vel)
        assert sorted(g["count"].tolist()) == sorted(s for s in sizes if s >= m)
