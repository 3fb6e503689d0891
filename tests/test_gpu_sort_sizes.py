"""GPU check of the build's radix sort at the edges of its tiles and of the sizes
where it changes them: the exported order against a stable sort of the exported
keys' definition on the host."""
import numpy as np
import pytest

from paper_2604_05885_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4097, 5119, 5120, 5121, 99999, 100000, 100353, 399999, 400000, 401408,
                               401409, 899999, 900000, 900097])
def test_sorted_order(n):
    import torch
    from paper_2604_05885_amd import api
    p = inputs.clustered(n, 9, 400)
    p[: n // 5] = p[n // 2]          # equal keys keep the input order
    with api.jz_build(torch.from_numpy(p).cuda(), api.default_opts(keep_keys=1)) as t:
        e = t.export(order=True, keys=True)
    order, keys = e["order"], e["keys"]
    assert np.array_equal(np.sort(order), np.arange(n))
    by_input = np.empty(n, np.uint64)
    by_input[order] = keys
    assert np.array_equal(order, np.argsort(by_input, kind="stable"))


@pytest.mark.parametrize("n", [1003520, 1003521, 2999999, 3000000, 3006463, 3006465])
def test_sorted_order_large_tiles(n):
    test_sorted_order(n)
