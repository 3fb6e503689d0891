"""Output rows of the kNN leaf stage at every alignment of the buffers and
every word size its stores use (4, 8 and 16 bytes), on guarded buffers."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2604_05885_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 3, 4, 6, 8, 10, 12, 14, 15, 16, 30, 32, 33, 34, 36, 64, 68])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_rows_at_every_alignment(k, shift):
    import torch
    from paper_2604_05885_amd import api
    n = 700
    p = inputs.uniform(n, 51)
    wi, wd = oracle.knn_bf(p, k)
    # rows start `shift` words into a buffer whose surroundings must stay as they are
    bi = torch.full((n * k + 8,), -7, dtype=torch.int32, device="cuda")
    bd = torch.full((n * k + 8,), -7.0, dtype=torch.float32, device="cuda")
    with api.jz_build(torch.from_numpy(p).cuda()) as t:
        st = api.lib.jz_knn(t.handle, k, ctypes.c_void_p(bi.data_ptr() + 4 * shift),
                            ctypes.c_void_p(bd.data_ptr() + 4 * shift), None)
        assert st == api.JZ_OK
    torch.cuda.synchronize()
    gi, gd = bi.cpu().numpy(), bd.cpu().numpy()
    assert np.array_equal(gi[shift:shift + n * k].reshape(n, k), wi)
    assert np.array_equal(gd[shift:shift + n * k].reshape(n, k).view(np.uint32), wd.view(np.uint32))
    for g in (gi, gd):
        assert np.all(g[:shift] == -7) and np.all(g[shift + n * k:] == -7)
