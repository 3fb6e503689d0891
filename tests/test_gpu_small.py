"""GPU parity of the one-launch build of small sets: its order, keys' splits and
leaf boxes against the general build (which keep_keys selects) and against the
oracle, around its largest size, for every option it accepts, and its errors."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2604_05885_amd import inputs

pytestmark = pytest.mark.gpu

SMALL = 4096


@pytest.fixture(scope="module")
def jz():
    from paper_2604_05885_amd import api
    return api


def sets(n):
    yield inputs.uniform(n, 300 + n)
    yield inputs.clustered(n, max(1, n // 700), 301 + n)
    p = inputs.uniform(n, 302 + n)
    p[n // 3:] = p[0]               # equal keys: splits by position
    yield p
    p = np.zeros((n, 3), np.float32)
    p[:, 1] = np.arange(n)           # a line
    yield p


@pytest.mark.parametrize("n", [1, 2, 3, 31, 63, 64, 65, 1023, 1024, 1025, 2048, 4095, SMALL, SMALL + 1])
def test_small_build_equals_general(jz, n):
    import torch
    for p in sets(n):
        d = torch.from_numpy(p).cuda()
        for o in ({}, {"leaf_max": 1}, {"leaf_max": 7, "ngr": 3}, {"key_bits": 1}, {"key_bits": 17},
                  {"key_bits": 18}):
            with jz.jz_build(d, jz.default_opts(**o)) as t, \
                    jz.jz_build(d, jz.default_opts(keep_keys=1, **o)) as g:
                a, b = t.stats(), g.stats()
                assert a["nodes"] == b["nodes"] and a["super_nodes"] == b["super_nodes"], (n, o)
                a, b = t.export(plane=0, order=True), g.export(plane=0, order=True)
                assert np.array_equal(a["order"], b["order"]), (n, o)
                assert np.array_equal(a["spl"], b["spl"]), (n, o)


@pytest.mark.parametrize("n", [5, 1000, SMALL, SMALL + 1])
def test_small_results(jz, n):
    import torch
    for i, p in enumerate(sets(n)):
        d = torch.from_numpy(p).cuda()
        k = min(9, n)
        b = inputs.linking_length(n, 0.4)
        with jz.jz_build(d, jz.default_opts(leaf_max=(64, 5, 32, 64)[i])) as t:
            gi, gd, gl = t.knn_fof(k, b)
        wi, wd = oracle.knn_bf(p, k)
        assert np.array_equal(gi.cpu().numpy(), wi) and np.array_equal(gl.cpu().numpy(), oracle.fof_bf(p, b))
        assert np.array_equal(gd.cpu().numpy().view(np.uint32), wd.view(np.uint32))


def test_small_errors(jz):
    import torch
    p = inputs.uniform(500, 310)
    for bad in (np.nan, np.inf, -np.inf):
        q = p.copy()
        q[321, 2] = bad
        with pytest.raises(jz.JzError) as e:
            jz.jz_build(torch.from_numpy(q).cuda())
        assert e.value.status == jz.JZ_E_NONFINITE
    for q in (p * 2, -p):
        with pytest.raises(jz.JzError) as e:
            jz.jz_build(torch.from_numpy(q).cuda(), jz.default_opts(period=1.0))
        assert e.value.status == jz.JZ_E_INVALID


def test_small_build_out_of_memory(jz):
    """Every allocation of a small build failing in turn: JZ_E_OOM, nothing left."""
    import torch
    d = torch.from_numpy(inputs.uniform(900, 311)).cuda()
    A = jz.TorchAllocator()
    state = {"fail": 0, "count": 0}
    types = [f[1] for f in jz.Allocator._fields_]

    def alloc(ctx, nbytes, stream):
        state["count"] += 1
        return None if state["count"] == state["fail"] else A._alloc(ctx, nbytes, stream)

    cb = (types[1](alloc), types[2](A._free))

    class Wrapped:
        struct = jz.Allocator(ctypes.c_void_p(None), *cb)

    with jz.jz_build(d, allocator=Wrapped()):
        n_alloc = state["count"]
    assert A.live == 0 and n_alloc > 4
    for m in range(1, n_alloc + 1):
        state.update(fail=m, count=0)
        with pytest.raises(jz.JzError) as e:
            jz.jz_build(d, allocator=Wrapped())
        assert e.value.status == jz.JZ_E_OOM and A.live == 0, m
