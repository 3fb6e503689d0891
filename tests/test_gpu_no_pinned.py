"""Calls in a process that gets no pinned host memory: a build of several
planes and calls whose lists grow read the device's counters several times, and
give the oracle's results, and the call that allocates nothing does not ask for
pinned memory either. (A stand-in for hipHostMalloc, loaded before the
library, refuses every block.)"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <stddef.h>
static int calls;
int hipHostMalloc(void **p, size_t n, unsigned f) { ++calls; *p = 0; return 2; /* hipErrorOutOfMemory */ }
int refused(void) { return calls; }
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np, torch, oracle
from paper_2604_05885_amd import api, inputs
n = 20000
p = inputs.clustered(n, 16, 41)
b = inputs.linking_length(n, 0.3)
wi, wl = oracle.knn_bf(p, 11)[0], oracle.fof_bf(p, b)
d = torch.from_numpy(p).cuda()
opts = api.default_opts(n_target=10, list_per_node=1.0)
with api.jz_build(d, opts) as t:
    assert t.stats()["planes"] > 1
    i, _ = t.knn(11)
    assert t.stats()["reruns"] > 0
    l = t.fof(b)
    assert t.stats()["reruns"] > 0
    assert np.array_equal(i.cpu().numpy(), wi) and np.array_equal(l.cpu().numpy(), wl)
    i, _, l = t.knn_fof(11, b)
    assert np.array_equal(i.cpu().numpy(), wi) and np.array_equal(l.cpu().numpy(), wl)
assert shim.refused() > 0
print("ok", shim.refused())
"""

NOALLOC = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np, torch, oracle
from paper_2604_05885_amd import api, inputs
p = inputs.clustered(20000, 16, 42)
idx = torch.empty((20000, 8), dtype=torch.int32, device="cuda")
d2 = torch.empty((20000, 8), dtype=torch.float32, device="cuda")
with api.jz_build(torch.from_numpy(p).cuda(), api.default_opts(list_per_node=1.0)) as t:
    before = shim.refused()
    st = api.lib.jz_knn_noalloc(t.handle, 8, ctypes.c_void_p(idx.data_ptr()), ctypes.c_void_p(d2.data_ptr()),
                                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == api.JZ_OK, api.lib.jz_last_error()
    asked = shim.refused() - before
assert np.array_equal(idx.cpu().numpy(), oracle.knn_bf(p, 8)[0])
assert before > 0 and asked == 0, (before, asked)
print("ok")
"""


@pytest.mark.parametrize("child", [CHILD, NOALLOC], ids=["calls", "noalloc"])
def test_without_pinned_memory(tmp_path, child):
    (tmp_path / "shim.c").write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(tmp_path / "shim.so"), str(tmp_path / "shim.c")], check=True)
    r = subprocess.run([sys.executable, "-c", child, str(tmp_path / "shim.so"), ROOT],
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.strip().splitlines()[-1].startswith("ok"), r.stdout + r.stderr
