"""Host check of the copies a call makes of device results (HostCopy), with the
HIP calls replaced by stand-ins: where no pinned memory is to be had, a copy
in pageable memory is read again like a pinned one, with any size."""
import os
import subprocess

import pytest

from paper_2604_05885_amd import build

MAIN = r"""
#include "jz_internal.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
static int g_pinned = 0, g_live = 0, g_calls = 0;  // whether there is pinned memory
extern "C" {
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    ++g_calls;
    if (!g_pinned) return hipErrorOutOfMemory;
    ++g_live;
    *p = malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { --g_live; free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
}
#define CHECK(x) do { if (!(x)) { printf("line %d: %s: %s\n", __LINE__, #x, jz_last_error()); return 1; } } while (0)
int main(int argc, char **argv) {
    g_pinned = atoi(argv[1]);
    std::vector<unsigned char> a(HOST_BLOCK * 3), b(HOST_BLOCK * 3);
    for (size_t i = 0; i < a.size(); ++i) { a[i] = (unsigned char)(i * 7 + 1); b[i] = (unsigned char)(i * 5 + 3); }
    // as a build reads: 9 words, then one per plane; as a rerun does: the same size
    const size_t sizes[][4] = {{36, 64, 8, 36}, {25000, 25000, 25000, 25000},
                               {8, HOST_BLOCK, HOST_BLOCK + 1, 8}, {3 * HOST_BLOCK, 4, 3 * HOST_BLOCK, HOST_BLOCK}};
    for (const auto &row : sizes) {
        HostCopy h;
        for (int i = 0; i < 4; ++i) {
            const unsigned char *src = i & 1 ? b.data() : a.data();
            CHECK(h.read(src, row[i], nullptr) == JZ_OK);
            CHECK(memcmp(h.as<unsigned char>(), src, row[i]) == 0);
        }
    }
    jz_release_cached();
    CHECK(g_live == 0);
    return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_copy")
    (d / "main.hip").write_text(MAIN)
    objs = []
    for src in (os.path.join(build.CSRC, "api.hip"), str(d / "main.hip")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.run([build.hipcc(), *build.HIPFLAGS, "--offload-host-only", "-c", src, "-o", objs[-1]],
                       check=True, capture_output=True)
    out = str(d / "main")
    # (the kernels' side of the library is not linked in: nothing here calls it)
    subprocess.run(["g++", "-no-pie", *objs, "-o", out, "-pthread", "-Wl,--unresolved-symbols=ignore-all"],
                   check=True, capture_output=True)
    return out


@pytest.mark.parametrize("pinned", [1, 0])
def test_read_again(exe, pinned):
    r = subprocess.run([exe, str(pinned)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
