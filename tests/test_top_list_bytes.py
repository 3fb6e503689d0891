"""Host check of the size of the dense super-node lists: for every number of
super nodes a tree can have, the byte count is exact, or the list is refused."""
import subprocess

import pytest

from paper_2604_05885_amd import build

MAIN = r"""
#include "jz_internal.h"
#include <cstdio>
#include <cstdlib>
int main(int, char **argv) {
    const int64_t S = atoll(argv[1]);
    size_t b = 0;
    if (top_list_bytes(S, b)) printf("%zu\n", b);
    else printf("refused\n");
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("top_list")
    (d / "main.hip").write_text(MAIN)
    out = d / "main"
    subprocess.run([build.hipcc(), *build.HIPFLAGS, "--offload-host-only", str(d / "main.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    return str(out)


# (2^61 = 1518500249.99^2 pairs of 8 bytes are 2^64 bytes)
@pytest.mark.parametrize("S", [1, 32, 46341, 189000, 1 << 20, 1 << 27, 1 << 30, 1518500249, 1518500250,
                               1518500260, 2 ** 31 - 2])
def test_bytes_or_refused(exe, S):
    r = subprocess.run([exe, str(S)], capture_output=True, text=True, timeout=60, check=True).stdout.strip()
    if 8 * S * S < 2 ** 40:  # what a device may hold
        assert r == str(8 * S * S)
    else:
        assert r == "refused" or int(r) == 8 * S * S
