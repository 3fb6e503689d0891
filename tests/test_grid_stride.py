"""Host check of the index arithmetic with which a grid of one wave per leaf
clears its counters: for every grid that can be launched (fewer than 2^32 work
items), the words touched are those of the array, each once."""
import os
import subprocess

import pytest

from paper_2604_05885_amd import build

MAIN = r"""
#include "jz_device.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
int main(int argc, char **argv) {
    const unsigned nblk = strtoul(argv[1], nullptr, 10), size = 64;
    const size_t n = strtoul(argv[2], nullptr, 10);
    std::vector<int> seen(n, 0);
    auto run = [&](unsigned blk, unsigned item) {
        size_t calls = 0;
        grid_stride(blk, size, nblk, item, n, [&](size_t i) {
            if (i >= n || ++calls > n) {
                printf("workgroup %u of %u, item %u: word %zd of %zu\n", blk, nblk, item, (ssize_t)i, n);
                exit(1);
            }
            ++seen[i];
        });
    };
    // (the first workgroups, which own all the words, those around every power of 2, the last)
    std::vector<unsigned> blks;
    for (unsigned b = 0; b < nblk && b < 64; ++b) blks.push_back(b);
    for (unsigned p = 128; p && p < nblk; p <<= 1)
        for (unsigned b = p - 2; b < p + 2; ++b)
            if (b < nblk) blks.push_back(b);
    if (nblk > 128) blks.push_back(nblk - 1);
    for (unsigned b : blks)
        for (unsigned item = 0; item < size; ++item) run(b, item);
    for (size_t i = 0; i < n; ++i)
        if (seen[i] != 1) { printf("word %zu touched %d times\n", i, seen[i]); return 1; }
    return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid_stride")
    (d / "main.hip").write_text(MAIN)
    out = d / "main"
    subprocess.run([build.hipcc(), *build.HIPFLAGS, "--offload-host-only", str(d / "main.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    return str(out)


@pytest.mark.parametrize("nblk", [1, 3, 21, 1000, 2 ** 25 - 1, 2 ** 25, 2 ** 25 + 1, 2 ** 26 - 1])
def test_words_of_a_launchable_grid(exe, nblk):
    r = subprocess.run([exe, str(nblk), "1288"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
