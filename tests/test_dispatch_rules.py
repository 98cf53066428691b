"""CPU: the library's rules that choose launch shapes, through a small host
program linked with it."""
import os
import subprocess

import pytest

from paper_2608_12780_amd import binding as B
from paper_2608_12780_amd import build

PROBE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "kernels.h"
int main(int argc, char **argv) {
  if (!strcmp(argv[1], "shares")) {  // cus most cost...
    const int nsub = argc - 4;
    double cost[8];
    int blocks[8];
    for (int m = 0; m < nsub; ++m) cost[m] = atof(argv[4 + m]);
    scope::km_block_shares(cost, nsub, atoi(argv[2]), atoll(argv[3]), blocks);
    for (int m = 0; m < nsub; ++m) printf("%d ", blocks[m]);
  }
}
"""


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    B.lib()
    d = tmp_path_factory.mktemp("probe")
    src, exe = d / "probe.cpp", d / "probe"
    src.write_text(PROBE)
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    cmd = ["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", f"{rocm}/include",
           "-I", build.CSRC, str(src), "-o", str(exe), B.LIB_PATH,
           f"-Wl,-rpath,{os.path.dirname(os.path.abspath(B.LIB_PATH))}", f"-Wl,-rpath,{rocm}/lib",
           f"-L{rocm}/lib", "-lamdhip64", "-Wl,--allow-shlib-undefined"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr

    def run(*args):
        out = subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True, check=True)
        return [int(x) for x in out.stdout.split()]
    return run


def _cost(c, dx):
    dxp = next(p for p in (16, 32, 48, 64, 128) if dx <= p)
    return (c + 31) // 32 * 32 * (4 * dxp + 256)


@pytest.mark.parametrize("cols", [
    [(333, 16), (333, 56), (333, 56)],      # rounded shares: 61 + 98 + 98 = 257
    [(333, 44), (333, 42), (333, 42)],
    [(333, 16)] * 8,
    [(10, 2)] * 5 + [(1000, 30)] * 2 + [(900, 58)],  # several shares below one block
    [(1, 1), (1024, 127)],
])
@pytest.mark.parametrize("cus", [256, 304, 8])
def test_subspaces_share_the_cus(probe, cols, cus):
    cost = [_cost(*c) for c in cols]
    blocks = probe("shares", cus, 1 << 40, *cost)
    assert len(blocks) == len(cols) and min(blocks) >= 1
    assert sum(blocks) == max(cus, len(cols))
    # no move of one block from a subspace to another shortens the longest
    longest = max(c / b for c, b in zip(cost, blocks))
    for i in range(len(cols)):
        for j in range(len(cols)):
            if i != j and blocks[i] > 1:
                moved = list(blocks)
                moved[i] -= 1
                moved[j] += 1
                assert max(c / b for c, b in zip(cost, moved)) >= longest * (1 - 1e-12)
    assert probe("shares", cus, 3, *cost) == [min(b, 3) for b in blocks]
