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
  } else if (!strcmp(argv[1], "lloyd")) {  // bf16 heads n (C dx)...: form, blocks, the plan's blocks
    const int nsub = (argc - 5) / 2;
    scope::KmProblem p[8] = {};
    int col0[8], dx[8], C[8], d = 0;
    for (int m = 0; m < nsub; ++m) {
      C[m] = atoi(argv[5 + 2 * m]);
      dx[m] = atoi(argv[6 + 2 * m]);
      col0[m] = d;
      d += dx[m];
    }
    for (int m = 0; m < nsub; ++m) {
      p[m].bf16 = atoi(argv[2]);
      p[m].heads = atoi(argv[3]);
      p[m].n = atoi(argv[4]);
      p[m].ld = d;
      p[m].col0 = col0[m];
      p[m].dx = dx[m];
      p[m].C = C[m];
      p[m].cpad = scope::km_cpad(C[m]);
      p[m].dxp = scope::km_dxp(dx[m]);
      p[m].mfma = scope::km_mfma_ok(p[m].bf16, d, col0[m], dx[m], C[m]);
    }
    scope::AccPlan plan;
    scope::km_accum_plan(nsub, col0, dx, C, p[0].heads, p[0].n, &plan);
    const scope::LloydForm f = scope::km_lloyd_form(p, nsub, plan);
    printf("%d %d %d", static_cast<int>(f.form), f.blocks, plan.blocks);
  } else if (!strcmp(argv[1], "attention")) {  // heads n d c_q: copies of fp32 K and V, block order
    const int heads = atoi(argv[2]), n = atoi(argv[3]), d = atoi(argv[4]), c_q = atoi(argv[5]);
    printf("%d %d", scope::attention_copies_kv(n, d, c_q, false), scope::attention_ordered(heads, n, d, c_q));
  } else if (!strcmp(argv[1], "alone")) {  // d slots waves
    printf("%d", scope::attention_runs_alone(atoi(argv[2]), atoll(argv[3]), atoll(argv[4])));
  } else if (!strcmp(argv[1], "finish")) {  // heads n C nsub dx
    const int heads = atoi(argv[2]), n = atoi(argv[3]), nsub = atoi(argv[5]), w = atoi(argv[6]);
    int col0[8], dx[8], C[8];
    for (int m = 0; m < nsub; ++m) {
      col0[m] = m * w;
      dx[m] = w;
      C[m] = atoi(argv[4]);
    }
    scope::AccPlan plan;
    scope::km_accum_plan(nsub, col0, dx, C, heads, n, &plan);
    printf("%d %d", plan.blocks, scope::km_finish_shared(plan, heads));
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


SEPARATE, ITERATION, ALL = 0, 1, 2


def _split(d, m):
    return [d // m // 2 * 2] * (m - 1) + [d - (m - 1) * (d // m // 2 * 2)]


@pytest.mark.parametrize("bf16,heads,n,c,widths,want", [
    (1, 3, 320, 32, [128], ALL),                  # ten slices
    (1, 3, 321, 32, [128], ITERATION),
    (1, 300, 330, 16, [128], ITERATION),          # one block each: queries ...
    (1, 300, 640, 16, [16, 56, 56], ALL),         # ... and narrower rows
    (1, 140, 1000, 16, [128], ITERATION),
    (1, 100, 1024, 16, [16, 56, 56], ALL),        # 32 slices
    (1, 100, 1025, 16, [16, 56, 56], ITERATION),
    (1, 130, 2900, 16, [64], SEPARATE),           # half the CUs
    (0, 60, 1600, 32, [16, 56, 56], ALL),
    (0, 50, 1900, 32, [16, 56, 56], SEPARATE),
    (0, 33, 2500, 32, [16] * 8, SEPARATE),        # 264 blocks: a nearly empty round
    (0, 24, 4096, 32, [16] * 8, ALL),
    (0, 24, 4097, 32, [16] * 8, SEPARATE),        # beyond 48 MiB
    (1, 3, 2185, 160, [128], SEPARATE),           # sums beyond the LDS
])
def test_lloyd_forms(probe, bf16, heads, n, c, widths, want):
    form, blocks, plan = probe("lloyd", bf16, heads, n, *[x for w in widths for x in (c, w)])
    assert form == want
    assert blocks == 1 if form == ALL else 0 <= blocks <= plan


def test_one_block_never_runs_alone_over_many_slices(probe):
    """One block per head and subspace takes more than 32 slices only where
    such blocks keep most CUs busy, and blocks never outnumber the slabs."""
    for bf16 in (0, 1):
        for m in (1, 3, 8):
            for heads in (1, 2, 7, 24, 33, 40, 86, 129, 140, 257, 300):
                for n in (200, 321, 700, 1024, 1025, 2000, 5000):
                    widths = _split(128, m)
                    form, blocks, plan = probe("lloyd", bf16, heads, n, *[x for w in widths for x in (16, w)])
                    assert 0 <= blocks <= plan
                    assert (blocks == 0) == (form == SEPARATE)
                    if blocks == 1 and n > 1024:
                        pairs = heads * m
                        rounds = -(-pairs // 256)
                        assert pairs >= 256 if bf16 else pairs >= 0.6 * 256 * rounds


@pytest.mark.parametrize("heads,n,d,c_q,want", [
    (1, 1023, 128, 1, (0, 0)), (1, 1024, 128, 1, (1, 0)), (1, 1024, 64, 1, (1, 0)),   # dense
    (8, 3071, 128, 17, (0, 0)), (8, 3072, 128, 17, (1, 0)),                           # sparse
    (8, 6143, 64, 37, (0, 0)), (8, 6144, 64, 37, (1, 0)),
    (8, 2304, 128, 38, (0, 0)), (8, 2304, 128, 39, (1, 0)),                           # many chunks
    (8, 2304, 64, 86, (0, 0)), (8, 2304, 64, 87, (1, 0)), (8, 1023, 128, 512, (0, 0)),
    (1, 4095, 128, 1, (1, 0)), (1, 4096, 128, 1, (1, 1)),
    (4, 8192, 128, 1, (1, 1)), (4, 8193, 128, 1, (1, 0)),      # 128 slots, 132 ...
    (8, 8192, 128, 1, (1, 0)), (8, 8193, 128, 1, (1, 1)),      # ... 256, 264
    (8, 16383, 64, 37, (1, 0)), (8, 16384, 64, 37, (1, 1)),
    (24, 118800, 128, 256, (1, 0)), (8, 65536, 128, 256, (1, 1)), (8, 65537, 128, 256, (1, 0)),
    (1, 1 << 24, 128, 256, (0, 0)),
])
def test_attention_forms(probe, heads, n, d, c_q, want):
    assert tuple(probe("attention", heads, n, d, c_q)) == want


@pytest.mark.parametrize("d,slots,waves,want", [
    # measured on both sides: calls whose remainders are faster alone ...
    (64, 57, 143, 1), (64, 351, 1194, 1), (64, 525, 1207, 1), (64, 633, 1456, 1), (64, 420, 2048, 1),
    (128, 109, 229, 1), (128, 226, 452, 1), (128, 256, 512, 1),
    # ... and paired
    (64, 557, 3286, 0), (64, 799, 2317, 0), (64, 769, 1538, 0), (64, 600, 2049, 0),
    (128, 201, 904, 0), (128, 226, 1446, 0), (128, 257, 500, 0), (128, 128, 513, 0),
    (64, 1 << 40, 1 << 43, 0), (128, 1 << 40, 1 << 43, 0),
])
def test_remainders_alone(probe, d, slots, waves, want):
    assert probe("alone", d, slots, waves) == [want]


@pytest.mark.parametrize("heads,n,c,nsub,dx,want", [
    (1, 42000, 32, 1, 128, 1),
    (16, 19721, 128, 1, 128, 1), (16, 19721, 129, 1, 128, 0),   # 2,048 rows, 2,064
    (31, 19721, 209, 3, 20, 0), (16, 2600, 209, 3, 20, 0),
    (40, 42000, 32, 1, 128, 0),                                 # fewer than 8 slabs
])
def test_slabs_of_a_row_are_shared_while_the_chip_has_room(probe, heads, n, c, nsub, dx, want):
    blocks, shared = probe("finish", heads, n, c, nsub, dx)
    assert shared == want and shared == (blocks >= 8 and heads * c * nsub <= 2048)
