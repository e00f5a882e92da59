"""The rules that give a direct sum its kernels and its split (csrc/direct_plan.h,
plain C++), on the CPU: the split covers every source, fits the scratch memory and
the launch, and the lines between the kernels lie where they were measured."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CAP = 8 * 131072                       # doubles of partial sums of a context
FEW, TILE, PLAIN = 0, 1, 2

MAIN = r"""
#include <cstdio>
#include "direct_plan.h"
int main() {
  long cap, n, nt;
  int nseg;
  while (std::scanf("%ld %ld %ld %d", &cap, &n, &nt, &nseg) == 4) {
    const tg::DirectPlan p = tg::direct_plan(cap, n, nt, nseg);
    std::printf("%d %d %ld %ld %d\n", (int)p.path, p.lane_targets, (long)p.chunk,
                (long)p.nchunks, (int)p.block_reduce);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "plan")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_1507_01009_amd", "csrc"),
                           str(d / "main.cpp"), "-o", exe])

    def ask(rows):
        text = "".join("%d %d %d %d\n" % r for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, x.split())) for x in out.splitlines()]
    return ask


def _sizes():
    rng = np.random.default_rng(4)
    edges = [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1024, 4095, 4096, 4097, 8191,
             8192, 8193, 65535, 65536, 131071, 131072, 262144, 1 << 20, (1 << 20) - 1]
    rows = [(CAP, n, nt, s) for n in [0] + edges + [1 << 22, 1 << 29] for nt in edges + [1 << 28]
            for s in (1, 2, 256)]
    rows += [(cap, int(n), int(nt), int(s)) for cap in (CAP, 1 << 19)
             for n, nt, s in zip(np.exp(rng.uniform(0, 19, 3000)), np.exp(rng.uniform(0, 17, 3000)),
                                 rng.choice([1, 3], 3000))]
    return rows


def test_splits_cover_and_fit(plan):
    rows = _sizes()
    for (cap, n, nt, nseg), (path, lt, chunk, k, _) in zip(rows, plan(rows)):
        r = (cap, n, nt, nseg, path, lt, chunk, k)
        assert chunk >= 1 and k >= (n > 0), r
        assert k * chunk >= n and (k - 1) * chunk < max(n, 1), r
        # the few-target kernel always stores partial sums, the others from two chunks on
        if path == FEW or k > 1:
            assert 8 * nt * k <= cap, r
        if path == FEW:
            assert nt <= 65535 and k < 1 << 31, r          # the launch's grid
        if path == TILE:
            assert nseg == 1 and chunk % 256 == 0 and k <= 65535, r


@pytest.mark.parametrize("n,nt,nseg,path", [
    # several segments: no tiles, so few-target blocks up to 4096 targets
    (20000, 128, 64, FEW), (8192, 256, 256, FEW), (131072, 128, 32, FEW), (8192, 4096, 256, FEW),
    (8192, 4097, 256, PLAIN), (8191, 256, 256, PLAIN), (4000, 256, 256, PLAIN),
    (1 << 20, 4096, 64, PLAIN),                            # partial sums beyond the scratch
    (262144, 64, 1, FEW), (262144, 8191, 1, TILE), (100, 63, 1, PLAIN), (63, 1000, 1, PLAIN)])
def test_lines(plan, n, nt, nseg, path):
    assert plan([(CAP, n, nt, nseg)])[0][0] == path


@pytest.mark.parametrize("n,nt,span", [(131072, 1, 1024), (1 << 20, 1, 1024), ((1 << 20) + 1, 1, 4096),
                                       (500000, 2, 1024), (50000, 24, 1024), (20000, 64, 1024), (131072, 12, 1024), (131072, 13, 4096),
                                       (250000, 24, 4096), (131072, 48, 4096), (8192, 127, 1024)])
def test_few_target_ranges(plan, n, nt, span):
    """Ranges of 1024 sources only where ranges of 4096 leave much of the chip idle."""
    path, _, chunk, _, _ = plan([(CAP, n, nt, 1)])[0]
    assert (path, chunk) == (FEW, span)


@pytest.mark.parametrize("n,nt,path", [(8192, 128, FEW), (20000, 200, FEW), (65535, 128, FEW),
                                       (65536, 128, TILE), (262144, 88, FEW), (262144, 89, TILE), (8192, 1023, FEW),
                                       (8192, 1024, TILE), (1 << 22, 64, FEW), (4096, 128, TILE)])
def test_line_of_one_segment(plan, n, nt, path):
    """Above 88 targets of one segment the tiles from 2^23 pairs on."""
    assert plan([(CAP, n, nt, 1)])[0][0] == path


@pytest.mark.parametrize("n,nt,block", [(8000, 64, True), (4096, 64, False), (4352, 64, True),
                                        (4000, 8191, False), (262144, 300, True)])
def test_who_adds_the_chunks(plan, n, nt, block):
    """A thread per target up to 16 chunks, a block beyond."""
    path, _, _, k, b = plan([(CAP, n, nt, 1)])[0]
    assert path == TILE and bool(b) == block == (k > 16)


@pytest.mark.parametrize("n,nt,path", [(64, 131072, TILE), (64, 131073, PLAIN), (95, 1000000, PLAIN),
                                       (96, 1000000, TILE), (64, 64, TILE)])
def test_line_of_many_targets(plan, n, nt, path):
    """A thread each for more targets than a round of tile blocks, on few sources."""
    assert plan([(CAP, n, nt, 1)])[0][0] == path
