"""Keys, stable sort and tree on each path of the sort: systems of one tile at
most (one block sorts each) at the edges of its particles per thread, merged
runs at the edges of runs, chunks and rounds, with runs that lie inside one gap
of another and runs of equal keys, and the radix passes just past the merges.
Coincident particles check that equal keys keep their order.  Everything is an
integer structure or a cube: bit-exact against the oracle."""
import sys

import numpy as np
import pytest

import oracle
from paper_1507_01009_amd import ics
from gpu_helpers import gpu_run

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _cloud(n, seed):
    pos = ics.plummer(max(n, 2), seed)[0][:n].copy()
    pick = np.random.default_rng(seed).integers(0, n, (2, n // 10))
    pos[pick[0]] = pos[pick[1]]
    return pos


def _check(pos, levels, sys_off=None):
    n = pos.shape[0]
    mass = np.random.default_rng(n).uniform(0.5, 1.5, n) / n
    g = gpu_run(pos, mass, 0.01, 0.5, 8, 64, sys_off=sys_off, key_levels=levels)["tree"]
    t = oracle.build_tree(pos, sys_off, 8, levels=levels)
    assert np.array_equal(g["cube"], t.cube)
    assert np.array_equal(g["skeys"], t.skeys)
    if levels == 42:
        assert np.array_equal(g["skeys_lo"], t.skeys_lo)
    assert np.array_equal(g["perm"], t.perm)
    for k in ("level", "first", "count", "child", "nchild", "parent"):
        assert np.array_equal(g[k], getattr(t, k)), k
    assert np.array_equal(g["groups"], oracle.groups(t, 64))


@pytest.mark.parametrize("levels", [21, 42])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1024, 1025, 2049, 4095, 4096, 4097])
def test_one_system(n, levels):
    say("sort", n, levels)
    _check(_cloud(n, 70 + n), levels)


@pytest.mark.parametrize("levels", [21, 42])
@pytest.mark.parametrize("sizes", [(1024, 1, 0, 700), (4096, 0, 1025, 3, 64), (4097, 900, 1)])
def test_batch(sizes, levels):
    say("sort batch", sizes, levels)
    _check(np.concatenate([_cloud(n, 7 + n) for n in sizes if n]), levels,
           [0] + list(np.cumsum(sizes)))


@pytest.mark.parametrize("levels", [21, 42])
@pytest.mark.parametrize("n", [6143, 8192, 8193, 8705, 32768, 32769, 70001])
def test_merged_runs(n, levels):
    say("merge", n, levels)
    _check(_cloud(n, 90 + n), levels)


@pytest.mark.parametrize("levels", [21, 42])
def test_merged_batch(levels):
    say("merge batch", levels)
    sizes = (9000, 0, 2048, 2049, 33000)
    _check(np.concatenate([_cloud(n, 11 + n) for n in sizes if n]), levels,
           [0] + list(np.cumsum(sizes)))


@pytest.mark.parametrize("levels", [21, 42])
@pytest.mark.parametrize("kind", ["gap", "equal", "sorted"])
def test_merged_runs_special(kind, levels):
    say("merge", kind, levels)
    rng = np.random.default_rng(5)
    if kind == "gap":        # runs 1 to 3 between two keys of run 0: more than is staged
        pos = rng.uniform(-1.0, 1.0, (9000, 3))
        pos[2048:8192] = 0.3 + 1e-5 * rng.uniform(0.0, 1.0, (6144, 3))
    elif kind == "equal":
        pos = np.full((9000, 3), 0.25)
        pos[4000:4500] = rng.uniform(-1.0, 1.0, (500, 3))
    else:
        pos = rng.uniform(-1.0, 1.0, (20000, 3))
        pos = pos[oracle.build_tree(pos, None, 8).perm]
    _check(pos, levels)


@pytest.mark.parametrize("sizes,levels", [(((3 << 19) + 1,), 21), ((1000003, 0, 5, 600001), 21),
                                          (((1 << 22) + 1,), 42)])
def test_radix_passes(sizes, levels):
    say("radix", sizes, levels)
    pos = np.random.default_rng(3).normal(size=(sum(sizes), 3))
    off = [0] + list(np.cumsum(sizes)) if len(sizes) > 1 else None
    _check(pos, levels, off)
