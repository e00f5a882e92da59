"""Keys, stable sort and tree where the sort takes another path: systems of one
tile at most (one block sorts each), at the edges of its particles per thread,
and one particle more than that.  Coincident particles check that equal keys
keep their order.  Everything is an integer structure or a cube: bit-exact
against the oracle."""
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
