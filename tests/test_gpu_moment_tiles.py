"""Moments at the edges of the particle tiles and of the runs of tiles in which
they are formed, and where a tile holds more internal nodes than are listed.
Leaves equal the oracle's bit for bit; an internal node equals its children's
parallel-axis sums, formed here in the kernel's order, bit for bit (a node
left out, or formed before its children, does not)."""
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


def _check(pos, mass, nl, sys_off=None, max_nodes=0):
    g = gpu_run(pos, mass, 0.01, 0.5, nl, 64, sys_off=sys_off, max_nodes=max_nodes)["tree"]
    t = oracle.build_tree(pos, sys_off, nl)
    sp, sm = oracle.sorted_arrays(t, pos, mass)
    mom = oracle.moments(t, sp, sm)
    leaf = t.nchild == 0
    assert np.array_equal(g["nchild"], t.nchild)
    assert np.array_equal(g["mom"][leaf, 0], mom[leaf, 0])
    assert np.array_equal(g["com"][leaf, :3], mom[leaf, 1:4])
    assert np.array_equal(g["mom"][leaf, 1:7], mom[leaf, 4:10])
    # internal nodes from their children's values
    v = np.flatnonzero(~leaf)
    k = np.arange(8)[None, :]
    has = k < t.nchild[v, None]
    c = np.where(has, t.child[v, None] + k, 0)
    oct_sum = lambda x: (((x[:, 0] + x[:, 1]) + (x[:, 2] + x[:, 3]))
                         + ((x[:, 4] + x[:, 5]) + (x[:, 6] + x[:, 7])))
    m = np.where(has, g["mom"][c, 0], 0.0)
    x = [np.where(has, g["com"][c, q], 0.0) for q in range(3)]
    M = oct_sum(m)
    com = [oct_sum(m * x[q]) / M for q in range(3)]
    assert np.array_equal(g["mom"][v, 0], M)
    assert np.array_equal(g["com"][v, :3], np.stack(com, 1))
    d = [x[q] - com[q][:, None] for q in range(3)]
    for s, (i, j) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
        S = np.where(has, g["mom"][c, 1 + s] + m * d[i] * d[j], 0.0)
        assert np.array_equal(g["mom"][v, 1 + s], oct_sum(S)), s


@pytest.mark.parametrize("n", [511, 512, 513, 1025, 32767, 32769, 70001])
def test_tile_and_run_edges(n):
    say("moment tiles", n)
    pos, _, _ = ics.plummer(n, 40 + n)
    _check(pos, np.random.default_rng(n).uniform(0.5, 1.5, n) / n, 8)


def test_more_internal_nodes_than_a_tile_lists():
    """Close pairs and leaves of one particle: chains of nodes with a single
    child, some 20 levels for each pair."""
    say("moment tiles, chains")
    rng = np.random.default_rng(6)
    a = rng.normal(size=(700, 3))
    _check(np.concatenate([a, a + 1e-5 * rng.normal(size=a.shape)]), np.full(1400, 1e-3), 1,
           max_nodes=60000)


def test_systems_across_tiles():
    say("moment tiles, batch")
    n = 9000
    off = np.array([0, 1, 700, 701, 701, 5000, n])
    pos = np.random.default_rng(7).normal(size=(n, 3)) ** 3
    _check(pos, np.full(n, 1e-3), 8, off)


@pytest.mark.parametrize("n", [16896, 16897, 24001, 32768])
def test_candidates_read_again_with_42_levels(n):
    """More candidates of nodes beyond their tile than are kept, with 42 levels
    from 34 tiles on.  Where no leaf reaches level 21, the tree and its moments
    are those of 21 levels, bit for bit; below it, where pairs fall together
    to the last levels, masses and centres are the oracle's."""
    say("moment tiles, 42 levels", n)
    pos, _, _ = ics.plummer(n, 90 + n)
    mass = np.random.default_rng(n).uniform(0.5, 1.5, n) / n
    a = gpu_run(pos, mass, 0.01, 0.5, 8, 64)["tree"]
    b = gpu_run(pos, mass, 0.01, 0.5, 8, 64, key_levels=42)["tree"]
    assert a["level"].max() < 21
    for k in ("level", "first", "count", "child", "com", "mom"):
        assert np.array_equal(a[k], b[k]), k
    # leaves of one particle: the pairs make chains of nodes down to their level
    rng = np.random.default_rng(n + 1)
    h = n // 8
    pos[n - h:] = pos[:h] + 1e-9 * rng.normal(size=(h, 3))
    g = gpu_run(pos, mass, 0.01, 0.5, 1, 64, key_levels=42, max_nodes=60 * n)["tree"]
    t = oracle.build_tree(pos, None, 1, levels=42)
    sp, sm = oracle.sorted_arrays(t, pos, mass)
    mom = oracle.moments(t, sp, sm)
    assert t.level.max() > 21 and np.array_equal(g["nchild"], t.nchild)
    # at most eight children a level over 42 levels, each sum rounded to 2^-53
    # of its magnitude (of the centre: the largest coordinate)
    tol = 8 * 42 * 2.0 ** -53
    assert np.max(np.abs(g["mom"][:, 0] / mom[:, 0] - 1.0)) <= tol
    assert np.max(np.abs(g["com"][:, :3] - mom[:, 1:4])) <= 2 * tol * np.abs(pos).max()
