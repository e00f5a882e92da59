"""Walk groups, formed with the nodes where a group is at least a leaf and by
kernels of their own below that: group sizes on both sides of the powers of two
of the window minima, runs of equal keys inside a tile, across tiles and over
more than the 4096 particles looked back at in one step.  Bit-exact against the
oracle."""
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


def _check(pos, nl, ng, levels=21, sys_off=None):
    n = pos.shape[0]
    g = gpu_run(pos, np.full(n, 1.0 / n), 0.01, 0.5, nl, ng, sys_off=sys_off, key_levels=levels)
    t = oracle.build_tree(pos, sys_off, nl, levels=levels)
    assert np.array_equal(g["tree"]["groups"], oracle.groups(t, ng))
    assert np.all(np.isfinite(g["acc"]))


@pytest.mark.parametrize("nl,ng", [(1, 1), (1, 2), (8, 4), (8, 7), (8, 8), (8, 15), (8, 31), (16, 16),
                                   (8, 63), (8, 64), (8, 65), (8, 127), (12, 128), (16, 3)])
def test_group_sizes(nl, ng):
    say("groups", nl, ng)
    _check(ics.plummer(5003, nl + ng)[0], nl, ng)


@pytest.mark.parametrize("levels", [21, 42])
@pytest.mark.parametrize("ng", [8, 48, 64, 128])
def test_runs_of_equal_keys(ng, levels):
    say("groups of equal keys", ng, levels)
    rng = np.random.default_rng(ng)
    pos = rng.uniform(-1.0, 1.0, (16000, 3))
    pos[:9500] = 0.3                     # 37 tiles
    pos[9500:9700] = -0.2                # inside one or two
    pos[9700:9700 + ng] = 0.11           # exactly a group, and one more
    pos[9900:9901 + ng] = -0.77
    _check(pos, 8, ng, levels)
    _check(np.concatenate([pos, pos[:700], pos[5000:9600]]), 8, ng, levels,
           [0, 16000, 16000, 16700, 21300])


def test_many_systems_smaller_than_a_group():
    say("groups of small systems")
    sizes = np.random.default_rng(2).integers(0, 200, 60)
    pos = np.concatenate([ics.plummer(max(int(m), 2), 5 + k)[0][:m] for k, m in enumerate(sizes)])
    _check(pos, 8, 64, 21, [0] + list(np.cumsum(sizes)))


@pytest.mark.parametrize("levels", [21, 42])
@pytest.mark.parametrize("nl,ng", [(8, 4), (16, 3)])
@pytest.mark.parametrize("n", [1, 5, 900, 1025, 4096])
def test_groups_below_a_leaf_in_one_block_systems(n, nl, ng, levels):
    """Smaller groups than leaves where a block sorts a system: the group
    starts are cleared by the sort."""
    say("groups below a leaf", n, nl, ng, levels)
    _check(ics.plummer(max(n, 2), n + ng)[0][:n], nl, ng, levels)


def test_groups_below_a_leaf_in_a_batch_of_small_systems():
    say("groups below a leaf, batch")
    sizes = np.random.default_rng(3).integers(0, 1500, 20)
    pos = np.concatenate([ics.plummer(max(int(m), 2), 9 + k)[0][:m] for k, m in enumerate(sizes)])
    _check(pos, 8, 4, 21, [0] + list(np.cumsum(sizes)))
