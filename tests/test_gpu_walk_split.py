"""The force walk with groups split into parts: how a group is split depends
on the number of targets of the whole walk, its lists and its sums inside a
tile do not."""
import sys

import numpy as np
import pytest

import oracle
from paper_1507_01009_amd import ics
from gpu_helpers import gpu_run, rel_err

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# Parts are sums of the same tiles (same FP32 values in mixed precision, the
# same terms in FP64) grouped differently in FP64: at most some 40 tiles of
# up to 64 slices each, so a few hundred roundings of 2^-53 of a sum of
# magnitudes that exceeds the result by less than a hundredfold.
TOL = 1e-12


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,ng,every,soft", [(7, 64, 1, None), (65, 1, 1, None),
                                             (700, 128, 1, None), (3001, 64, 1, "spline"),
                                             (9000, 16, 7, None), (9000, 128, 50, None),
                                             (40000, 64, 1, None)])
def test_results_do_not_depend_on_the_split(n, ng, every, soft, precision):
    """A system alone (few targets: its groups are split) and in a batch with
    a much larger one (split into fewer parts or not at all)."""
    say("split", n, ng, every, soft, precision)
    pos, _, m = ics.plummer(n, 300 + n)
    act = None if every == 1 else np.arange(0, n, every, dtype=np.int32)
    rows = slice(0, n) if act is None else act
    alone = gpu_run(pos, m, 0.01, 0.5, 8, ng, active=act, precision=precision, softening=soft)
    big = 300000
    rng = np.random.default_rng(n)
    act2 = None if act is None else np.concatenate([act, np.arange(n, n + big, dtype=np.int32)])
    both = gpu_run(np.concatenate([pos, rng.normal(size=(big, 3))]),
                   np.concatenate([m, np.full(big, 1.0 / big)]), 0.01, 0.5, 8, ng, active=act2,
                   sys_off=np.array([0, n, n + big]), precision=precision, softening=soft)
    e = rel_err(both["acc"][rows], alone["acc"][rows]).max()
    p = np.max(np.abs(both["pot"][rows] / alone["pot"][rows] - 1.0))
    say("  acc %.3g pot %.3g" % (e, p))
    assert e <= TOL and p <= TOL
    if precision == 0 and soft is None:
        ev = oracle.tree_forces(pos, m, 0.01, 0.5, 8, ng, active=act)
        assert rel_err(alone["acc"][rows], ev.acc[rows]).max() <= 1e-12
        assert (alone["counts"]["n_p2p"], alone["counts"]["n_p2m"]) == (ev.n_p2p, ev.n_p2m)


def test_one_context_over_changing_active_sets():
    """Walks of one context with few, many and no active targets in turn: each
    is split on its own, and rows that are not active keep their values."""
    import torch
    from paper_1507_01009_amd import binding as B
    from gpu_helpers import to_dev
    n = 20000
    pos, _, m = ics.plummer(n, 77)
    full = gpu_run(pos, m, 0.01, 0.5, precision=0)
    ctx = B.Context(n)
    ctx.build_tree(to_dev(pos))
    ctx.compute_moments(to_dev(m))
    for count in (3, 20000, 150, 0, 5000):
        say("active", count)
        idx = np.sort(np.random.default_rng(count).choice(n, count, replace=False)).astype(np.int32)
        acc = torch.full((n, 3), 7.0, dtype=torch.float64, device="cuda")
        ctx.tree_forces(0.01, 0.5, acc, None, to_dev(idx if count else np.zeros(1, np.int32)),
                        to_dev(np.array([count], np.int32)))
        ctx.sync()
        a = acc.cpu().numpy()
        rest = np.setdiff1d(np.arange(n), idx)
        assert np.all(a[rest] == 7.0)
        assert ctx.get_counts()["n_targets"] == count
        if count == n:
            assert rel_err(a, full["acc"]).max() <= TOL
        elif count:      # the active targets' boxes differ, so do the lists: the truncation error
            assert np.median(rel_err(a[idx], full["acc"][idx])) <= 1e-2
    ctx.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_replayed_walk_on_a_tree_of_other_sizes(precision):
    """A captured evaluation replayed after the tree was built again with larger
    and smaller groups gives what an eager one gives on that tree."""
    import torch
    from paper_1507_01009_amd import binding as B
    from gpu_helpers import to_dev
    n = 3001
    pos, _, m = ics.plummer(n, 41)
    dp, dm = to_dev(pos), to_dev(m)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx = B.Context(n, leaf_size=8, group_size=16, precision=precision, stream=s)
        out = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
        ref = torch.zeros_like(out)
        ctx.build_tree(dp); ctx.compute_moments(dm); ctx.tree_forces(0.01, 0.5, out)
        ctx.sync()
        ctx.graph_begin()
        ctx.tree_forces(0.01, 0.5, out)
        graph = ctx.graph_end()
        for nl, ng in ((8, 128), (8, 16), (16, 100), (4, 64)):
            say("replayed walk", precision, nl, ng)
            ctx.set_sizes(nl, ng)
            ctx.build_tree(dp); ctx.compute_moments(dm); ctx.tree_forces(0.01, 0.5, ref)
            out.zero_()
            graph.launch(s)
            s.synchronize()
            assert torch.equal(out, ref), (nl, ng)
        del graph
        ctx.close()


@pytest.mark.parametrize("alpha", [None, 1e-3])
def test_fp64_walks_on_both_sides_of_the_even_line(alpha):
    """147456 particles take the FP64 kernel without the limit on a SIMD's
    waves, one fewer the other: the same terms and tiles."""
    n = 147455
    say("even", n, alpha)
    pos, _, m = ics.plummer(n, 77)
    old = None if alpha is None else np.full((n, 3), 0.3)
    a = gpu_run(pos, m, 0.01, 0.5, 8, 64, alpha=alpha, acc_old=old)
    far = np.full((1, 3), 50.0)
    b = gpu_run(np.concatenate([pos, far]), np.append(m, 1.0), 0.01, 0.5, 8, 64,
                sys_off=np.array([0, n, n + 1]), alpha=alpha,
                acc_old=None if old is None else np.concatenate([old, far]))
    e = rel_err(b["acc"][:n], a["acc"]).max()
    say("  acc %.3g" % e)
    assert e <= TOL
    assert (a["counts"]["n_p2p"], a["counts"]["n_p2m"]) == (b["counts"]["n_p2p"], b["counts"]["n_p2m"])


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("soft,alpha", [(None, None), ("spline", None), (None, 1e-3), ("spline", 1e-3)])
@pytest.mark.parametrize("n,ng,every", [(9000, 64, 1), (20000, 128, 3), (33000, 64, 1)])
def test_few_waves_give_the_same_bits(n, ng, every, soft, alpha, precision):
    """One, two and four waves per CU, which take split groups as a whole where
    each has several (20000 stars: 900 groups, 256 waves), against all waves."""
    say("few waves", n, ng, every, soft, alpha, precision)
    pos, _, m = ics.plummer(n, 500 + n)
    act = None if every == 1 else np.arange(0, n, every, dtype=np.int32)
    old = None if alpha is None else np.random.default_rng(n).normal(size=(n, 3))
    runs = [gpu_run(pos, m, 0.01, 0.5, 8, ng, active=act, precision=precision, softening=soft,
                    alpha=alpha, acc_old=old, waves_per_cu=w) for w in (0, 1, 2, 4)]
    for r in runs[1:]:
        assert np.array_equal(r["acc"], runs[0]["acc"], equal_nan=True)
        assert np.array_equal(r["pot"], runs[0]["pot"], equal_nan=True)
        assert r["counts"] == runs[0]["counts"]


def test_time_with_one_wave_per_cu():
    """One wave per CU takes 3.9 times as long on 20000 stars as all waves (6.6
    times where it takes the parts of a group one by one, each with the whole
    traversal); the limit lies between."""
    import torch
    from paper_1507_01009_amd import binding as B
    from gpu_helpers import to_dev
    n = 20000
    pos, _, m = ics.plummer(n, 3)
    dp, dm = to_dev(pos), to_dev(m)
    acc = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    us = []
    for w in (0, 1):
        say("few waves, time", w)
        ctx = B.Context(n, precision=B.TG_MIXED, waves_per_cu=w)
        ctx.build_tree(dp)
        ctx.compute_moments(dm)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        best = 1e9
        for _ in range(8):
            ev[0].record()
            for _ in range(10):
                ctx.tree_forces(0.01, 0.5, acc)
            ev[1].record()
            ev[1].synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]) * 100.0)
        us.append(best)
        ctx.close()
    say("  %.1f and %.1f us" % tuple(us))
    assert us[1] <= 5.2 * us[0]
