"""The FP64 direct sum's tiled path (64 or 128 targets to a block, source
tiles in LDS) at the edges of its blocks, tiles and splits, against the same
sums in extended precision."""
import sys

import numpy as np
import pytest

import oracle
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _inputs(nt, ns, own, seed):
    rng = np.random.default_rng(seed)
    sp = rng.normal(size=(ns, 3)) ** 3
    sm = rng.uniform(0.5, 1.5, ns) / ns
    se = rng.choice([0.0, 1e-3, 0.02], ns)
    if own:
        return sp, sm, se, sp, se
    return sp, sm, se, rng.normal(size=(nt, 3)) ** 3, rng.choice([0.0, 0.01], nt)


def _run(a, softening="plummer", acc0=None, pot0=None, **kw):
    import torch
    from paper_1507_01009_amd import binding as B
    nt = a[3].shape[0]
    ctx = B.Context(1)
    ctx.set_softening(softening)
    acc = to_dev(acc0) if acc0 is not None else torch.full((nt, 3), float("nan"),
                                                           dtype=torch.float64, device="cuda")
    pot = to_dev(pot0) if pot0 is not None else torch.full((nt,), float("nan"),
                                                           dtype=torch.float64, device="cuda")
    ctx.direct_fp64(*[to_dev(x) for x in a], acc, pot, **kw)
    ctx.sync()
    ctx.close()
    return acc.cpu().numpy(), pot.cpu().numpy()


def _extended(a, own):
    """(acc, pot, sums of the terms' magnitudes) in long double."""
    sp, sm, se, tp, te = [x.astype(np.longdouble) for x in a]
    acc = np.zeros((tp.shape[0], 3), np.longdouble)
    pot = np.zeros(tp.shape[0], np.longdouble)
    sa, spt = np.zeros_like(acc), np.zeros_like(pot)
    for i in range(tp.shape[0]):
        d = tp[i] - sp
        D1 = 1.0 / np.sqrt((d * d).sum(1) + np.maximum(se, te[i]) ** 2)
        if own:
            D1[i] = 0.0
        w = (sm * D1 ** 3)[:, None] * d
        acc[i], sa[i] = -w.sum(0), np.abs(w).sum(0)
        pot[i] = spt[i] = (sm * D1).sum()
    return acc, -pot, sa, spt


# rounding of one term: the difference 1 u, r^2 6 u (3 u in D1), D1 2 u more,
# its cube 15 u with the three products' 3 u and the last one's 1 u: below
# 24 u of the term, and the compensated sum adds about 2 u
TOL = 26 * 2.0 ** -53


@pytest.mark.parametrize("nt,ns,own", [(64, 64, True), (65, 65, True), (64, 257, False),
                                       (127, 8191, False), (128, 255, False), (129, 256, False),
                                       (129, 70001, False), (300, 300, True), (4097, 512, False),
                                       (2500, 2500, True)])
def test_tiles_match_extended_precision(nt, ns, own):
    say("direct tiles", nt, ns, own)
    a = _inputs(nt, ns, own, nt + ns)
    acc, pot = _run(a, self_pairs=own)
    ra, rp, sa, sp = _extended(a, own)
    say("  acc %.3g pot %.3g of the bound" % (np.max(np.abs(acc - ra) / sa) / TOL,
                                             np.max(np.abs(pot - rp) / sp) / TOL))
    assert np.all(np.abs(acc - ra) <= TOL * sa)
    assert np.all(np.abs(pot - rp) <= TOL * sp)


@pytest.mark.parametrize("nt,ns,own", [(1, 1, True), (1, 1, False), (2, 2, True), (63, 63, True),
                                       (63, 1000, False), (3, 8191, False), (700, 63, False)])
def test_a_thread_per_target(nt, ns, own):
    """The plain kernel, below the sizes of the others: no source, one, and chunks."""
    say("direct plain", nt, ns, own)
    a = _inputs(nt, ns, own, nt + ns)
    acc, pot = _run(a, self_pairs=own)
    ra, rp, sa, sp = _extended(a, own)
    assert np.all(np.abs(acc - ra) <= TOL * sa) and np.all(np.abs(pot - rp) <= TOL * sp)


@pytest.mark.parametrize("nt,ns", [(100, 3000), (500, 5001)])
def test_tiles_spline_and_accumulation(nt, ns):
    say("direct tiles spline", nt, ns)
    a = _inputs(nt, ns, False, 3 * nt)
    acc, pot = _run(a, softening="spline")
    ra, rp = oracle.direct_pairs(*a, softening="spline")
    assert np.max(np.linalg.norm(acc - ra, axis=1) / np.linalg.norm(ra, axis=1)) <= 1e-12
    assert np.max(np.abs(pot - rp) / np.abs(rp)) <= 1e-12
    rng = np.random.default_rng(1)
    a0, p0 = rng.normal(size=(nt, 3)), rng.normal(size=nt)
    acc2, pot2 = _run(a, softening="spline", acc0=a0, pot0=p0, accumulate=True)
    assert np.array_equal(acc2, a0 + acc) and np.array_equal(pot2, p0 + pot)


def test_coincident_unsoftened_pairs_as_the_formula():
    """r = 0 without softening: an infinite potential and no finite force,
    also where the pair is one of many; its own pair is left out."""
    a = [x.copy() for x in _inputs(70, 300, False, 9)]
    a[2][:], a[4][:] = 0.0, 0.0
    a[3][5] = a[0][17]
    acc, pot = _run(a)
    assert np.all(np.isnan(acc[5])) and not np.isfinite(pot[5])
    rest = np.arange(70) != 5
    assert np.all(np.isfinite(acc[rest])) and np.all(np.isfinite(pot[rest]))
    b = (a[0], a[1], a[2], a[0], a[2])
    acc, pot = _run(b, self_pairs=True)
    assert np.all(np.isfinite(acc)) and np.all(np.isfinite(pot))


def _segmented(sizes, per, seed):
    rng = np.random.default_rng(seed)
    off, tof = np.concatenate([[0], np.cumsum(sizes)]), per * np.arange(len(sizes) + 1)
    a = (rng.normal(size=(off[-1], 3)) ** 3, rng.uniform(0.5, 1.5, off[-1]) / off[-1],
         rng.choice([0.0, 1e-3], off[-1]), rng.normal(size=(tof[-1], 3)),
         rng.choice([0.0, 0.01], tof[-1]))
    return a, [int(x) for x in off], [int(x) for x in tof]


@pytest.mark.parametrize("sizes,per", [((8192,) + (300, 0, 9000) * 21, 2),      # 128 targets
                                       ((8191, 100) * 70, 1), ((20000, 1), 65)])
def test_many_targets_of_several_segments(sizes, per):
    """From 128 targets in all, with segments long enough for the few-target
    kernel and without, empty and short segments between."""
    say("direct segments", len(sizes), per)
    a, so, to = _segmented(sizes, per, len(sizes))
    acc, pot = _run(a, src_seg=so, tgt_seg=to)
    for s in range(len(sizes)):
        i, j = slice(to[s], to[s + 1]), slice(so[s], so[s + 1])
        ra, rp, sa, sp = _extended((a[0][j], a[1][j], a[2][j], a[3][i], a[4][i]), False)
        assert np.all(np.abs(acc[i] - ra) <= TOL * sa) and np.all(np.abs(pot[i] - rp) <= TOL * sp)


def _time(ctx, a, **kw):
    """Least time of a call in us, from windows of 20 calls."""
    import torch
    d = [to_dev(x) for x in a]
    acc = torch.zeros((a[3].shape[0], 3), dtype=torch.float64, device="cuda")
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = 1e9
    for _ in range(8):
        ev[0].record()
        for _ in range(20):
            ctx.direct_fp64(*d, acc, **kw)
        ev[1].record()
        ev[1].synchronize()
        best = min(best, ev[0].elapsed_time(ev[1]) * 50.0)
    return best


def test_time_of_many_targets_of_several_segments():
    """64 systems with two targets each take about as long as 63 such systems
    (126 targets; a thread per target and chunk took six times as long)."""
    from paper_1507_01009_amd import binding as B
    ctx = B.Context(1)
    us = []
    for systems in (63, 64):
        say("direct segments, time", systems)
        a, so, to = _segmented((20000,) * systems, 2, 1)
        us.append(_time(ctx, a, src_seg=so, tgt_seg=to))
    say("  %.1f and %.1f us" % tuple(us))
    assert us[1] <= 2.5 * us[0]


def test_time_of_a_hundred_targets_on_few_sources():
    """128 targets on 8192 sources take about as long as 60 (tiles, whose 32
    chunks a thread per target added up, took 2.7 times as long)."""
    from paper_1507_01009_amd import binding as B
    ctx = B.Context(1)
    us = [_time(ctx, _inputs(nt, 8192, False, nt)) for nt in (60, 128)]
    say("direct few sources, time  %.1f and %.1f us" % tuple(us))
    assert us[1] <= 1.8 * us[0]


@pytest.mark.parametrize("nt,ns", [(65, 8192), (128, 65535), (128, 65536), (700, 9000),
                                   (64, 4097), (200, 8191)])
def test_lines_of_one_segment(nt, ns):
    """Both sides of the lines between the few-target blocks, the tiles, and the
    two ways to add up the tiles' chunks."""
    say("direct lines", nt, ns)
    a = _inputs(nt, ns, False, nt + ns)
    acc, pot = _run(a)
    ra, rp, sa, sp = _extended(a, False)
    assert np.all(np.abs(acc - ra) <= TOL * sa) and np.all(np.abs(pot - rp) <= TOL * sp)


@pytest.mark.parametrize("nt,ns", [(131073, 65), (131072, 95), (131080, 96)])
def test_many_targets_on_few_sources(nt, ns):
    """Both sides of the line between tiles and a thread per target: the first and
    last blocks' targets."""
    say("direct many targets", nt, ns)
    a = _inputs(nt, ns, False, nt + ns)
    acc, pot = _run(a)
    pick = np.r_[0:130, nt // 2:nt // 2 + 130, nt - 130:nt]
    ra, rp, sa, sp = _extended((a[0], a[1], a[2], a[3][pick], a[4][pick]), False)
    assert np.all(np.abs(acc[pick] - ra) <= TOL * sa) and np.all(np.abs(pot[pick] - rp) <= TOL * sp)
    assert np.all(np.isfinite(acc)) and np.all(np.isfinite(pot))
