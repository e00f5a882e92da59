"""SMBH sums of an evaluation (stars and the other SMBHs in two launches up to 63
SMBHs) against the same sums by tg_direct_fp64, and idle block substeps (totals,
mutual pull and the next move in one launch up to 4 SMBHs) against single
substeps.  Both orders of operations are the same: bit for bit."""
import sys

import numpy as np
import pytest

from paper_1507_01009_amd import ics
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _system(n, nb, sizes=None, softening="plummer"):
    import torch
    from paper_1507_01009_amd import binding as B
    rng = np.random.default_rng(n + nb)
    off = None if sizes is None else [0] + list(np.cumsum(sizes))
    seg = None if sizes is None else [nb * k for k in range(len(sizes) + 1)]
    S = 1 if sizes is None else len(sizes)
    d = {"pos": to_dev(ics.plummer(n, 3)[0]), "vel": to_dev(0.3 * rng.normal(size=(n, 3))),
         "mass": to_dev(rng.uniform(0.5, 1.5, n) / n), "bpos": to_dev(rng.normal(size=(S * nb, 3))),
         "bvel": to_dev(0.2 * rng.normal(size=(S * nb, 3))),
         "bmass": to_dev(rng.uniform(0.01, 0.02, S * nb)),
         "beps": to_dev(rng.uniform(0.005, 0.02, S * nb))}
    z = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda")
    d.update(acc=z(n, 3), pot=z(n), bacc=z(S * nb, 3), bpot=z(S * nb))
    ctx = B.Context(n, max_systems=S)
    ctx.set_softening(softening)
    d["sys"] = ctx.make_system(d["pos"], d["vel"], d["acc"], d["mass"], 0.01, 0.5, pot=d["pot"],
                               sys_off=off, bh_pos=d["bpos"], bh_vel=d["bvel"], bh_acc=d["bacc"],
                               bh_mass=d["bmass"], bh_eps=d["beps"], bh_pot=d["bpot"], bh_seg=seg)
    return ctx, d, off, seg


@pytest.mark.parametrize("softening", ["plummer", "spline"])
@pytest.mark.parametrize("nb,sizes", [(1, None), (2, None), (5, None), (63, None), (64, None),
                                      (3, (9000, 0, 700, 8300))])
def test_sums_equal_the_direct_kernels(nb, sizes, softening):
    import torch
    n = 9001 if sizes is None else sum(sizes)
    say("smbh sums", nb, sizes, softening)
    ctx, d, off, seg = _system(n, nb, sizes, softening)
    ctx.forces(d["sys"])
    acc, pot = torch.zeros_like(d["bacc"]), torch.zeros_like(d["bpot"])
    eps = torch.full((n,), 0.01, dtype=torch.float64, device="cuda")
    ctx.direct_fp64(d["pos"], d["mass"], eps, d["bpos"], d["beps"], acc, pot=pot, src_seg=off,
                    tgt_seg=seg)
    ctx.direct_fp64(d["bpos"], d["bmass"], d["beps"], d["bpos"], d["beps"], acc, pot=pot,
                    src_seg=seg, tgt_seg=seg, self_pairs=True, accumulate=True)
    ctx.sync()
    assert torch.equal(d["bacc"], acc) and torch.equal(d["bpot"], pot)
    assert bool((acc.abs().sum(1) > 0).all())


@pytest.mark.parametrize("nb", [1, 2, 4, 5])
def test_idle_substeps_equal_single_ones(nb):
    import torch
    say("idle substeps", nb)
    out = []
    for driver in (False, True):
        ctx, d, _, _ = _system(9001, nb)
        i32 = dict(dtype=torch.int32, device="cuda")
        blk = [torch.zeros(9001, dtype=torch.uint8, device="cuda"),
               torch.full((9001,), 0.3 ** 4 * 1e-4, dtype=torch.float64, device="cuda"),
               torch.zeros(9001, **i32), torch.zeros(1, **i32),
               torch.zeros(1, dtype=torch.int64, device="cuda")]
        b = ctx.make_blocks(*blk, 2.0 ** -6, 8)
        ctx.forces(d["sys"])
        idle = 0
        if driver:
            idle = ctx.step_blocks(d["sys"], b, 40)
        else:
            for _ in range(40):
                ctx.step_block(d["sys"], b)
        ctx.sync()
        out.append([d[k].clone() for k in ("pos", "vel", "acc", "bpos", "bvel", "bacc", "bpot")]
                   + [blk[0].clone(), blk[4].clone()])
    assert idle > 20
    for x, y in zip(*out):
        assert torch.equal(x, y)


def test_mutual_sums_captured_after_an_evaluation():
    """An eager evaluation makes the SMBHs' own segment table known, also where their
    mutual pull comes with the stars' sums: the direct call on them can be captured."""
    import torch
    say("captured mutual sums")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx, d, _, seg = _system(9001, 2)
        ctx.forces(d["sys"])
        ctx.sync()
        acc, ref = torch.zeros_like(d["bacc"]), torch.zeros_like(d["bacc"])
        ctx.graph_begin()
        ctx.direct_fp64(d["bpos"], d["bmass"], d["beps"], d["bpos"], d["beps"], acc, self_pairs=True)
        graph = ctx.graph_end()
        ctx.direct_fp64(d["bpos"], d["bmass"], d["beps"], d["bpos"], d["beps"], ref, self_pairs=True)
        graph.launch(s)
        s.synchronize()
        assert torch.equal(acc, ref) and bool((acc != 0).any())
        del graph
        ctx.close()
