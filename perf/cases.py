"""Workloads that measure the library through its public entry points.

`listed()` names the fixed ones, `draw(rng)` gives further ones of the same
ranges, `prepare` makes the inputs and the context that a program keeps,
`run` is one pass (a force evaluation, an integrator step, a run of block
substeps, a hybrid step or a direct sum), `work` its unavoidable bytes and
flops and `exact` the same outputs from a plain FP64 direct sum.

Stars are drawn on the GPU: Plummer or Dehnen spheres (G = M = scale radius
= 1), equal masses, isotropic Gaussian velocities near the local circular
speed, SMBHs at the centre as in the benchmark workloads.
"""
import math

import numpy as np
import torch

from paper_1507_01009_amd import binding as B

_F64 = {"dtype": torch.float64, "device": "cuda"}


def _case(name, kind, n, **more):
    """Every case has every field, so that drawn and listed ones are alike."""
    c = {"name": name, "kind": kind, "n": n, "model": "dehnen", "gamma": 1.5, "fraction": 0.99,
         "precision": "mixed", "eps": 1e-3, "theta": 0.5, "alpha": 0.0, "softening": "plummer",
         "leaf": 8, "group": 64, "levels": 21, "n_bh": 0, "systems": 1, "active": 1.0,
         "substeps": 0, "n_src": 0, "dt": 1e-5, "r_chain0": 0.0}
    c.update(more)
    return c


def listed():
    return [
        # a small cluster, evaluated call by call (build, moments, forces): latency and launches
        _case("forces_1021_mixed", "forces", 1021, model="plummer", eps=0.01),
        # the Plummer sphere of the parity tests, in double precision
        _case("plummer_4096_fp64", "forces", 4096, model="plummer", precision="fp64", eps=0.01),
        # KDK steps of a galaxy with one SMBH, the energy-conservation run, in both precisions
        _case("hernquist_131072_kdk_mixed", "kdk", 131072, gamma=1.0, eps=0.01, n_bh=1, dt=1e-3),
        _case("hernquist_131072_kdk_fp64", "kdk", 131072, gamma=1.0, eps=0.01, n_bh=1, dt=1e-3,
              precision="fp64"),
        # the benchmark step: a dense cusp with an SMBH binary, in both precisions
        _case("cusp_1048576_kdk_mixed", "kdk", 1048576, n_bh=2),
        _case("cusp_1048576_kdk_fp64", "kdk", 1048576, n_bh=2, precision="fp64"),
        # the paper's own tree settings: relative opening test, drift-kick-drift (odd size)
        _case("relative_250007_dkd_mixed", "dkd", 250007, gamma=1.0, eps=0.01, n_bh=2, dt=1e-3,
              alpha=1e-3),
        # an untruncated cusp on 42-level keys with spline softening, in double precision (odd size)
        _case("spline_deep_100003_fp64", "forces", 100003, fraction=1.0 - 1e-9, levels=42,
              softening="spline", precision="fp64"),
        # 32 realisations of different sizes and slopes in one launch sequence
        _case("batch_32_kdk_mixed", "kdk", 4194304, gamma=0.0, eps=0.01, n_bh=1, systems=32,
              dt=1e-3),
        # one cycle of block substeps of a large galaxy through the host driver
        _case("hernquist_4194304_blocks", "blocks", 4194304, gamma=1.0, eps=0.01, n_bh=1,
              substeps=128, dt=2.0 ** -6),
        # the FP64 direct sum that tree forces are checked with: sampled targets, all sources
        _case("direct_8191_of_262144", "direct", 8191, n_src=262144, precision="fp64"),
        # the hybrid step: tree, host AR-chain around the SMBH, coupling and membership (a small
        # step, so that the chain changes little over a run of passes)
        _case("hybrid_131072_mixed", "hybrid", 131072, n_bh=1, r_chain0=0.003, dt=1e-6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forces", "forces", "active", "kdk", "kdk", "dkd", "batch", "blocks",
                       "direct", "hybrid"])
    prec = rng.choice(["mixed", "mixed", "fp64"])
    gamma = rng.choice([0.5, 1.0, 1.5])
    soft = rng.choice(["plummer", "plummer", "plummer", "spline"])
    leaf, group = rng.choice([(8, 64), (8, 64), (8, 48), (12, 64), (16, 32)])
    more = dict(precision=prec, gamma=gamma, softening=soft, leaf=leaf, group=group,
                eps=0.01 if gamma < 1.5 else 1e-3)
    if kind == "forces":
        deep = rng.random() < 0.25
        n = _log_int(rng, 512, 1500000)
        c = _case("", kind, n, model=rng.choice(["plummer", "dehnen"]),
                  levels=42 if deep else 21, fraction=1.0 - 1e-9 if deep else 0.99, **more)
    elif kind == "active":
        c = _case("", kind, _log_int(rng, 4096, 1500000), n_bh=1,
                  active=math.exp(rng.uniform(math.log(1e-3), math.log(0.5))), **more)
    elif kind == "kdk":
        c = _case("", kind, _log_int(rng, 1000, 1500000), n_bh=rng.choice([0, 1, 2]), dt=1e-4,
                  **more)
    elif kind == "dkd":
        c = _case("", kind, _log_int(rng, 1000, 1500000), n_bh=rng.choice([0, 1, 2]), dt=1e-4,
                  alpha=rng.choice([0.0, 1e-3, 5e-3]), **more)
    elif kind == "batch":
        s = rng.randint(2, 40)
        more["eps"] = 0.01
        c = _case("", "kdk", s * _log_int(rng, 2000, 30000), systems=s, n_bh=1, dt=1e-4, **more)
    elif kind == "blocks":
        c = _case("", kind, _log_int(rng, 20000, 1500000), n_bh=1, dt=2.0 ** -6,
                  substeps=rng.choice([64, 128]), **more)
    elif kind == "direct":
        more["precision"] = "fp64"
        c = _case("", kind, _log_int(rng, 300, 16000), n_src=_log_int(rng, 3000, 200000), **more)
    else:
        more.update(softening="plummer", gamma=1.5, eps=1e-3)
        c = _case("", kind, _log_int(rng, 30000, 200000), n_bh=1, r_chain0=0.003, dt=1e-6,
                  **more)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _sizes(case):
    """Stars per system: log-uniform over [2^14, 2^19] (scaled to the total)."""
    s, n = case["systems"], case["n"]
    if s == 1:
        return [n]
    w = [32.0 ** (((k * 0.6180339887498949) % 1.0)) for k in range(s)]
    out = [int(n * x / sum(w)) for x in w]
    out[0] += n - sum(out)
    return out


def _sphere(case, n, gamma, g):
    """(pos, vel) of one system, centred on the origin."""
    u = torch.rand(n, generator=g, **_F64).clamp_(min=1e-15)
    if case["model"] == "plummer":
        r = (u.clamp(max=1.0 - 1e-12) ** (-2.0 / 3.0) - 1.0).clamp_(min=1e-30) ** -0.5
        m = u
    else:
        y = (u * case["fraction"]) ** (1.0 / (3.0 - gamma))
        r = y / (1.0 - y)
        m = u * case["fraction"]
    cth = 2.0 * torch.rand(n, generator=g, **_F64) - 1.0
    phi = 2.0 * math.pi * torch.rand(n, generator=g, **_F64)
    sth = (1.0 - cth * cth).sqrt()
    pos = torch.stack([r * sth * phi.cos(), r * sth * phi.sin(), r * cth], 1)
    bh = 0.01 if case["n_bh"] else 0.0
    sigma = ((m + bh) / r.clamp(min=case["eps"]) / 3.0).sqrt()
    vel = torch.randn(n, 3, generator=g, **_F64) * sigma[:, None]
    return pos.contiguous(), vel.contiguous()


def _stars(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    sizes = _sizes(case)
    gam = [case["gamma"] or (0.5, 1.0, 1.5)[k % 3] for k in range(len(sizes))]
    parts = [_sphere(case, n, y, g) for n, y in zip(sizes, gam)]
    pos = torch.cat([p for p, _ in parts]).contiguous()
    vel = torch.cat([v for _, v in parts]).contiguous()
    mass = torch.cat([torch.full((n,), 1.0 / n, **_F64) for n in sizes])
    off = [0]
    for n in sizes:
        off.append(off[-1] + n)
    return pos, vel, mass, off, g


def _holes(case):
    """SMBHs of every system: one at rest at the centre, or a binary."""
    s, nb = case["systems"], case["n_bh"]
    if nb == 0:
        return None
    if nb == 1:
        bp, bv, bm = [[0.0, 0.0, 0.0]] * s, [[0.0, 0.0, 0.0]] * s, [0.01] * s
    else:
        v = math.sqrt(0.005 * (0.005 / 0.01 ** 2 + 0.005 ** 1.5 / 0.005 ** 2))
        bp = [[0.005, 0.0, 0.0], [-0.005, 0.0, 0.0]] * s
        bv = [[0.0, v, 0.0], [0.0, -v, 0.0]] * s
        bm = [0.005, 0.005] * s
    t = lambda x: torch.tensor(x, **_F64)
    return t(bp), t(bv), t(bm), t([case["eps"]] * len(bm))


class _State:
    pass


def prepare(case, seed):
    st = _State()
    st.case = case
    if case["kind"] == "direct":
        src = dict(case, n=case["n_src"])
        st.spos, _, st.smass, _, g = _stars(src, seed)
        pick = torch.randperm(case["n_src"], generator=g, device="cuda")
        pick = pick.repeat(-(-case["n"] // case["n_src"]))[:case["n"]]
        # checked positions near stars, not on them
        st.tpos = (st.spos[pick] * 1.001 + 1e-4).contiguous()
        st.seps = torch.full((case["n_src"],), case["eps"], **_F64)
        st.teps = torch.full((case["n"],), case["eps"], **_F64)
        st.acc, st.pot = torch.zeros((case["n"], 3), **_F64), torch.zeros(case["n"], **_F64)
        st.ctx = B.Context(1, precision=B.TG_FP64)
        st.ctx.set_softening(case["softening"])
        return st
    st.pos, st.vel, st.mass, off, g = _stars(case, seed)
    n = case["n"]
    st.acc, st.pot = torch.zeros((n, 3), **_F64), torch.zeros(n, **_F64)
    st.ctx = B.Context(n, max_systems=case["systems"], leaf_size=case["leaf"],
                       group_size=case["group"], key_levels=case["levels"],
                       precision=B.TG_FP64 if case["precision"] == "fp64" else B.TG_MIXED)
    st.ctx.set_softening(case["softening"])
    if case["kind"] == "forces":
        return st
    holes = _holes(case)
    bh = {}
    if holes is not None:
        st.bpos, st.bvel, st.bmass, st.beps = holes
        st.bacc, st.bpot = torch.zeros_like(st.bpos), torch.zeros_like(st.bmass)
        nb = case["n_bh"]
        bh = dict(bh_pos=st.bpos, bh_vel=st.bvel, bh_acc=st.bacc, bh_mass=st.bmass,
                  bh_eps=st.beps, bh_pot=st.bpot,
                  bh_seg=[nb * k for k in range(case["systems"] + 1)])
    st.sys = st.ctx.make_system(st.pos, st.vel, st.acc, st.mass, case["eps"], case["theta"],
                                pot=st.pot, sys_off=off, **bh)
    if case["kind"] == "hybrid":
        st.hy = B.Hybrid(st.ctx, st.sys, r_chain0=case["r_chain0"])
        st.hy.begin()
        return st
    st.ctx.forces(st.sys)          # the forces a program starts its steps from
    if case["alpha"] > 0.0:
        st.ctx.set_mac(relative=True, alpha=case["alpha"])
    if case["kind"] == "active":
        m = max(1, int(case["active"] * n))
        r2 = (st.pos * st.pos).sum(1)
        # the innermost stars, as block steps have them, in ascending order
        st.idx = torch.argsort(r2)[:m].sort().values.to(torch.int32).contiguous()
        st.na = torch.tensor([m], dtype=torch.int32, device="cuda")
    elif case["kind"] == "blocks":
        st.level = torch.zeros(n, dtype=torch.uint8, device="cuda")
        st.t4e2 = torch.full((n,), 0.3 ** 4 * case["eps"] ** 2, **_F64)
        st.idx = torch.zeros(n, dtype=torch.int32, device="cuda")
        st.na = torch.zeros(1, dtype=torch.int32, device="cuda")
        st.k = torch.zeros(1, dtype=torch.int64, device="cuda")
        st.blk = st.ctx.make_blocks(st.level, st.t4e2, st.idx, st.na, st.k, case["dt"], 8)
    return st


def run(st):
    case, ctx = st.case, st.ctx
    kind = case["kind"]
    if kind == "direct":
        ctx.direct_fp64(st.spos, st.smass, st.seps, st.tpos, st.teps, st.acc, pot=st.pot)
        return {"acc": st.acc, "pot": st.pot}
    if kind == "forces":
        ctx.build_tree(st.pos)
        ctx.compute_moments(st.mass)
        ctx.tree_forces(case["eps"], case["theta"], st.acc, st.pot)
        return {"acc": st.acc, "pot": st.pot}
    if kind == "active":
        ctx.forces(st.sys, st.idx, st.na)
    elif kind == "kdk":
        ctx.step_kdk(st.sys, case["dt"])
    elif kind == "dkd":
        ctx.step_dkd(st.sys, case["dt"])
    elif kind == "blocks":
        ctx.step_blocks(st.sys, st.blk, case["substeps"])
    else:
        st.hy.step(case["dt"])
    out = {"pos": st.pos, "vel": st.vel, "acc": st.acc, "pot": st.pot}
    if case["n_bh"]:
        out.update(bh_pos=st.bpos, bh_vel=st.bvel, bh_acc=st.bacc, bh_pot=st.bpot)
    if kind == "blocks":
        out.update(level=st.level, k=st.k)
    if kind == "hybrid":
        # the chain's members, in arrays of the largest chain's length (rows past the end -1 and 0)
        s = st.hy.state()
        m = len(s["members"])
        ids, x, v = np.full(256, -1, np.int32), np.zeros((256, 3)), np.zeros((256, 3))
        ids[:m], x[:m], v[:m] = s["members"], s["x"], s["v"]
        out.update(members=ids, member_x=x, member_v=v)
    return out


# -------------------------------------------------------------------- work
def _pair_flops(case, n):
    """Flops of one target's evaluation: 19 per particle pair and 54 per cell
    pair, whose counts grow with log N (measured counts of the opening angle
    0.5 at leaf 8; the relative test at 1e-3 needs about half)."""
    d = math.log2(max(n, 512))
    p2p, p2m = min(n, 550.0), max(0.0, 299.0 * (d - 9.86))
    return (19.0 * p2p + 54.0 * p2m) * (0.5 if case["alpha"] > 0.0 else 1.0)


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "direct":
        return {"bytes": 40.0 * case["n_src"] + 64.0 * n, "flops": 19.0 * n * case["n_src"]}
    flops = sum(m * _pair_flops(case, m) for m in _sizes(case))
    if kind == "forces":
        return {"bytes": 64.0 * n, "flops": flops}
    if kind == "active":
        return {"bytes": 32.0 * n + 36.0 * case["active"] * n, "flops": flops * case["active"]}
    if kind == "blocks":
        # a star's drift in every substep and its forces once a cycle of 128
        return {"bytes": 80.0 * n * case["substeps"], "flops": flops * case["substeps"] / 128.0}
    return {"bytes": 160.0 * n, "flops": flops}


# ------------------------------------------------------------------- exact
def _psi(r2, h, soft):
    """psi and psi_1 of pairs at squared distance r2 (r2 = 0: a star itself)."""
    if soft == "plummer":
        p = (r2 + h * h).rsqrt()
        return p, p * p * p
    r = r2.sqrt()
    far = r.clamp(min=1e-300).reciprocal()
    u = r / h
    inner = (1.4 + u * u * (-2.0 / 3.0 + u * u * (0.3 - 0.1 * u))) / h
    inner1 = (4.0 / 3.0 + u * u * (-1.2 + 0.5 * u)) / h ** 3
    uu = u.clamp(min=1.0)
    outer = (1.6 + uu * uu * (-4.0 / 3.0 + uu * (1.0 + uu * (-0.3 + uu / 30.0)))
             - 1.0 / (15.0 * uu)) / h
    outer1 = (8.0 / 3.0 + uu * (-3.0 + uu * (1.2 - uu / 6.0)) - 1.0 / (15.0 * uu ** 3)) / h ** 3
    p = torch.where(u < 1.0, inner, torch.where(u < 2.0, outer, far))
    p1 = torch.where(u < 1.0, inner1, torch.where(u < 2.0, outer1, far ** 3))
    return p, p1


def _direct(tpos, spos, smass, eps, soft, own):
    """Sums over all sources; own: targets are the sources (no self pair)."""
    acc, pot = torch.empty_like(tpos), torch.empty(tpos.shape[0], **_F64)
    rows = max(1, (1 << 26) // max(1, spos.shape[0]))
    for a in range(0, tpos.shape[0], rows):
        b = min(a + rows, tpos.shape[0])
        d = [tpos[a:b, k, None] - spos[None, :, k] for k in range(3)]
        p, p1 = _psi(d[0] * d[0] + d[1] * d[1] + d[2] * d[2], eps, soft)
        if own:
            i = torch.arange(a, b, device=tpos.device)
            p[i - a, i] = 0.0
        pot[a:b] = -(p @ smass)
        for k in range(3):
            acc[a:b, k] = -((p1 * d[k]) @ smass)
    return acc, pot


def _all_forces(case, pos, mass, off, holes):
    """Forces on stars and SMBHs at given positions."""
    soft, eps = case["softening"], case["eps"]
    nb = case["n_bh"]
    acc, pot = torch.empty_like(pos), torch.empty_like(mass)
    if holes is not None:
        bpos, bmass = holes[0], holes[2]
        bacc, bpot = torch.zeros_like(bpos), torch.zeros_like(bmass)
    for s in range(len(off) - 1):
        a, b = off[s], off[s + 1]
        acc[a:b], pot[a:b] = _direct(pos[a:b], pos[a:b], mass[a:b], eps, soft, True)
        if holes is not None:
            h = slice(nb * s, nb * (s + 1))
            da, dp = _direct(pos[a:b], bpos[h], bmass[h], eps, soft, False)
            acc[a:b] += da
            pot[a:b] += dp
            ba, bp = _direct(bpos[h], pos[a:b], mass[a:b], eps, soft, False)
            ca, cp = _direct(bpos[h], bpos[h], bmass[h], eps, soft, True)
            bacc[h], bpot[h] = ba + ca, bp + cp
    return (acc, pot, bacc, bpot) if holes is not None else (acc, pot, None, None)


def exact(case, seed):
    """Direct sums: the tree's forces differ from them by the truncation of
    the multipole expansion, the direct kernel's by rounding alone."""
    kind, dt = case["kind"], case["dt"]
    if kind == "direct":
        st = prepare(case, seed)
        acc, pot = _direct(st.tpos, st.spos, st.smass, case["eps"], case["softening"], False)
        return {"acc": acc, "pot": pot}
    if kind in ("blocks", "hybrid") or sum(m * m for m in _sizes(case)) > 7e10:
        return None
    pos, vel, mass, off, _ = _stars(case, seed)
    if kind == "forces":
        acc, pot = _direct(pos, pos, mass, case["eps"], case["softening"], True)
        return {"acc": acc, "pot": pot}
    holes = _holes(case)
    if kind == "active":
        return None                 # inactive rows keep the tree's earlier forces
    if kind == "kdk":
        acc, _, bacc, _ = _all_forces(case, pos, mass, off, holes)
        vel = vel + 0.5 * dt * acc
        pos = pos + dt * vel
        if holes is not None:
            holes = (holes[0], holes[1] + 0.5 * dt * bacc) + holes[2:]
            holes = (holes[0] + dt * holes[1],) + holes[1:]
    else:
        pos = pos + 0.5 * dt * vel
        if holes is not None:
            holes = (holes[0] + 0.5 * dt * holes[1],) + holes[1:]
    acc, pot, bacc, bpot = _all_forces(case, pos, mass, off, holes)
    w = 0.5 * dt if kind == "kdk" else dt
    vel = vel + w * acc
    if kind == "dkd":
        pos = pos + 0.5 * dt * vel
    out = {"pos": pos, "vel": vel, "acc": acc, "pot": pot}
    if holes is not None:
        bpos, bvel = holes[0], holes[1] + w * bacc
        if kind == "dkd":
            bpos = bpos + 0.5 * dt * bvel
        out.update(bh_pos=bpos, bh_vel=bvel, bh_acc=bacc, bh_pot=bpot)
    return out
