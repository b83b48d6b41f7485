"""The work that users of the kd-tree FMM library have it do, as measurable cases.

A case is a dict of plain values:

    op         what one pass does
               step     one force evaluation of a time step: build, moments,
                        walk, far and near field, momentum statistics
               kdk      two kick-drift-kick steps (three force evaluations)
               grad     accelerations and their vector-Jacobian product (a
                        training step through the forces), by autograd
               adjoint  kick-drift-kick steps with checkpoints, then the
                        reverse sweep through them
               census   forces, statistics and the census of asymmetric pairs
                        (one point of a sweep over N and theta)
    dist       plummer (untruncated, fixed h), star (n = 1 polytrope), binary
               (two of them), clumpy (uniform cube with Gaussian clumps and
               log-normal masses)
    n          particles
    fp32       the FP32 form instead of FP64
    mutual     the symmetric walk instead of leaf <- cell
    dehnen     the second expansion form
    com        the tree cut through the centre of mass
    theta, leaf

Inputs follow paper_2502_01496_amd/workloads.py, drawn on the GPU; the
smoothing lengths of all but the Plummer sphere come from the analytic number
density, h = 1.2 n^(-1/3) (57.9 neighbours in 2 h), which stands in for the
58-neighbour search of that module.
"""
import math

import torch

from paper_2502_01496_amd import fmm as F
from paper_2502_01496_amd import leapfrog as LF

DEV = "cuda:0"
DT = 1e-3         # time step of the KDK cases
STEPS = 2         # their steps


def _case(name, op, dist, n, **kw):
    c = dict(op=op, dist=dist, n=n, fp32=False, mutual=False, dehnen=False, com=False,
             theta=0.5, leaf=8)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small cluster integrated with a few thousand steps: launch latency
        _case("step_plummer_1000", "step", "plummer", 1000),
        # gradient of a short trajectory of a small cluster (fits of initial
        # conditions): many small force evaluations and reverse passes
        _case("adjoint_plummer_4096", "adjoint", "plummer", 4096),
        # a ragged star at PHANTOM's leaf size in the FP32 form: ordinary
        # production size of the low-resolution runs
        _case("kdk_star_30011_fp32", "kdk", "star", 30011, fp32=True, leaf=10),
        # one point of the sweep of |sum F| and the asymmetry estimates over N
        _case("census_star_131072", "census", "star", 131072, theta=0.7),
        # the polytrope binary of the KDK series
        _case("step_binary_524288", "step", "binary", 524288),
        _case("kdk_binary_524288_fp32", "kdk", "binary", 524288, fp32=True),
        # training step through the forces of the binary
        _case("grad_binary_524288", "grad", "binary", 524288),
        # the momentum-conserving walk, ragged size
        _case("mutual_binary_300007", "step", "binary", 300007, mutual=True),
        # the tree as the paper words it (cuts through the centre of mass)
        _case("com_clumpy_200003", "step", "clumpy", 200003, com=True, leaf=10),
        # the benchmark's default workload
        _case("step_clumpy_4194304", "step", "clumpy", 4194304),
        # concentrated cluster with an untruncated halo: FP32 forces and the
        # reverse pass (the list slots of twice as many particles would not
        # leave room for other states on the card)
        _case("grad_plummer_524288_fp32", "grad", "plummer", 524288, fp32=True),
        # the largest binary of the configurations, FP32 form
        _case("step_binary_16777216_fp32", "step", "binary", 16777216, fp32=True),
    ]


# largest n a drawn case takes, by operation and distribution: the halo of the
# untruncated Plummer sphere makes its lists long, the reverse pass and the
# mutual walk cost a few force evaluations each, and the centre-of-mass tree
# keeps buffers for 2n - 1 cells.  A large binary has two equal stars: with an
# odd particle one leaf spans both, takes every leaf as near, and the list
# slots of every leaf grow to that length.
_MOST = {"step": 1 << 23, "kdk": 1 << 21, "grad": 1 << 20, "adjoint": 1 << 17, "census": 1 << 20}


def draw(rng):
    op = rng.choice(["step", "step", "step", "kdk", "grad", "grad", "adjoint", "census"])
    dist = rng.choice(["plummer", "star", "binary", "clumpy"])
    mutual = rng.random() < 0.2
    com = rng.random() < 0.15
    most = _MOST[op]
    if dist == "plummer":
        most = min(most, 1 << 18)
    if mutual or com:
        most = min(most, 1 << 20)
    n = int(math.exp(rng.uniform(math.log(700), math.log(most))))
    if dist == "binary" and n > 1 << 17:
        n -= n % 2
    return _case(None, op, dist, n, fp32=rng.random() < 0.4, mutual=mutual,
                 dehnen=rng.random() < 0.15, com=com,
                 theta=rng.choice([0.3, 0.5, 0.5, 0.5, 0.7]) if n <= 1 << 17 else 0.5,
                 leaf=rng.choice([8, 8, 8, 10, 5, 16]))


# ------------------------------------------------------------------ inputs
def _directions(n, g):
    v = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    return v / v.norm(dim=1, keepdim=True)


def _star(n, g):
    """n particles of an n = 1 polytrope of radius 1 and their radii."""
    r = torch.linspace(0, 1, 65537, device=DEV, dtype=torch.float64)
    f = (torch.sin(math.pi * r) - math.pi * r * torch.cos(math.pi * r)) / math.pi
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    k = torch.searchsorted(f, u).clamp_(1, 65536)
    f0, f1 = f[k - 1], f[k]
    rr = r[k - 1] + (u - f0) / (f1 - f0).clamp_min(1e-300) * (r[1] - r[0])
    return rr[:, None] * _directions(n, g), rr


def _star_h(r, n):
    """h of a star of n particles from its density, at most the radius that
    holds 58 particles at the surface."""
    dens = n * (math.pi / 4) * torch.sinc(r.clamp_max(1.0))
    h = 1.2 * dens.clamp_min(1e-300) ** (-1.0 / 3.0)
    return h.clamp_max((5.87 / n) ** 0.25)


def _particles(case, seed):
    n, dist = case["n"], case["dist"]
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    if dist == "plummer":
        u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64).clamp_(1e-12, 1 - 1e-12)
        r = 1.0 / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
        x = r[:, None] * _directions(n, g)
        m = torch.full((n,), 1.0 / n, device=DEV, dtype=torch.float64)
        h = torch.full((n,), 0.01, device=DEV, dtype=torch.float64)
    elif dist == "star":
        x, r = _star(n, g)
        m = torch.full((n,), 1.0 / n, device=DEV, dtype=torch.float64)
        h = _star_h(r, n)
    elif dist == "binary":
        na = n // 2
        xa, ra = _star(na, g)
        xb, rb = _star(n - na, g)
        xa[:, 0] -= 2.0
        xb[:, 0] += 2.0
        x = torch.cat([xa, xb])
        m = torch.full((n,), 2.0 / n, device=DEV, dtype=torch.float64)
        h = torch.cat([_star_h(ra, na), _star_h(rb, n - na)])
    else:
        nc, sig, kc = int(0.3 * n), 0.02, 64
        centres = torch.rand(kc, 3, generator=g, device=DEV, dtype=torch.float64)
        which = torch.arange(nc, device=DEV) % kc
        xc = centres[which] + sig * torch.randn(nc, 3, generator=g, device=DEV,
                                                dtype=torch.float64)
        xb = torch.rand(n - nc, 3, generator=g, device=DEV, dtype=torch.float64)
        x = torch.cat([xc, xb])
        w = torch.exp(0.5 * torch.randn(n, generator=g, device=DEV, dtype=torch.float64))
        m = torch.empty(n, device=DEV, dtype=torch.float64)
        m[:nc] = w[:nc] * (0.3 / w[:nc].sum())
        m[nc:] = w[nc:] * (0.7 / w[nc:].sum())
        dens = torch.full((n,), float(n - nc), device=DEV, dtype=torch.float64)
        for k in range(kc):
            d2 = ((x - centres[k]) ** 2).sum(1)
            dens += (nc / kc) * (2 * math.pi * sig * sig) ** -1.5 * torch.exp(-d2 / (2 * sig * sig))
        h = 1.2 * dens ** (-1.0 / 3.0)
    return x.contiguous(), m, h, g


def prepare(case, seed):
    x, m, h, g = _particles(case, seed)
    n = case["n"]
    prec = F.FMM_FP32 if case["fp32"] else F.FMM_FP64
    field = LF.ForceField(theta=case["theta"], leaf_size=case["leaf"], precision=prec,
                          walk=F.FMM_WALK_MUTUAL if case["mutual"] else F.FMM_WALK_PHANTOM,
                          expansion=(F.FMM_EXPANSION_DEHNEN if case["dehnen"]
                                     else F.FMM_EXPANSION_PHANTOM),
                          tree_shape=F.FMM_TREE_COM if case["com"] else F.FMM_TREE_MEDIAN)
    s = dict(op=case["op"], field=field, x=x, m=m, h=h)
    if case["op"] in ("kdk", "adjoint", "step"):
        s["v"] = 0.3 * torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    if case["op"] == "grad":
        s["abar"] = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64).to(field.dtype)
    if case["op"] == "adjoint":
        s["xbar"] = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
        s["vbar"] = torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    if case["op"] in ("step", "census"):
        s["a"] = torch.empty(n, 3, device=DEV, dtype=field.dtype)
        s["stats"] = torch.empty(16, device=DEV, dtype=torch.float64)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    op, field, x, m, h = s["op"], s["field"], s["x"], s["m"], s["h"]
    if op == "step":
        field.forces(x, m, h, out=s["a"])
        F.fmm_momentum_stats_async(x, s["v"], m, s["a"], s["stats"])
        return {"a": s["a"], "stats": s["stats"]}
    if op == "census":
        field.forces(x, m, h, out=s["a"])
        st = F.fmm_momentum_stats(x, None, m, s["a"])
        c = F.fmm_asymmetry_estimate(field.g.tree)
        return {"a": s["a"], "sumF": st["sumF"], "sumAbsF": st["sumAbsF"], "F33": c["F33"],
                "F46": c["F46"], "pairs": [c["n_asym"], c["n_asym_super"]]}
    if op == "kdk":
        xT, vT, _ = LF.kdk_forward(x, s["v"], m, h, DT, STEPS, field, keep=False)
        return {"x": xT, "v": vT}
    if op == "grad":
        xg, mg = x.detach().requires_grad_(True), m.detach().requires_grad_(True)
        a = LF.FmmForce.apply(xg, mg, h, field)
        gx, gm = torch.autograd.grad(a, (xg, mg), s["abar"])
        return {"a": a.detach(), "x_bar": gx, "m_bar": gm}
    xT, vT, ckpt = LF.kdk_forward(x, s["v"], m, h, DT, STEPS, field)
    xbar, vbar, mbar = LF.kdk_backward(ckpt, m, h, DT, field, s["xbar"], s["vbar"])
    return {"x": xT, "v": vT, "x_bar": xbar, "v_bar": vbar, "m_bar": mbar}


# ------------------------------------------------------------------ work
def _counts(case):
    """Near-field pairs and far-field (M2L) interactions per particle, from
    the lists of each distribution at theta = 0.5 and leaf 8, scaled as
    theta^-3 (a bound of the order of magnitude, not a census)."""
    n, th = case["n"], (0.5 / case["theta"]) ** 3
    near, far = {"plummer": (1100.0 + 3550.0 * n / (1 << 20), 130.0 + 280.0 * n / (1 << 20)),
                 "star": (360.0, 41.0), "binary": (360.0, 41.0),
                 "clumpy": (730.0, 44.0)}[case["dist"]]
    return min(float(n), near * max(1.0, th)), far * th * 8.0 / case["leaf"]


def work(case):
    n, w = case["n"], 4 if case["fp32"] else 8
    near, far = _counts(case)
    force = n * (20.0 * near + 300.0 * far)            # flops of one evaluation
    fb = n * (5 * 8 + 3 * w)                           # x, m, h in, a out
    op = case["op"]
    if op == "step":
        return {"bytes": fb + n * 24.0, "flops": force}
    if op == "census":
        return {"bytes": float(fb), "flops": force}
    if op == "kdk":
        return {"bytes": n * (8 * 8 + 6 * 8.0), "flops": (STEPS + 1) * force}
    if op == "grad":
        return {"bytes": fb + n * 7.0 * w, "flops": 3.5 * force}
    return {"bytes": n * (14 * 8 + 13 * 8.0), "flops": (STEPS + 1) * 3.5 * force}


# ------------------------------------------------------------------ reference
def _m4(r, h):
    """phi'/r of the M4 kernel of smoothing length h."""
    q = r / h
    inner = (4 / 3 - 1.2 * q ** 2 + 0.5 * q ** 3) / h ** 3
    outer = (8 / 3 - 3 * q + 1.2 * q ** 2 - q ** 3 / 6) / h ** 3 - 1 / (15 * r ** 3)
    return torch.where(q < 1, inner, torch.where(q < 2, outer, r ** -3.0))


def _direct_rows(x, m, h, i0, i1):
    """Accelerations of the particles i0..i1 by the direct sum the FMM
    approximates."""
    d = x[i0:i1, None, :] - x[None, :, :]
    r2 = (d * d).sum(2)
    r2 = torch.where(r2 == 0, torch.ones_like(r2), r2)  # the particle itself: d = 0
    r = torch.sqrt(r2)
    gij = 0.5 * (_m4(r, h[i0:i1, None]) + _m4(r, h[None, :]))
    return -((m[None, :] * gij)[:, :, None] * d).sum(1)


def _direct(x, m, h):
    n = len(m)
    c = max(1, min(n, (1 << 26) // n))
    return torch.cat([_direct_rows(x, m, h, i, min(n, i + c)) for i in range(0, n, c)])


def _direct_vjp(x, m, h, abar):
    n = len(m)
    c = max(1, min(n, (1 << 24) // n))
    gx, gm = torch.zeros_like(x), torch.zeros_like(m)
    for i in range(0, n, c):
        xg, mg = x.detach().requires_grad_(True), m.detach().requires_grad_(True)
        a = _direct_rows(xg, mg, h, i, min(n, i + c))
        u, v = torch.autograd.grad((a * abar[i:i + c]).sum(), (xg, mg))
        gx += u
        gm += v
    return gx, gm


def exact(case, seed):
    """The direct sum that the FMM approximates, in 64 bits: its distance from
    the outputs is the method's truncation error, the same for every correct
    implementation.  None where it takes too long."""
    n, op = case["n"], case["op"]
    if n > (1 << 18 if op in ("step", "census") else 1 << 15 if op == "kdk" else 1 << 14):
        return None
    s = prepare(case, seed)
    x, m, h = s["x"], s["m"], s["h"]
    if op in ("step", "census"):
        a = _direct(x, m, h)
        if op == "census":
            f = m[:, None] * a
            return {"a": a, "sumF": None, "sumAbsF": float(f.norm(dim=1).sum()), "F33": None,
                    "F46": None, "pairs": None}
        return {"a": a, "stats": None}
    if op == "grad":
        gx, gm = _direct_vjp(x, m, h, s["abar"].double())
        return {"a": _direct(x, m, h), "x_bar": gx, "m_bar": gm}
    x, v = x.clone(), s["v"].clone()
    ckpt, a = [x.clone()], _direct(x, m, h)
    for _ in range(STEPS):
        v += 0.5 * DT * a
        x += DT * v
        a = _direct(x, m, h)
        v += 0.5 * DT * a
        ckpt.append(x.clone())
    if op == "kdk":
        return {"x": x, "v": v}
    xbar, vbar, mbar = s["xbar"].clone(), s["vbar"].clone(), torch.zeros_like(m)
    for k in range(STEPS, -1, -1):
        if k < STEPS:
            vbar = vbar + DT * xbar
        c = DT if 0 < k < STEPS else 0.5 * DT
        gx, gm = _direct_vjp(ckpt[k], m, h, c * vbar)
        xbar = xbar + gx
        mbar = mbar + gm
    return {"x": x, "v": v, "x_bar": xbar, "v_bar": vbar, "m_bar": mbar}
