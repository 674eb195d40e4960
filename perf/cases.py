"""The work that a user of this framework has it do, as cases to be timed.

Every case goes through the public binding (``paper_1407_2052_amd.amrvac``):
time steps, right-hand sides, the div B monitor and the adjoint of the time
integration, on block lists from one 512-cell block (launch latency) to the
25-million-cell uneven list and the 256^3 periodic box, in 1D, 2D and 3D, for
hydro, ideal MHD, GLM-MHD and Hall MHD, with MP5 and LIM03 and all three
Runge-Kutta schemes.  Everything is FP64, the only type the framework has.

Fields are seeded smooth perturbations of a uniform state, as in the
framework's own inputs: rho and p carry scalar modes, v and B solenoidal ones.
``exact`` evaluates the same scheme in plain torch, on whole arrays.
"""
import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_1407_2052_amd import amrvac

NG = 3
GAMMA = {"hd": 1.4, "mhd": 5.0 / 3.0, "glm": 5.0 / 3.0, "hall": 5.0 / 3.0}
SCHEMES = {"rk3": amrvac.RK3, "ssprk43": amrvac.SSPRK43, "ssprk54": amrvac.SSPRK54}
STAGES = {"rk3": 3, "ssprk43": 4, "ssprk54": 5}
CFL = 0.4
ETA_H = 0.01
GLM_CR = 0.18


def _case(op, ndim, physics, recon, scheme, blocks, size, steps=1, ragged=0, uneven=0, ckpt=0, tune=False):
    blocks = tuple(blocks) + (1,) * (3 - len(blocks))
    size = tuple(size) + (1,) * (3 - len(size))
    return {"op": op, "ndim": ndim, "physics": physics, "recon": recon, "scheme": scheme,
            "bx": blocks[0], "by": blocks[1], "bz": blocks[2], "nx": size[0], "ny": size[1], "nz": size[2],
            "steps": steps, "ragged": ragged, "uneven": uneven, "ckpt": ckpt, "tune": tune}


def listed():
    return [
        # the smallest call: one RK3 step of the 512-cell 1D Euler problem, as
        # a program that couples every step to something else makes it
        dict(_case("step", 1, "hd", "mp5", "rk3", [1], [512]), name="euler1d_512_step"),
        # a 1D MHD tube run to an output time in one call
        dict(_case("run", 1, "mhd", "mp5", "ssprk54", [8], [64], steps=40), name="mhd1d_512_run"),
        # 2D Euler 256^2 in 256 blocks of 16^2, run to an output time
        dict(_case("run", 2, "hd", "mp5", "ssprk54", [16, 16], [16, 16], steps=20), name="euler2d_256_run"),
        # 2D MHD 512^2 in 1024 blocks of 16^2, shape chosen by the autotuner
        dict(_case("step", 2, "mhd", "mp5", "ssprk54", [32, 32], [16, 16], steps=4, tune=True), name="mhd2d_512_steps"),
        # the benchmark's list: 4096 uneven blocks with caller-filled faces
        dict(_case("step", 3, "mhd", "mp5", "ssprk54", [1], [1], uneven=4096), name="mhd3d_uneven4096_step"),
        # the uniform 256^3 box in 4096 blocks of 16^3
        dict(_case("step", 3, "mhd", "mp5", "ssprk54", [16, 16, 16], [16, 16, 16]), name="mhd3d_256_step"),
        # the paper's other combination, RK3 + LIM03, on a quarter of the list
        dict(_case("step", 3, "mhd", "lim03", "rk3", [1], [1], steps=2, uneven=1024), name="lim03_uneven1024_steps"),
        # GLM-MHD with the div B monitor read after the step
        dict(_case("monitor", 3, "glm", "mp5", "ssprk54", [8, 8, 8], [16, 16, 16]), name="glm3d_128_monitor"),
        # Hall MHD: the current pre-pass before every stage
        dict(_case("step", 3, "hall", "mp5", "ssprk54", [6, 6, 6], [16, 16, 16]), name="hall3d_96_step"),
        # a right-hand side alone, for a caller's own integrator: 3D hydro on
        # blocks of many odd sizes
        dict(_case("rhs", 3, "hd", "mp5", "rk3", [5, 6, 4], [13, 11, 17], ragged=4), name="rhs3d_ragged"),
        # gradient of a 2D Euler run with respect to its initial state
        dict(_case("adjoint", 2, "hd", "mp5", "ssprk54", [16, 16], [16, 16], steps=40, ckpt=20), name="adjoint2d_256"),
        # gradient of a 3D MHD run
        dict(_case("adjoint", 3, "mhd", "mp5", "ssprk54", [8, 8, 8], [16, 16, 16], steps=4, ckpt=2), name="adjoint3d_128"),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["1d", "2d", "2d", "3d", "3d", "uneven", "glm", "hall", "rhs", "adj2", "adj3"])
    rec, sch = rng.choice([("mp5", "ssprk54"), ("mp5", "ssprk54"), ("mp5", "ssprk43"), ("mp5", "rk3"), ("lim03", "rk3"),
                           ("lim03", "ssprk43")])
    ragged = rng.choice([0, 0, 3])
    if kind == "1d":
        n = logint(16, 512)
        nb = logint(1, max(1, 2048 // n))
        return _case(rng.choice(["step", "run"]), 1, rng.choice(["hd", "mhd"]), rec, sch, [nb], [n], steps=logint(1, 40),
                     ragged=ragged if n > 8 else 0)
    if kind == "2d":
        n, m = logint(8, 40), logint(8, 40)
        return _case(rng.choice(["step", "run"]), 2, rng.choice(["hd", "mhd", "mhd"]), rec, sch,
                     [max(1, logint(32, 640) // n), max(1, logint(32, 640) // m)], [n, m], steps=logint(1, 20), ragged=ragged)
    n = [logint(8, 33) for _ in range(3)]
    nb = [max(1, logint(24, 128) // k) for k in n]
    if kind == "3d":
        return _case("step", 3, rng.choice(["hd", "mhd", "mhd"]), rec, sch, nb, n, steps=rng.choice([1, 1, 2]), ragged=ragged)
    if kind == "uneven":
        return _case("step", 3, "mhd", rec, sch, [1], [1], uneven=logint(14, 1400))
    if kind == "glm":
        return _case("monitor", 3, "glm", rec, sch, nb, n, ragged=ragged)
    if kind == "hall":
        return _case("step", 3, "hall", rec, sch, nb, n, ragged=ragged)
    if kind == "rhs":
        d = rng.choice([2, 3])
        return _case("rhs", d, rng.choice(["hd", "mhd"]), rec, sch, nb[:d], n[:d], ragged=rng.choice([0, 4]))
    if kind == "adj2":
        a, b = logint(8, 33), logint(8, 33)
        k = logint(4, 30)
        return _case("adjoint", 2, rng.choice(["hd", "mhd"]), "mp5", sch, [max(1, logint(32, 300) // a), max(1, logint(32, 300) // b)],
                     [a, b], steps=k, ckpt=rng.choice([max(1, k // 2), k]))
    nb = [max(1, logint(24, 96) // k) for k in n]
    return _case("adjoint", 3, rng.choice(["hd", "mhd"]), "mp5", sch, nb, n, steps=2, ckpt=rng.choice([1, 2]))


# ---------------------------------------------------------------------------
# Geometry: block extents and where each block sits.
# ---------------------------------------------------------------------------
def _nvar(case):
    return {"hd": 2 + case["ndim"], "mhd": 8, "glm": 9, "hall": 8}[case["physics"]]


def _widths(case):
    """Block widths along each direction; a ragged list varies them by up to +-ragged/2."""
    out = []
    for d, (b, n) in enumerate((("bx", "nx"), ("by", "ny"), ("bz", "nz"))):
        r = case["ragged"] if d < case["ndim"] else 0
        out.append([case[n] + ((3 * i + d) % (r + 1) - r // 2 if r else 0) for i in range(case[b])])
    return out


def _uneven_sizes(nb):
    """32^3 : 16^3 : 8^3 in the ratio 1 : 2 : 4 by count, largest first."""
    a = nb // 7
    return [32] * a + [16] * (2 * a) + [8] * (nb - 3 * a)


def _cells(case):
    if case["uneven"]:
        return sum(s ** 3 for s in _uneven_sizes(case["uneven"]))
    w = _widths(case)
    return sum(w[0]) * sum(w[1]) * sum(w[2])


def work(case):
    """Bytes: the state in and out once (twice the work arrays for the other
    operations).  Operations, arithmetic and selections: 30 per MP5 and 15 per
    LIM03 reconstruction, two reconstructions per interface and variable, the
    primitives, one flux and split per direction, the stage combination; the
    reverse of a stage counts as two forward ones."""
    nv, nd, cells = _nvar(case), case["ndim"], _cells(case)
    stage = nd * (2 * nv * (30 if case["recon"] == "mp5" else 15) + 30 + 4 * nv) + 30 + 6 * nv
    evals = 1 if case["op"] == "rhs" else STAGES[case["scheme"]] * case["steps"]
    state = 8.0 * nv * cells
    if case["op"] == "adjoint":
        return {"bytes": 3 * state, "flops": 3.0 * evals * stage * cells}
    return {"bytes": 2 * state + (8.0 * cells if case["op"] == "monitor" else 0.0), "flops": 1.0 * evals * stage * cells}


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
class _Modes:
    """Seeded primitive fields on the periodic unit box: 8 modes with |k_d| <= 4."""

    def __init__(self, case, seed):
        rng = np.random.default_rng(seed)
        nd, self.mhd, self.glm = case["ndim"], case["physics"] != "hd", case["physics"] == "glm"
        self.gamma, self.nd, nm = GAMMA[case["physics"]], nd, 8
        ks = []
        while len(ks) < nm:
            k = rng.integers(-4, 5, size=nd)
            if np.any(k):
                ks.append(np.concatenate([k, np.zeros(3 - nd, np.int64)]))
        self.k, self.ph = np.array(ks, np.float64), rng.uniform(0.0, 2.0 * math.pi, nm)
        a = rng.uniform(0.5, 1.0, (9, nm))
        a = a / a.sum(axis=1, keepdims=True) * rng.choice([-1.0, 1.0], (9, nm))
        amp = np.zeros((9, nm))   # rho v p B psi
        amp[0], amp[4], amp[8] = 0.1 * a[0], 0.1 * a[4], 0.02 * a[8]
        for rows in ((1, 2, 3), (5, 6, 7)):
            e = rng.normal(size=(nm, 3))
            if nd > 1:   # perpendicular to k; in 1D the perturbation keeps B_x uniform
                e -= self.k * ((e * self.k).sum(1) / (self.k ** 2).sum(1))[:, None]
            elif rows[0] == 5:
                e[:, 0] = 0.0
            e /= np.linalg.norm(e, axis=1, keepdims=True)
            for q, r in enumerate(rows):
                amp[r] = 0.1 * a[rows[0]] * e[:, q]
        self.amp = amp
        self.base = [1.0, 0.3, -0.2, 0.1, 1.0, 0.9, 0.4, -0.3, 0.0]

    def conserved(self, x, y, z):
        """Conserved variables (first axis) at broadcastable coordinates."""
        w = [None] * 9
        for m in range(len(self.ph)):
            s = torch.sin(2 * math.pi * (self.k[m, 0] * x + self.k[m, 1] * y + self.k[m, 2] * z) + self.ph[m])
            for q in range(9):
                if self.amp[q, m] != 0.0 and (q < 5 or self.mhd):
                    w[q] = (self.base[q] if w[q] is None else w[q]) + float(self.amp[q, m]) * s
        w = [torch.full_like(w[0], self.base[q]) if w[q] is None else w[q] for q in range(9)]
        rho, nc = w[0], 3 if self.mhd else self.nd
        u = [rho] + [rho * w[1 + q] for q in range(nc)]
        e = w[4] / (self.gamma - 1.0) + 0.5 * rho * sum(w[1 + q] * w[1 + q] for q in range(nc))
        if self.mhd:
            e = e + 0.5 * (w[5] * w[5] + w[6] * w[6] + w[7] * w[7])
        u.append(e)
        if self.mhd:
            u += [w[5], w[6], w[7]]
        if self.glm:
            u.append(w[8])
        return torch.stack(u)


def _padded(n, nd):
    return [n[d] + 2 * NG if d < nd else 1 for d in range(3)]


def _layout(case, seed):
    """The block list: n, dx, xlo, nbr per block, the flat state on the device
    and, per block, its offset and padded extents."""
    dev, nd = ("cuda" if torch.cuda.is_available() else "cpu"), case["ndim"]
    f, nv = _Modes(case, seed), _nvar(case)
    if case["uneven"]:
        N, sizes = 256, _uneven_sizes(case["uneven"])
        org = np.random.default_rng([seed, 1]).integers(0, N, (len(sizes), 3))
        n = np.array([[s] * 3 for s in sizes], np.int64)
        dx, xlo, nbr = np.full((len(sizes), 3), 1.0 / N), org / N, np.full((len(sizes), 6), -1, np.int64)
        parts = []
        for s in (32, 16, 8):
            o = torch.as_tensor(org[n[:, 0] == s], dtype=torch.float64, device=dev)
            i = (torch.arange(-NG, s + NG, dtype=torch.float64, device=dev) + 0.5)
            for q in range(0, len(o), 256):
                c = (o[q:q + 256, :, None] + i[None, None, :]) / N
                u = f.conserved(c[:, 0, None, None, :], c[:, 1, None, :, None], c[:, 2, :, None, None])
                parts.append(u.transpose(0, 1).reshape(-1))
        flat = torch.cat(parts)
    else:
        w = _widths(case)
        N = [sum(x) for x in w]
        starts = [np.concatenate([[0], np.cumsum(x)]) for x in w]
        x = [(torch.arange(N[d], dtype=torch.float64, device=dev) + 0.5) / N[d] if d < nd
             else torch.zeros(1, dtype=torch.float64, device=dev) for d in range(3)]
        u = f.conserved(x[0][None, None, :], x[1][None, :, None], x[2][:, None, None])
        h = 1.0 / max(N[:nd])   # cubic cells: the box is the unit box along its longest side
        n, xlo, nbr, parts = [], [], [], []
        nb = [len(a) for a in w]
        idx = [[(torch.arange(starts[d][q] - NG, starts[d][q] + w[d][q] + NG, device=dev) % N[d]) if d < nd
                else torch.zeros(1, dtype=torch.int64, device=dev) for q in range(nb[d])] for d in range(3)]
        for bz in range(nb[2]):
            uz = u.index_select(1, idx[2][bz])
            for by in range(nb[1]):
                uy = uz.index_select(2, idx[1][by])
                for bx in range(nb[0]):
                    b = (bx, by, bz)
                    parts.append(uy.index_select(3, idx[0][bx]).reshape(-1))
                    n.append([w[d][b[d]] for d in range(3)])
                    xlo.append([starts[d][b[d]] * h if d < nd else 0.0 for d in range(3)])
                    row = [-1] * 6
                    for d in range(nd):
                        for side, step in ((0, -1), (1, 1)):
                            c = list(b)
                            c[d] = (c[d] + step) % nb[d]
                            row[2 * d + side] = (c[2] * nb[1] + c[1]) * nb[0] + c[0]
                    nbr.append(row)
        flat = torch.cat(parts)
        n, xlo, nbr = np.array(n), np.array(xlo), np.array(nbr)
        dx = np.where(np.arange(3)[None, :] < nd, h, 1.0) * np.ones((len(n), 1))
    shapes = [[nv] + _padded(q, nd)[::-1] for q in n]
    offs = np.concatenate([[0], np.cumsum([int(np.prod(s)) for s in shapes])])
    return n, dx, xlo, nbr, flat, shapes, offs


def _views(flat, shapes, offs):
    return [flat[int(offs[b]):int(offs[b + 1])].view(*s) for b, s in enumerate(shapes)]


def _cotangent(case, seed, flat):
    g = torch.Generator(device=flat.device).manual_seed(int(seed) + 77)
    return torch.randn(flat.shape, generator=g, dtype=torch.float64, device=flat.device)


def _dt(case):
    """Fixed step of the adjoint: CFL 0.4 at a signal speed of 2.5 per direction."""
    return CFL / (2.5 * case["ndim"] * max(sum(w) for w in _widths(case)[:case["ndim"]]))


def prepare(case, seed):
    n, dx, xlo, nbr, flat, shapes, offs = _layout(case, seed)
    ph = case["physics"]
    ctx = amrvac.Context(case["ndim"], {"hd": False, "mhd": True, "hall": True, "glm": 2}[ph], GAMMA[ph],
                         amrvac.EXEC_BATCHED_SINGLE if case["uneven"] else amrvac.EXEC_BATCHED,
                         recon=amrvac.LIM03 if case["recon"] == "lim03" else amrvac.MP5,
                         eta_h=ETA_H if ph == "hall" else 0.0)
    ctx.set_blocks(_views(flat, shapes, offs), n, dx, xlo, nbr)
    s = {"case": case, "ctx": ctx, "flat": flat}
    if case["tune"]:
        ctx.autotune(SCHEMES[case["scheme"]], 2)
    if case["op"] == "rhs":
        sizes = [_nvar(case) * int(np.prod(q)) for q in n]
        s["out"] = torch.empty(sum(sizes), dtype=torch.float64, device=flat.device)
        o = np.concatenate([[0], np.cumsum(sizes)])
        s["outs"] = [s["out"][int(o[b]):int(o[b + 1])] for b in range(len(n))]
    if case["op"] == "adjoint":
        s["cot"] = _cotangent(case, seed, flat)
        s["lam"] = torch.empty_like(flat)
        s["lams"] = _views(s["lam"], shapes, offs)
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    scheme = SCHEMES[case["scheme"]]
    if case["op"] == "step":
        ctx.ssprk_step(scheme, case["steps"], cfl=CFL, t=None)
        return s["flat"]
    if case["op"] == "run":
        t = ctx.ssprk_step(scheme, case["steps"], cfl=CFL, t=0.0)
        return {"u": s["flat"], "t": t}
    if case["op"] == "monitor":
        ctx.ssprk_step(scheme, case["steps"], cfl=CFL, t=None)
        div, mean = ctx.divb()
        return {"u": s["flat"], "div": torch.cat([x.reshape(-1) for x in div]), "mean": mean}
    if case["op"] == "rhs":
        _, cmax = ctx.fd_rhs(s["outs"])
        return {"rhs": s["out"], "cmax": cmax}
    s["lam"].copy_(s["cot"])
    ctx.ssprk_adjoint(scheme, _dt(case), case["steps"], case["ckpt"], s["lams"])
    return s["lam"]


# ---------------------------------------------------------------------------
# The same scheme in plain torch on whole arrays, in 64 bits.
# ---------------------------------------------------------------------------
def _axis(d):
    return 4 - d   # arrays are (block, variable, z, y, x)


def _prim(u, nd, mhd, gamma):
    nc = 3 if mhd else nd
    rho = u[:, 0]
    v = [u[:, 1 + q] / rho for q in range(nc)]
    e = u[:, 1 + nc] - 0.5 * sum(u[:, 1 + q] * v[q] for q in range(nc))
    B = [u[:, 5 + q] for q in range(3)] if mhd else None
    b2 = B[0] * B[0] + B[1] * B[1] + B[2] * B[2] if mhd else None
    if mhd:
        e = e - 0.5 * b2
    return rho, v, (gamma - 1.0) * e, B, b2


def _speed(u, d, c):
    rho, v, p, B, b2 = _prim(u, c["nd"], c["mhd"], c["gamma"])
    a2 = c["gamma"] * p / rho
    if not c["mhd"]:
        return v[d].abs() + a2.sqrt()
    s = a2 + b2 / rho
    cf = (0.5 * (s + (s * s - 4.0 * a2 * B[d] * B[d] / rho).clamp(min=0.0).sqrt())).sqrt()
    if c["eta"]:
        cf = torch.maximum(cf, c["eta"] * b2.sqrt() / rho * (math.pi / c["dx"]))
    return v[d].abs() + cf


def _flux(u, d, c, ch, J):
    rho, v, p, B, b2 = _prim(u, c["nd"], c["mhd"], c["gamma"])
    if not c["mhd"]:
        F = [u[:, 1 + d]] + [u[:, 1 + q] * v[d] + (p if q == d else 0.0) for q in range(c["nd"])]
        return torch.stack(F + [v[d] * (u[:, 1 + c["nd"]] + p)], 1)
    pt, bv = p + 0.5 * b2, B[0] * v[0] + B[1] * v[1] + B[2] * v[2]
    F = [u[:, 1 + d]] + [u[:, 1 + q] * v[d] - B[d] * B[q] + (pt if q == d else 0.0) for q in range(3)]
    F.append(v[d] * (u[:, 4] + pt) - B[d] * bv)
    F += [torch.zeros_like(rho) if q == d else v[d] * B[q] - B[d] * v[q] for q in range(3)]
    if J is not None:
        h, jb = c["eta"] / rho, J[:, 0] * B[0] + J[:, 1] * B[1] + J[:, 2] * B[2]
        for q in range(3):
            F[5 + q] = F[5 + q] + h * (B[d] * J[:, q] - J[:, d] * B[q])
        F[4] = F[4] + h * (jb * B[d] - b2 * J[:, d])
    if c["glm"]:
        F[5 + d] = F[5 + d] + u[:, 8]
        F.append(ch * ch * B[d])
    return torch.stack(F, 1)


def _minmod4(w, x, y, z):
    same = (torch.sign(w) == torch.sign(x)) & (torch.sign(w) == torch.sign(y)) & (torch.sign(w) == torch.sign(z))
    m = torch.minimum(torch.minimum(w.abs(), x.abs()), torch.minimum(y.abs(), z.abs()))
    return torch.where(same, torch.sign(w).detach() * m, torch.zeros_like(m))


def _mp5(a, b, c, d, e):
    fl = (2.0 * a - 13.0 * b + 47.0 * c + 27.0 * d - 3.0 * e) / 60.0
    dm, d0, dp = a - 2.0 * b + c, b - 2.0 * c + d, c - 2.0 * d + e
    mp, mm = _minmod4(4.0 * d0 - dp, 4.0 * dp - d0, d0, dp), _minmod4(4.0 * d0 - dm, 4.0 * dm - d0, d0, dm)
    ul, md, lc = c + 4.0 * (c - b), 0.5 * (c + d) - 0.5 * mp, c + 0.5 * (c - b) + 4.0 / 3.0 * mm
    lo = torch.maximum(torch.minimum(torch.minimum(c, d), md), torch.minimum(torch.minimum(c, ul), lc))
    hi = torch.minimum(torch.maximum(torch.maximum(c, d), md), torch.maximum(torch.maximum(c, ul), lc))
    return torch.minimum(torch.maximum(fl, lo), hi)


def _lim03(b, c, d, h):
    dm, dp = c - b, d - c
    p3 = (2.0 * dp + dm) / 3.0
    s, zero = torch.sign(dp), torch.zeros_like(dp)
    lo = torch.minimum(s * p3, torch.maximum(-0.5 * s * dm, torch.minimum(torch.minimum(2.0 * s * dm, s * p3), 1.6 * s * dp)))
    return c + 0.5 * torch.where((dm * dm + dp * dp) / (h * h) <= 1.0, p3, s * torch.maximum(zero, lo))


def _difference(ue, Je, cm, ch, d, c):
    """-(Fhat_{i+1/2} - Fhat_{i-1/2}) / dx along d from the state extended by 3 cells along d."""
    ax, n = _axis(d), ue.shape[_axis(d)] - 2 * NG
    F = _flux(ue, d, c, ch, Je)
    fp, fm = 0.5 * (F + cm * ue), 0.5 * (F - cm * ue)
    P = [fp.narrow(ax, q, n + 1) for q in range(6)]
    M = [fm.narrow(ax, q, n + 1) for q in range(6)]
    if c["lim"]:
        g = _lim03(P[1], P[2], P[3], c["dx"]) + _lim03(M[4], M[3], M[2], c["dx"])
    else:
        g = _mp5(*P[:5]) + _mp5(M[5], M[4], M[3], M[2], M[1])
    return -(g.narrow(ax, 1, n) - g.narrow(ax, 0, n)) / c["dx"]


def _extend(u, ghost, d):
    ax = _axis(d)
    n = u.shape[ax]
    if ghost is None:   # periodic; a box narrower than the halo wraps more than once
        k = torch.arange(-NG, n + NG, device=u.device) % n
        return u.index_select(ax, k)
    return torch.cat([ghost[d][0], u, ghost[d][1]], ax)


def _current(u, c):
    B, J = [u[:, 5 + q] for q in range(3)], []

    def der(q, d):
        if d >= c["nd"]:
            return torch.zeros_like(B[q])
        r = lambda k: torch.roll(B[q], -k, 3 - d)  # noqa: E731
        return (-r(2) + 8.0 * r(1) - 8.0 * r(-1) + r(-2)) / (12.0 * c["dx"])
    for q in range(3):
        J.append(der((q + 2) % 3, (q + 1) % 3) - der((q + 1) % 3, (q + 2) % 3))
    return torch.stack(J, 1)


def _cmax(us, c):
    cm = [max_of([_speed(u, d, c).amax() for u in us]) for d in range(c["nd"])]
    return [max_of(cm)] * c["nd"] if c["glm"] else cm


def max_of(v):
    return v[0] if len(v) == 1 else torch.stack(list(v)).amax()


def _rhs(us, ghosts, c, cm=None):
    cm = _cmax(us, c) if cm is None else cm
    out = []
    for u, g in zip(us, ghosts):
        J = _current(u, c) if c["eta"] else None
        L = 0.0
        for d in range(c["nd"]):
            def part(u, cmd, d=d, g=g, J=J):
                return _difference(_extend(u, g, d), None if J is None else _extend(J, None, d), cmd, cmd, d, c)
            L = L + (checkpoint(part, u, cm[d], use_reentrant=False) if u.requires_grad else part(u, cm[d]))
        out.append(L)
    return out, cm


def _tables(scheme):
    if scheme == "rk3":
        return ({1: {0: 1.0}, 2: {0: 0.75, 1: 0.25}, 3: {0: 1 / 3, 2: 2 / 3}}, {1: {0: 1.0}, 2: {1: 0.25}, 3: {2: 2 / 3}})
    if scheme == "ssprk43":
        return ({1: {0: 1.0}, 2: {1: 1.0}, 3: {0: 2 / 3, 2: 1 / 3}, 4: {3: 1.0}}, {1: {0: 0.5}, 2: {1: 0.5}, 3: {2: 1 / 6}, 4: {3: 0.5}})
    a52, a53, a54 = 0.51723167208978, 0.12759831133288, 0.34833675773694
    return ({1: {0: 1.0}, 2: {0: 0.44437049406734, 1: 0.55562950593266}, 3: {0: 0.62010185138540, 2: 0.37989814861460},
             4: {0: 0.17807995410773, 3: 0.82192004589227}, 5: {0: 1.0 - (a52 + a53 + a54), 2: a52, 3: a53, 4: a54}},
            {1: {0: 0.39175222700392}, 2: {1: 0.36841059262959}, 3: {2: 0.25189177424738}, 4: {3: 0.54497475021237},
             5: {3: 0.08460416338212, 4: 0.22600748319395}})


def _step(us, ghosts, c, dt=None):
    al, be = _tables(c["scheme"])
    cm, ch = _cmax(us, c), None
    if dt is None:
        dt = CFL / sum(x / c["dx"] for x in cm)
    ch = cm[0]
    U, L = {0: us}, {}
    for i in range(1, len(al) + 1):
        L[i - 1], _ = _rhs(U[i - 1], ghosts, c, cm if i == 1 else None)
        U[i] = [sum(a * U[k][q] for k, a in al[i].items()) + dt * sum(b * L[k][q] for k, b in be[i].items())
                for q in range(len(us))]
    new = U[len(al)]
    if c["glm"]:
        decay = torch.exp(-dt * ch / GLM_CR)
        new = [torch.cat([u[:, :8], u[:, 8:] * decay], 1) for u in new]
    return new, dt


def exact(case, seed):
    n, dx, _, _, flat, shapes, offs = _layout(case, seed)
    nd, nv = case["ndim"], _nvar(case)
    c = {"nd": nd, "mhd": case["physics"] != "hd", "glm": case["physics"] == "glm", "gamma": GAMMA[case["physics"]],
         "eta": ETA_H if case["physics"] == "hall" else 0.0, "lim": case["recon"] == "lim03", "dx": float(dx[0, 0]),
         "scheme": case["scheme"]}
    inner = [slice(NG, -NG) if d < nd else slice(None) for d in (2, 1, 0)]
    if case["uneven"]:   # one array per block size, with its ghost layers
        us, ghosts = [], []
        for s in (32, 16, 8):
            b = np.flatnonzero(n[:, 0] == s)
            P = flat[int(offs[b[0]]):int(offs[b[-1] + 1])].view(len(b), nv, s + 6, s + 6, s + 6)
            us.append(P[(slice(None), slice(None), *inner)].clone())
            g = []
            for d in range(3):
                pick = list(inner)
                pick[2 - d] = slice(None)
                Q = P[(slice(None), slice(None), *pick)]
                g.append((Q.narrow(_axis(d), 0, NG).clone(), Q.narrow(_axis(d), s + NG, NG).clone()))
            ghosts.append(g)

        def put(us, into):
            for s, u in zip((32, 16, 8), us):
                b = np.flatnonzero(n[:, 0] == s)
                P = into[int(offs[b[0]]):int(offs[b[-1] + 1])].view(len(b), nv, s + 6, s + 6, s + 6)
                P[(slice(None), slice(None), *inner)] = u
            return into
    else:
        w = _widths(case)
        st = [np.concatenate([[0], np.cumsum(x)]) for x in w]
        nb = [len(x) for x in w]
        views = _views(flat, shapes, offs)

        def boxes():
            for b in range(len(n)):
                q = (b % nb[0], b // nb[0] % nb[1], b // (nb[0] * nb[1]))
                yield b, [slice(int(st[d][q[d]]), int(st[d][q[d] + 1])) for d in (2, 1, 0)]

        def gather(vs):
            u = torch.empty((1, nv, *[sum(x) for x in w[::-1]]), dtype=torch.float64, device=flat.device)
            for b, box in boxes():
                u[(0, slice(None), *box)] = vs[b][(slice(None), *inner)]
            return u

        def put(us, into):
            vs = _views(into, shapes, offs)
            for b, box in boxes():
                vs[b][(slice(None), *inner)] = us[0][(0, slice(None), *box)]
            return into

        def interiors(u):
            return torch.cat([u[(0, slice(None), *box)].reshape(-1) for _, box in boxes()])
        us, ghosts = [gather(views)], [None]
    if case["op"] == "rhs":
        L, cm = _rhs(us, ghosts, c)
        return {"rhs": interiors(L[0]), "cmax": np.array([float(x) for x in cm] + [0.0] * (3 - nd))}
    if case["op"] == "adjoint":
        if _cells(case) * case["steps"] * nv > 1.5e8:
            return None
        states, dt = [us[0]], _dt(case)
        for _ in range(case["steps"] - 1):
            states.append(_step([states[-1]], ghosts, c, dt)[0][0])
        lam = gather(_views(_cotangent(case, seed, flat), shapes, offs))
        for u in reversed(states):
            u = u.detach().requires_grad_(True)
            new, _ = _step([u], ghosts, c, dt)
            lam, = torch.autograd.grad(new[0], u, lam)
        return put([lam], torch.zeros_like(flat))
    t = 0.0
    for _ in range(case["steps"]):
        us, dt = _step(us, ghosts, c)
        t += float(dt)
    u = put(us, flat)
    if case["op"] == "step":
        return u
    if case["op"] == "run":
        return {"u": u, "t": t}
    div = 0.0
    for d in range(nd):
        r = lambda k: torch.roll(us[0][:, 5 + d], -k, 3 - d)  # noqa: E731
        div = div + (8.0 * (r(1) - r(-1)) - (r(2) - r(-2))) / (12.0 * c["dx"])
    div = div.unsqueeze(1)
    return {"u": u, "div": interiors(div), "mean": float(div.abs().mean())}
