"""Timing cases of the Newton multigrid solver: the calls a user's program makes, from one small
channel to the full-size wedge, each through the package's public entry points.

listed() names the fixed cases, draw(rng) gives further ones of the same ranges, prepare() makes
what a program holds before the call, run() is one pass, work() the bytes and operations no
implementation can do without, and exact() the same outputs in plain FP64 torch written from the
paper's formulas (no code of the package).
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

import swe_workloads as W

DEV = "cuda"

# Kinds of cases
#   step1d    residual, then Jacobian, of one channel (two calls a program makes per iteration)
#   vcycle1d  linear solve of one channel: operator set-up and the Newton step's two V-cycles
#   solve1d   whole Newton solve of one channel
#   batch1d   whole Newton solve of a batch of equal channels (the flagship workload)
#   uneven1d  whole Newton solve of a batch of channels of many sizes and widths
#   step2d    residual, then Jacobian, of one 2D problem
#   vcycle2d  linear solve of one 2D system: operator set-up and the Newton step's three V-cycles
#   newton2d  the first Newton steps of a 2D solve (every step does the same work)


def listed():
    return [
        # the smallest call: one smooth channel of 200 cells, launch latency only
        {"name": "step1d_200", "kind": "step1d", "n": 200, "levels": 3, "jac": 3},
        # one linear solve of a benchmark-sized channel, as a program with its own Newton loop does
        {"name": "vcycle1d_12800", "kind": "vcycle1d", "n": 12800, "levels": 8, "jac": 3, "prec": 0},
        # one channel solved alone (interactive use; latency of a chain of small launches)
        {"name": "solve1d_12800", "kind": "solve1d", "n": 12800, "levels": 8, "jac": 3, "prec": 0},
        # the flagship benchmark: 256 hump channels of 12800 cells in one batch, FP64
        {"name": "batch1d_256x12800", "kind": "batch1d", "count": 256, "n": 12800, "levels": 8, "jac": 3, "prec": 0},
        # a served mix of channels, 256 to 16384 cells, FP32 multigrid
        {"name": "uneven1d_512_fp32", "kind": "uneven1d", "count": 512, "prec": 1},
        # smallest 2D grid that is served
        {"name": "step2d_64x32", "kind": "step2d", "cx": 8, "cy": 4, "k": 3, "jac": 9},
        # full-size 2D residual and Jacobian
        {"name": "step2d_1024x512", "kind": "step2d", "cx": 8, "cy": 4, "k": 7, "jac": 9},
        # linear solve on a ragged middle grid with FP32 multigrid (served requests use it)
        {"name": "vcycle2d_160x96_fp32", "kind": "vcycle2d", "cx": 5, "cy": 3, "k": 5, "jac": 9, "prec": 1},
        # linear solve at full size in FP64
        {"name": "vcycle2d_1024x512", "kind": "vcycle2d", "cx": 8, "cy": 4, "k": 7, "jac": 9, "prec": 0},
        # Newton steps on the smallest served 2D grid, FP32 multigrid
        {"name": "newton2d_64x32_fp32", "kind": "newton2d", "cx": 8, "cy": 4, "k": 3, "jac": 9, "prec": 1, "steps": 4},
        # Newton steps with the full 21-cell stencil (the paper's comparison solver), FP64
        {"name": "newton2d_j21_128x64", "kind": "newton2d", "cx": 8, "cy": 4, "k": 4, "jac": 21, "prec": 0, "steps": 2},
        # Newton steps on the largest served 2D grid, FP32 multigrid
        {"name": "newton2d_512x256_fp32", "kind": "newton2d", "cx": 8, "cy": 4, "k": 6, "jac": 9, "prec": 1, "steps": 2},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step1d", "vcycle1d", "solve1d", "batch1d", "uneven1d", "step2d", "vcycle2d", "newton2d"])
    if kind in ("step1d", "vcycle1d", "solve1d", "batch1d"):
        # n = m 2^(levels-1) with a coarsest grid of 25 to 120 cells, odd ones among them
        target = _log_int(rng, 200, 16384 if kind != "batch1d" else 12800)
        m = rng.randint(25, 120)
        k = max(0, min(9, int(round(math.log2(target / m)))))
        if kind in ("solve1d", "batch1d"):
            k = max(k, 1)
        n = m << k
        case = {"kind": kind, "n": n, "levels": k + 1, "jac": 5 if k > 0 and rng.random() < 0.25 else 3}
        if kind != "step1d":
            case["prec"] = int(rng.random() < 0.4)
        if kind == "batch1d":
            case["count"] = min(_log_int(rng, 2, 256), max(2, 256 * 12800 // n))
        return case
    if kind == "uneven1d":
        return {"kind": kind, "count": _log_int(rng, 4, 512), "prec": int(rng.random() < 0.6)}
    # 2D grids: cx 2^k x cy 2^k with at most 40 coarsest cells, up to 1024 x 512
    cx, cy = rng.randint(4, 8), rng.randint(3, 4)
    case = {"kind": kind, "cx": cx, "cy": cy, "k": rng.randint(1, 7), "jac": 9}
    if kind == "newton2d":
        case["k"] = rng.randint(2, 6)
        case["steps"] = rng.randint(1, 2)
    if case["k"] <= 5 and rng.random() < 0.25:
        case["jac"] = 21
    if kind != "step2d":
        case["prec"] = int(rng.random() < 0.5)
    return case


# ---- inputs --------------------------------------------------------------------------------

def _problem1d(case, seed, i=0):
    """Channel i of a case: up to 2048 cells a served channel (smooth bump, varying width), above
    it the seeded hump of the benchmark."""
    n, s = case["n"], 1000 * seed + i
    if n <= 2048:
        p = W.config4_instance(s)
        return dataclasses.replace(p, n=n, levels=case["levels"],
                                   params=dataclasses.replace(p.params, eps=W.eps_for_n(n)))
    return W.config2(s, n=n, levels=case["levels"])


def _uneven(case, seed):
    """The uneven batch: the seeded sizes of the benchmark's batch, channels drawn from the seed."""
    out = []
    for i in range(case["count"]):
        size, p = W.config4_instance(i), W.config4_instance(1000 * seed + i)
        out.append(dataclasses.replace(p, n=size.n, levels=size.levels, params=size.params))
    return out


def _problem2d(case, seed):
    nx, ny = case["cx"] << case["k"], case["cy"] << case["k"]
    return W.wedge_problem(nx, ny, levels=case["k"] + 1, seed=seed)


def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(7919 * seed + salt)
    return g


def _perturbed(U, seed):
    """A state away from the initial guess: every component within 1% of it, seeded."""
    U = torch.tensor(np.ascontiguousarray(U), dtype=torch.float64, device=DEV)
    r = torch.rand(U.shape, dtype=torch.float64, device=DEV, generator=_gen(seed, 1))
    return U * (1.0 + 0.02 * (r - 0.5))


OFF9 = [(0, 0), (-2, 0), (-1, 0), (1, 0), (2, 0), (0, -2), (0, -1), (0, 1), (0, 2)]
OFF21 = (OFF9 + [(di, dj) for dj in (-1, 1) for di in (-2, -1, 1, 2)]
         + [(di, dj) for di in (-1, 1) for dj in (-2, 2)])
OFF5 = [(0, 0), (-1, 0), (1, 0), (0, -1), (0, 1)]


def _operator1d(case, seed):
    """Block operator and right-hand side with the shape of the 1D Jacobian, dominant diagonal."""
    n, nb = case["n"], case["jac"]
    g = _gen(seed, 2)
    J = 0.2 * (torch.rand((nb, 2, 2, n), dtype=torch.float64, device=DEV, generator=g) - 0.5)
    h = nb // 2
    J[h, 0, 0] += 3.0
    J[h, 1, 1] += 3.0
    for b in range(nb):
        d = b - h
        if d < 0:
            J[b, :, :, :-d] = 0.0
        elif d > 0:
            J[b, :, :, n - d:] = 0.0
    rhs = 2.0 * torch.rand((2, n), dtype=torch.float64, device=DEV, generator=g) - 1.0
    return J, rhs


def _operator2d(case, seed):
    """Block operator and right-hand side with the shape of the 2D Jacobian, dominant diagonal."""
    nx, ny, nb = case["cx"] << case["k"], case["cy"] << case["k"], case["jac"]
    g = _gen(seed, 3)
    J = torch.rand((nb, 3, 3, ny, nx), dtype=torch.float64, device=DEV, generator=g)
    J -= 0.5
    J *= 0.2
    for c in range(3):
        J[0, c, c] += 3.0
    for b, (di, dj) in enumerate(OFF9 if nb == 9 else OFF21):
        if di < 0:
            J[b, :, :, :, :-di] = 0.0
        elif di > 0:
            J[b, :, :, :, nx - di:] = 0.0
        if dj < 0:
            J[b, :, :, :-dj] = 0.0
        elif dj > 0:
            J[b, :, :, ny - dj:] = 0.0
    rhs = 2.0 * torch.rand((3, ny, nx), dtype=torch.float64, device=DEV, generator=g) - 1.0
    return J, rhs


# ---- the calls -----------------------------------------------------------------------------

def prepare(case, seed):
    import paper_2505_10857_amd as P
    kind = case["kind"]
    if kind == "step1d":
        s = P.Solver1D(_problem1d(case, seed), device=DEV, jac=case["jac"])
        return {"kind": kind, "s": s, "U": _perturbed(s.dev.prob.initial_guess(), seed)}
    if kind == "step2d":
        s = P.Solver2D(_problem2d(case, seed), device=DEV, jac=case["jac"])
        return {"kind": kind, "s": s, "U": _perturbed(s.dev.prob.initial_guess(), seed)}
    if kind in ("vcycle1d", "vcycle2d"):
        if kind == "vcycle1d":
            s = P.Solver1D(_problem1d(case, seed), device=DEV, jac=case["jac"], precision=case["prec"])
            J, rhs = _operator1d(case, seed)
        else:
            s = P.Solver2D(_problem2d(case, seed), device=DEV, jac=case["jac"], precision=case["prec"])
            J, rhs = _operator2d(case, seed)
        if case["prec"]:
            rhs = rhs.float()
        s.workspace()
        return {"kind": kind, "s": s, "J": J, "rhs": rhs, "dU": torch.zeros_like(rhs), "cycles": s.p.nu3}
    if kind == "solve1d":
        s = P.Solver1D(_problem1d(case, seed), device=DEV, jac=case["jac"], precision=case["prec"])
        s.workspace()
        U0 = s.state()
        return {"kind": kind, "s": s, "U0": U0, "U": torch.empty_like(U0)}
    if kind == "newton2d":
        s = P.Solver2D(_problem2d(case, seed), device=DEV, jac=case["jac"], precision=case["prec"],
                       n_max=case["steps"])
        s.workspace()
        U0 = s.state()
        return {"kind": kind, "s": s, "U0": U0, "U": torch.empty_like(U0)}
    if kind == "batch1d":
        probs = [_problem1d(case, seed, i) for i in range(case["count"])]
    else:
        probs = _uneven(case, seed)
    b = P.BatchSolver1D(probs, device=DEV, jac=case.get("jac", 3), precision=case["prec"])
    U0 = torch.cat([u.reshape(-1) for u in b.states()])
    U = torch.empty_like(U0)
    views, o = [], 0
    for p in probs:
        views.append(U[o:o + 2 * p.n].view(2, p.n))
        o += 2 * p.n
    return {"kind": kind, "s": b, "U0": U0, "U": U, "views": views}


def run(state):
    kind, s = state["kind"], state["s"]
    if kind in ("step1d", "step2d"):
        R, rn, res = s.residual(state["U"])
        return [R, rn, res, s.jacobian(state["U"], R, rn)]
    if kind in ("vcycle1d", "vcycle2d"):
        dU = state["dU"].zero_()
        for c in range(state["cycles"]):
            s.vcycle(state["J"] if c == 0 else None, state["rhs"], dU, setup=(c == 0))
        return [dU]
    state["U"].copy_(state["U0"])
    if kind in ("solve1d", "newton2d"):
        st, _ = s.newton_solve(state["U"])
        return [state["U"], st.iters, st.status, st.res]
    rep = s.solve(state["views"])
    return [state["U"], np.array([r[0] for r in rep]), np.array([r[1] for r in rep]), np.array([r[2] for r in rep])]


def work(case):
    """Inputs read once, outputs written once; operations of the formulas (an FP64 reconstruction
    about 20, a flux about 45; a block product 2 b^2) over about 25 Newton steps for a solve."""
    kind, nb = case["kind"], case.get("jac", 3)
    if kind.endswith("1d"):
        cells = case["n"] * case.get("count", 1) if "n" in case else 3950 * case["count"]
        rj = 350 + 2 * nb * 100                                   # residual and Jacobian, per cell
        cycle = 2 * (8 * nb * 4 * 4 + 8 * nb + 40)                # one V-cycle, all levels
        if kind == "step1d":
            return {"bytes": cells * (16 + 56 + 16 + 8 + 32 * nb), "flops": cells * rj}
        if kind == "vcycle1d":
            return {"bytes": cells * (32 * nb + (32 if case["prec"] == 0 else 16)), "flops": 2 * cells * cycle}
        return {"bytes": cells * (16 + 56 + 16), "flops": 25 * cells * (rj + 2 * cycle)}
    nx, ny = case["cx"] << case["k"], case["cy"] << case["k"]
    cells = nx * ny
    nu = 10 if nx <= 16 else (15 if nx <= 32 else 20)
    rj = 4000 + 3 * nb * 1200
    cycle = 2 * nu * 4 * 18 * (nb + 5 // 3) + 2 * 18 * nb
    if kind == "step2d":
        return {"bytes": cells * (24 + 64 + 24 + 8 + 72 * nb), "flops": cells * rj}
    if kind == "vcycle2d":
        return {"bytes": cells * (72 * nb + (48 if case["prec"] == 0 else 24)), "flops": 3 * cells * cycle}
    return {"bytes": cells * (24 + 64 + 24), "flops": case["steps"] * cells * (rj + 3 * cycle)}


# ---- the same outputs in plain FP64 torch --------------------------------------------------

ZETA = 1e-6


def _weno(um, u0, up, plus):
    """Third-order WENO value at the face on the cell's left (plus) or right (minus), eq. 7-8."""
    b0, b1 = (up - u0) ** 2, (u0 - um) ** 2
    if plus:
        c0, c1, d0, d1 = 1.5 * u0 - 0.5 * up, 0.5 * um + 0.5 * u0, 1.0 / 3.0, 2.0 / 3.0
    else:
        c0, c1, d0, d1 = 0.5 * u0 + 0.5 * up, -0.5 * um + 1.5 * u0, 2.0 / 3.0, 1.0 / 3.0
    a0, a1 = d0 / (ZETA + b0) ** 2, d1 / (ZETA + b1) ** 2
    return (a0 * c0 + a1 * c1) / (a0 + a1)


def _cubic_weights():
    t = (-1.5, -0.5, 0.5, 1.5)
    out = []
    for x in (-0.5 / math.sqrt(3.0), 0.5 / math.sqrt(3.0)):
        out.append([math.prod((x - t[m]) / (t[k] - t[m]) for m in range(4) if m != k) for k in range(4)])
    return out


CW = _cubic_weights()


class _Channel:
    """A batch of equal-sized channels with discharge imposed upstream and depth downstream."""

    def __init__(self, probs):
        self.p, self.n, self.dx, self.g = probs[0].params, probs[0].n, probs[0].dx, probs[0].g
        self.levels = probs[0].levels

        def geo(f):
            return torch.tensor(np.stack([f(p) for p in probs]), dtype=torch.float64, device=DEV)

        def gauss(p, q):
            return p.x0 + (np.arange(p.n) + 0.5) * p.dx + (q - 0.5) * p.dx / math.sqrt(3.0)

        self.sf = geo(lambda p: p.width(p.x0 + np.arange(p.n + 1) * p.dx)[0])
        self.sg = [geo(lambda p, q=q: p.width(gauss(p, q))[0]) for q in (0, 1)]
        self.sx = [geo(lambda p, q=q: p.width(gauss(p, q))[1]) for q in (0, 1)]
        self.bx = [geo(lambda p, q=q: p.bottom(gauss(p, q))[1]) for q in (0, 1)]
        self.q = geo(lambda p: np.array([p.bc_left.q]))
        self.h = geo(lambda p: np.array([p.bc_right.h]))
        self.omega = geo(lambda p: np.array([p.params.omega]))

    def residual(self, U):
        H, Q = U[:, 0], U[:, 1]
        sR = self.sf[:, -1:]
        Hn, Qn = H[:, -1:], Q[:, -1:]
        HR = torch.where((Qn / Hn) ** 2 < self.g * Hn / sR, sR * self.h, Hn)
        H = torch.cat([H[:, :1], H[:, :1], H, HR, HR], 1)
        Q = torch.cat([self.q, self.q, Q, Qn, Qn], 1)
        um, u0, up = slice(0, -2), slice(1, -1), slice(2, None)     # cells -1 .. N
        Hp, Hm = _weno(H[:, um], H[:, u0], H[:, up], True), _weno(H[:, um], H[:, u0], H[:, up], False)
        Qp, Qm = _weno(Q[:, um], Q[:, u0], Q[:, up], True), _weno(Q[:, um], Q[:, u0], Q[:, up], False)
        HL, QL, HR, QR = Hm[:, :-1], Qm[:, :-1], Hp[:, 1:], Qp[:, 1:]   # faces 0 .. N
        g, s = self.g, self.sf
        hL, hR, uL, uR = HL / s, HR / s, QL / HL, QR / HR
        cL, cR = torch.sqrt(g * hL), torch.sqrt(g * hR)
        SL, SR = torch.minimum(uL - cL, uR - cR), torch.maximum(uL + cL, uR + cR)
        F = []
        for fL, fR, vL, vR in ((QL, QR, HL, HR),
                               (QL * uL + 0.5 * g * s * hL * hL, QR * uR + 0.5 * g * s * hR * hR, QL, QR)):
            mid = (SR * fL - SL * fR + SL * SR * (vR - vL)) / (SR - SL)
            F.append(torch.where(SL >= 0, fL, torch.where(SR <= 0, fR, mid)))
        S = 0.0
        for q in (0, 1):
            Hg = (CW[q][0] * Hp[:, :-2] + CW[q][1] * Hp[:, 1:-1] + CW[q][2] * Hm[:, 1:-1] + CW[q][3] * Hm[:, 2:])
            hg = Hg / self.sg[q]
            S = S + 0.5 * g * hg * hg * self.sx[q] - g * self.sg[q] * hg * self.bx[q]
        return torch.stack([F[0][:, 1:] - F[0][:, :-1], F[1][:, 1:] - F[1][:, :-1] - 0.5 * self.dx * S], 1)

    def jacobian(self, U, R, nb):
        """[B, nb, 2, 2, n]: every fifth cell perturbed at once (a row sees five cells)."""
        B, n, h = U.shape[0], self.n, nb // 2
        J = torch.zeros((B, nb, 2, 2, n), dtype=torch.float64, device=DEV)
        for m in range(2):
            for a in range(5):
                V = U.clone()
                V[:, m, a::5] += self.p.eps
                D = (self.residual(V) - R) / self.p.eps
                for r in range(5):
                    d = (a - r + 2) % 5 - 2
                    if abs(d) <= h:
                        J[:, d + h, :, m, r::5] = D[:, :, r::5]
        for b in range(nb):
            d = b - h
            if d < 0:
                J[:, b, :, :, :-d] = 0.0
            elif d > 0:
                J[:, b, :, :, n - d:] = 0.0
        rn = R.abs().sum(1)
        for c in range(2):
            J[:, h, c, c] += self.p.alpha * rn
        return J


def _apply1(J, x, skip_diag):
    nb, n = J.shape[1], x.shape[2]
    h = nb // 2
    out = torch.zeros_like(x)
    for b in range(nb):
        d = b - h
        if d == 0 and skip_diag:
            continue
        lo, hi = max(0, -d), n - max(0, d)
        out[:, :, lo:hi] += (J[:, b, :, :, lo:hi] * x[:, None, :, lo + d:hi + d]).sum(2)
    return out


def _coarsen1(J):
    nb = J.shape[1]
    h = nb // 2
    C = torch.zeros(J.shape[:1] + (3, 2, 2, J.shape[-1] // 2), dtype=torch.float64, device=DEV)
    for f in (0, 1):
        for b in range(nb):
            d = (f + b - h) // 2
            if abs(d) <= 1:
                C[:, d + 1] += J[:, b, :, :, f::2]
    return C


class _Mg1:
    def __init__(self, J, levels, omega, nu1, nu2):
        self.J, self.omega, self.nu = [J], omega.reshape(-1, 1, 1), (nu1, nu2)
        for _ in range(levels - 1):
            self.J.append(_coarsen1(self.J[-1]))
        self.Di = [torch.linalg.inv(j[:, j.shape[1] // 2].permute(0, 3, 1, 2)).permute(0, 2, 3, 1) for j in self.J]
        j, n = self.J[-1], self.J[-1].shape[-1]
        A = torch.zeros((j.shape[0], n, 2, n, 2), dtype=torch.float64, device=DEV)
        i = torch.arange(n, device=DEV)
        for b in range(j.shape[1]):
            k = i + b - j.shape[1] // 2
            ok = (k >= 0) & (k < n)
            A[:, i[ok], :, k[ok], :] = j[:, b].permute(3, 0, 1, 2)[ok]
        self.lu = torch.linalg.lu_factor(A.reshape(j.shape[0], 2 * n, 2 * n))

    def smooth(self, l, rhs, x, nu):
        C = 3 if self.J[l].shape[1] == 5 else 2
        for _ in range(nu):
            for c in list(range(C)) + list(range(C - 1, -1, -1)):
                r = rhs + _apply1(self.J[l], x, True)
                t = (self.Di[l] * r[:, None]).sum(2)
                x[:, :, c::C] = ((1 - self.omega) * x - self.omega * t)[:, :, c::C]

    def cycle(self, rhs, x, l=0):
        if l == len(self.J) - 1:
            B, _, n = x.shape
            y = torch.linalg.lu_solve(*self.lu, -rhs.permute(0, 2, 1).reshape(B, 2 * n, 1))
            return y.reshape(B, n, 2).permute(0, 2, 1).contiguous()
        self.smooth(l, rhs, x, self.nu[0])
        r = rhs + _apply1(self.J[l], x, False)
        rc = r[:, :, 0::2] + r[:, :, 1::2]
        x = x + self.cycle(rc, torch.zeros_like(rc), l + 1).repeat_interleave(2, 2)
        self.smooth(l, rhs, x, self.nu[1])
        return x


def _solve1(probs, jac):
    ch = _Channel(probs)
    p, B = ch.p, len(probs)
    U = torch.tensor(np.stack([q.initial_guess() for q in probs]), dtype=torch.float64, device=DEV)
    R = ch.residual(U)
    res = R.abs().sum(1).mean(1)
    active = torch.ones(B, dtype=torch.bool, device=DEV)
    iters, step = torch.zeros(B, dtype=torch.int64, device=DEV), 0
    while step < p.n_max and bool(active.any()):
        mg = _Mg1(ch.jacobian(U, R, jac), ch.levels, ch.omega, p.nu1, p.nu2)
        x = torch.zeros_like(U)
        for _ in range(p.nu3):
            x = mg.cycle(R, x)
        U = torch.where(active[:, None, None], U + p.tau * x, U)
        R = ch.residual(U)
        res = torch.where(active, R.abs().sum(1).mean(1), res)
        iters += active
        active = active & ~(res < p.tol)
        step += 1
    return U, iters, torch.where(res < p.tol, 0, 1), res


class _Wedge:
    """The wedge problem: state inflow left and top, extrapolation right, split bottom side."""

    def __init__(self, p):
        self.prob, self.p, self.g = p, p.params, p.g
        self.nx, self.ny, self.dx, self.dy = p.nx, p.ny, p.dx, p.dy
        xc = p.x0 + (np.arange(p.nx) + 0.5) * p.dx
        yc = p.y0 + (np.arange(p.ny) + 0.5) * p.dy
        self.b = {}
        for be in (0, 1):
            for ga in (0, 1):
                X, Y = np.meshgrid(xc + (ga - 0.5) * p.dx / math.sqrt(3.0), yc + (be - 0.5) * p.dy / math.sqrt(3.0))
                _, bx, by = p.bottom(X, Y)
                self.b[be, ga] = [torch.tensor(v, device=DEV) for v in (bx, by)]
        i = p.bc[0]
        self.inflow = torch.tensor([i.h, i.h * i.u, i.h * i.v], dtype=torch.float64, device=DEV).reshape(3, 1, 1)
        self.wall = torch.tensor(xc >= p.wall_x, device=DEV)

    def ghosts(self, U):
        nx, ny = self.nx, self.ny
        flip = torch.tensor([1.0, 1.0, -1.0], dtype=torch.float64, device=DEV).reshape(3, 1, 1)
        low = torch.where(self.wall, flip * U[:, [1, 0]], U[:, [0, 0]])
        V = torch.cat([low, U, self.inflow.expand(3, 2, nx)], 1)
        return torch.cat([self.inflow.expand(3, ny + 4, 2), V, V[:, :, -1:], V[:, :, -1:]], 2)

    def _states(self, V):
        """Characteristic face states along the last axis (component 1 normal): minus states of
        faces -1..n, plus states of faces -2..n-1 for n cells and two ghosts each side."""
        out = []
        for plus in (False, True):
            S = [V[:, :, 0:-2], V[:, :, 1:-1], V[:, :, 2:]]
            M = 0.5 * (S[0] + S[1]) if plus else 0.5 * (S[1] + S[2])
            h, un, ut = M[0], M[1] / M[0], M[2] / M[0]
            c = torch.sqrt(self.g * h)
            w = []
            for f in range(3):
                q = [((un + c) * s[0] - s[1]) / (2 * c) if f == 0 else
                     (-ut * s[0] + s[2] if f == 1 else (-(un - c) * s[0] + s[1]) / (2 * c)) for s in S]
                w.append(_weno(*q, plus))
            out.append(torch.stack([w[0] + w[2], (un - c) * w[0] + (un + c) * w[2], ut * w[0] + w[1] + ut * w[2]]))
        return out

    def _direction(self, V):
        """Flux difference along the last axis and the cubic's depths at its Gauss points
        ([Gauss line][point]) for the rows 1 .. -1 of V's middle axis (one extra each side)."""
        m, p = self._states(V)
        g, t = self.g, 0.5 / math.sqrt(3.0)
        F, depths = 0.0, []
        for s in (-t, t):
            gp = [v[:, 1:-1] + s * 0.5 * (v[:, 2:] - v[:, :-2]) for v in (m, p)]
            L, R = gp[0][:, :, :-1], gp[1][:, :, 1:]              # faces -1 .. n-1
            fl, sp = [], []
            for q in (L, R):
                u = q[1] / q[0]
                fl.append(torch.stack([q[1], q[1] * u + 0.5 * g * q[0] * q[0], q[2] * u]))
                sp.append(u.abs() + torch.sqrt(g * q[0]))
            F = F + 0.25 * (fl[0] + fl[1] - torch.maximum(*sp) * (R - L))
            hm, hp = gp[0][0], gp[1][0]
            # the four depths of cell i: plus i-3/2, plus i-1/2, minus i+1/2, minus i+3/2
            four = [hp[:, :-2], hp[:, 1:-1], hm[:, 1:-1], hm[:, 2:]]
            depths.append([sum(CW[q][k] * four[k] for k in range(4)) for q in (0, 1)])
        return F[:, :, 1:] - F[:, :, :-1], depths

    def residual(self, U):
        V = self.ghosts(U)
        Fx, hx = self._direction(V[:, 1:-1])
        Vt = V[[0, 2, 1]][:, :, 1:-1].transpose(1, 2)
        Fy, hy = self._direction(Vt)
        Fy = Fy[[0, 2, 1]].transpose(1, 2)
        R = Fx / self.dx + Fy / self.dy
        for be in (0, 1):
            for ga in (0, 1):
                bx, by = self.b[be, ga]
                R[1] += 0.25 * self.g * hx[be][ga] * bx
                R[2] += 0.25 * self.g * hy[ga][be].transpose(0, 1) * by
        return R

    def jacobian(self, U, R, nb):
        off = {o: b for b, o in enumerate(OFF9 if nb == 9 else OFF21)}
        J = torch.zeros((nb, 3, 3, self.ny, self.nx), dtype=torch.float64, device=DEV)
        eps = self.p.eps
        for a in range(5):
            for c in range(5):
                for m in range(3):
                    V = U.clone()
                    V[m, c::5, a::5] += eps
                    D = (self.residual(V) - R) / eps
                    for i in range(5):
                        for j in range(5):
                            b = off.get(((a - i + 2) % 5 - 2, (c - j + 2) % 5 - 2))
                            if b is not None:
                                J[b, :, m, j::5, i::5] = D[:, j::5, i::5]
        for (di, dj), b in off.items():
            if di < 0:
                J[b, :, :, :, :-di] = 0.0
            elif di > 0:
                J[b, :, :, :, self.nx - di:] = 0.0
            if dj < 0:
                J[b, :, :, :-dj] = 0.0
            elif dj > 0:
                J[b, :, :, self.ny - dj:] = 0.0
        rn = R.abs().sum(0)
        for k in range(3):
            J[0, k, k] += self.p.alpha * rn
        return J


def _offsets(J):
    return {5: OFF5, 9: OFF9, 21: OFF21}[J.shape[0]]


def _apply2(J, x, skip_diag):
    ny, nx = x.shape[1:]
    out = torch.zeros_like(x)
    for b, (di, dj) in enumerate(_offsets(J)):
        if b == 0 and skip_diag:
            continue
        j0, j1, i0, i1 = max(0, -dj), ny - max(0, dj), max(0, -di), nx - max(0, di)
        if j1 <= j0 or i1 <= i0:
            continue
        out[:, j0:j1, i0:i1] += (J[b, :, :, j0:j1, i0:i1] * x[None, :, j0 + dj:j1 + dj, i0 + di:i1 + di]).sum(1)
    return out


class _Mg2:
    def __init__(self, J, levels, omega, nu1, nu2):
        self.J, self.omega, self.nu = [J], omega, (nu1, nu2)
        for _ in range(levels - 1):
            f = self.J[-1]
            C = torch.zeros((5, 3, 3, f.shape[3] // 2, f.shape[4] // 2), dtype=torch.float64, device=DEV)
            for b, (di, dj) in enumerate(_offsets(f)):
                for pj in (0, 1):
                    for pi in (0, 1):
                        o = ((pi + di) // 2, (pj + dj) // 2)
                        if o in OFF5:
                            C[OFF5.index(o)] += f[b, :, :, pj::2, pi::2]
            self.J.append(C)
        self.Di = [torch.linalg.inv(j[0].permute(2, 3, 0, 1)).permute(2, 3, 0, 1).contiguous() for j in self.J]
        self.mask = []
        for j in self.J:
            jj, ii = torch.meshgrid(torch.arange(j.shape[3], device=DEV), torch.arange(j.shape[4], device=DEV),
                                    indexing="ij")
            nb = j.shape[0]
            col = ii % 3 + 3 * (jj % 3) if nb == 21 else (ii + jj) % (3 if nb == 9 else 2)
            self.mask.append([col == c for c in range({5: 2, 9: 3, 21: 9}[nb])])
        j = self.J[-1]
        ny, nx = j.shape[3:]
        A = torch.zeros((ny * nx, 3, ny * nx, 3), dtype=torch.float64, device=DEV)
        for b, (di, dj) in enumerate(_offsets(j)):
            for y in range(max(0, -dj), ny - max(0, dj)):
                for x in range(max(0, -di), nx - max(0, di)):
                    A[y * nx + x, :, (y + dj) * nx + x + di, :] = j[b, :, :, y, x]
        self.lu = torch.linalg.lu_factor(A.reshape(3 * ny * nx, 3 * ny * nx))

    def smooth(self, l, rhs, x, nu):
        m = self.mask[l]
        for _ in range(2 * nu):
            for c in list(range(len(m))) + list(range(len(m) - 1, -1, -1)):
                r = rhs + _apply2(self.J[l], x, True)
                t = (self.Di[l] * r[None]).sum(1)
                x = torch.where(m[c], (1 - self.omega) * x - self.omega * t, x)
        return x

    def cycle(self, rhs, x, l=0):
        if l == len(self.J) - 1:
            y = torch.linalg.lu_solve(*self.lu, -rhs.permute(1, 2, 0).reshape(-1, 1))
            return y.reshape(rhs.shape[1], rhs.shape[2], 3).permute(2, 0, 1).contiguous()
        x = self.smooth(l, rhs, x, self.nu[0])
        r = rhs + _apply2(self.J[l], x, False)
        rc = r[:, 0::2, 0::2] + r[:, 0::2, 1::2] + r[:, 1::2, 0::2] + r[:, 1::2, 1::2]
        e = self.cycle(rc, torch.zeros_like(rc), l + 1)
        x = x + e.repeat_interleave(2, 1).repeat_interleave(2, 2)
        return self.smooth(l, rhs, x, self.nu[1])


def exact(case, seed):
    kind = case["kind"]
    if kind == "uneven1d":        # hundreds of different grids one by one: too slow in plain torch
        return None
    if kind == "step1d":
        prob = _problem1d(case, seed)
        ch, U = _Channel([prob]), _perturbed(prob.initial_guess(), seed)[None]
        R = ch.residual(U)
        rn = R.abs().sum(1)
        return [R[0], rn[0], rn.mean(), ch.jacobian(U, R, case["jac"])[0]]
    if kind == "step2d":
        prob = _problem2d(case, seed)
        w, U = _Wedge(prob), _perturbed(prob.initial_guess(), seed)
        R = w.residual(U)
        rn = R.abs().sum(0)
        return [R, rn, rn.mean(), w.jacobian(U, R, case["jac"])]
    if kind == "vcycle1d":
        p = _problem1d(case, seed).params
        J, rhs = _operator1d(case, seed)
        if case["prec"]:
            rhs = rhs.float().double()
        mg = _Mg1(J[None], case["levels"], torch.full((1,), p.omega, dtype=torch.float64, device=DEV), p.nu1, p.nu2)
        x = torch.zeros_like(rhs)[None]
        for _ in range(p.nu3):
            x = mg.cycle(rhs[None], x)
        return [x[0]]
    if kind == "vcycle2d":
        p = _problem2d(case, seed).params
        J, rhs = _operator2d(case, seed)
        if case["prec"]:
            rhs = rhs.float().double()
        mg = _Mg2(J, case["k"] + 1, p.omega, p.nu1, p.nu2)
        x = torch.zeros_like(rhs)
        for _ in range(p.nu3):
            x = mg.cycle(rhs, x)
        return [x]
    if kind == "newton2d":
        prob = _problem2d(case, seed)
        w, p = _Wedge(prob), prob.params
        U = torch.tensor(prob.initial_guess(), dtype=torch.float64, device=DEV)
        for _ in range(case["steps"]):
            R = w.residual(U)
            mg = _Mg2(w.jacobian(U, R, case["jac"]), prob.levels, p.omega, p.nu1, p.nu2)
            x = torch.zeros_like(U)
            for _ in range(p.nu3):
                x = mg.cycle(R, x)
            U = U + p.tau * x
        res = float(w.residual(U).abs().sum(0).mean())
        return [U, case["steps"], 1, res]
    if kind == "solve1d":
        U, it, st, res = _solve1([_problem1d(case, seed)], case["jac"])
        return [U[0], int(it[0]), int(st[0]), float(res[0])]
    probs = [_problem1d(case, seed, i) for i in range(case["count"])]
    parts = [_solve1(probs[o:o + 32], case["jac"]) for o in range(0, len(probs), 32)]
    U, it, st, res = (torch.cat([p[k].reshape(-1) for p in parts]) for k in range(4))
    return [U, it.cpu().numpy(), st.cpu().numpy(), res.cpu().numpy()]
