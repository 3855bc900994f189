"""Timed cases of the shallow-water solver: what a program using it has it do.

A case is one of four kinds of call sequence through the public binding
(``paper_2311_11348_amd.swe``):

* ``run``    a context in hand (mesh, bathymetry, orders, state set): advance
             it by the run's number of steps and read the state back, the
             loop of a simulation that writes its state out;
* ``solve``  a whole request from the caller's arrays to the result: create
             the context, set mesh, bathymetry, forcing and initial state,
             step, read the state back (what a served request pays);
* ``batch``  several instances resident in one batch: advance all of them
             and read every member's state back;
* ``rhs``    one evaluation of the semi-discrete right-hand side.

States come back in the precision the context computes in (a program that
chose FP32 keeps FP32 fields).  ``exact`` evaluates the same method in 64 bits
by quadrature, in plain torch.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2311_11348_amd import flops, swe
from paper_2311_11348_amd import inputs as I

FP64, FP32 = swe.SWE_FP64, swe.SWE_FP32_WB
KS = (1, 3, 6, 10)
DEG = (0, 1, 1, 2, 2, 2, 3, 3, 3, 3)
MONO = ((0, 0), (1, 0), (0, 1), (2, 0), (1, 1), (0, 2), (3, 0), (2, 1), (1, 2), (0, 3))


def _case(name, kind, problem, n, p, fp32, steps, scheme="fused", count=1):
    c = dict(kind=kind, problem=problem, n=n, p=p, fp32=fp32, steps=steps, scheme=scheme, count=count)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: a dozen steps' worth of launches on a toy mesh (a check run, an interactive try)
        _case("smoke_p2_fp64", "run", "bump", 12, 2, False, 10),
        # the plain small run: 2,048 elements, p = 1, the bump, its 100 steps
        _case("bump_p1_fp64", "run", "bump", 32, 1, False, 100),
        # the full tidal workload, its 500 steps, in its headline precision
        _case("tidal_p2_fp32", "run", "tidal", 512, 2, True, 500),
        # the same in FP64, on a mesh whose side is odd
        _case("tidal_p2_fp64", "run", "tidal", 361, 2, False, 200),
        # the lowest linear order in FP32 and the highest in both, closed basin with a hump
        _case("hump_p1_fp32", "run", "hump", 301, 1, True, 200),
        _case("hump_p3_fp64", "run", "hump", 180, 3, False, 100),
        # adaptive tsunami: orders 1-3 re-chosen every step; the paper's separated scheme
        # in FP32 at full size, the partitioned one in FP64 on a smaller odd mesh
        _case("tsunami_p13_fp32", "run", "tsunami", 256, 3, True, 200, "separated"),
        _case("tsunami_p13_fp64", "run", "tsunami", 97, 3, False, 100, "partitioned"),
        # the dam break with every 32nd element at p = 2 (static order map), its 100 steps
        _case("dambreak_p12_fp64", "run", "dambreak", 320, 2, False, 100, "partitioned"),
        # a served request, from arrays to result
        _case("request_p3_fp32", "solve", "tidal", 105, 3, True, 300),
        # eight instances of all orders in one batch
        _case("batch_fp32", "batch", "instances", 110, 3, True, 100, "fused", 8),
        # one right-hand-side evaluation (an outer integrator's or a test's call)
        _case("rhs_p2_fp64", "rhs", "tidal", 128, 2, False, 1),
    ]


def draw(rng):
    """One more case: every kind, order, precision and scheme, sides 8 to 360 (log-uniform, odd ones
    among them), steps 10 to 300; element-steps bounded by the largest listed case's."""
    kind = rng.choice(["run"] * 7 + ["solve", "batch", "rhs"])
    fp32 = rng.random() < 0.5
    n = int(round(math.exp(rng.uniform(math.log(8), math.log(360)))))
    steps = int(round(math.exp(rng.uniform(math.log(10), math.log(300)))))
    if kind == "batch":
        count = rng.randint(2, 10)
        n = min(n, 90)
        steps = min(steps, 100)
        return _case("", kind, "instances", n, 3, fp32, steps, "fused", count)
    if kind != "run":
        n = min(n, 200)
        return _case("", kind, rng.choice(["tidal", "hump"]), n, rng.choice([1, 2, 3]), fp32,
                     1 if kind == "rhs" else steps)
    prob = rng.choice(["bump", "tidal", "hump", "shallow", "dambreak", "tsunami"])
    scheme, p = "fused", rng.choice([0, 1, 1, 2, 2, 3])
    if prob == "dambreak":
        p = rng.choice([1, 2])
        scheme = rng.choice(["separated", "partitioned"])
    elif prob == "tsunami":
        p, n = 3, min(n, 256)
        scheme = "separated" if fp32 else rng.choice(["separated", "partitioned"])
        steps = min(steps, 100)
    elif prob == "shallow":
        p = rng.choice([1, 2])
    if n > 250:
        steps = min(steps, 200)
    if p == 3:
        n = min(n, 200)
        steps = min(steps, 100)
    return _case("", kind, prob, n, p, fp32, steps, scheme)


# ------------------------------------------------------------------ inputs
def _members(case, seed):
    """(problem, initial amplitude of the added waves, start time) of each instance of a case."""
    rng = np.random.default_rng([int(seed), 17])
    ms = int(rng.integers(0, 2 ** 31 - 1))
    t0 = float(rng.uniform(0.0, I.TIDE_PERIOD))
    n, p, kind = case["n"], case["p"], case["problem"]
    if kind == "bump":
        return [(I.config_c1(n=n, p=p), 0.02, 0.0)]
    if kind == "tidal":
        return [(I.config_c2(n=n, p=p, seed=ms), 0.3, t0)]
    if kind == "hump":
        prob = I.config_c3(n=n, seed=ms)
        prob.p[:] = p
        prob.p_base, prob.p_max, prob.adapt = p, p, 0
        return [(prob, 0.05, 0.0)]
    if kind == "tsunami":
        return [(I.config_c3(n=n, seed=ms), 0.005, 0.0)]
    if kind == "shallow":
        return [(I.config_shallow(n=n, p=p, seed=ms), 0.002, 0.0)]
    if kind == "dambreak":
        return [(I.config_dambreak(n=n, p_lo=p - 1, p_hi=p, every=32, seed=ms), 0.01, 0.0)]
    out = []
    for i in range(case["count"]):
        # sides from half to twice the case's, spread over their logarithm; orders in turn, tidal and hump alternating
        side = 2 * n * 4.0 ** -((0.5 + 0.618 * i) % 1.0)
        out.append((I.instance_problem(rng, 2.0 * side * side, 1 + i % case["p"], i % 2 == 0, case["steps"], f"inst{i}"),
                    0.1, t0 if i % 2 == 0 else 0.0))
    return out


def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _initial(prob, amp, seed):
    """Coefficients [ne][3][K] of the problem's initial state plus three long waves of amplitude amp
    (m) running in random directions (q = c xi along each, c the long-wave speed), by quadrature."""
    rng = np.random.default_rng([int(seed), 23])
    T = _ref(prob.p_max)
    P = torch.as_tensor(prob.mesh.vxy, device=_dev())[torch.as_tensor(prob.mesh.tri, device=_dev()).long()]
    xr, yr, w = T["qx"], T["qy"], T["qw"]
    x = P[:, 0, None, 0] + xr * (P[:, 1, None, 0] - P[:, 0, None, 0]) + yr * (P[:, 2, None, 0] - P[:, 0, None, 0])
    y = P[:, 0, None, 1] + xr * (P[:, 1, None, 1] - P[:, 0, None, 1]) + yr * (P[:, 2, None, 1] - P[:, 0, None, 1])
    ic = prob.ic(x.cpu().numpy(), y.cpu().numpy())
    xi, U, V = (torch.as_tensor(np.ascontiguousarray(f), device=_dev()) for f in ic)
    hb = torch.as_tensor(prob.hb_vertex, device=_dev())[torch.as_tensor(prob.mesh.tri, device=_dev()).long()]
    c = torch.sqrt(prob.g * hb.mean(1, keepdim=True))
    L = prob.mesh.length
    for _ in range(3):
        a, th, ph = amp * rng.uniform(0.3, 1.0), rng.uniform(0, 2 * np.pi), rng.uniform(0, 2 * np.pi)
        k = 2 * np.pi * rng.uniform(1.0, 4.0) / L
        s = a * torch.sin(k * (np.cos(th) * x + np.sin(th) * y) + ph)
        xi, U, V = xi + s, U + c * np.cos(th) * s, V + c * np.sin(th) * s
    det = (P[:, 1, 0] - P[:, 0, 0]) * (P[:, 2, 1] - P[:, 0, 1]) - (P[:, 2, 0] - P[:, 0, 0]) * (P[:, 1, 1] - P[:, 0, 1])
    m = torch.sqrt(det)[:, None, None] * torch.stack([(f * w) @ T["phi"].T for f in (xi, U, V)], 1)
    K = torch.as_tensor([KS[int(q)] for q in prob.p], device=_dev())
    m *= (torch.arange(m.shape[2], device=_dev())[None, :] < K[:, None])[:, None, :]
    return np.ascontiguousarray(m.cpu().numpy())


def _scheme(case):
    return {"fused": 0, "separated": 1, "partitioned": 2}[case["scheme"]]


def _precision(case):
    return FP32 if case["fp32"] else FP64


def prepare(case, seed):
    s = dict(case=case, members=[])
    for i, (prob, amp, t0) in enumerate(_members(case, seed)):
        c0 = _initial(prob, amp, seed * 100 + i)
        ctx = None
        if case["kind"] != "solve":
            ctx = swe.context_for(prob, precision=_precision(case), separate=_scheme(case))
            if case["kind"] != "rhs":
                ctx.set_state(c0, t0)
        s["members"].append(dict(prob=prob, c0=c0, t0=t0, dt=prob.dt(), ctx=ctx))
    if case["kind"] == "batch":
        s["batch"] = swe.Batch(precision=_precision(case), budget_bytes=16 << 30, max_instances=64)
        for m in s["members"]:
            s["batch"].admit(m["ctx"], 2 ** 30, m["dt"])
    return s


def _out(case, c, t):
    return {"state": c.astype(np.float32) if case["fp32"] else c, "t": t}


def run(state):
    case, m = state["case"], state["members"][0]
    if case["kind"] == "rhs":
        r = m["ctx"].rhs(m["t0"], m["c0"])
        return {"rhs": r.astype(np.float32) if case["fp32"] else r}
    if case["kind"] == "solve":
        with swe.context_for(m["prob"], precision=_precision(case), separate=_scheme(case)) as ctx:
            ctx.set_state(m["c0"], m["t0"])
            ctx.step(case["steps"], m["dt"])
            ctx.sync()
            return _out(case, *ctx.state())
    if case["kind"] == "batch":
        state["batch"].tick(case["steps"])
        state["batch"].sync()
        return [_out(case, *q["ctx"].state()) for q in state["members"]]
    m["ctx"].step(case["steps"], m["dt"])
    m["ctx"].sync()
    out = _out(case, *m["ctx"].state())
    if m["prob"].adapt and not case["fp32"]:
        out["order"] = m["ctx"].order()
    return out


def work(case):
    """Per step: the state (three fields) read and written once, the element's vertex and neighbour ids
    and its share of the vertices read once, two stages' operations; the caller's arrays once per pass."""
    w = 4 if case["fp32"] else 8
    total = dict(bytes=0.0, flops=0.0)
    sizes = [(2 * case["n"] ** 2, case["p"])]
    if case["kind"] == "batch":
        sizes = [(2 * case["n"] ** 2, 1 + i % case["p"]) for i in range(case["count"])]
    for ne, p in sizes:
        q = 1 if case["problem"] == "tsunami" else p - 1 if case["problem"] == "dambreak" else p   # most elements' order
        stages = 1 if case["kind"] == "rhs" else 2 * case["steps"]
        total["flops"] += ne * flops.stage_flops(q)["total"] * stages
        total["bytes"] += ne * ((6 * KS[q] * w + 40) * (stages / 2) + 3 * KS[p] * w)
        if case["kind"] in ("solve", "rhs"):
            total["bytes"] += ne * 3 * KS[p] * 8
    return total


# ------------------------------------------------------------------ the method in 64 bits
@functools.lru_cache(maxsize=None)
def _ref(p):
    """Basis values on quadrature points of the reference triangle and its edges, order p: rules exact
    for every integrand of the method at that order."""
    def gauss(m):
        t, w = np.polynomial.legendre.leggauss(m)
        return 0.5 * (t + 1.0), 0.5 * w

    def tri(m):
        t, w = gauss(m)
        X, Y = [a.ravel() for a in np.meshgrid(t, t, indexing="ij")]
        W = np.outer(w, w).ravel() * (1.0 - X)
        return X, Y * (1.0 - X), W

    # orthonormal basis: Gram-Schmidt of the monomials in the L2 product of the reference triangle
    f = math.factorial
    G = np.array([[f(a + c) * f(b + d) / f(a + b + c + d + 2) for c, d in MONO] for a, b in MONO])
    B = np.linalg.inv(np.linalg.cholesky(G))[:KS[p]]          # rows: basis functions in monomials

    def values(x, y):
        return B @ np.array([x ** a * y ** b for a, b in MONO])

    def gradients(x, y):
        gx = np.array([a * x ** max(a - 1, 0) * y ** b for a, b in MONO])
        gy = np.array([b * x ** a * y ** max(b - 1, 0) for a, b in MONO])
        return B @ gx, B @ gy

    d = _dev()
    T = {}
    X, Y, W = tri(6)                                          # projection and C: exact to degree 10
    T["qx"], T["qy"], T["qw"] = (torch.as_tensor(a, device=d) for a in (X, Y, W))
    T["phi"] = torch.as_tensor(values(X, Y), device=d)
    ph, K = values(X, Y), KS[p]
    C = np.einsum("q,nq,iq,jq->ijn", W, ph, ph, ph)
    trunc = C.copy()                                          # u H = q: depth modes up to max(deg i, deg j)
    for i in range(K):
        for j in range(K):
            trunc[i, j, KS[max(DEG[i], DEG[j])]:] = 0.0
    T["trunc"] = torch.as_tensor(trunc.reshape(K * K, K), device=d)
    T["full"] = torch.as_tensor(np.ascontiguousarray(C[:, :, :3]).reshape(K * K, -1), device=d)
    X, Y, W = tri((3 * p) // 2 + 1)
    v, (gx, gy) = values(X, Y), gradients(X, Y)
    T["v"] = torch.as_tensor(np.ascontiguousarray(v.T), device=d)
    T["gx"], T["gy"] = torch.as_tensor(gx * W, device=d), torch.as_tensor(gy * W, device=d)
    T["hat"] = torch.as_tensor(np.stack([1 - X - Y, X, Y], 1), device=d)
    t, w = gauss((3 * p + 2) // 2 + 1)
    corner = np.array([[0.0, 0.0], [1.0, 0.0], [0.0, 1.0]])
    T["edge"], T["lift"] = [], []
    for k in range(3):
        a, b = corner[(k + 1) % 3], corner[(k + 2) % 3]
        e = values(a[0] + t * (b[0] - a[0]), a[1] + t * (b[1] - a[1]))
        T["edge"].append(torch.as_tensor(np.ascontiguousarray(e.T), device=d))
        T["lift"].append(torch.as_tensor(e * w, device=d))
    T["t"] = torch.as_tensor(t, device=d)
    T["mid"] = [values(*[np.array([0.5 * (corner[(k + 1) % 3][i] + corner[(k + 2) % 3][i])]) for i in (0, 1)])[:3, 0].tolist()
                for k in range(3)] if p >= 1 else None
    chk = [(0, 0), (1, 0), (0, 1)] + [tuple(0.5 * (corner[(k + 1) % 3] + corner[(k + 2) % 3])) for k in range(3)]
    T["check"] = torch.as_tensor(np.ascontiguousarray(values(np.array([c[0] for c in chk]), np.array([c[1] for c in chk])).T), device=d)
    T["hatmode"] = torch.as_tensor(values(*[np.asarray(a) for a in tri(6)[:2]])[:3]
                                   @ (tri(6)[2][:, None] * np.stack([1 - tri(6)[0] - tri(6)[1], tri(6)[0], tri(6)[1]], 1)), device=d)
    return T


class _Method:
    """The semi-discrete method on one problem; coefficients [3][K][ne], scaled by 1 / sqrt(|det B|)."""

    def __init__(self, prob):
        d = _dev()
        self.prob, self.T, self.K = prob, _ref(prob.p_max), KS[prob.p_max]
        tri = torch.as_tensor(prob.mesh.tri, device=d).long().T
        xy = torch.as_tensor(prob.mesh.vxy, device=d)
        self.X, self.Y = xy[tri, 0], xy[tri, 1]
        self.h = torch.as_tensor(prob.hb_vertex, device=d)[tri]
        X, Y, h = self.X, self.Y, self.h
        self.det = (X[1] - X[0]) * (Y[2] - Y[0]) - (X[2] - X[0]) * (Y[1] - Y[0])
        self.b00, self.b01 = (Y[2] - Y[0]) / self.det, -(X[2] - X[0]) / self.det
        self.b10, self.b11 = -(Y[1] - Y[0]) / self.det, (X[1] - X[0]) / self.det
        self.hx = self.b00 * (h[1] - h[0]) + self.b10 * (h[2] - h[0])
        self.hy = self.b01 * (h[1] - h[0]) + self.b11 * (h[2] - h[0])
        hm = self.T["hatmode"] @ h
        self.hb = hm[:min(3, self.K)]
        self.hbM = (self.T["full"][:, :hm.shape[0]] @ hm).reshape(self.K, self.K, -1)
        # neighbour across each edge, from equal vertex pairs
        t = prob.mesh.tri
        ne = t.shape[0]
        a, b = t[:, [1, 2, 0]], t[:, [2, 0, 1]]
        key = (np.minimum(a, b).astype(np.int64) * prob.mesh.nv + np.maximum(a, b)).T.ravel()   # [3][ne]
        order = np.argsort(key, kind="stable")
        same = np.nonzero(key[order][1:] == key[order][:-1])[0]
        other = np.full(3 * ne, -1, np.int64)
        other[order[same]], other[order[same + 1]] = order[same + 1], order[same]
        tag = prob.mesh.tag.T.ravel()
        self.inner = torch.as_tensor((other >= 0).reshape(3, ne), device=d)
        self.open = torch.as_tensor(((other < 0) & (tag == I.TAG_OPEN)).reshape(3, ne), device=d)
        self.other = torch.as_tensor(np.maximum(other, 0), device=d)
        self.order = torch.as_tensor(prob.p.astype(np.int64), device=d)

    def mask(self):
        Ke = torch.as_tensor(KS, device=_dev())[self.order]
        return torch.arange(self.K, device=_dev())[:, None] < Ke[None, :]

    def velocity(self, c):
        K = self.K
        M = (self.T["trunc"] @ c[0]).reshape(K, K, -1) + self.hbM
        if int(self.order.min()) < self.prob.p_max:
            live = self.mask()
            both = live[:, None, :] & live[None, :, :]
            M = torch.where(both, M, torch.eye(K, device=M.device, dtype=M.dtype)[:, :, None])
        r = c[1:3].clone().transpose(0, 1).contiguous()                    # [K][2][ne]
        for j in range(K - 1):                                             # Gaussian elimination
            f = M[j + 1:, j] / M[j, j]
            M[j + 1:, j + 1:] -= f[:, None] * M[j, j + 1:][None]
            r[j + 1:] -= f[:, None] * r[j][None]
        for i in range(K - 1, -1, -1):
            if i + 1 < K:
                r[i] -= (M[i, i + 1:, None] * r[i + 1:]).sum(0)
            r[i] /= M[i, i]
        return r.transpose(0, 1)

    def forcing(self, t):
        f = self.prob.forcing
        return float(sum(a * math.sin(w * t + p) for a, w, p in zip(f.amp, f.omega, f.phase)))

    def rhs(self, c, t):
        T, pr, K, ne = self.T, self.prob, self.K, c.shape[2]
        g, xhat = pr.g, self.forcing(t)
        u = self.velocity(c)
        f = torch.cat([c, u])                                              # xi U V u v
        L = torch.zeros_like(c)
        q = torch.matmul(T["v"], f)                                        # [5][Q][ne]
        hb = T["hat"] @ self.h
        pres = g * q[0] * (0.5 * q[0] + hb)
        for j, (fx, fy) in enumerate(((q[1], q[2]), (q[1] * q[3] + pres, q[1] * q[4]), (q[2] * q[3], q[2] * q[4] + pres))):
            L[j] = T["gx"] @ (self.b00 * fx + self.b01 * fy) + T["gy"] @ (self.b10 * fx + self.b11 * fy)
        L[1] += g * self.hx * c[0] + pr.f_coriolis * c[2]
        L[2] += g * self.hy * c[0] - pr.f_coriolis * c[1]
        if pr.friction == I.FRICTION_QUADRATIC:
            L[1:3] -= pr.friction_coef * math.sqrt(2.0) * torch.sqrt(u[0, 0] ** 2 + u[1, 0] ** 2) * u
        elif pr.friction == I.FRICTION_LINEAR:
            L[1:3] -= pr.friction_coef * c[1:3]
        tr = torch.stack([torch.matmul(T["edge"][k], f) for k in range(3)], 2)      # [5][Qe][3][ne]
        across = tr.flip(1).reshape(5, -1, 3 * ne)
        mean = math.sqrt(2.0) * f[:, 0]
        s = T["t"][:, None]
        for k in range(3):
            ka, kb = (k + 1) % 3, (k + 2) % 3
            dx, dy = self.X[kb] - self.X[ka], self.Y[kb] - self.Y[ka]
            ln = torch.sqrt(dx * dx + dy * dy)
            nx, ny = dy / ln, -dx / ln
            hm, hs = 0.5 * (self.h[ka] + self.h[kb]), self.h[ka] + s * (self.h[kb] - self.h[ka])
            idx = self.other.reshape(3, ne)[k]
            m = tr[:, :, k]
            o = across[:, :, idx]
            inner, opn = self.inner[k], self.open[k]
            land = ~(inner | opn)
            mm = mean[:, idx % ne]
            un, qn = m[3] * nx + m[4] * ny, m[1] * nx + m[2] * ny
            uno, qno = o[3] * nx + o[4] * ny, o[1] * nx + o[2] * ny
            xo = torch.where(inner, o[0], torch.where(opn, torch.full_like(m[0], xhat), m[0]))
            Uo = torch.where(inner, o[1], torch.where(opn, m[1], m[1] - 2.0 * qn * nx))
            Vo = torch.where(inner, o[2], torch.where(opn, m[2], m[2] - 2.0 * qn * ny))
            uno = torch.where(inner, uno, torch.where(opn, un, -un))
            qno = torch.where(inner, qno, torch.where(opn, qn, -qn))
            ub = (mean[3] * nx + mean[4] * ny).abs()
            ubo = torch.where(inner, (mm[3] * nx + mm[4] * ny).abs(), ub)
            xb = torch.maximum(mean[0], torch.where(inner, mm[0], torch.where(opn, torch.full_like(ub, xhat), mean[0])))
            lam = torch.maximum(ub, ubo) + torch.sqrt(g * (xb + hm))
            P = 0.5 * g * (m[0] ** 2 + xo ** 2) + g * (m[0] + xo) * hs
            F = [torch.where(land, torch.zeros_like(qn), qn + qno + lam * (m[0] - xo)),
                 m[1] * un + Uo * uno + P * nx + lam * (m[1] - Uo),
                 m[2] * un + Vo * uno + P * ny + lam * (m[2] - Vo)]
            for j in range(3):
                L[j] -= T["lift"][k] @ (0.5 * F[j] * (ln / self.det))
        if int(self.order.min()) < pr.p_max:
            L *= self.mask()
        return L

    def limit(self, c):
        """Minimum depth control: the depth's deviation from its mean scaled until every check point has h_min."""
        h, hmin = self.h, self.prob.h_min
        low = (self.T["check"] @ c[0] + torch.cat([h, torch.stack([0.5 * (h[(k + 1) % 3] + h[(k + 2) % 3]) for k in range(3)])])).amin(0)
        mean = math.sqrt(2.0) * c[0, 0] + h.mean(0)
        th = torch.where(mean > hmin, (mean - hmin) / (mean - low), torch.zeros_like(mean))
        th = torch.where((low < hmin) & (self.order > 0), th, torch.ones_like(th))
        c = c.clone()
        c[:, 1:] *= th
        c[0, 1:3] += (th - 1.0) * self.hb[1:3]
        return c

    def adapt(self, c, t):
        """Orders from the jumps of the linear part of xi at the edge midpoints; dropped modes cleared."""
        ne = c.shape[2]
        mids = torch.stack([sum(self.T["mid"][k][i] * c[0, i] for i in range(3)) for k in range(3)])
        o = torch.where(self.inner, mids.reshape(-1)[self.other].reshape(3, ne), mids)
        o = torch.where(self.open, torch.full_like(mids, self.forcing(t)), o)
        jump = (mids - o).abs().amax(0)
        lo, hi = self.prob.p_base, self.prob.p_max
        new, thr = torch.full_like(self.order, lo), self.prob.adapt_tau
        bands = []
        for p in range(hi, lo, -1):
            bands.append((p, thr))
            thr *= 0.1
        for p, x in reversed(bands):
            new = torch.where(jump >= x, torch.full_like(new, p), new)
        self.order = new
        return c * self.mask()

    def advance(self, c, t0, steps, dt):
        c = (c * self.mask()) if not self.prob.adapt else c
        for s in range(steps):
            t = t0 + s * dt
            if self.prob.adapt:
                c = self.adapt(c, t)
            c1 = c + dt * self.rhs(c, t)
            c1 = self.limit(c1) if self.prob.h_min > 0.0 and self.prob.p_max > 0 else c1
            c = 0.5 * c + 0.5 * (c1 + dt * self.rhs(c1, t + dt))
            c = self.limit(c) if self.prob.h_min > 0.0 and self.prob.p_max > 0 else c
        return c

    def scaled(self, coef):
        return (torch.as_tensor(coef, device=_dev()) / torch.sqrt(self.det)[:, None, None]).permute(1, 2, 0).contiguous()

    def plain(self, c):
        return (c.permute(2, 0, 1) * torch.sqrt(self.det)[:, None, None]).contiguous().cpu().numpy()


def exact(case, seed):
    out = []
    for i, (prob, amp, t0) in enumerate(_members(case, seed)):
        M = _Method(prob)
        c = M.scaled(_initial(prob, amp, seed * 100 + i))
        if case["kind"] == "rhs":
            return {"rhs": M.plain(M.rhs(c * M.mask(), t0))}
        c = M.advance(c, t0, case["steps"], prob.dt())
        out.append({"state": M.plain(c), "t": t0 + case["steps"] * prob.dt()})
        if prob.adapt and not case["fp32"]:
            out[-1]["order"] = None
    return out if case["kind"] == "batch" else out[0]
