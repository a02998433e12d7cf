"""Cases on which the framework's speed is measured.

Each case is one call (or the short sequence of calls) that a program using
the package makes per iteration: an SLSQP-like solver that hands over a
least-squares subproblem, a server that solves again with a factor it keeps,
a batch of uneven subproblems, a thin QR, an equality-constrained subproblem,
a Hessian factor and its rank-one update.

The factorizations work in place, so a pass first copies the iteration's
matrix into the buffer that is overwritten, as such a solver does with its
new Jacobian; buffers, workspace and batch plan are kept between passes.
"""
import math

import torch

import paper_2506_09463_amd as hqr

F64 = torch.float64


def listed():
    return [
        # the smallest subproblem a solver hands over: a few variables
        {"name": "lsq 20x8", "op": "lsq", "m": 20, "n": 8, "nrhs": 1, "pad": 0, "kappa": 0.0},
        # the small configuration of the benchmark
        {"name": "lsq 128x64", "op": "lsq", "m": 128, "n": 64, "nrhs": 1, "pad": 0, "kappa": 0.0},
        # an ordinary ragged subproblem inside a larger buffer (leading dimension > rows)
        {"name": "lsq 701x333 r3", "op": "lsq", "m": 701, "n": 333, "nrhs": 3, "pad": 4, "kappa": 0.0},
        # the upper part of the served range
        {"name": "lsq 3000x2000 r4", "op": "lsq", "m": 3000, "n": 2000, "nrhs": 4, "pad": 0, "kappa": 0.0},
        # the large configuration of the benchmark (its shape; conditioned columns)
        {"name": "lsq 8192x4096", "op": "lsq", "m": 8192, "n": 4096, "nrhs": 1, "pad": 0, "kappa": 1e5},
        # thin QR: factor, then the leading n columns of Q
        {"name": "thin qr 6001x700", "op": "thinq", "m": 6001, "n": 700, "pad": 0},
        # the batched configuration of the benchmark
        {"name": "batch 2000", "op": "batch", "count": 2000, "nmin": 16, "nmax": 512, "nrhs": 8, "factored": 0.0},
        # continuous batching of small served requests: two of three reuse a stored factor
        {"name": "batch 300 reuse", "op": "batch", "count": 300, "nmin": 16, "nmax": 400, "nrhs": 3, "factored": 0.67},
        # a served request on a cached factor: Q^T b and back-substitution
        {"name": "stored 2047x1500 r3", "op": "stored", "m": 2047, "n": 1500, "nrhs": 3, "pad": 0},
        # a served mixed-precision request with FP64 refinement, nothing waiting on the host
        {"name": "mixed 3000x2048 r2", "op": "mixed", "m": 3000, "n": 2048, "nrhs": 2, "pad": 0, "kappa": 100.0},
        # SLSQP's subproblem with linearized equality constraints
        {"name": "lse 1500x700 p120", "op": "lse", "m": 1500, "n": 700, "p": 120},
        # the Hessian's factor and its rank-one update
        {"name": "cholesky 2000 update", "op": "chol", "n": 2000},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["lsq", "lsq", "lsq", "lsq", "thinq", "batch", "batch", "stored", "mixed", "lse", "chol"])
    pad = rng.choice([0, 0, 1, 2, 3, 8])
    if op == "lsq":
        n = _log(rng, 4, 4096)
        m = min(8192, n + int(n * rng.uniform(0.02, 1.5)) + 1)
        kappa = rng.choice([0.0, 1e3, 1e5]) if n >= 1000 else 0.0
        return {"op": op, "m": m, "n": n, "nrhs": rng.randint(1, 4), "pad": pad, "kappa": kappa}
    if op == "thinq":
        n = _log(rng, 20, 1200)
        return {"op": op, "m": min(8000, int(n * math.exp(rng.uniform(0.1, 2.5))) + 1), "n": n, "pad": pad}
    if op == "batch":
        return {"op": op, "count": _log(rng, 10, 1500), "nmin": 16, "nmax": rng.randint(40, 512),
                "nrhs": rng.randint(1, 8), "factored": rng.choice([0.0, 0.5, 0.67])}
    if op == "stored":
        n = _log(rng, 16, 3000)
        return {"op": op, "m": n + int(n * rng.uniform(0.02, 0.5)) + 1, "n": n, "nrhs": rng.randint(1, 4), "pad": pad}
    if op == "mixed":
        n = _log(rng, 513, 2500)
        return {"op": op, "m": n + int(n * rng.uniform(0.02, 0.5)) + 1, "n": n, "nrhs": rng.randint(1, 4), "pad": pad,
                "kappa": rng.choice([10.0, 100.0])}
    if op == "lse":
        n = _log(rng, 20, 1200)
        return {"op": op, "m": n + int(n * rng.uniform(0.02, 1.5)) + 1, "n": n, "p": max(1, int(n * rng.uniform(0.02, 0.4)))}
    return {"op": "chol", "n": _log(rng, 16, 3000)}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, m, n, pad=0):
    """m x n column-major N(0, 1) with leading dimension m + pad (zeros in the pad)."""
    base = torch.zeros((n, m + pad), dtype=F64, device="cuda")
    base[:, :m] = torch.randn((n, m), generator=g, dtype=F64, device="cuda")
    return base.t()[:m]


def _cosine(n):
    """The orthogonal n x n cosine matrix (type IV)."""
    k = torch.arange(n, dtype=F64, device="cuda") + 0.5
    return torch.cos(math.pi / n * k[:, None] * k[None, :]) * math.sqrt(2.0 / n)


def _matrix(g, c):
    """A: Gaussian, or U diag(1 .. 1/kappa) V^T with orthonormal U and V."""
    m, n, pad = c["m"], c["n"], c["pad"]
    A = _randn(g, m, n, pad)
    if c.get("kappa"):
        U = A.contiguous()
        for _ in range(2):
            L = torch.linalg.cholesky(U.t() @ U)
            U = torch.linalg.solve_triangular(L, U.t().contiguous(), upper=False).t().contiguous()
        sign = torch.where(torch.rand(n, generator=g, dtype=F64, device="cuda") < 0.5, -1.0, 1.0).to(F64)
        sigma = torch.logspace(0.0, -math.log10(c["kappa"]), n, dtype=F64, device="cuda")
        mix = torch.randperm(n, generator=g, device="cuda")
        A.copy_((U * sigma) @ (_cosine(n)[:, mix] * sign))
    return A


def _rhs(g, c, A):
    """b: N(0, 1); for a conditioned A near its range, as a solver's is."""
    m, n, r = c["m"], c["n"], c["nrhs"]
    if not c.get("kappa"):
        return _randn(g, m, r, c["pad"])
    x = torch.randn((n, r), generator=g, dtype=F64, device="cuda")
    B = _randn(g, m, r, c["pad"])
    B.copy_(A @ x + 1e-6 * B)
    return B


def _like(t):
    """A buffer of t's shape and leading dimension."""
    return torch.zeros((t.shape[1], t.stride(1) if t.shape[1] > 1 else t.shape[0]), dtype=F64, device="cuda").t()[: t.shape[0]]


def _shapes(c):
    """(rows, columns, whether a factor is kept) of every problem of the batch."""
    g = torch.Generator()
    g.manual_seed(c["count"])
    n = torch.randint(c["nmin"], c["nmax"] + 1, (c["count"],), generator=g)
    m = n + (torch.rand(c["count"], generator=g) * (n + 1)).to(torch.int64)
    new = c["count"] - int(c["count"] * c["factored"])       # the new problems first, then those with a kept factor
    return m.tolist(), n.tolist(), [k >= new for k in range(c["count"])]


class _Arena:
    """Column-major matrices of several shapes one after another in one buffer."""

    def __init__(self, ms, ns):
        self.shapes = list(zip(ms, ns))
        self.off = [0]
        for m, n in self.shapes:
            self.off.append(self.off[-1] + m * n)
        self.flat = None

    def views(self, flat):
        self.flat = flat
        return [flat[o:o + m * n].view(n, m).t() for (m, n), o in zip(self.shapes, self.off)]


def _inputs(c, seed):
    """What the caller has before the call: new tensors, from the seed alone."""
    g = _gen(seed)
    op = c["op"]
    if op in ("lsq", "mixed", "stored"):
        A = _matrix(g, c)
        return {"A": A, "B": _rhs(g, c, A)}
    if op == "thinq":
        return {"A": _matrix(g, c)}
    if op == "batch":
        m, n, f = _shapes(c)
        A, B = _Arena(m, n), _Arena(m, [c["nrhs"]] * len(m))
        d = {"m": m, "n": n, "factored": f}
        d["As"] = A.views(torch.randn(A.off[-1], generator=g, dtype=F64, device="cuda"))
        d["Bs"] = B.views(torch.randn(B.off[-1], generator=g, dtype=F64, device="cuda"))
        d["A"], d["B"] = A.flat, B.flat
        return d
    if op == "lse":
        m, n, p = c["m"], c["n"], c["p"]
        v = lambda k: torch.randn(k, generator=g, dtype=F64, device="cuda")
        return {"A": _randn(g, m, n), "C": _randn(g, p, n), "b": v(m), "d": v(p)}
    n = c["n"]
    G = torch.randn((n, n + 8), generator=g, dtype=F64, device="cuda")
    S = torch.zeros((n, n), dtype=F64, device="cuda").t()
    S.copy_(G @ G.t() / n)
    S.diagonal().add_(0.1)
    return {"S": S, "v": torch.randn(n, generator=g, dtype=F64, device="cuda")}


def prepare(case, seed):
    c, op = case, case["op"]
    s = {"case": c, "in": _inputs(c, seed)}
    i = s["in"]
    s["info"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    work = lambda b: torch.empty(b // 8 + 1, dtype=F64, device="cuda")
    if op in ("lsq", "mixed"):
        s["A"], s["B"] = _like(i["A"]), _like(i["B"])
        s["up"] = torch.zeros(c["n"], dtype=F64, device="cuda")
        s["res"] = torch.zeros(c["nrhs"], dtype=F64, device="cuda")
        s["iters"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        prec = hqr.HQR_PREC_MIXED if op == "mixed" else hqr.HQR_PREC_FP64
        s["work"] = work(hqr.workspace_size(c["m"], c["n"], c["nrhs"], prec))
    elif op == "thinq":
        s["A"], s["Q"] = _like(i["A"]), _like(i["A"])
        s["up"] = torch.zeros(c["n"], dtype=F64, device="cuda")
        s["work"] = work(hqr.workspace_size(c["m"], c["n"], c["n"]))
    elif op == "stored":
        s["B"] = _like(i["B"])
        s["up"], _ = hqr.qr_factor(i["A"])          # i["A"] now holds the factor the server keeps
    elif op == "batch":
        mA, mB = _Arena(i["m"], i["n"]), _Arena(i["m"], [c["nrhs"]] * len(i["m"]))
        keep = any(i["factored"])
        if keep:
            f = [k for k, y in enumerate(i["factored"]) if y]
            ups, _, _ = hqr.qr_lsq_solve_batched([i["As"][k] for k in f],
                                                 [torch.zeros((1, i["m"][k]), dtype=F64, device="cuda").t() for k in f])
            kept = dict(zip(f, ups))
        else:
            kept = {}
        s["A"] = torch.zeros_like(i["A"])
        s["B"] = torch.zeros_like(i["B"])
        s["A"].copy_(i["A"])
        As, Bs = mA.views(s["A"]), mB.views(s["B"])
        s["up"] = torch.zeros(sum(i["n"]), dtype=F64, device="cuda")
        ups = list(torch.split(s["up"], i["n"]))
        for k, u in kept.items():
            ups[k].copy_(u[: i["n"][k]])
        s["res"] = torch.zeros(len(As) * c["nrhs"], dtype=F64, device="cuda")
        s["info"] = torch.zeros(len(As), dtype=torch.int32, device="cuda")
        s["work"] = work(hqr.batched_workspace_size(len(As)))
        s["plan"] = hqr.BatchPlan(As, Bs, ups=ups, resnorms=list(torch.split(s["res"], c["nrhs"])), info=s["info"],
                                  work=s["work"], factored=i["factored"] if keep else None)
        # the new problems' matrices, copied in on every pass
        s["new"] = sum(m * n for m, n, y in zip(i["m"], i["n"], i["factored"]) if not y)
    elif op == "lse":
        s["A"], s["C"] = _like(i["A"]), _like(i["C"])
        s["b"] = torch.zeros_like(i["b"])
        s["x"] = torch.zeros(c["n"], dtype=F64, device="cuda")
        s["work"] = work(hqr.load().hqr_lse_workspace_size(c["m"], c["n"], c["p"]))
    else:
        s["S"], s["v"] = _like(i["S"]), torch.zeros_like(i["v"])
        s["work"] = work(32768)
    return s


def run(state):
    s, i, c = state, state["in"], state["case"]
    op = c["op"]
    if op == "lsq":
        s["A"].copy_(i["A"])
        s["B"].copy_(i["B"])
        hqr.qr_lsq_solve(s["A"], s["B"], up=s["up"], resnorm=s["res"], info=s["info"], iters=s["iters"], work=s["work"])
        return {"A": s["A"], "up": s["up"], "B": s["B"], "res": s["res"], "info": s["info"]}
    if op == "mixed":
        s["A"].copy_(i["A"])
        s["B"].copy_(i["B"])
        hqr.qr_lsq_solve(s["A"], s["B"], up=s["up"], resnorm=s["res"], info=s["info"], iters=s["iters"], work=s["work"],
                         precision=hqr.HQR_PREC_MIXED, A_orig=i["A"], no_fallback=True)
        # the call's results; the factor behind them is one of 32-bit accuracy, and B's rows past n are left by it
        return {"x": s["B"][: c["n"]], "res": s["res"], "info": s["info"], "iters": s["iters"]}
    if op == "thinq":
        s["A"].copy_(i["A"])
        hqr.qr_factor(s["A"], up=s["up"], info=s["info"], work=s["work"])
        hqr.qr_form_q(s["A"], s["up"], Q=s["Q"], work=s["work"])
        return {"A": s["A"], "up": s["up"], "Q": s["Q"], "info": s["info"]}
    if op == "stored":
        A, n = i["A"], c["n"]
        s["B"].copy_(i["B"])
        hqr.qr_apply_qt(A, s["up"], s["B"])
        hqr.qr_backsolve(A[:n, :n], s["B"], info=s["info"])
        return {"B": s["B"], "info": s["info"]}
    if op == "batch":
        s["A"][: s["new"]].copy_(i["A"][: s["new"]])
        s["B"].copy_(i["B"])
        s["plan"].run()
        return {"A": s["A"], "up": s["up"], "B": s["B"], "res": s["res"], "info": s["info"]}
    if op == "lse":
        s["A"].copy_(i["A"])
        s["C"].copy_(i["C"])
        s["b"].copy_(i["b"])
        hqr.qr_lse_solve(s["A"], s["C"], s["b"], i["d"], x=s["x"], info=s["info"], work=s["work"])
        return {"x": s["x"], "info": s["info"]}
    s["S"].copy_(i["S"])
    s["v"].copy_(i["v"])
    hqr.cholesky(s["S"], info=s["info"], work=s["work"])
    hqr.chol_update(s["S"], s["v"])
    return {"R": s["S"], "info": s["info"]}


def work(case):
    c, op = case, case["op"]
    fac = lambda m, n: 2.0 * m * n * n - 2.0 / 3.0 * n ** 3
    if op in ("lsq", "mixed"):
        m, n, r = c["m"], c["n"], c["nrhs"]
        return {"bytes": 8.0 * (2 * m * n + 2 * m * r + n + r), "flops": fac(m, n) + 4.0 * m * n * r + n * n * r}
    if op == "thinq":
        m, n = c["m"], c["n"]
        return {"bytes": 8.0 * (3 * m * n + n), "flops": 2 * fac(m, n)}
    if op == "stored":
        m, n, r = c["m"], c["n"], c["nrhs"]
        return {"bytes": 8.0 * (m * n + 2 * m * r + n), "flops": 4.0 * m * n * r - n * n * r}
    if op == "batch":
        by = fl = 0.0
        for m, n, f in zip(*_shapes(c)):
            r = c["nrhs"]
            by += 8.0 * ((1 if f else 2) * m * n + 2 * m * r + n + r)
            fl += (0.0 if f else fac(m, n)) + 4.0 * m * n * r - n * n * r
        return {"bytes": by, "flops": fl}
    if op == "lse":
        m, n, p = c["m"], c["n"], c["p"]
        return {"bytes": 8.0 * (m * n + p * n + m + n + p), "flops": fac(n, p) + 4.0 * m * n * p - 2.0 * m * p * p + fac(m, n - p)}
    n = c["n"]
    return {"bytes": 8.0 * n * n, "flops": n ** 3 / 3.0 + 3.0 * n * n}


# ------------------------------------------------------- 64-bit references
def _geqrf(A):
    """(A in the package's storage, up, LAPACK's factor, tau) by LAPACK: the
    package keeps a reflector's tail unnormalised and its leading component
    in up."""
    F, tau = torch.geqrf(A)
    n = A.shape[1]
    up = -tau * F.diagonal()[:n]
    low = torch.tril(torch.ones_like(F, dtype=torch.bool), -1)
    return torch.where(low, F * up, F), up, F, tau


def _lsq(A, B):
    """The least-squares call's outputs."""
    n = A.shape[1]
    st, up, F, tau = _geqrf(A)
    QB = torch.ormqr(F, tau, B, left=True, transpose=True)
    res = QB[n:].norm(dim=0)
    QB[:n] = torch.linalg.solve_triangular(torch.triu(F[:n]), QB[:n].clone(), upper=True)
    return st, up, QB, res


def exact(case, seed):
    c, op = case, case["op"]
    i = _inputs(c, seed)
    if op in ("lsq", "mixed", "stored"):
        A, B = i["A"].cpu(), i["B"].cpu()
        st, up, QB, res = _lsq(A, B)
        if op == "lsq":
            return {"A": st, "up": up, "B": QB, "res": res, "info": None}
        if op == "mixed":
            return {"x": QB[: c["n"]], "res": res, "info": None, "iters": None}
        return {"B": QB, "info": None}
    if op == "thinq":
        st, up, F, tau = _geqrf(i["A"].cpu())
        return {"A": st, "up": up, "Q": torch.linalg.householder_product(F, tau), "info": None}
    if op == "batch":
        oa, ou, ob, orr = [], [], [], []
        A, B = i["A"].cpu(), i["B"].cpu()
        As, Bs = _Arena(i["m"], i["n"]).views(A), _Arena(i["m"], [c["nrhs"]] * len(i["m"])).views(B)
        for a, b in zip(As, Bs):
            st, up, QB, res = _lsq(a, b)
            oa.append(st.t().reshape(-1))
            ou.append(up)
            ob.append(QB.t().reshape(-1))
            orr.append(res)
        return {"A": torch.cat(oa), "up": torch.cat(ou), "B": torch.cat(ob), "res": torch.cat(orr), "info": None}
    if op == "lse":
        A, C, b, d = (i[k].cpu() for k in ("A", "C", "b", "d"))
        p = c["p"]
        F, tau = torch.geqrf(C.t().contiguous())
        y1 = torch.linalg.solve_triangular(torch.triu(F[:p]).t(), d[:, None], upper=False)
        AQ = torch.ormqr(F, tau, A.t().contiguous(), left=True, transpose=True).t()
        y2 = _lsq(AQ[:, p:].contiguous(), b[:, None] - AQ[:, :p] @ y1)[2][: c["n"] - p]
        return {"x": torch.ormqr(F, tau, torch.cat([y1, y2]), left=True, transpose=False)[:, 0], "info": None}
    S, v = i["S"].cpu(), i["v"].cpu()
    R = torch.linalg.cholesky(S + v[:, None] * v[None, :]).t()
    return {"R": torch.triu(R) + torch.tril(S, -1), "info": None}
