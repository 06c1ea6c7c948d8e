"""The work that a user of this library has it do, case by case, for timing and for comparing results.

Every case is one call of a public entry point of `paper_1807_07132_amd.nadmm` on data resident on the GPU: a
Hessian-vector product, objective and gradient, a CG solve, a line search, a whole local Newton-CG solve, or the ADMM
outer solver.  The shapes are those of the benchmark configurations (`workloads.py`), of the tests and of the library's
own documentation, from calls that only launches bound to the largest data share; `draw` spreads over the ranges they
stand for.

Ranges: dense A of 500 to 2,000,000 rows and 4 to 4096 columns (at most 90 million elements when drawn), row stride equal
to the number of columns (odd ones among them) or padded, 2 to 33 classes; sparse A of 2,000 to 60,000 rows, 2,000 to
300,000 columns and at most 12 million drawn positions when drawn.  Features are of order one, logits of order one to ten,
penalty 1, so that a few CG iterations reduce the residual by some orders of magnitude.
"""
import math

import torch

from paper_1807_07132_amd import nadmm

BETA, GAMMA, MAX_LS = 1e-4, 0.5, 10


def listed():
    return [
        # the smallest problem of the benchmark configurations: one Newton step of 10 CG iterations; launches and latency
        dict(name="tiny_solve", op="newton", data="gauss", n=1000, p=20, C=3, newton=1, cg=10),
        # objective and gradient on a small share with an ordinary number of columns
        dict(name="small_grad", op="grad", data="gauss", n=9001, p=260, C=10),
        # tabular data: a few dozen columns, several classes, rows that are not 16-byte aligned; CG of one Newton iteration
        dict(name="tabular_cg", op="cg", data="gauss", n=100000, p=70, C=7, cg=10),
        # the headline benchmark: Hessian-vector product on the image-like share
        dict(name="image_hessvec", op="hessvec", data="image", n=60000, p=784, C=10),
        # the x-update of one ADMM worker on it, as configured: 10 Newton iterations of 10 CG iterations
        dict(name="image_solve", op="newton", data="image", n=60000, p=784, C=10, newton=10, cg=10),
        # the same data with a constant column appended: odd rows; one line search that has to reduce its step
        dict(name="image_bias_search", op="search", data="image", n=60000, p=785, C=10),
        # two outer iterations of the ADMM solver with the image-like rows split over four workers
        dict(name="image_admm", op="admm", data="image", n=60000, p=784, C=10, workers=4, outer=2, newton=10, cg=10),
        # wide rows of unit length: CG of one Newton iteration
        dict(name="wide_cg", op="cg", data="unit", n=50000, p=3072, C=10, cg=10),
        # the largest share: many rows, many columns, 20 classes
        dict(name="multiclass_hessvec", op="hessvec", data="mixture", n=250000, p=2000, C=20),
        # tall two-class data: a whole x-update
        dict(name="binary_solve", op="newton", data="gauss", n=1375000, p=28, C=2, newton=10, cg=10),
        # tall two-class data with a constant column: odd short rows
        dict(name="binary_bias_grad", op="grad", data="gauss", n=1375000, p=29, C=2),
        # counts in sparse storage, one of 32 workers' shares of a data set with 279,998 features and 20 classes
        dict(name="sparse_hessvec", op="hessvec", data="counts", n=40628, p=279998, C=20, per_row=2000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["tabular", "tabular", "image", "wide", "classes", "sparse"])
    op = rng.choice(["hessvec", "grad", "cg", "newton", "search"])
    if family == "sparse":
        c = dict(data="counts", n=_log_int(rng, 2000, 60000), p=_log_int(rng, 2000, 300000), C=rng.randint(2, 33))
        c["per_row"] = max(8, min(400, 12000000 // c["n"], c["p"] // 8))
    else:
        if family == "tabular":
            p, C, data = _log_int(rng, 4, 128), rng.randint(2, 12), "gauss"
        elif family == "image":
            p, C, data = _log_int(rng, 129, 960), rng.randint(2, 17), "image"
        elif family == "wide":
            p, C, data = _log_int(rng, 961, 4096), rng.randint(2, 33), rng.choice(["unit", "mixture"])
        else:
            p, C, data = _log_int(rng, 16, 960), rng.randint(18, 33), "gauss"
        most = min(2000000, 90000000 // p)
        c = dict(data=data, n=_log_int(rng, max(500, min(most, 2 * p)), most), p=p, C=C)
        if rng.random() < 0.2:
            c["pad"] = rng.randint(1, 7)  # rows are a slice of a wider array
    c["op"] = op
    if op == "newton":
        c["newton"] = rng.randint(1, 3)
    if op in ("cg", "newton"):  # fewer than there are unknowns: the residual stays one
        c["cg"] = min(rng.randint(2, 4) if op == "cg" else rng.randint(3, 8), max(2, c["p"] * (c["C"] - 1) // 3))
    return c


# ---- inputs, from the seed alone ----

def _dense(case, gen):
    n, p, C = case["n"], case["p"], case["C"]
    wide = torch.empty((n, p + case.get("pad", 0)), device="cuda")
    if case["data"] == "image":  # values in [0, 1), four fifths of them zero
        wide.uniform_(0.0, 5.0, generator=gen)
        wide.mul_(wide < 1.0)
    else:  # columns of different scale
        wide.normal_(generator=gen)
        wide.mul_(torch.exp(torch.rand(wide.shape[1], generator=gen, device="cuda") * 2.3 - 1.15))
    A = wide[:, :p]
    if case["data"] in ("gauss", "image"):  # labels from a linear model, logits of order two
        W = torch.randn((p, C), generator=gen, device="cuda") * (2.0 / math.sqrt(p * (0.067 if case["data"] == "image" else 1.0)))
        u = torch.rand((n, C), generator=gen, device="cuda").clamp_(1e-7, 1.0 - 1e-7)
        labels = torch.argmax(A @ W - torch.log(-torch.log(u)), 1).int()
    else:                                   # a mean for every class
        labels = torch.randint(0, C, (n,), generator=gen, device="cuda", dtype=torch.int32)
        means = torch.randn((C, p), generator=gen, device="cuda") * (0.5 if case["data"] == "unit" else math.sqrt(0.1))
        for r0 in range(0, n, 16384):
            A[r0:r0 + 16384] += means[labels[r0:r0 + 16384].long()]
        if case["data"] == "unit":
            A /= torch.linalg.vector_norm(A, dim=1, keepdim=True)
    return A, labels


def _counts(case, gen):
    """Positions with replacement from log-normal column weights, repeats merged; values log(1 + k) of geometric counts.
    Both compressed views, entries in order."""
    n, p = case["n"], case["p"]
    labels = torch.randint(0, case["C"], (n,), generator=gen, device="cuda", dtype=torch.int32)
    w = torch.exp(2.0 * torch.randn(p, generator=gen, device="cuda", dtype=torch.float64))
    cdf = torch.cumsum(w / w.sum(), 0)
    total = n * case["per_row"]
    keys = []
    for k0 in range(0, total, 1 << 24):
        m = min(1 << 24, total - k0)
        cols = torch.searchsorted(cdf, torch.rand(m, generator=gen, device="cuda", dtype=torch.float64)).clamp_(max=p - 1)
        keys.append(torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int64) * p + cols)
    key = torch.unique(torch.cat(keys))
    del keys
    rows, cols = torch.div(key, p, rounding_mode="floor"), key % p
    u = torch.rand(key.numel(), generator=gen, device="cuda").clamp_(min=1e-7)
    val = torch.log1p(torch.floor(torch.log2(1.0 / u)) + 1.0)
    order = torch.sort(cols * n + rows)[1]

    def pointers(idx, m):
        ptr = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
        ptr[1:] = torch.cumsum(torch.bincount(idx, minlength=m), 0)
        return ptr

    A = nadmm.SparseA(n, p, pointers(rows, n), cols.int(), val, pointers(cols, p), rows[order].int(), val[order])
    return A, labels


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    sparse = case["data"] == "counts"
    A, labels = _counts(case, gen) if sparse else _dense(case, gen)
    d = (case["p"], case["C"] - 1)
    # a point whose logits are of order one (rows have length 1, 0.26 sqrt(p) or about sqrt(p))
    length = {"unit": 0.3, "image": 0.26 * math.sqrt(case["p"]), "counts": 1.4 * math.sqrt(case.get("per_row", 1))}
    X = torch.randn(d, generator=gen, device="cuda") / length.get(case["data"], math.sqrt(case["p"]))
    z = 0.3 * torch.randn(d, generator=gen, device="cuda") / length.get(case["data"], math.sqrt(case["p"]))
    y = 0.1 * torch.randn(d, generator=gen, device="cuda") / length.get(case["data"], math.sqrt(case["p"]))
    V = torch.randn(d, generator=gen, device="cuda")
    return dict(A=A, labels=labels, X=X, z=z, y=y, V=V)


LAM, RHO = 1e-3, 1.0


def _direction(case, t):
    """What CG and the line search are given: the gradient at X, and a descent direction long enough that the full
    step is not taken."""
    P = _Plain(case, t)
    _, g = P.loss_grad(t["X"].double())
    length = 3.0 * math.sqrt(case["p"]) if case["data"] != "unit" else 400.0
    return g.float(), (-length * g / torch.linalg.vector_norm(g)).float()


def prepare(case, seed):
    t = _inputs(case, seed)
    n, C, op = case["n"], case["C"], case["op"]
    state = dict(case=case, t=t)
    if op == "admm":
        N = case["workers"]
        cut = [n * i // N for i in range(N + 1)]
        state["workers"] = [nadmm.Problem(t["A"][cut[i]:cut[i + 1]], t["labels"][cut[i]:cut[i + 1]], C, 1.0 / n, 0.0, RHO)
                            for i in range(N)]
        state["params"] = nadmm.make_admm_params(case["outer"], nadmm.make_params(case["newton"], case["cg"], MAX_LS,
                                                                                  0.0, 0.0, BETA, GAMMA))
        need = nadmm.nadmm_admm_workspace_bytes(state["workers"], state["params"])
        state["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        state["x"] = t["X"].expand(N, *t["X"].shape).contiguous()
        return state
    prob = state["prob"] = nadmm.Problem(t["A"], t["labels"], C, 1.0 / n, LAM, RHO, t["z"], t["y"])
    if op == "newton":
        state["params"] = nadmm.make_params(case["newton"], case["cg"], MAX_LS, 0.0, 0.0, BETA, GAMMA)
        prob.workspace(state["params"])
    else:
        prob.workspace()
    if op in ("cg", "search"):
        state["g"], state["step"] = _direction(case, t)
    return state


def run(state):
    case, t = state["case"], state["t"]
    op = case["op"]
    if op == "admm":
        x = state["x"].clone()
        z, u, _ = nadmm.nadmm_admm_solve(state["workers"], LAM, x, state["params"], want_stats=False, ws=state["ws"])
        return x, z, u
    prob = state["prob"]
    if op == "hessvec":
        return nadmm.nadmm_hessvec(prob, t["X"], t["V"])
    if op == "grad":
        return nadmm.nadmm_loss_grad(prob, t["X"])
    if op == "cg":
        return nadmm.nadmm_cg_solve(prob, t["X"], state["g"], case["cg"], 0.0)
    if op == "search":
        return nadmm.nadmm_line_search(prob, t["X"], state["step"], state["g"], beta=BETA, gamma=GAMMA, max_ls=MAX_LS)
    X = t["X"].clone()
    nadmm.nadmm_local_newton(prob, X, state["params"], want_stats=False)
    return X


# ---- what a pass cannot do without ----

def work(case):
    n, p, NC, op = case["n"], case["p"], case["C"] - 1, case["op"]
    if case["data"] == "counts":
        # positions drawn with replacement: about a tenth of them are merged (at the full size 73.6 of 81.3 million stay)
        entries = 0.905 * n * case["per_row"]
        once = 8.0 * entries + 8.0 * (n + 1)
    else:
        entries = float(n) * p
        once = 4.0 * entries
    vec = 4.0 * p * NC
    product = 2.0 * entries * NC
    if op == "hessvec":   # A V and A^T D, and the probabilities from A X
        return {"bytes": once + 3 * vec, "flops": 3 * product}
    if op == "grad":
        return {"bytes": once + 4.0 * n + 4 * vec, "flops": 2 * product}
    if op == "cg":        # one pass over A for each iteration; A X once
        return {"bytes": case["cg"] * once + 3 * vec, "flops": (2 * case["cg"] + 1) * product}
    if op == "search":    # A X and A p in one pass
        return {"bytes": once + 4.0 * n + 5 * vec, "flops": 2 * product}
    # a Newton iteration: one pass for the gradient, one for each CG iteration (A p is a sum of the A d of those)
    passes = case["newton"] * (case["cg"] + 1) * case.get("outer", 1)
    return {"bytes": passes * once + 4.0 * n + 4 * vec * case.get("workers", 1), "flops": 2 * passes * product}


def tolerance(case):
    """About four times the largest error against `exact` over several hundred drawn cases: float32 sums of products whose
    factors carry 16 or more bits (A V, A^T D) or 24 (A X).  A CG solve also returns the norm of its residual, whose error
    is that of the residual itself, a difference of larger vectors."""
    return {"hessvec": {"rel": 2e-6}, "grad": {"rel": 2e-6}, "search": {"rel": 4e-6}, "cg": {"rel": 3e-4},
            "newton": {"rel": 1e-4}, "admm": {"rel": 2e-5}}[case["op"]]


# ---- the same in 64 bits, with plain torch ----

class _Plain:
    def __init__(self, case, t, rows=slice(None), s=None, lam=LAM, rho=RHO, z=None, y=None):
        self.sparse = case["data"] == "counts"
        self.A = t["A"] if self.sparse else t["A"][rows]
        self.b, self.C = t["labels"][rows].long(), case["C"]
        self.s, self.lam, self.rho = 1.0 / case["n"] if s is None else s, lam, rho
        self.z = t["z"].double() if z is None else z
        self.y = t["y"].double() if y is None else y
        if self.sparse:
            ptr, self.col, self.val = self.A.tensors[0], self.A.tensors[1].long(), self.A.tensors[2].double()
            self.row = torch.repeat_interleave(torch.arange(case["n"], device="cuda"), ptr[1:] - ptr[:-1])
        else:
            self.chunk = max(1, (1 << 26) // case["p"])

    def mul(self, X):      # A X
        if not self.sparse:
            return torch.cat([self.A[r:r + self.chunk].double() @ X for r in range(0, self.A.shape[0], self.chunk)])
        out = torch.zeros((self.A.shape[0], X.shape[1]), dtype=torch.float64, device="cuda")
        return self._scatter(out, self.row, self.col, X)

    def tmul(self, D):     # A^T D
        out = torch.zeros((self.A.shape[1], D.shape[1]), dtype=torch.float64, device="cuda")
        if not self.sparse:
            for r in range(0, self.A.shape[0], self.chunk):
                out += self.A[r:r + self.chunk].double().T @ D[r:r + self.chunk]
            return out
        return self._scatter(out, self.col, self.row, D)

    def _scatter(self, out, to, of, B):
        for k in range(0, self.val.numel(), 1 << 22):
            e = slice(k, k + (1 << 22))
            out.index_add_(0, to[e], self.val[e, None] * B[of[e]])
        return out

    def probs(self, Z):
        M = Z.max(1, keepdim=True)[0].clamp_(min=0.0)
        E = torch.exp(Z - M)
        alpha = E.sum(1, keepdim=True) + torch.exp(-M)
        return E / alpha, (M + torch.log(alpha))[:, 0]

    def _mine(self):
        return (torch.arange(self.C - 1, device="cuda")[None, :] == self.b[:, None]).double()

    def loss_at(self, Z, X):
        _, lse = self.probs(Z)
        u = X - self.z + self.y / self.rho
        return self.s * (lse - (Z * self._mine()).sum(1)).sum() + 0.5 * self.lam * (X * X).sum() + 0.5 * self.rho * (u * u).sum()

    def loss_grad(self, X):
        Z = self.mul(X)
        P, _ = self.probs(Z)
        g = self.s * self.tmul(P - self._mine()) + self.lam * X + self.rho * (X - self.z) + self.y
        return self.loss_at(Z, X), g

    def hessvec(self, P, V):
        T = P * self.mul(V)
        return self.s * self.tmul(T - P * T.sum(1, keepdim=True)) + (self.lam + self.rho) * V

    def cg(self, X, g, iters):
        P, _ = self.probs(self.mul(X))
        p, r, d = torch.zeros_like(g), -g, -g
        rr = (r * r).sum()
        gg = rr.clone()
        for _ in range(iters):
            q = self.hessvec(P, d)
            a = rr / (d * q).sum()
            p = p + a * d
            r = r - a * q
            new = (r * r).sum()
            d = r + (new / rr) * d
            rr = new
        return p, torch.sqrt(rr / gg)

    def search(self, X, p, g):
        Z, W = self.mul(X), self.mul(p)
        f0, slope, a = self.loss_at(Z, X), (p * g).sum(), 1.0
        for k in range(MAX_LS + 2):
            f = self.loss_at(Z + a * W, X + a * p)
            if bool(f <= f0 + a * BETA * slope):
                return a, f, 1
            if k == MAX_LS + 1:
                return a, f, 0
            a *= GAMMA

    def newton(self, X, newton, cg):
        for _ in range(newton):
            _, g = self.loss_grad(X)
            p, _ = self.cg(X, g, cg)
            X = X + self.search(X, p, g)[0] * p
        return X


def exact(case, seed):
    t = _inputs(case, seed)
    op, X = case["op"], t["X"].double()
    if op == "admm":
        N, n = case["workers"], case["n"]
        cut = [n * i // N for i in range(N + 1)]
        x, u = X.expand(N, *X.shape).clone(), torch.zeros((N, *X.shape), dtype=torch.float64, device="cuda")
        z = torch.zeros_like(X)
        for _ in range(case["outer"]):
            for i in range(N):
                W = _Plain(case, t, slice(cut[i], cut[i + 1]), 1.0 / n, 0.0, RHO, z, u[i])
                x[i] = W.newton(x[i], case["newton"], case["cg"])
            z = (RHO * x + u).sum(0) / (LAM + N * RHO)
            u = u + RHO * (x - z)
        return x, z, u
    P = _Plain(case, t)
    if op == "hessvec":
        return P.hessvec(P.probs(P.mul(X))[0], t["V"].double())
    if op == "grad":
        return P.loss_grad(X)
    if op == "newton":
        return P.newton(X, case["newton"], case["cg"])
    g, step = _direction(case, t)
    if op == "cg":
        p, relres = P.cg(X, g.double(), case["cg"])
        return p, torch.tensor(case["cg"], dtype=torch.int32), relres
    a, f, ok = P.search(X, step.double(), g.double())
    return torch.tensor(a, dtype=torch.float64), f, torch.tensor(ok, dtype=torch.int32)
