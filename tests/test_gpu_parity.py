"""GPU parity: every entry point of the C ABI against the float64 CPU oracle,
element by element, on the same seeded inputs.

Tolerances (the benchmark spec): loss, gradient and Hessian-vector product within 1e-4
relative (L2) error; Newton-CG iterates after the fixed iteration budget within
1e-3.  Step sizes and iteration counts are integers decided by floating-point
comparisons: both sides must agree unless the comparison is a tie (see
parity_utils.oracle_newton_following).
"""
import dataclasses
import math

import numpy as np
import pytest
import scipy.sparse as sp
import torch

from oracle import nadmm_oracle as orc
from paper_1807_07132_amd import nadmm, workloads
from parity_utils import TOL_ITERATE, TOL_PRIMITIVE, oracle_newton_following, oracle_problem, rel_abs, rel_l2

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.detach().cpu().numpy()


# (name, workload factory): sizes span several row tiles and column tiles with ragged tails
CASES = {
    "tiny": lambda: workloads.tiny(0),
    "image_like_3k": lambda: workloads.image_like(0, n=3111),
    "wide_700": lambda: workloads.wide(0, n=700),
    "tall_binary_50k": lambda: workloads.tall_binary(0, n=50021),
    "large_multiclass_900": lambda: workloads.large_multiclass(0, n=900),
    "ragged_1237x45_C5": lambda: workloads.generic(1237, 45, 5, seed=3),
    "ragged_333x130_C12": lambda: workloads.generic(333, 130, 12, seed=4, mean=True),
    "ragged_517x65_C3": lambda: workloads.generic(517, 65, 3, seed=5),
    "max_classes_200x33_C33": lambda: workloads.generic(200, 33, 33, seed=6, x_std=0.1),
    "single_row_1x7_C4": lambda: workloads.generic(1, 7, 4, seed=7),
    "single_feature_300x1_C2": lambda: workloads.generic(300, 1, 2, seed=8),
    "rows_64": lambda: workloads.generic(64, 32, 3, seed=9),
    "rows_65": lambda: workloads.generic(65, 33, 3, seed=10),
    # shapes the fused single-pass kernel takes (row stride a multiple of 4, C-1 <= 16, p <= 960)
    "fused_2000x100_C7": lambda: workloads.generic(2000, 100, 7, seed=12),
    "fused_9001x260_C10": lambda: workloads.generic(9001, 260, 10, seed=13, mean=True),
    "fused_4100x36_C17": lambda: workloads.generic(4100, 36, 17, seed=14, x_std=0.2),
    "fused_130x960_C4": lambda: workloads.generic(130, 960, 4, seed=15, x_std=0.05),
    "fused_8200x64_C2": lambda: workloads.generic(8200, 64, 2, seed=16),
    # rows that are not 16-byte aligned (odd p, lda = p) on the matrix-core paths: their any-stride instantiations
    "fused_any_3000x785_C10": lambda: workloads.generic(3000, 785, 10, seed=41, x_std=0.03, mean=True),
    "sliced_any_700x1101_C4": lambda: workloads.generic(700, 1101, 4, seed=42, x_std=0.05),
    # shapes the thin-data kernel takes (p <= 32, p % 4 == 0, C-1 <= 3, contiguous rows)
    "thin_5000x4_C2": lambda: workloads.generic(5000, 4, 2, seed=17),
    "thin_70001x32_C3": lambda: workloads.generic(70001, 32, 3, seed=18, mean=True),
    "thin_300x12_C4": lambda: workloads.generic(300, 12, 4, seed=19),
    "thin_256x8_C2": lambda: workloads.generic(256, 8, 2, seed=20),
    # shapes the column-sliced two-sweep path takes (p > 960 or C-1 > 16, row stride a multiple of 4)
    "sliced_3000x100_C26": lambda: workloads.generic(3000, 100, 26, seed=24, x_std=0.1),
    "sliced_1500x1100_C4": lambda: workloads.generic(1500, 1100, 4, seed=25, x_std=0.05),
    "sliced_33x1604_C33": lambda: workloads.generic(33, 1604, 33, seed=26, x_std=0.03),
    "sliced_300x36_C33": lambda: workloads.generic(300, 36, 33, seed=27, x_std=0.2),    # 32 free classes: two full class blocks
    "sliced_200x964_C3": lambda: workloads.generic(200, 964, 3, seed=28, x_std=0.05),  # one step past the fused kernel's limit
    # several tiles per workgroup and column slice in sweep 1 (row ranges of 79 and 36 rows cut into equal tiles of 27 and 18)
    "sliced_20000x1100_C4": lambda: workloads.generic(20000, 1100, 4, seed=43, x_std=0.05),
    "sliced_9000x200_C20": lambda: workloads.generic(9000, 200, 20, seed=44, x_std=0.1),
    # the same with rows that are only 4-byte aligned, and a shape whose logits Z and W of 1/256 of the rows do not fit the LDS
    # together (32 free classes, 100000 rows: sweep 1 then runs on 512 row ranges)
    "sliced_any_9000x1101_C4": lambda: workloads.generic(9000, 1101, 4, seed=45, x_std=0.05),
    "sliced_100000x36_C33": lambda: workloads.generic(100000, 36, 33, seed=46, x_std=0.2),
    # d = p (C-1) = 280000: the long-vector forms of the reduction, the CG update and the line-search tail
    "long_vectors_40x70000_C5": lambda: workloads.generic(40, 70000, 5, seed=29, x_std=0.01, mean=True),
}

# 1 = two-pass vector kernels forced, 2 = fused matrix-core kernel forced, 4 = column-sliced two-sweep path forced,
# 0 = automatic (the thin-data path is the automatic choice wherever it applies)
PATHS = [1, 2, 4, 0]


@pytest.fixture(scope="module")
def cache():
    return {}


def setup_case(cache, name):
    if name not in cache:
        w = CASES[name]()
        cache[name] = (w, nadmm.Problem.from_workload(w), oracle_problem(w))
    return cache[name]


def force_path(gp, path):
    """Select a kernel path; skip the test if this problem's shape is outside that path's limits."""
    nadmm.nadmm_set_kernel_path(path)
    try:
        nadmm.nadmm_query_kernel_path(gp)
    except nadmm.NadmmError as e:
        assert e.code == nadmm.NADMM_EUNSUPPORTED
        pytest.skip("shape outside the limits of the forced kernel path")


@pytest.fixture(autouse=True)
def _reset_path():
    yield
    nadmm.nadmm_set_kernel_path(0)


def x_for(w):
    X = w.X0
    if not X.any():
        X = (np.random.default_rng(11).standard_normal(X.shape) * 0.2).astype(np.float32)
    return X


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("name", list(CASES))
def test_loss_and_gradient(cache, name, path):
    w, gp, op = setup_case(cache, name)
    force_path(gp, path)
    for X in (x_for(w), np.zeros_like(w.X0)):
        loss, grad = nadmm.nadmm_loss_grad(gp, dev(X))
        loss_only, none = nadmm.nadmm_loss_grad(gp, dev(X), want_grad=False)
        assert none is None
        f_ref, g_ref = orc.loss_grad(op, X)
        assert rel_abs(loss.item(), f_ref) <= TOL_PRIMITIVE
        assert rel_abs(loss_only.item(), f_ref) <= TOL_PRIMITIVE
        assert rel_l2(host(grad), g_ref) <= TOL_PRIMITIVE


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("name", list(CASES))
def test_hessvec(cache, name, path):
    w, gp, op = setup_case(cache, name)
    force_path(gp, path)
    X = x_for(w)
    hv = nadmm.nadmm_hessvec(gp, dev(X), dev(w.V))
    assert rel_l2(host(hv), orc.hessvec(op, X, w.V)) <= TOL_PRIMITIVE
    # bit-identical on repetition (fixed-order reductions)
    hv2 = nadmm.nadmm_hessvec(gp, dev(X), dev(w.V))
    assert torch.equal(hv, hv2)


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("name", ["tiny", "image_like_3k", "tall_binary_50k", "ragged_1237x45_C5", "ragged_333x130_C12",
                                  "fused_2000x100_C7", "fused_130x960_C4", "thin_5000x4_C2", "thin_256x8_C2", "sliced_1500x1100_C4",
                                  "sliced_33x1604_C33", "wide_700", "long_vectors_40x70000_C5", "fused_any_3000x785_C10",
                                  "sliced_any_700x1101_C4"])
def test_cg_fixed_iterations(cache, name, path):
    w, gp, op = setup_case(cache, name)
    force_path(gp, path)
    X = x_for(w)
    g_ref = orc.grad(op, X)
    g32 = g_ref.astype(np.float32)
    for K in (1, 5):
        p, iters, relres = nadmm.nadmm_cg_solve(gp, dev(X), dev(g32), K, 0.0)
        p_ref, k_ref, rel_ref = orc.cg(op, X, g32, K, 0.0)
        assert iters.item() == k_ref == K
        assert rel_l2(host(p), p_ref) <= TOL_ITERATE
        if rel_ref > 1e-5:
            assert relres.item() == pytest.approx(rel_ref, rel=5e-3)
        else:                               # converged to rounding level: only the level is comparable
            assert relres.item() < 1e-5


# The sums over d of a line search on vectors of more than 8192 elements: one element beyond, whole and part chunks of 2048, more than 256
# of them, and no z or y.
@pytest.mark.parametrize("missing", ["", "z", "y", "zy"])
@pytest.mark.parametrize("p,C", [(8193, 2), (3072, 5), (2341, 6), (65537, 9)])
def test_line_search_on_long_vectors(p, C, missing):
    w = workloads.generic(24, p, C, seed=p + C, x_std=0.5 / math.sqrt(p), mean=True)
    z = None if "z" in missing else w.z
    y = None if "y" in missing else w.y
    op = orc.Problem(w.A, w.b, w.C, s=w.s, lam=0.3, rho=0.2, z=z, y=y)
    gp = nadmm.Problem(dev(w.A), dev(w.b), w.C, w.s, 0.3, 0.2, None if z is None else dev(z), None if y is None else dev(y))
    g = orc.grad(op, w.X0)
    for scale in (1.0, 3000.0):
        d = (-scale * g).astype(np.float32)
        g32 = g.astype(np.float32)
        a_ref, f_ref, ok_ref, _ = orc.line_search(op, w.X0, d, g32, w.beta, w.gamma, 20)
        alpha, f_new, ok = nadmm.nadmm_line_search(gp, dev(w.X0), dev(d), dev(g32), math.nan, w.beta, w.gamma, 20)
        assert alpha.item() == pytest.approx(a_ref, rel=1e-6) and bool(ok.item()) == ok_ref
        assert rel_abs(f_new.item(), f_ref) <= TOL_PRIMITIVE


@pytest.mark.parametrize("name", ["tiny", "ragged_1237x45_C5"])
def test_cg_tolerance_mode(cache, name):
    w, gp, op = setup_case(cache, name)
    X = x_for(w)
    g32 = orc.grad(op, X).astype(np.float32)
    for tol in (1e-3, 1e-4):
        p, iters, relres = nadmm.nadmm_cg_solve(gp, dev(X), dev(g32), 60, tol)
        p_ref, k_ref, _ = orc.cg(op, X, g32, 60, tol)
        k = iters.item()
        assert 0 < k < 60 and abs(k - k_ref) <= 1
        # eq. (inexact), checked with the oracle's Hessian on the GPU's direction
        res = np.linalg.norm(orc.hessvec(op, X, host(p)) + g32) / np.linalg.norm(g32)
        assert res <= tol * 1.05
        if k == k_ref:
            assert rel_l2(host(p), p_ref) <= TOL_ITERATE
    # zero right-hand side: zero iterations, zero direction
    p, iters, _ = nadmm.nadmm_cg_solve(gp, dev(X), dev(np.zeros_like(g32)), 5, 0.0)
    assert iters.item() == 0 and not host(p).any()


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("name", ["tiny", "image_like_3k", "tall_binary_50k", "ragged_517x65_C3", "fused_8200x64_C2",
                                  "thin_70001x32_C3", "sliced_3000x100_C26", "long_vectors_40x70000_C5"])
def test_line_search(cache, name, path):
    w, gp, op = setup_case(cache, name)
    force_path(gp, path)
    X = x_for(w)
    g = orc.grad(op, X)
    for scale, max_ls in ((1.0, 10), (30.0, 10), (3000.0, 20), (-1.0, 4), (-1.0, 0)):
        p = (-scale * g).astype(np.float32)      # scale < 0: ascent direction, Armijo can never hold
        g32 = g.astype(np.float32)
        a_ref, f_ref, ok_ref, _ = orc.line_search(op, X, p, g32, w.beta, w.gamma, max_ls)
        for f0 in (math.nan, orc.loss(op, X)):
            alpha, f_new, ok = nadmm.nadmm_line_search(gp, dev(X), dev(p), dev(g32), f0, w.beta, w.gamma, max_ls)
            assert alpha.item() == pytest.approx(a_ref, rel=1e-6)
            assert bool(ok.item()) == ok_ref
            assert rel_abs(f_new.item(), f_ref) <= TOL_PRIMITIVE


# The line search evaluated by the sweep itself (up to 16 step sizes with the one for F(X)) and, from 17 on, by a kernel on stored
# logits.  Path 2: one and several tiles of 32 rows with remainders, one and several column steps, 1, 9 and 16 class lanes, any stride.
# Path 3: part of a chunk of 64 rows, one and several chunks per wave, rows of quads and others, 1 to 3 free classes.
@pytest.mark.parametrize("n,p,C,path", [(1, 20, 2, 2), (33, 129, 10, 2), (8193, 260, 10, 2), (8450, 785, 17, 2), (300, 960, 3, 2), (9001, 100, 17, 2),
                                        (50, 8, 2, 3), (2049, 29, 2, 3), (16385, 7, 4, 3), (70001, 32, 2, 3), (262209, 20, 4, 3)])
def test_line_search_in_the_sweep(n, p, C, path):
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / math.sqrt(p), mean=True)
    gp, op = nadmm.Problem.from_workload(w), oracle_problem(w)
    force_path(gp, path)
    f0, g = orc.loss(op, w.X0), orc.grad(op, w.X0)
    g32 = g.astype(np.float32)
    for scale, max_ls in ((1.0, 10), (40.0, 13), (40.0, 14), (4000.0, 15), (-1.0, 13), (-1.0, 0)):
        pdir = (-scale * g).astype(np.float32)
        a_ref, f_ref, ok_ref, _ = orc.line_search(op, w.X0, pdir, g32, 1e-4, 0.5, max_ls)
        for given in (math.nan, f0):
            alpha, f_new, ok = nadmm.nadmm_line_search(gp, dev(w.X0), dev(pdir), dev(g32), given, 1e-4, 0.5, max_ls)
            assert alpha.item() == a_ref and bool(ok.item()) == ok_ref
            # the losses here are mostly the step's own logits: the product A p in three terms (relative error below 4 * 2^-17) on path 2,
            # float32 sums of at most 32 products on path 3, some of whose 33 roundings of 2^-24 add up
            assert rel_abs(f_new.item(), f_ref) <= (4 * 2.0 ** -17 if path == 2 else 33 * 2.0 ** -24)
    # a Newton iteration with as many step sizes as the pass that forms A p evaluates, and with two more (on path 3 that pass takes more than
    # 2048 rows: fewer are solved in one launch, which tries the step sizes in turn)
    for max_ls in (13, 15):
        X = dev(w.X0)
        st = nadmm.nadmm_local_newton(gp, X, nadmm.make_params(2, 3, max_ls))
        w.max_newton, w.max_cg, w.max_ls = 2, 3, max_ls
        assert rel_l2(host(X), oracle_newton_following(op, w.X0, w, st["alpha"])[0]) <= TOL_ITERATE


# A direction along which one row's logit overflows: its loss is NaN where that logit is +inf, on every path, and a step size with it is taken
# (Algorithm 2's test does not fail against NaN).  Path 1 evaluates stored logits.
@pytest.mark.parametrize("label", ["first", "reference"])
@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("n,p,C", [(3000, 28, 2), (2500, 29, 2), (50, 8, 2), (3000, 12, 4)])
def test_line_search_where_a_logit_overflows(n, p, C, sign, label):
    w = workloads.generic(n, p, C, seed=n + p)
    w.A[n // 2, :2] = 4.0
    w.b[n // 2] = 0 if label == "first" else C - 1
    X, pdir = np.zeros_like(w.X0), np.zeros_like(w.X0)
    pdir[:2, 0] = sign * 6e37                  # 2 * 4 * 6e37 is beyond float32
    w.A[np.arange(n) != n // 2, :2] = 0.0
    gp = nadmm.Problem.from_workload(w)
    got = {}
    for path in (3, 1):
        force_path(gp, path)
        for f0 in (0.0, 1e80):                 # below and above what the penalty adds
            got[path, f0] = [v.item() for v in nadmm.nadmm_line_search(gp, dev(X), dev(pdir), dev(X), f0, 1e-4, 0.5, 3)]
    for f0 in (0.0, 1e80):
        assert got[3, f0] == pytest.approx(got[1, f0], rel=1e-6, nan_ok=True), f0
        assert math.isnan(got[1, f0][1]) == (sign > 0)


NEWTON_CASES = ["tiny", "image_like_3k", "wide_700", "tall_binary_50k", "large_multiclass_900", "ragged_1237x45_C5",
                "fused_any_3000x785_C10", "sliced_any_700x1101_C4",
                "single_row_1x7_C4", "fused_9001x260_C10", "fused_4100x36_C17", "thin_70001x32_C3", "thin_300x12_C4", "sliced_3000x100_C26",
                "sliced_1500x1100_C4", "sliced_20000x1100_C4", "sliced_9000x200_C20", "sliced_any_9000x1101_C4", "sliced_100000x36_C33",
                "long_vectors_40x70000_C5"]


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("name", NEWTON_CASES)
def test_local_newton(cache, name, path):
    w, gp, op = setup_case(cache, name)
    force_path(gp, path)
    T = min(w.max_newton, 4)
    K = min(w.max_cg, 10)
    params = nadmm.make_params(T, K, w.max_ls, 0.0, 0.0, w.beta, w.gamma)
    X = dev(w.X0.copy())
    st = nadmm.nadmm_local_newton(gp, X, params)
    w2 = dataclasses.replace(w, max_cg=K)
    X_ref, st_ref, _ = oracle_newton_following(op, w.X0, w2, st["alpha"], max_newton=T)
    assert st["newton_iters"] == st_ref["newton_iters"] == T
    assert st["cg_iters_total"] == st_ref["cg_iters_total"]
    assert st["alpha"] == pytest.approx([it["alpha"] for it in st_ref["iters"]], rel=1e-6)
    assert rel_l2(host(X), X_ref) <= TOL_ITERATE
    assert rel_abs(st["loss_initial"], st_ref["loss_initial"]) <= TOL_PRIMITIVE
    assert rel_abs(st["loss_final"], st_ref["loss_final"]) <= TOL_PRIMITIVE
    assert st["loss"] == pytest.approx([it["loss"] for it in st_ref["iters"]], rel=TOL_PRIMITIVE)
    # whether the i_max break was taken is decided by comparisons of objective values; where the predicted
    # decrease <p,g> is below the float32 resolution of the objective the decision is noise on both sides
    ties = [it for it in st_ref["iters"] if abs(float(np.sum(it["p"] * it["g"]))) <= 1e-6 * max(1.0, abs(it["loss"]))]
    assert abs(st["armijo_failed"] - st_ref["armijo_failed"]) <= len(ties), (
        st, [(it["alpha"], it["armijo_ok"], it["loss"], it["grad_norm"]) for it in st_ref["iters"]])


# (case, CG iterations, theta, bound on the iterates).  8, 12, 16 or 32 history buffers go into one launch.
# fused_130x960_C4 has 130 rows for 2880 unknowns: float32 CG loses conjugacy there after some 16 iterations and the
# iterates leave the float64 oracle's by 1.3e-2 (measured, the same with and without the history); the bound says so.
HISTORY_CASES = [("image_like_3k", 12, 0.0, TOL_ITERATE), ("image_like_3k", 12, 3e-2, TOL_ITERATE), ("wide_700", 12, 0.0, TOL_ITERATE),
                 ("image_like_3k", 20, 0.0, TOL_ITERATE), ("image_like_3k", 29, 0.0, TOL_ITERATE),
                 ("fused_130x960_C4", 1, 0.0, TOL_ITERATE), ("fused_130x960_C4", 2, 0.0, TOL_ITERATE),
                 ("fused_130x960_C4", 5, 0.0, TOL_ITERATE), ("fused_130x960_C4", 12, 3e-2, TOL_ITERATE),
                 ("fused_130x960_C4", 16, 0.0, TOL_ITERATE), ("fused_130x960_C4", 32, 0.0, 3e-2)]


@pytest.mark.parametrize("name,K,cg_tol,bound", HISTORY_CASES)
def test_local_newton_with_and_without_the_history_of_directional_logits(cache, name, K, cg_tol, bound):
    """A workspace sized for the solve's parameters lets the fused path put A p together from the A d_k its CG sweeps
    leave behind (p = sum_k alpha_k d_k) instead of another pass over A; one sized without parameters takes that
    pass.  Both must follow the oracle, also when CG stops early and leaves part of the history unused."""
    w, gp, op = setup_case(cache, name)
    force_path(gp, 2)
    T = 3
    params = nadmm.make_params(T, K, w.max_ls, cg_tol, 0.0, w.beta, w.gamma)
    small, large = nadmm.nadmm_workspace_bytes(gp), nadmm.nadmm_workspace_bytes(gp, params)
    assert large >= small + K * w.n * (w.C - 1) * 4      # this shape qualifies for the history
    w2 = dataclasses.replace(w, max_cg=K, cg_tol=cg_tol)
    out = []
    for nbytes in (small, large):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        ws.fill_(0xFF)                                   # NaN patterns: nothing may be read before it is written
        X = dev(w.X0.copy())
        st = nadmm.nadmm_local_newton(gp, X, params, ws=ws)
        X_ref, st_ref, _ = oracle_newton_following(op, w.X0, w2, st["alpha"], max_newton=T)
        assert st["newton_iters"] == T
        assert st["cg_iters"] == [it["cg_iters"] for it in st_ref["iters"]]
        if cg_tol > 0 and name == "image_like_3k":
            assert min(st["cg_iters"]) < K               # the early stop is really exercised
        assert st["alpha"] == pytest.approx([it["alpha"] for it in st_ref["iters"]], rel=1e-6)
        assert rel_l2(host(X), X_ref) <= bound
        if bound == TOL_ITERATE:
            assert rel_abs(st["loss_final"], st_ref["loss_final"]) <= TOL_PRIMITIVE
        out.append((host(X), st))
    assert out[0][1]["alpha"] == out[1][1]["alpha"]
    assert rel_l2(out[0][0], out[1][0]) <= 1e-4


@pytest.mark.parametrize("path,grad_tol", [(1, 1e-4), (2, 2e-3)])
def test_local_newton_stops_on_gradient_tolerance(cache, path, grad_tol):
    """Stopping test of Algorithm 3.  ||g|| is 585 at the start; close to the minimiser the gradient is a small difference
    of large sums, so the tolerance that can be met depends on the products' accuracy: 1e-4 on the fp32 vector kernels,
    while the matrix-core kernels stall at 2e-4 .. 4e-4 and are asked for 2e-3."""
    w, gp, op = setup_case(cache, "ragged_1237x45_C5")
    force_path(gp, path)
    params = nadmm.make_params(30, 50, 10, 1e-6, grad_tol, w.beta, w.gamma)
    X = dev(w.X0.copy())
    st = nadmm.nadmm_local_newton(gp, X, params)
    assert 0 < st["newton_iters"] < 30
    assert st["grad_norm_final"] < grad_tol
    g = orc.grad(op, host(X))
    assert np.linalg.norm(g) < 2 * grad_tol
    # the minimiser is unique: compare with the oracle run to convergence
    X_ref, _ = orc.local_newton(op, w.X0, 50, 200, 1e-10, 1e-10, w.beta, w.gamma, 10)
    assert rel_l2(host(X), X_ref) <= TOL_ITERATE * (1 if path == 1 else 5)
    # warm start at the solution: no iteration is taken
    st2 = nadmm.nadmm_local_newton(gp, X, params)
    assert st2["newton_iters"] == 0


def test_sum_scaling_and_missing_z_y(cache):
    w = workloads.generic(700, 40, 6, seed=21)
    op = orc.Problem(w.A, w.b, w.C, s=1.0, lam=0.5, rho=2.0)
    gp = nadmm.Problem(dev(w.A), dev(w.b), w.C, 1.0, 0.5, 2.0, None, None)
    X = w.X0
    loss, grad = nadmm.nadmm_loss_grad(gp, dev(X))
    assert rel_abs(loss.item(), orc.loss(op, X)) <= TOL_PRIMITIVE
    assert rel_l2(host(grad), orc.grad(op, X)) <= TOL_PRIMITIVE
    assert rel_l2(host(nadmm.nadmm_hessvec(gp, dev(X), dev(w.V))), orc.hessvec(op, X, w.V)) <= TOL_PRIMITIVE


@pytest.mark.parametrize("missing", ["", "z", "y", "zy"])
def test_vectors_that_are_only_4_byte_aligned(cache, missing):
    """X, z, y and the outputs may start at any multiple of 4 bytes; a missing z or y counts as zeros.  (The workgroup
    that finishes the objective beside the gradient's reduction reads them 16 bytes at a time where it can.)"""
    w = workloads.generic(700, 40, 6, seed=23)
    z = None if "z" in missing else w.z
    y = None if "y" in missing else w.y
    op = orc.Problem(w.A, w.b, w.C, s=w.s, lam=w.lam, rho=w.rho, z=z, y=y)

    def off(a, k):   # a device copy that starts k floats into a 256-byte aligned buffer
        if a is None:
            return None
        buf = torch.zeros(a.size + 8, dtype=torch.float32, device="cuda")
        view = buf[k:k + a.size].view(a.shape)
        view.copy_(torch.from_numpy(np.ascontiguousarray(a)))
        assert view.data_ptr() % 16 == (4 * k) % 16
        return view

    f_ref, g_ref = orc.loss_grad(op, w.X0)
    for kx, kz, ky in ((1, 2, 3), (0, 1, 0), (0, 0, 0)):
        gp = nadmm.Problem(dev(w.A), dev(w.b), w.C, w.s, w.lam, w.rho, off(z, kz), off(y, ky))
        X = off(w.X0, kx)
        grad_out = off(np.zeros_like(w.X0), 3)
        loss, grad = nadmm.nadmm_loss_grad(gp, X, grad_out=grad_out)
        assert rel_abs(loss.item(), f_ref) <= TOL_PRIMITIVE
        assert rel_l2(host(grad), g_ref) <= TOL_PRIMITIVE
        hv = nadmm.nadmm_hessvec(gp, X, off(w.V, 1))
        assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE


@pytest.mark.parametrize("stride", [64, 53])   # rows 16-byte aligned or not: every path applies either way
def test_row_stride_larger_than_p(cache, stride):
    w = workloads.generic(900, 50, 4, seed=22)
    op = oracle_problem(w)
    big = torch.zeros((w.n, stride), dtype=torch.float32, device="cuda")
    big[:, : w.p] = dev(w.A)
    big[:, w.p:] = float("nan")             # padding must never be read as data
    gp = nadmm.Problem(big[:, : w.p], dev(w.b), w.C, w.s, w.lam, w.rho, dev(w.z), dev(w.y))
    ran = 0
    for path in PATHS:
        nadmm.nadmm_set_kernel_path(path)
        nadmm.nadmm_query_kernel_path(gp)
        ran += 1
        loss, grad = nadmm.nadmm_loss_grad(gp, dev(w.X0))
        assert rel_abs(loss.item(), orc.loss(op, w.X0)) <= TOL_PRIMITIVE
        assert rel_l2(host(grad), orc.grad(op, w.X0)) <= TOL_PRIMITIVE
        assert rel_l2(host(nadmm.nadmm_hessvec(gp, dev(w.X0), dev(w.V))), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE
        params = nadmm.make_params(2, 5, w.max_ls, 0.0, 0.0, w.beta, w.gamma)
        X = dev(w.X0.copy())
        st = nadmm.nadmm_local_newton(gp, X, params)
        X_ref, st_ref, _ = oracle_newton_following(op, w.X0, dataclasses.replace(w, max_cg=5), st["alpha"], max_newton=2)
        assert rel_l2(host(X), X_ref) <= TOL_ITERATE
    assert ran == 4


@pytest.mark.parametrize("shape", [(400, 30, 5), (400, 32, 5), (700, 32, 3), (300, 1000, 4)])
def test_large_logits_do_not_overflow(cache, shape):
    """Logits far beyond the float32 range of exp() on every kernel path the shape admits (vector kernels,
    fused, thin-data, column-sliced): the log-sum-exp shift of Section 2.2 keeps loss and gradient finite."""
    n, p, C = shape
    w = workloads.generic(n, p, C, seed=23, scale=6.0, x_std=3.0 if p < 100 else 0.6)
    op = oracle_problem(w)
    assert np.abs(orc.logits(op, w.X0)).max() > 150
    gp = nadmm.Problem.from_workload(w)
    ran = 0
    for path in (1, 2, 3, 4, 0):
        nadmm.nadmm_set_kernel_path(path)
        try:
            nadmm.nadmm_query_kernel_path(gp)
        except nadmm.NadmmError:
            continue
        ran += 1
        loss, grad = nadmm.nadmm_loss_grad(gp, dev(w.X0))
        assert math.isfinite(loss.item()) and torch.isfinite(grad).all()
        assert rel_abs(loss.item(), orc.loss(op, w.X0)) <= TOL_PRIMITIVE
        assert rel_l2(host(grad), orc.grad(op, w.X0)) <= TOL_PRIMITIVE
        hv = nadmm.nadmm_hessvec(gp, dev(w.X0), dev(w.V))
        assert torch.isfinite(hv).all()
        # exp() turns the absolute error of a logit into a relative error of P, so logits of size 150 need the
        # full float32 accuracy of the product Z = A X: the matrix-core paths take that one product with
        # three bf16 parts per operand, and every path meets the bar of the primitives here too
        assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE
    assert ran >= 2


@pytest.mark.parametrize("shape", [(300, 64, 17), (2100, 200, 17), (500, 1000, 17)])
def test_all_logits_strongly_negative_with_16_free_classes(cache, shape):
    """C - 1 = 16 fills every lane of a 16-lane class group, so the 0 of M = max{0, Z_1..Z_{C-1}} (eq. max_x) has to be
    put in explicitly: with every free-class logit below -88, exp(-M) overflows without it and the row loss is infinite."""
    n, p, C = shape
    w = workloads.generic(n, p, C, seed=31, scale=1.0, x_std=1.0)
    A = np.abs(w.A) + 0.5                      # non-negative data
    X = ((-np.abs(w.X0) - 0.2) * (300.0 / p)).astype(np.float32)   # every weight negative: all logits near -400
    w = dataclasses.replace(w, A=A.astype(np.float32), X0=X)
    op = oracle_problem(w)
    Z = orc.logits(op, w.X0)
    assert Z.max() < -100
    gp = nadmm.Problem.from_workload(w)
    ran = 0
    for path in (1, 2, 4, 0):
        nadmm.nadmm_set_kernel_path(path)
        try:
            nadmm.nadmm_query_kernel_path(gp)
        except nadmm.NadmmError:
            continue
        ran += 1
        loss, grad = nadmm.nadmm_loss_grad(gp, dev(w.X0))
        assert math.isfinite(loss.item()) and torch.isfinite(grad).all()
        assert rel_abs(loss.item(), orc.loss(op, w.X0)) <= TOL_PRIMITIVE
        assert rel_l2(host(grad), orc.grad(op, w.X0)) <= TOL_PRIMITIVE
        hv = nadmm.nadmm_hessvec(gp, dev(w.X0), dev(w.V))
        assert torch.isfinite(hv).all()
        assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE
    assert ran >= 3


def test_non_default_stream(cache):
    w, gp, op = setup_case(cache, "ragged_1237x45_C5")
    s = torch.cuda.Stream()
    X, V = dev(w.X0), dev(w.V)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        hv = nadmm.nadmm_hessvec(gp, X, V, stream=s)
    s.synchronize()
    assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE


@pytest.mark.parametrize("sized_for_params", [False, True])
def test_local_newton_replays_from_a_hip_graph(cache, sized_for_params):
    """The whole local solve is enqueued without host synchronisation or allocation, so it can be captured
    once and replayed; every replay (with eager work in between) must give the eager result bit for bit.
    With a workspace sized for the parameters the solve keeps the directional logits of its CG sweeps (another
    set of kernels and launches)."""
    w, gp, op = setup_case(cache, "fused_2000x100_C7")
    params = nadmm.make_params(2, 5, w.max_ls, 0.0, 0.0, w.beta, w.gamma)
    nbytes = nadmm.nadmm_workspace_bytes(gp, params if sized_for_params else None)
    assert (nbytes > nadmm.nadmm_workspace_bytes(gp)) == sized_for_params
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    X0 = dev(w.X0.copy())
    X_eager = X0.clone()
    nadmm.nadmm_local_newton(gp, X_eager, params, want_stats=False, ws=ws)   # also the warm-up (kernel attributes)
    torch.cuda.synchronize()
    X = X0.clone()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            nadmm.nadmm_local_newton(gp, X, params, want_stats=False, ws=ws, stream=side)
    for _ in range(3):
        X.copy_(X0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(X, X_eager)
        hv = nadmm.nadmm_hessvec(gp, X0, dev(w.V), ws=ws)                      # eager work between the replays
        assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE


@pytest.mark.parametrize("shape", [(260, 64, 4), (300, 28, 2), (150, 1000, 3), (90, 21, 6)])
def test_degenerate_inputs(cache, shape):
    """All-zero data (every probability 1/C), one-class labels (reference class only / one free class only),
    zero direction, no regulariser: closed forms and the oracle on every kernel path the shape admits."""
    n, p, C = shape
    w = workloads.generic(n, p, C, seed=40)
    X, V = w.X0 if w.X0.any() else x_for(w), w.V
    variants = {
        "zero_data": (np.zeros_like(w.A), w.b),
        "reference_class_only": (w.A, np.full_like(w.b, C - 1)),
        "first_class_only": (w.A, np.zeros_like(w.b)),
    }
    for vname, (A, b) in variants.items():
        op = orc.Problem(A, b, C, s=w.s, lam=0.0, rho=w.rho, z=w.z, y=w.y)
        gp = nadmm.Problem(dev(A), dev(b), C, w.s, 0.0, w.rho, dev(w.z), dev(w.y))
        for path in (1, 2, 3, 4):
            nadmm.nadmm_set_kernel_path(path)
            try:
                nadmm.nadmm_query_kernel_path(gp)
            except nadmm.NadmmError:
                continue
            loss, grad = nadmm.nadmm_loss_grad(gp, dev(X))
            assert rel_abs(loss.item(), orc.loss(op, X)) <= TOL_PRIMITIVE, (vname, path)
            assert rel_l2(host(grad), orc.grad(op, X)) <= TOL_PRIMITIVE, (vname, path)
            hv = nadmm.nadmm_hessvec(gp, dev(X), dev(V))
            assert rel_l2(host(hv), orc.hessvec(op, X, V)) <= TOL_PRIMITIVE, (vname, path)
            if vname == "zero_data":     # H = rho I when A = 0 and lambda = 0
                assert rel_l2(host(hv), w.rho * V.astype(np.float64)) <= 1e-6
            hv0 = nadmm.nadmm_hessvec(gp, dev(X), dev(np.zeros_like(V)))
            assert not host(hv0).any()


def test_zero_iteration_budgets_and_longest_line_search(cache):
    w, gp, op = setup_case(cache, "ragged_1237x45_C5")
    X = x_for(w)
    g32 = orc.grad(op, X).astype(np.float32)
    # no CG iteration: the zero start is returned
    p, iters, relres = nadmm.nadmm_cg_solve(gp, dev(X), dev(g32), 0, 0.0)
    assert iters.item() == 0 and not host(p).any() and relres.item() == pytest.approx(1.0)
    # no Newton iteration: X untouched
    Xd = dev(X)
    st = nadmm.nadmm_local_newton(gp, Xd, nadmm.make_params(0, 5, w.max_ls, 0.0, 0.0, w.beta, w.gamma))
    assert st["newton_iters"] == 0 and np.array_equal(host(Xd), X)
    # Newton iterations without CG: p = 0, the step changes nothing
    st = nadmm.nadmm_local_newton(gp, Xd, nadmm.make_params(2, 0, w.max_ls, 0.0, 0.0, w.beta, w.gamma))
    assert st["newton_iters"] == 2 and st["cg_iters_total"] == 0 and np.array_equal(host(Xd), X)
    # the longest line search the library compiles for, on an ascent direction: i_max + 1 reductions, then the break
    max_ls = nadmm.NADMM_MAX_LS
    pdir = g32.copy()
    alpha, f_new, ok = nadmm.nadmm_line_search(gp, dev(X), dev(pdir), dev(g32), math.nan, w.beta, 0.9, max_ls)
    a_ref, f_ref, ok_ref, _ = orc.line_search(op, X, pdir, g32, w.beta, 0.9, max_ls)
    assert not ok.item() and not ok_ref
    assert alpha.item() == pytest.approx(0.9 ** (max_ls + 1), rel=1e-5) == pytest.approx(a_ref, rel=1e-5)
    assert rel_abs(f_new.item(), f_ref) <= TOL_PRIMITIVE


def test_two_streams_with_their_own_workspaces_do_not_interfere(cache):
    w1, gp1, op1 = setup_case(cache, "fused_2000x100_C7")
    w2, gp2, op2 = setup_case(cache, "ragged_1237x45_C5")
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    params = nadmm.make_params(2, 5, 10, 0.0, 0.0, 1e-4, 0.5)
    X1, X2 = dev(w1.X0.copy()), dev(w2.X0.copy())
    ref1, ref2 = X1.clone(), X2.clone()
    nadmm.nadmm_local_newton(gp1, ref1, params, want_stats=False)
    nadmm.nadmm_local_newton(gp2, ref2, params, want_stats=False)
    torch.cuda.synchronize()
    for _ in range(3):
        X1.copy_(dev(w1.X0)); X2.copy_(dev(w2.X0))
        torch.cuda.synchronize()
        with torch.cuda.stream(s1):
            nadmm.nadmm_local_newton(gp1, X1, params, want_stats=False, stream=s1)
        with torch.cuda.stream(s2):
            nadmm.nadmm_local_newton(gp2, X2, params, want_stats=False, stream=s2)
        s1.synchronize(); s2.synchronize()
        assert torch.equal(X1, ref1) and torch.equal(X2, ref2)


# Single-pass kernel for wide rows (kernel path 4, sweeps with a transpose product): numbers of column steps at which waves
# hold different counts (513 = 16 steps and one column; 1024 = 4 steps per wave exactly; 1025; 2049; 3072 = the widest), rows at
# the edges of a tile of 16 and of the 256 row ranges, rows that are only 4-byte aligned, one and two blocks of classes, and
# shapes on either side of the limits (3073 and 2049 columns with 25 classes take two sweeps).
WIDE_SHAPES = [(1, 513, 2), (15, 544, 10), (16, 1024, 17), (17, 1025, 5), (257, 1100, 10), (4096, 640, 3), (4097, 1537, 9),
               (300, 2049, 10), (129, 2561, 16), (530, 3072, 10), (40, 3071, 2), (35, 3073, 4),
               (33, 290, 18), (129, 2048, 20), (257, 1500, 19), (50, 700, 18), (4100, 330, 20), (70, 513, 33), (48, 1025, 25), (31, 2048, 33), (31, 2049, 25)]


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("n,p,C", WIDE_SHAPES)
def test_wide_single_pass(n, p, C, pad):
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / math.sqrt(p), mean=True)
    A = torch.full((n, p + pad), float("nan"), device="cuda")  # what lies between the rows must not matter
    A[:, :p] = dev(w.A)
    gp = nadmm.Problem(A[:, :p], dev(w.b), C, w.s, w.lam, w.rho, dev(w.z), dev(w.y))
    op = oracle_problem(w)
    force_path(gp, 4)
    loss, grad = nadmm.nadmm_loss_grad(gp, dev(w.X0))
    f_ref, g_ref = orc.loss_grad(op, w.X0)
    # 16-bit products summed in float32: relative error 2^-16 per term, averaged over the sum; TOL_PRIMITIVE is the API's bar
    assert rel_abs(loss.item(), f_ref) <= TOL_PRIMITIVE and rel_l2(host(grad), g_ref) <= TOL_PRIMITIVE
    hv = nadmm.nadmm_hessvec(gp, dev(w.X0), dev(w.V))
    assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE
    assert torch.equal(hv, nadmm.nadmm_hessvec(gp, dev(w.X0), dev(w.V)))
    p_out, it, _ = nadmm.nadmm_cg_solve(gp, dev(w.X0), dev(g_ref.astype(np.float32)), 3, 0.0)  # cached probabilities
    p_ref, it_ref, _ = orc.cg(op, w.X0, g_ref.astype(np.float32).astype(np.float64), 3, 0.0)
    assert it.item() == it_ref and rel_l2(host(p_out), p_ref) <= TOL_ITERATE


# 17 to 32 free classes from 97 columns on: 4 to 9 column steps for eight waves, of which some hold none with 4 to 7; fewer than 7 steps take two sweeps
# from 12289 rows on.  Four waves form the probabilities of a tile (with X): tiles of 1 to 16 rows, one and two blocks of classes, extra classes.
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("n,p,C", [(1, 97, 18), (33, 100, 20), (257, 128, 33), (4099, 129, 21), (12288, 190, 19), (12289, 190, 19), (300, 192, 26), (70, 193, 18),
                                   (12300, 200, 33), (530, 224, 20), (47, 256, 25), (1030, 257, 19), (31, 288, 33)])
def test_wide_single_pass_with_few_steps(n, p, C, pad):
    test_wide_single_pass(n, p, C, pad)


# Sweeps with X of 17 to 32 free classes at numbers of rows and columns where one sweep or two may be the faster (up to 16
# column steps; two blocks of classes over 48 steps): gradient, objective, Newton (whose head adds up the row losses that the sweep left).
@pytest.mark.parametrize("n,p,C", [(12288, 330, 20), (12289, 330, 20), (12289, 481, 18), (22528, 290, 21), (22529, 290, 21), (4096, 1550, 26), (4097, 1550, 26),
                                   (4097, 1550, 25)])
def test_wide_or_two_sweeps_with_many_classes(n, p, C):
    w = workloads.generic(n, p, C, seed=n + C, x_std=0.5 / math.sqrt(p), mean=True)
    gp, op = nadmm.Problem.from_workload(w), oracle_problem(w)
    loss, grad = nadmm.nadmm_loss_grad(gp, dev(w.X0))
    f_ref, g_ref = orc.loss_grad(op, w.X0)
    # products with 2^-16 per term (gradient) and 2^-22 (objective): the API's bar, and a tenth of it for the objective
    assert rel_abs(loss.item(), f_ref) <= 0.1 * TOL_PRIMITIVE and rel_l2(host(grad), g_ref) <= TOL_PRIMITIVE
    assert rel_l2(host(nadmm.nadmm_hessvec(gp, dev(w.X0), dev(w.V))), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE
    X = dev(w.X0)
    st = nadmm.nadmm_local_newton(gp, X, nadmm.make_params(1, 2, 10))
    assert rel_abs(st["loss_initial"], f_ref) <= 0.1 * TOL_PRIMITIVE
    w.max_newton, w.max_cg = 1, 2
    assert rel_l2(host(X), oracle_newton_following(op, w.X0, w, st["alpha"])[0]) <= TOL_ITERATE


# Long vectors of wide rows: the CG update's kernel lays out the next direction's operands.  A solve of ten
# iterations that is stopped on the way by its tolerance and one that is not, one block of classes, extra classes, two blocks.
@pytest.mark.parametrize("tol", [0.0, 0.05])
@pytest.mark.parametrize("n,p,C", [(300, 2740, 10), (200, 1310, 20), (210, 1030, 25)])
def test_wide_cg_on_long_vectors(n, p, C, tol):
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / math.sqrt(p), mean=True)
    gp = nadmm.Problem(dev(w.A), dev(w.b), C, w.s, 0.1, 0.1, dev(w.z), dev(w.y))
    op = oracle_problem(w)
    op.lam, op.rho = 0.1, 0.1
    _, g = orc.loss_grad(op, w.X0)
    g = g.astype(np.float32)
    force_path(gp, 4)
    p_out, it, rel = nadmm.nadmm_cg_solve(gp, dev(w.X0), dev(g), 10, tol)
    p_ref, it_ref, rel_ref = orc.cg(op, w.X0, g.astype(np.float64), 10, tol)
    assert it.item() == it_ref and rel_l2(host(p_out), p_ref) <= TOL_ITERATE
    assert (it_ref < 10) == (tol > 0.0)


# Iterations behind the one that met the tolerance leave everything as it is, however many there are (the update's state alternates between
# two slots): one launch (general kernels, wide rows, sparse storage) and two, and a gradient of zero, where no iteration is made.
@pytest.mark.parametrize("n,p,C,path", [(60, 1000, 6, 1), (300, 1100, 4, 4), (300, 1103, 2, 4), (300, 2740, 10, 4), (24, 131073, 2, 1), (60, 2000, 3, 5)])
def test_cg_iterations_behind_the_last(n, p, C, path):
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / math.sqrt(p), mean=True)
    op = oracle_problem(w)
    A = dev(w.A)
    if path == 5:
        csr = sp.csr_matrix(w.A)
        A = nadmm.SparseA.from_scipy(csr, csr.tocsc())
    gp = nadmm.Problem(A, dev(w.b), C, w.s, op.lam, op.rho, dev(w.z), dev(w.y))
    g = orc.loss_grad(op, w.X0)[1].astype(np.float32)
    force_path(gp, path)
    tol = 0.3
    it_ref = orc.cg(op, w.X0, g.astype(np.float64), 20, tol)[1]
    assert it_ref < 20
    want = [t.clone() for t in nadmm.nadmm_cg_solve(gp, dev(w.X0), dev(g), it_ref, tol)]
    for more in (1, 2, 3, 30):
        got = nadmm.nadmm_cg_solve(gp, dev(w.X0), dev(g), it_ref + more, tol)
        assert all(torch.equal(a, b) for a, b in zip(got, want)) and got[1].item() == it_ref
        p_out, it, _ = nadmm.nadmm_cg_solve(gp, dev(w.X0), torch.zeros_like(dev(g)), more, tol)
        assert it.item() == 0 and not p_out.any()


# CG updates made by several workgroups, each of which takes the norm of the new residual from sums of the old one and of what the
# data leave of H (path 1: the general kernels).  Vectors of 1 and several workgroups and up to one, at and beyond the length where two kernels take over; a linear term that
# is small, as large as the data and far above them.  None of these sums cancels (a thousandth of the terms and more is left).
# Bounds: those of the other solves of fixed length; a residual at rounding level has only that level.
@pytest.mark.parametrize("reg", [0.05, 0.5, 1e4])
@pytest.mark.parametrize("n,p,C,path", [(30, 2048, 2, 1), (60, 1000, 6, 1), (24, 131072, 2, 1), (50, 8193, 9, 1), (300, 1400, 10, 4), (24, 131073, 2, 1)])
def test_cg_update_of_several_workgroups(n, p, C, path, reg):
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / math.sqrt(p), mean=True)
    gp = nadmm.Problem(dev(w.A), dev(w.b), C, w.s, reg, reg, dev(w.z), dev(w.y))
    op = oracle_problem(w)
    op.lam, op.rho = reg, reg
    g = orc.loss_grad(op, w.X0)[1].astype(np.float32)
    force_path(gp, path)
    for K in (1, 2, 6):
        p_out, it, rel = nadmm.nadmm_cg_solve(gp, dev(w.X0), dev(g), K, 0.0)
        p_ref, it_ref, rel_ref = orc.cg(op, w.X0, g.astype(np.float64), K, 0.0)
        assert it.item() == it_ref and rel_l2(host(p_out), p_ref) <= TOL_ITERATE
        assert abs(rel.item() - rel_ref) <= 5e-3 * rel_ref + 1e-6


# Rows of up to 128 columns: the kernel for narrow rows (1 to 4 column steps, one and two blocks of classes, tiles of 16, 32 and
# 64 rows with remainders, more rows than one round of 512 workgroups) and the thin-data kernel on rows that are no whole number
# of 16-byte pieces (lda = p odd, a few elements of padding, one row, the last piece of the matrix at every offset).
NARROW_SHAPES = [(1, 5, 6), (17, 31, 7), (65, 4, 17), (130, 33, 5), (2049, 47, 16), (33000, 36, 10), (50001, 97, 4), (49152, 128, 17),
                 (40000, 64, 2), (63, 32, 33), (1000, 65, 20), (500, 96, 33), (33001, 45, 18), (49151, 112, 3), (49151, 113, 3),
                 (1, 8, 2), (2, 3, 2), (255, 29, 2), (256, 30, 3), (257, 31, 2), (1025, 13, 4), (70001, 21, 3), (3, 32, 2), (40, 1, 2)]


@pytest.mark.parametrize("pad", [0, 1, 3])
@pytest.mark.parametrize("n,p,C", NARROW_SHAPES)
def test_narrow_rows(n, p, C, pad):
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / math.sqrt(p), mean=True)
    # ends with the last row (16-byte aligned rows: up to three elements later, as the header asks); NaN between the rows
    flat = torch.full(((n - 1) * (p + pad) + (p if (p + pad) % 4 else (p + 3) // 4 * 4),), float("nan"), device="cuda")
    A = flat.as_strided((n, p), (p + pad, 1))
    A.copy_(dev(w.A))
    gp = nadmm.Problem(A, dev(w.b), C, w.s, w.lam, w.rho, dev(w.z), dev(w.y))
    op = oracle_problem(w)
    X, V = dev(w.X0), dev(w.V)
    loss, grad = nadmm.nadmm_loss_grad(gp, X)
    loss_only, _ = nadmm.nadmm_loss_grad(gp, X, want_grad=False)
    f_ref, g_ref = orc.loss_grad(op, w.X0)
    # products of full float32 accuracy summed in float32: some 2^-22 of the terms' absolute sum (test_narrow_rows_keep_float32_accuracy);
    # here the API's bar
    assert rel_abs(loss.item(), f_ref) <= 1e-6 and rel_abs(loss_only.item(), f_ref) <= 1e-6
    assert rel_l2(host(grad), g_ref) <= TOL_PRIMITIVE
    hv = nadmm.nadmm_hessvec(gp, X, V)
    assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE
    assert torch.equal(hv, nadmm.nadmm_hessvec(gp, X, V))
    g32 = g_ref.astype(np.float32)
    k = min(3, p * (C - 1))
    p_out, it, _ = nadmm.nadmm_cg_solve(gp, X, dev(g32), k, 0.0)
    p_ref, it_ref, _ = orc.cg(op, w.X0, g32.astype(np.float64), k, 0.0)
    assert it.item() == it_ref and rel_l2(host(p_out), p_ref) <= TOL_ITERATE
    Xn = X.clone()
    st = nadmm.nadmm_local_newton(gp, Xn, nadmm.make_params(2, k, 10))
    w.max_newton, w.max_cg = 2, k
    X_ref, _, _ = oracle_newton_following(op, w.X0, w, st["alpha"])
    assert rel_l2(host(Xn), X_ref) <= TOL_ITERATE


# The kernel for narrow rows and the thin-data kernel work to float32 accuracy (every operand in three bf16 parts and six terms, or float32
# itself).  On one to four rows nothing averages out: with two parts of V, of D or of the tile in either product the relative
# error is 1.2e-6 to 1e-5 at these shapes (computed in float64 with rounded operands), while some ten float32 roundings per
# element, exp() and its sum among them, give about 3e-7.  lambda, rho, z and y do not hide it.
FLOAT32_ACCURACY = 8e-7


@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("n,p,C", [(1, 5, 6), (3, 33, 18), (1, 70, 7), (2, 47, 33), (1, 128, 17), (4, 64, 33), (1, 101, 4), (3, 64, 9), (2, 29, 3), (4, 21, 4),
                                   (2, 31, 3), (1, 7, 2), (1, 15, 4), (3000, 31, 3), (2049, 11, 4), (4097, 27, 2)])
def test_narrow_rows_keep_float32_accuracy(n, p, C, pad):
    w = workloads.generic(n, p, C, seed=n + p, x_std=1.0 / math.sqrt(p), mean=True, lam=0.0, rho=1e-30)
    w = dataclasses.replace(w, z=np.zeros_like(w.z), y=np.zeros_like(w.y))
    thin = p <= 32 and C <= 4
    if C <= 17 and not thin and (p >= 48 or (p + pad) % 4 == 0):   # fewer rows would go to the fused kernel
        reps = 49152 // n + 1
        w = dataclasses.replace(w, A=np.tile(w.A, (reps, 1)), b=np.tile(w.b, reps), s=1.0 / (n * reps))
    A = torch.full((w.A.shape[0], p + pad), float("nan"), device="cuda")
    A[:, :p] = dev(w.A)
    gp = nadmm.Problem(A[:, :p], dev(w.b), C, w.s, w.lam, w.rho, None, None)
    op = oracle_problem(dataclasses.replace(w, A=w.A[:n], b=w.b[:n], s=1.0 / n))   # repeated rows: the same mean
    X, V = dev(w.X0), dev(w.V)
    errs = (rel_l2(host(nadmm.nadmm_hessvec(gp, X, V)), orc.hessvec(op, w.X0, w.V)),
            rel_l2(host(nadmm.nadmm_loss_grad(gp, X)[1]), orc.grad(op, w.X0)))
    print(f"narrow accuracy {n}x{p} C{C} pad{pad}: {errs[0]:.1e} {errs[1]:.1e}", flush=True)
    assert max(errs) <= FLOAT32_ACCURACY


# A CG or Newton solve of a small thin problem in one launch: rows at the limits of one workgroup (4 rows for 256 or 512 threads; 2049
# rows take the general path), all numbers of classes, columns that are no whole number of 16-byte pieces, CG that stops early.
@pytest.mark.parametrize("tol", [0.0, 3e-2])
@pytest.mark.parametrize("n,p,C", [(1, 4, 2), (3, 1, 2), (255, 32, 3), (1000, 20, 3), (1023, 21, 4), (1024, 7, 2), (1025, 16, 4), (2047, 29, 2),
                                   (2048, 32, 3), (2049, 32, 3)])
def test_small_cg(n, p, C, tol):
    w = workloads.generic(n, p, C, seed=n, x_std=0.5 / math.sqrt(p), mean=True)
    gp, op = nadmm.Problem.from_workload(w), oracle_problem(w)
    d = p * (C - 1)
    k = min(10, d)
    g32 = orc.grad(op, w.X0).astype(np.float32)
    got, it, relres = nadmm.nadmm_cg_solve(gp, dev(w.X0), dev(g32), k, tol)
    ref, it_ref, rel_ref = orc.cg(op, w.X0, g32.astype(np.float64), k, tol)
    assert it.item() == it_ref and rel_l2(host(got), ref) <= TOL_ITERATE
    assert abs(relres.item() - rel_ref) <= 1e-5 + 1e-3 * rel_ref
    X = dev(w.X0)
    st = nadmm.nadmm_local_newton(gp, X, nadmm.make_params(2, k, 10, cg_tol=tol))
    w.max_newton, w.max_cg, w.cg_tol = 2, k, tol
    X_ref, st_ref, forced = oracle_newton_following(op, w.X0, w, st["alpha"])
    assert rel_l2(host(X), X_ref) <= TOL_ITERATE
    assert forced or st["cg_iters"] == [i["cg_iters"] for i in st_ref["iters"]]


# The same with few iterations.
@pytest.mark.parametrize("n,p,C,k", [(2048, 32, 2, 4), (2048, 32, 2, 5), (1000, 20, 3, 1), (1000, 20, 3, 2), (2048, 29, 3, 3), (2048, 29, 3, 4), (512, 31, 2, 1)])
def test_small_cg_with_few_iterations(n, p, C, k):
    w = workloads.generic(n, p, C, seed=n + k, x_std=0.5 / math.sqrt(p), mean=True)
    gp, op = nadmm.Problem.from_workload(w), oracle_problem(w)
    g32 = orc.grad(op, w.X0).astype(np.float32)
    got, it, relres = nadmm.nadmm_cg_solve(gp, dev(w.X0), dev(g32), k, 0.0)
    ref, it_ref, rel_ref = orc.cg(op, w.X0, g32.astype(np.float64), k, 0.0)
    assert it.item() == it_ref == k and rel_l2(host(got), ref) <= TOL_ITERATE
    assert abs(relres.item() - rel_ref) <= 1e-5 + 1e-3 * rel_ref
    X = dev(w.X0)
    st = nadmm.nadmm_local_newton(gp, X, nadmm.make_params(2, k, 10))
    w.max_newton, w.max_cg = 2, k
    assert rel_l2(host(X), oracle_newton_following(op, w.X0, w, st["alpha"])[0]) <= TOL_ITERATE
    assert st["cg_iters"] == [k, k]


# The stopping test of Algorithm 3 at every iteration of a solve: the iterate is that of a solve of so many iterations, bit for bit, and
# nothing after it takes a step.  The heads of kernels of their own, beside the first reduction and in the first CG sweep.
@pytest.mark.parametrize("n,p,C,path", [(2100, 28, 2, 3), (70001, 21, 3, 3), (3000, 100, 7, 2), (9001, 260, 10, 2), (40000, 64, 3, 2), (700, 90, 20, 4),
                                        (300, 1100, 4, 4), (300, 40, 3, 1)])
def test_newton_ends_at_every_iteration(n, p, C, path):
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / math.sqrt(p), mean=True)
    gp = nadmm.Problem.from_workload(w)
    force_path(gp, path)
    X = dev(w.X0)
    st = nadmm.nadmm_local_newton(gp, X, nadmm.make_params(5, 2, 10))
    gn = st["grad_norm"]
    assert all(b < 0.99 * a for a, b in zip(gn, gn[1:]))
    for stop in range(5):
        Xs, Xr = dev(w.X0), dev(w.X0)
        got = nadmm.nadmm_local_newton(gp, Xs, nadmm.make_params(8, 2, 10, grad_tol=1.001 * gn[stop]))
        ref = nadmm.nadmm_local_newton(gp, Xr, nadmm.make_params(stop, 2, 10))
        assert torch.equal(Xs, Xr)
        assert got["newton_iters"] == stop and got["cg_iters_total"] == ref["cg_iters_total"] and got["ls_evals_total"] == ref["ls_evals_total"]
        assert got["grad_norm_final"] == gn[stop] and (stop == 0 or got["loss_final"] == ref["loss_final"])


# Rounds of the kernel for narrow rows dealt out to its workgroups: the last counts before and the first with 512 uneven ones (3 to 8
# rounds of 256, 128 and 64 rows), one row more than a whole number of rounds, one row less, the first count past 8.  The same with two
# blocks of classes (rounds of 128 and 64 rows).
@pytest.mark.parametrize("n,p,C", [(65536, 100, 3), (65537, 100, 3), (98305, 70, 17), (131071, 65, 4), (131073, 40, 3), (262145, 9, 6), (262145, 70, 3),
                                   (65536, 84, 29), (65537, 84, 29), (98303, 36, 18), (131073, 9, 20), (262145, 64, 22)])
def test_narrow_rounds(n, p, C):
    w = workloads.generic(n, p, C, seed=n % 991 + p, x_std=0.5 / math.sqrt(p), mean=True)
    gp, op = nadmm.Problem.from_workload(w), oracle_problem(w)
    X, V = dev(w.X0), dev(w.V)
    loss, grad = nadmm.nadmm_loss_grad(gp, X)
    f_ref, g_ref = orc.loss_grad(op, w.X0)
    assert rel_abs(loss.item(), f_ref) <= 1e-6 and rel_l2(host(grad), g_ref) <= FLOAT32_ACCURACY
    hv = nadmm.nadmm_hessvec(gp, X, V)
    assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= FLOAT32_ACCURACY
    assert torch.equal(hv, nadmm.nadmm_hessvec(gp, X, V))


# The thin-data kernel's chunks of 64 rows dealt out to 256 workgroups of 8 or 16 waves: the last chunk full, of one row, one row more
# than a chunk per workgroup and than one per wave; rows of quads and others; CG with its update in the next sweep, to the end and
# stopped early; every call twice, bit for bit.
@pytest.mark.parametrize("tol", [0.0, 3e-2])
@pytest.mark.parametrize("n,p,C", [(2049, 29, 2), (2112, 32, 3), (16384, 20, 4), (16385, 13, 3), (131073, 31, 3), (262145, 28, 2), (262144, 7, 4)])
def test_thin_chunks(n, p, C, tol):
    w = workloads.generic(n, p, C, seed=n % 997 + p, x_std=0.5 / math.sqrt(p), mean=True)
    gp, op = nadmm.Problem.from_workload(w), oracle_problem(w)
    assert nadmm.nadmm_query_kernel_path(gp) == 3
    X, V = dev(w.X0), dev(w.V)
    loss, grad = nadmm.nadmm_loss_grad(gp, X)
    f_ref, g_ref = orc.loss_grad(op, w.X0)
    # float32 products and sums, of at most 3e5 terms in groups of a lane's, a wave's, a workgroup's and all workgroups'
    assert rel_abs(loss.item(), f_ref) <= 1e-6 and rel_l2(host(grad), g_ref) <= 1e-6
    hv = nadmm.nadmm_hessvec(gp, X, V)
    assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= 1e-6
    assert torch.equal(hv, nadmm.nadmm_hessvec(gp, X, V)) and torch.equal(grad, nadmm.nadmm_loss_grad(gp, X)[1])
    g32 = g_ref.astype(np.float32)
    got, it, relres = nadmm.nadmm_cg_solve(gp, X, dev(g32), 5, tol)
    ref, it_ref, rel_ref = orc.cg(op, w.X0, g32.astype(np.float64), 5, tol)
    assert it.item() == it_ref and rel_l2(host(got), ref) <= TOL_ITERATE
    assert abs(relres.item() - rel_ref) <= 1e-5 + 1e-3 * rel_ref
    assert torch.equal(got, nadmm.nadmm_cg_solve(gp, X, dev(g32), 5, tol)[0])
    Xn = X.clone()
    st = nadmm.nadmm_local_newton(gp, Xn, nadmm.make_params(2, 5, 10, cg_tol=tol))
    w.max_newton, w.max_cg, w.cg_tol = 2, 5, tol
    X_ref, st_ref, forced = oracle_newton_following(op, w.X0, w, st["alpha"])
    assert rel_l2(host(Xn), X_ref) <= TOL_ITERATE
    assert forced or st["cg_iters"] == [i["cg_iters"] for i in st_ref["iters"]]
    # objective and stopping test of the head, which the first CG sweep makes: before the first iteration and before the second
    assert rel_abs(st["loss_initial"], f_ref) <= 1e-6 and rel_abs(st["grad_norm"][0], np.linalg.norm(g_ref)) <= 1e-6
    assert st["grad_norm"][1] < st["grad_norm"][0]
    for stop, tol_g in ((0, 1.01 * st["grad_norm"][0]), (1, 1.01 * st["grad_norm"][1])):
        Xs = X.clone()
        st1 = nadmm.nadmm_local_newton(gp, Xs, nadmm.make_params(3, 5, 10, cg_tol=tol, grad_tol=tol_g))
        assert st1["newton_iters"] == stop and (stop > 0 or torch.equal(Xs, X))
        assert st1["grad_norm_final"] == st["grad_norm"][stop]


# The one launch of a small Newton solve: line searches that reduce their step (sum scaling, far from the minimiser), a row block of
# which A starts on any 4-byte boundary, and the stopping test of Algorithm 3 before the first and between iterations.
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n,p,C", [(257, 12, 3), (1024, 20, 3), (1500, 31, 2), (2048, 13, 4)])
def test_small_newton(n, p, C, shift):
    w = workloads.generic(n, p, C, seed=n + p, x_std=6.0 / math.sqrt(p))
    flat = torch.empty(shift + n * p, device="cuda")
    A = flat[shift:].as_strided((n, p), (p, 1), shift)
    A.copy_(dev(w.A))
    gp = nadmm.Problem(A, dev(w.b), C, w.s, w.lam, w.rho, dev(w.z), dev(w.y))
    op = oracle_problem(w)
    k = 6
    X = dev(w.X0)
    st = nadmm.nadmm_local_newton(gp, X, nadmm.make_params(4, k, 10))
    w.max_newton, w.max_cg = 4, k
    X_ref, st_ref, forced = oracle_newton_following(op, w.X0, w, st["alpha"])
    assert rel_l2(host(X), X_ref) <= TOL_ITERATE
    assert st["newton_iters"] == 4 and st["cg_iters"] == [i["cg_iters"] for i in st_ref["iters"]]
    assert min(st["alpha"]) < 1.0                  # a step was reduced
    assert rel_abs(st["loss_initial"], orc.loss(op, w.X0)) <= 1e-6 and rel_abs(st["loss_final"], orc.loss(op, host(X))) <= 1e-5
    X1 = dev(w.X0)                                 # without statistics: the same iterate, bit for bit
    nadmm.nadmm_local_newton(gp, X1, nadmm.make_params(4, k, 10), want_stats=False)
    assert torch.equal(X, X1)
    gn = st["grad_norm"]
    X2 = dev(w.X0)
    st2 = nadmm.nadmm_local_newton(gp, X2, nadmm.make_params(4, k, 10, grad_tol=2.0 * max(gn)))
    assert st2["newton_iters"] == 0 and st2["cg_iters_total"] == 0 and torch.equal(X2, dev(w.X0))
    assert rel_abs(st2["grad_norm_final"], gn[0]) <= 1e-12
    stop = min(range(4), key=lambda i: gn[i])      # the first iteration whose gradient is below the tolerance ends the solve
    st3 = nadmm.nadmm_local_newton(gp, dev(w.X0), nadmm.make_params(4, k, 10, grad_tol=1.0000001 * gn[stop]))
    assert st3["newton_iters"] == stop


# Thin rows with a stride of whole quads and padding, 16-byte aligned or not (A four bytes further): the thin-data kernel by force, which
# lays them out row by row in LDS, and the automatic choice (the same kernel, under path number 2 on 2049 to 65535 aligned ones).
# Rows at the edges of four chunks of 64, the last piece of the matrix, every number of quads.
@pytest.mark.parametrize("path", [0, 3])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n,p,lda,C", [(3, 3, 4, 4), (255, 5, 8, 3), (256, 8, 8, 2), (257, 11, 12, 4), (2048, 13, 16, 3), (2049, 16, 16, 2), (511, 17, 20, 4),
                                       (70001, 23, 24, 2), (1025, 26, 28, 3), (513, 31, 32, 3), (5000, 32, 32, 2), (66000, 7, 8, 4), (2049, 27, 28, 2), (2065, 5, 8, 4),
                                       (65535, 18, 20, 4), (33001, 31, 32, 3), (5000, 29, 32, 2)])
def test_thin_rows_of_whole_quads(n, p, lda, C, shift, path):
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / math.sqrt(p), mean=True)
    flat = torch.full((shift + n * lda,), float("nan"), device="cuda")    # NaN between the rows; ends with the last row's quads
    A = flat[shift:].as_strided((n, p), (lda, 1), shift)
    A.copy_(dev(w.A))
    gp = nadmm.Problem(A, dev(w.b), C, w.s, w.lam, w.rho, dev(w.z), dev(w.y))
    op = oracle_problem(w)
    force_path(gp, path)
    X, V = dev(w.X0), dev(w.V)
    loss, grad = nadmm.nadmm_loss_grad(gp, X)
    f_ref, g_ref = orc.loss_grad(op, w.X0)
    # float32 products and sums, of at most 1e5 terms in groups; the API's bar for the iterates
    assert rel_abs(loss.item(), f_ref) <= 1e-6 and rel_l2(host(grad), g_ref) <= TOL_PRIMITIVE
    assert rel_l2(host(nadmm.nadmm_hessvec(gp, X, V)), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE
    g32 = g_ref.astype(np.float32)
    k = min(3, p * (C - 1))
    p_out, it, _ = nadmm.nadmm_cg_solve(gp, X, dev(g32), k, 0.0)
    p_ref, it_ref, _ = orc.cg(op, w.X0, g32.astype(np.float64), k, 0.0)
    assert it.item() == it_ref and rel_l2(host(p_out), p_ref) <= TOL_ITERATE
    Xn = X.clone()
    st = nadmm.nadmm_local_newton(gp, Xn, nadmm.make_params(2, k, 10))
    w.max_newton, w.max_cg = 2, k
    assert rel_l2(host(Xn), oracle_newton_following(op, w.X0, w, st["alpha"])[0]) <= TOL_ITERATE


# The reduction of the partial sums of A^T D takes them in batches of 128 and the rest in one of 32, 64 or 128: numbers of
# partials (one per tile of 32 rows here) at the edges of these, a d that is no multiple of the 32 elements of a workgroup.
@pytest.mark.parametrize("parts", [1, 7, 8, 9, 31, 32, 33, 64, 65, 127, 128, 129, 160, 161, 193, 255, 256])
def test_reduction_of_any_number_of_partials(parts):
    w = workloads.generic(32 * parts - 5, 129, 4, seed=parts, x_std=0.05)
    gp, op = nadmm.Problem.from_workload(w), oracle_problem(w)
    force_path(gp, 2)
    X, V = dev(w.X0), dev(w.V)
    # float32 sums of up to 256 partials on top of the products' accuracy: the API's bar
    assert rel_l2(host(nadmm.nadmm_loss_grad(gp, X)[1]), orc.grad(op, w.X0)) <= TOL_PRIMITIVE
    hv = nadmm.nadmm_hessvec(gp, X, V)
    assert rel_l2(host(hv), orc.hessvec(op, w.X0, w.V)) <= TOL_PRIMITIVE
    assert torch.equal(hv, nadmm.nadmm_hessvec(gp, X, V))
