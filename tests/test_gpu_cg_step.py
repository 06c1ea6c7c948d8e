"""The CG update that several workgroups make in one launch, called by itself on vectors made for it: the norm of the new residual comes from four
sums over the old vectors, or, where those cancel, from the vectors.  Against the same in numpy, float64 sums of float32 vectors."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import nadmm_oracle as orc
from paper_1807_07132_amd import nadmm, workloads
from parity_utils import TOL_ITERATE, oracle_problem, rel_l2

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include <cstring>
#include "nadmm_internal.h"
using namespace nadmm;
extern "C" {
long state_bytes() { return sizeof(DevState); }
void set_state(DevState* st, int slot, double rr, double gg, int active) {
  std::memset(st, 0x5a, sizeof(DevState));
  st->gg_cg = gg;
  st->cgs[slot] = CgSlot{rr, active, 7, 0, 0};
}
void get_state(const DevState* st, int slot, double* rr, int* v) {
  rr[0] = st->cgs[slot].rr; rr[1] = st->rr;
  v[0] = st->cgs[slot].active; v[1] = st->cgs[slot].iters; v[2] = st->cg_active; v[3] = st->cg_iters;
}
long operand_bytes(int p, int NC) {
  Shape s{}; s.n = 1; s.p = p; s.NC = NC; s.d = (int64_t)p * NC;
  return (long)wide_operand_bytes(s);
}
int step(void* st, int slot, float* pdir, float* r, float* r_out, float* dvec, const float* q, const double* dot, int ndot, int p, int NC, float tol,
         float lambda, float rho, const float* rho_scale, void* operands, void* stream) {
  CgUpdateArgs a{};
  a.st = static_cast<DevState*>(st); a.slot_in = slot; a.pdir = pdir; a.r = r; a.r_out = r_out; a.dvec = dvec; a.q = q; a.dot_part = dot; a.ndot = ndot;
  a.d = (int64_t)p * NC; a.tol = tol; a.lambda = lambda; a.rho = rho; a.rho_scale = rho_scale;
  Shape s{}; s.n = 1; s.p = p; s.NC = NC; s.d = a.d;
  return (int)(operands != nullptr ? launch_wide_direction(a, s, operands, (hipStream_t)stream) : launch_cg_update(a, (hipStream_t)stream));
}
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    nadmm.lib()
    d = tmp_path_factory.mktemp("shim")
    (d / "shim.cpp").write_text(SHIM)
    so = d / "shim.so"
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{os.path.join(ROOT, 'include')}",
                           f"-I{os.path.join(ROOT, 'paper_1807_07132_amd', 'csrc')}", "-Wno-unused-result", "-shared", "-fPIC", str(d / "shim.cpp"),
                           nadmm.LIB_PATH, f"-Wl,-rpath,{os.path.dirname(nadmm.LIB_PATH)}", "-o", str(so)])
    L = C.CDLL(str(so))
    vp, i, f = C.c_void_p, C.c_int, C.c_float
    L.state_bytes.restype = L.operand_bytes.restype = C.c_long
    L.operand_bytes.argtypes = [i, i]
    L.set_state.argtypes = [vp, i, C.c_double, C.c_double, i]
    L.get_state.argtypes = [vp, i, vp, vp]
    L.step.argtypes = [vp, i, vp, vp, vp, vp, vp, vp, i, i, i, f, f, f, vp, vp, vp]
    return L


def run_step(L, slot, r, d, pdir, q, sums, ndot, p, NC, tol, lam, rho, scale, rr, gg, active, wide):
    st = np.zeros(L.state_bytes(), np.uint8)
    L.set_state(st.ctypes.data, slot, rr, gg, active)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    t = dict(st=dev(st), r=dev(r), d=dev(d), p=dev(pdir), q=dev(q), out=torch.full((len(r),), float("nan"), device="cuda"))
    parts = np.zeros((4, ndot))                     # the four sums, spread unevenly
    w = np.arange(1, ndot + 1) / (ndot * (ndot + 1) / 2)
    for k in range(4):
        parts[k] = sums[k] * w
        if np.isfinite(sums[k]):
            parts[k, -1] += sums[k] - parts[k].sum()
    dot, sc = dev(parts.reshape(-1)), dev(np.array([scale], np.float32))
    ops = torch.zeros(L.operand_bytes(p, NC), dtype=torch.uint8, device="cuda") if wide else None
    torch.cuda.synchronize()
    rc = L.step(t["st"].data_ptr(), slot, t["p"].data_ptr(), t["r"].data_ptr(), t["out"].data_ptr(), t["d"].data_ptr(), t["q"].data_ptr(), dot.data_ptr(), ndot,
                p, NC, tol, lam, rho, sc.data_ptr(), ops.data_ptr() if wide else None, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    out = t["st"].cpu().numpy()
    rrs, v = np.zeros(2), np.zeros(4, np.int32)
    L.get_state(out.ctypes.data, slot ^ 1, rrs.ctypes.data, v.ctypes.data)
    assert torch.equal(t["r"].cpu(), torch.from_numpy(r))          # read only
    return rrs, v, {k: t[k].cpu().numpy() for k in ("out", "d", "p")}


# p, NC, sums, wide: one element, parts of a workgroup's 2048, several workgroups, up to the last length; more sums than threads read at once
SHAPES = [(1, 1, 1, False), (255, 1, 8, False), (2048, 1, 64, False), (683, 3, 1023, False), (65535, 2, 4096, False), (131072, 1, 4096, False),
          (1000, 2, 63, True), (3072, 9, 864, True), (1500, 19, 891, True), (2048, 32, 2048, True),
          # one free class: 16-byte pieces of the vectors, the last one of 4, 1, 2 and 3 elements
          (3072, 1, 96, True), (961, 1, 31, True), (1810, 1, 57, True), (2051, 1, 65, True)]


@pytest.mark.parametrize("p,NC,ndot,wide", SHAPES)
@pytest.mark.parametrize("cancel", ["none", "edge", "deep", "all"])
def test_norm_of_the_new_residual(shim, p, NC, ndot, wide, cancel):
    d = p * NC
    rng = np.random.default_rng(d + len(cancel))
    slot = d & 1
    lam, rho, scale = np.float32(0.125), np.float32(0.25), np.float32(0.5)          # lambda + rho_scale rho = 1/4 exactly
    r = (rng.standard_normal(d) + 3).astype(np.float32)
    # q of step length 1 (<d, q> is given as <r, r>): the residual that is left is r - q, exact in float32 where q is close to r
    left = {"none": 0.5, "edge": 4e-4, "deep": 0.0, "all": 0.0}[cancel] * rng.standard_normal(d)
    q = (r - left * r).astype(np.float32)
    if cancel == "deep":                                                            # a unit in the last place, up or down, in a third of them
        ulp = np.nextafter(r, np.float32(np.inf)) - r
        q = (r + ulp * rng.integers(-1, 2, size=d)).astype(np.float32)
        q[0] = r[0] + ulp[0]
    dv, pd = rng.standard_normal(d).astype(np.float32), rng.standard_normal(d).astype(np.float32)
    R, Q = r.astype(np.float64), q.astype(np.float64)
    T = Q - 0.25 * R
    rr = float(R @ R)
    sums = [rr, float(R @ T), float(T @ T), rr]
    new = (R - Q).astype(np.float32)
    want = float(new.astype(np.float64) @ new.astype(np.float64))
    size = 0.75 ** 2 * rr + float(T @ T)
    by_sums = size - 2 * 0.75 * float(R @ T)
    if cancel in ("deep", "all"):
        assert want < 1e-12 * size                                                  # the vectors are read again ...
        assert d < 1000 or abs(by_sums - want) >= 0.02 * want                       # ... and have to be (all: the sums give their rounding for 0)
    elif d > 1000:                                                                  # edge: a little above the line, 1e-7 of the terms
        assert 1.1e-7 < want / size < 2e-7 if cancel == "edge" else want / size > 1e-2
    tol = 0.0
    rrs, v, t = run_step(shim, slot, r, dv, pd, q, sums, ndot, p, NC, tol, lam, rho, scale, rr, 4 * rr, 1, wide)
    # sums of 2^17 float64 terms against numpy's in another order: 1e-12; the identity: some 20 roundings of terms of which 1e-7 is left, 20 2^-53 10^7
    bound = 1e-12 if cancel in ("deep", "all") else (2e-8 if d > 1000 else 1e-6)    # d < 1000: the share that is left is not checked above
    assert abs(rrs[0] - want) <= bound * want and rrs[1] == rrs[0]
    stop = cancel == "all"                                                          # a residual of zero meets a tolerance of zero
    assert list(v) == [0 if stop else 1, 8, 0 if stop else 1, 8]
    assert np.array_equal(t["out"], new)
    assert np.array_equal(t["p"], (pd.astype(np.float64) + dv).astype(np.float32))
    be = np.float64(np.float32(rrs[0] / rr))
    fma = dv if stop else (be * dv + new).astype(np.float32)                        # be and dv have 24 bits each: the product is exact in float64
    assert rel_l2(t["d"], fma.astype(np.float64)) <= 1e-7


@pytest.mark.parametrize("p,NC,ndot,wide", [(2049, 1, 65, False), (3072, 9, 864, True), (1810, 1, 57, True)])
@pytest.mark.parametrize("dq,active", [(0.0, 1), (-1.0, 1), (float("nan"), 1), (float("inf"), 1), (1.0, 0)])
def test_update_that_is_not_made(shim, p, NC, ndot, wide, dq, active):
    """No positive curvature, or CG has stopped before: the iterate stays, the other slot says that CG has stopped."""
    d = p * NC
    rng = np.random.default_rng(3)
    r, q, dv, pd = (rng.standard_normal(d).astype(np.float32) for _ in range(4))
    rr = float(r.astype(np.float64) @ r)
    rrs, v, t = run_step(shim, 0, r, dv, pd, q, [dq * rr, 0.3, 1.0, rr], ndot, p, NC, 0.0, np.float32(0.1), np.float32(0.2), np.float32(1), rr, rr, active, wide)
    assert v[0] == 0 and v[1] == 7 and rrs[0] == rr
    assert np.array_equal(t["p"], pd) and np.array_equal(t["d"], dv) and np.isnan(t["out"]).all()


@pytest.mark.parametrize("reg", [0.05, 0.5])
@pytest.mark.parametrize("n,p,C,path", [(2, 2048, 2, 1), (3, 2048, 2, 1), (2, 3072, 3, 4)])
def test_solve_that_exhausts_its_krylov_space(n, p, C, path, reg):
    """n (C-1) directions in which the data act and the linear term: after one iteration more the residual is what rounding leaves, and the
    sums of the last update cancel.  What rounding leaves: an error eps of a product (2^-24 of its terms on path 1, 2^-16 on path 4) enters the residual
    as alpha ||q|| eps and is carried on as the residual grows from then on; four times that for the sums inside a product."""
    K = n * (C - 1) + 1
    w = workloads.generic(n, p, C, seed=n + p, x_std=0.5 / p ** 0.5, mean=True)
    op = oracle_problem(w)
    op.lam, op.rho = reg, reg
    g = orc.loss_grad(op, w.X0)[1].astype(np.float32)
    # the oracle's iteration, vectors rounded to float32: what is left of the terms in the last update
    r, least = -g.astype(np.float64), []
    dv, terms, norms = r.copy(), 0.0, [np.linalg.norm(r)]
    for _ in range(K):
        q = orc.hessvec(op, w.X0, dv).astype(np.float32).astype(np.float64)
        rr, mu = (r * r).sum(), 2 * reg
        a = np.float64(np.float32(rr / (dv * q).sum()))
        t = q - mu * r
        new = (r - a * q).astype(np.float32).astype(np.float64)
        least.append((new * new).sum() / ((1 - a * mu) ** 2 * rr + a * a * (t * t).sum()))
        dv = (new + np.float64(np.float32((new * new).sum() / rr)) * dv).astype(np.float32).astype(np.float64)
        r = new
        terms += a * np.linalg.norm(q)
        norms.append(np.linalg.norm(r))
    assert least[-1] < 1e-7
    growth = max(b / a for i, a in enumerate(norms) for b in norms[i:])
    bound = 4 * (2.0 ** -24 if path == 1 else 2.0 ** -16) * terms * growth / norms[0]
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    gp = nadmm.Problem(dev(w.A), dev(w.b), C, w.s, reg, reg, dev(w.z), dev(w.y))
    nadmm.nadmm_set_kernel_path(path)
    try:
        p_out, it, rel = nadmm.nadmm_cg_solve(gp, dev(w.X0), dev(g), K, 0.0)
    finally:
        nadmm.nadmm_set_kernel_path(0)
    p_ref = orc.cg(op, w.X0, g.astype(np.float64), K, 0.0)[0]
    assert it.item() == K and rel_l2(p_out.cpu().numpy(), p_ref) <= TOL_ITERATE
    assert 0 <= rel.item() <= bound
