"""Host-only checks of the C ABI: the library loads, exports every declared
symbol, its structs match the header as a C compiler lays them out, and
argument validation returns the documented codes before anything is enqueued
(no GPU is touched)."""
import ctypes as C
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "nadmm.h")

from paper_1807_07132_amd import nadmm  # noqa: E402


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(nadmm.LIB_PATH):
        from paper_1807_07132_amd import build
        build.build(verbose=False)
    return nadmm.lib()


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(nadmm_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = declared_functions()
    assert {"nadmm_loss_grad", "nadmm_hessvec", "nadmm_cg_solve", "nadmm_line_search", "nadmm_local_newton",
            "nadmm_workspace_bytes"} <= set(names)
    for name in names:
        assert hasattr(lib, name), name
    assert lib.nadmm_version() >= 100
    assert lib.nadmm_status_string(0) == b"ok"
    assert b"workspace" in lib.nadmm_status_string(nadmm.NADMM_EWORKSPACE)


def test_struct_layout_matches_the_header(tmp_path):
    src = tmp_path / "sizes.c"
    src.write_text(
        '#include <stdio.h>\n#include <stddef.h>\n#include "nadmm.h"\n'
        "int main(void){printf(\"%zu %zu %zu %zu %zu %zu %zu %zu %zu %zu %zu %zu %zu %zu %zu %zu\\n\", sizeof(nadmm_problem), sizeof(nadmm_params),"
        " sizeof(nadmm_stats), offsetof(nadmm_problem, d_labels), offsetof(nadmm_problem, d_z),"
        " offsetof(nadmm_stats, loss_initial), offsetof(nadmm_stats, grad_norm), sizeof(nadmm_admm_params),"
        " sizeof(nadmm_admm_stats), offsetof(nadmm_admm_params, local), offsetof(nadmm_admm_stats, d_trace),"
        " offsetof(nadmm_problem, sparse), sizeof(nadmm_sparse), offsetof(nadmm_sparse, d_val_t),"
        " offsetof(nadmm_admm_params, rb_tau), offsetof(nadmm_admm_stats, rho_scale_trace));return 0;}\n")
    exe = tmp_path / "sizes"
    subprocess.check_call(["gcc", "-std=c99", "-Wall", "-Werror", f"-I{os.path.join(ROOT, 'include')}", str(src), "-o", str(exe)])
    got = [int(v) for v in subprocess.check_output([str(exe)]).split()]
    want = [C.sizeof(nadmm.nadmm_problem), C.sizeof(nadmm.nadmm_params), C.sizeof(nadmm.nadmm_stats),
            nadmm.nadmm_problem.d_labels.offset, nadmm.nadmm_problem.d_z.offset,
            nadmm.nadmm_stats.loss_initial.offset, nadmm.nadmm_stats.grad_norm.offset,
            C.sizeof(nadmm.nadmm_admm_params), C.sizeof(nadmm.nadmm_admm_stats), nadmm.nadmm_admm_params.local.offset,
            nadmm.nadmm_admm_stats.d_trace.offset, nadmm.nadmm_problem.sparse.offset, C.sizeof(nadmm.nadmm_sparse),
            nadmm.nadmm_sparse.d_val_t.offset, nadmm.nadmm_admm_params.rb_tau.offset,
            nadmm.nadmm_admm_stats.rho_scale_trace.offset]
    assert got == want


def fake_problem(n=1000, p=20, Cc=3, lda=None, rho=1.0, lam=1e-3, A=0x1000, labels=0x2000):
    return nadmm.nadmm_problem(A, n, p, p if lda is None else lda, labels, Cc, 1.0, lam, rho, None, None, None)


def fake_sparse(nnz=5000, **kw):
    f = dict(nnz=nnz, d_row_ptr=0x4000, d_col_idx=0x5000, d_val=0x6000, d_col_ptr=0x7000, d_row_idx=0x8000,
             d_val_t=0x9000)
    f.update(kw)
    return nadmm.nadmm_sparse(f["nnz"], f["d_row_ptr"], f["d_col_idx"], f["d_val"], f["d_col_ptr"], f["d_row_idx"],
                              f["d_val_t"])


def sparse_problem(sp, **kw):
    prob = fake_problem(A=None, **kw)
    prob.sparse = C.pointer(sp)
    return prob


def test_sparse_problems_on_the_host(lib):
    fake = C.c_void_p(0x3000)
    sp = fake_sparse()
    prob = sparse_problem(sp, n=1000, p=3000, Cc=5)
    need = lib.nadmm_workspace_bytes(C.byref(prob), None)
    assert need > 0 and need % 256 == 0
    assert lib.nadmm_query_kernel_path(C.byref(prob)) == 5
    # no dense array is needed, and a dense problem never takes the sparse path
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem())) in (1, 2, 3, 4)
    prev = lib.nadmm_set_kernel_path(5)
    try:
        assert lib.nadmm_query_kernel_path(C.byref(fake_problem())) == nadmm.NADMM_EUNSUPPORTED
        assert lib.nadmm_query_kernel_path(C.byref(prob)) == 5
        lib.nadmm_set_kernel_path(1)
        assert lib.nadmm_query_kernel_path(C.byref(prob)) == nadmm.NADMM_EUNSUPPORTED
    finally:
        lib.nadmm_set_kernel_path(prev)
    # more stored entries need more windows, hence more workspace
    sp_big = fake_sparse(nnz=50_000_000)
    assert lib.nadmm_workspace_bytes(C.byref(sparse_problem(sp_big, n=1000, p=3000, Cc=5)), None) > need
    for bad in (fake_sparse(nnz=-1), fake_sparse(d_row_ptr=None), fake_sparse(d_col_ptr=None), fake_sparse(d_val=None),
                fake_sparse(d_row_idx=None), fake_sparse(d_val_t=None), fake_sparse(d_col_idx=None)):
        pb = sparse_problem(bad, n=1000, p=3000, Cc=5)
        assert lib.nadmm_workspace_bytes(C.byref(pb), None) == 0
        assert lib.nadmm_hessvec(C.byref(pb), fake, fake, fake, fake, 1 << 30, None) == nadmm.NADMM_EINVAL
    # an empty matrix needs no index or value arrays
    empty = fake_sparse(nnz=0, d_col_idx=None, d_val=None, d_row_idx=None, d_val_t=None)
    assert lib.nadmm_workspace_bytes(C.byref(sparse_problem(empty, n=1000, p=3000, Cc=5)), None) > 0
    huge = sparse_problem(sp, n=(1 << 31), p=30, Cc=3)
    assert lib.nadmm_hessvec(C.byref(huge), fake, fake, fake, fake, 1 << 30, None) == nadmm.NADMM_EUNSUPPORTED
    assert lib.nadmm_hessvec(C.byref(prob), fake, fake, fake, fake, need - 1, None) == nadmm.NADMM_EWORKSPACE


def test_sparse_scratch_holds_what_the_kernels_use(lib):
    """Sparse storage: logits [Z | W], the packed operand (into which the rows of D go as well), one partial sum and the windows' tables; no
    further n (C-1) floats.  112000 x 30, C = 21 fits the built-in buffer with these and not with those."""
    for n, p, cls, group in ((112000, 30, 21, 8), (100000, 2000, 17, 4), (50000, 9000, 5, 1)):
        nc = cls - 1
        sp = fake_sparse(nnz=3 * n)
        prob = sparse_problem(sp, n=n, p=p, Cc=cls)
        used = 4 * (2 * n * nc + 4 * group * max(2 * p, n) + p * nc)
        tables = 1 << 19 if nc <= 4 else 2 << 20     # at most 4096 windows: 2 first rows, 2 tickets and 4 (C-1) floats each, rounded up
        assert used < lib.nadmm_hessvec_static_bytes(C.byref(prob)) <= used + tables, (n, p, cls)
    fits = sparse_problem(fake_sparse(nnz=336000), n=112000, p=30, Cc=21)
    assert lib.nadmm_hessvec_static_bytes(C.byref(fits)) <= lib.nadmm_static_scratch_bytes()


@pytest.mark.parametrize("missing", [("_cuda_getCurrentRawStream",), ("_cuda_getDevice",), ("_cuda_getCurrentRawStream", "_cuda_getDevice")])
def test_current_stream_without_torch_s_private_functions(monkeypatch, missing):
    import importlib.util
    import torch
    for name in missing:
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: type("Stream", (), {"cuda_stream": 0x1234567890})())
    spec = importlib.util.spec_from_file_location("paper_1807_07132_amd.nadmm_again", nadmm.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    assert again._stream(None) == 0x1234567890
    assert again._stream(type("Stream", (), {"cuda_stream": 7})()) == 7


def test_workspace_bytes(lib):
    small = lib.nadmm_workspace_bytes(C.byref(fake_problem()), None)
    big = lib.nadmm_workspace_bytes(C.byref(fake_problem(n=60000, p=784, Cc=10)), None)
    assert small > 0 and big > small and small % 256 == 0
    assert big >= 4 * 60000 * 9 * 4                      # four n x (C-1) row buffers
    assert big < 1 << 30
    assert lib.nadmm_workspace_bytes(C.byref(fake_problem(n=0)), None) == 0
    assert lib.nadmm_workspace_bytes(None, None) == 0


def test_workspace_bytes_with_parameters(lib):
    """With parameters the size may add the history of directional logits (max_cg arrays of n (C-1) floats) where the
    single-pass matrix-core path applies and the history is cheaper than the pass over A it replaces."""
    rows = 60000 * 9 * 4
    head = fake_problem(n=60000, p=784, Cc=10)
    base = lib.nadmm_workspace_bytes(C.byref(head), None)
    for max_cg, kept in ((10, True), (29, True), (30, False), (0, False), (33, False)):   # 3 max_cg (C-1) <= p, max_cg <= 32
        pr = nadmm.make_params(10, max_cg, 10, 0.0, 0.0, 1e-4, 0.5)
        need = lib.nadmm_workspace_bytes(C.byref(head), C.byref(pr))
        assert need % 256 == 0
        if kept:
            assert max_cg * rows <= need - base < max_cg * (rows + 256)
        else:
            assert need == base
    pr = nadmm.make_params(10, 10, 10, 0.0, 0.0, 1e-4, 0.5)
    for other in (fake_problem(n=1375000, p=28, Cc=2),            # thin-data path
                  fake_problem(n=50000, p=3072, Cc=10),           # column-sliced path
                  fake_problem(n=50000, p=3072, Cc=10, lda=3073)):  # the same on rows that are not 16-byte aligned
        assert lib.nadmm_workspace_bytes(C.byref(other), C.byref(pr)) == lib.nadmm_workspace_bytes(C.byref(other), None)


@pytest.mark.parametrize("kw,code", [
    (dict(n=0), nadmm.NADMM_EINVAL),
    (dict(p=0), nadmm.NADMM_EINVAL),
    (dict(Cc=1), nadmm.NADMM_EINVAL),
    (dict(lda=19), nadmm.NADMM_EINVAL),
    (dict(rho=0.0), nadmm.NADMM_EINVAL),
    (dict(rho=float("nan")), nadmm.NADMM_EINVAL),
    (dict(lam=-1.0), nadmm.NADMM_EINVAL),
    (dict(A=None), nadmm.NADMM_EINVAL),
    (dict(Cc=40), nadmm.NADMM_EUNSUPPORTED),
])
def test_invalid_problems_are_rejected_on_the_host(lib, kw, code):
    prob = fake_problem(**kw)
    fake = C.c_void_p(0x3000)
    assert lib.nadmm_hessvec(C.byref(prob), fake, fake, fake, fake, 1 << 30, None) == code
    assert lib.nadmm_loss_grad(C.byref(prob), fake, fake, fake, fake, 1 << 30, None) == code
    params = nadmm.make_params()
    assert lib.nadmm_local_newton(C.byref(prob), fake, C.byref(params), None, fake, 1 << 30, None) == code


def test_null_arguments_and_workspace_errors(lib):
    prob = fake_problem()
    fake = C.c_void_p(0x3000)
    need = lib.nadmm_workspace_bytes(C.byref(prob), None)
    assert lib.nadmm_hessvec(C.byref(prob), None, fake, fake, fake, need, None) == nadmm.NADMM_EINVAL
    assert lib.nadmm_hessvec(C.byref(prob), fake, fake, None, fake, need, None) == nadmm.NADMM_EINVAL
    assert lib.nadmm_hessvec(C.byref(prob), fake, fake, fake, None, need, None) == nadmm.NADMM_EWORKSPACE
    assert lib.nadmm_hessvec(C.byref(prob), fake, fake, fake, fake, need - 1, None) == nadmm.NADMM_EWORKSPACE
    assert lib.nadmm_hessvec(C.byref(prob), fake, fake, fake, C.c_void_p(0x3010), need, None) == nadmm.NADMM_EWORKSPACE
    # labels are required by the objective but not by the Hessian-vector product
    nolab = fake_problem(labels=None)
    assert lib.nadmm_loss_grad(C.byref(nolab), fake, fake, fake, fake, need, None) == nadmm.NADMM_EINVAL
    assert lib.nadmm_cg_solve(C.byref(prob), fake, fake, fake, -1, 0.0, None, None, fake, need, None) == nadmm.NADMM_EINVAL
    assert lib.nadmm_cg_solve(C.byref(prob), fake, None, fake, 5, 0.0, None, None, fake, need, None) == nadmm.NADMM_EINVAL


@pytest.mark.parametrize("beta,gamma,max_ls,code", [
    (0.0, 0.5, 10, nadmm.NADMM_EINVAL), (1.0, 0.5, 10, nadmm.NADMM_EINVAL),
    (1e-4, 0.0, 10, nadmm.NADMM_EINVAL), (1e-4, 1.0, 10, nadmm.NADMM_EINVAL),
    (1e-4, 0.5, -1, nadmm.NADMM_EINVAL), (1e-4, 0.5, 63, nadmm.NADMM_EUNSUPPORTED),
])
def test_line_search_parameters_are_validated(lib, beta, gamma, max_ls, code):
    prob = fake_problem()
    fake = C.c_void_p(0x3000)
    need = lib.nadmm_workspace_bytes(C.byref(prob), None)
    rc = lib.nadmm_line_search(C.byref(prob), fake, fake, fake, 1.0, beta, gamma, max_ls, fake, fake, fake, fake, need, None)
    assert rc == code
    params = nadmm.make_params(armijo_beta=beta, backtrack_gamma=gamma, max_ls=max_ls)
    assert lib.nadmm_local_newton(C.byref(prob), fake, C.byref(params), None, fake, need, None) == code


def test_kernel_path_switch(lib):
    prev = lib.nadmm_set_kernel_path(1)
    assert prev in (0, 1, 2, 3, 4)
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem())) == 1
    assert lib.nadmm_set_kernel_path(7) == nadmm.NADMM_EINVAL
    lib.nadmm_set_kernel_path(0)
    # automatic selection: thin data -> 3, medium width -> 2, wide or many classes -> 4, whatever the alignment of the rows
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=1000, p=20, Cc=3))) == 3
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=60000, p=784, Cc=10))) == 2
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=50000, p=3072, Cc=10))) == 4
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=250000, p=2000, Cc=20))) == 4
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=45, Cc=5))) == 2
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=49, Cc=5))) == 2
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=48, Cc=5, A=0x1004))) == 2      # 4-byte aligned A
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=36, Cc=5))) == 2                 # aligned rows: any p
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=2001, Cc=5))) == 4               # wide and unaligned
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=49, Cc=20))) == 4                # many classes and unaligned
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=45, Cc=20))) == 4
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=49, Cc=20, A=0x1002))) == 1      # A not 4-byte aligned
    # forced: the any-stride variants take narrow rows too, down to one 16-byte piece
    lib.nadmm_set_kernel_path(2)
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=45, Cc=5))) == 2
    assert lib.nadmm_query_kernel_path(C.byref(fake_problem(n=500, p=3, Cc=5))) == nadmm.NADMM_EUNSUPPORTED
    lib.nadmm_set_kernel_path(0)
    # a forced path that cannot take the shape is reported, on the host
    lib.nadmm_set_kernel_path(3)
    fake = C.c_void_p(0x3000)
    wide = fake_problem(n=60000, p=784, Cc=10)
    need = lib.nadmm_workspace_bytes(C.byref(wide), None)
    assert lib.nadmm_hessvec(C.byref(wide), fake, fake, fake, fake, need, None) == nadmm.NADMM_EUNSUPPORTED
    lib.nadmm_set_kernel_path(prev)


# Rows that are not 16-byte aligned or padded: the number is that of the path that runs, so that forcing it is possible and takes
# the same path with the same workspace.
@pytest.mark.parametrize("kw,path", [
    (dict(n=1375000, p=29, Cc=2), 3), (dict(n=1000, p=30, Cc=2), 3),
    # 16-byte aligned rows with padding: number 2 on 2049 to 65535 (393215) of them with more than 16 padded unknowns
    (dict(n=2048, p=30, lda=32, Cc=2), 3), (dict(n=2049, p=30, lda=32, Cc=2), 2), (dict(n=65535, p=15, lda=16, Cc=4), 2),
    (dict(n=65536, p=15, lda=16, Cc=4), 3), (dict(n=393215, p=30, lda=32, Cc=3), 2), (dict(n=393216, p=30, lda=32, Cc=3), 3),
    (dict(n=5000, p=15, lda=16, Cc=2), 3), (dict(n=5000, p=5, lda=8, Cc=4), 2), (dict(n=5000, p=5, lda=8, Cc=3), 3),
    (dict(n=5000, p=15, lda=16, Cc=3, A=0x1004), 3), (dict(n=300, p=3, lda=4, Cc=2), 3), (dict(n=40000, p=3, lda=4, Cc=4), 3),
    (dict(n=1000, p=32, Cc=3, A=0x1004), 3),
    (dict(n=1000, p=24, Cc=4), 2), (dict(n=60000, p=45, Cc=5), 2), (dict(n=60000, p=45, Cc=20), 4), (dict(n=300, p=5, lda=9, Cc=2), 2),
    (dict(n=300, p=3, lda=5, Cc=2), 1), (dict(n=300, p=3, Cc=6), 1), (dict(n=300, p=3, lda=4, Cc=6), 2), (dict(n=1, p=3, Cc=2), 1),
    (dict(n=1000, p=29, Cc=2, A=0x1002), 1), (dict(n=60000, p=785, Cc=10), 2), (dict(n=50000, p=3073, Cc=10), 4)])
def test_queried_path_is_the_one_that_runs(lib, kw, path):
    prob = fake_problem(**kw)
    assert lib.nadmm_query_kernel_path(C.byref(prob)) == path
    need = lib.nadmm_workspace_bytes(C.byref(prob), None)
    lib.nadmm_set_kernel_path(path)
    try:
        assert lib.nadmm_query_kernel_path(C.byref(prob)) == path
        assert lib.nadmm_workspace_bytes(C.byref(prob), None) == need
    finally:
        lib.nadmm_set_kernel_path(0)


def test_static_scratch_entry_point_validates_on_the_host(lib):
    """nadmm_hessvec_static rejects invalid arguments and problems beyond its built-in buffer before any device call."""
    fake = C.c_void_p(0x3000)
    cap = lib.nadmm_static_scratch_bytes()
    assert cap == 32 << 20
    head = fake_problem(n=60000, p=784, Cc=10)
    assert 0 < lib.nadmm_hessvec_static_bytes(C.byref(head)) < 20 << 20           # the headline shape fits
    assert lib.nadmm_hessvec_static_bytes(C.byref(head)) < lib.nadmm_workspace_bytes(C.byref(head), None)
    assert lib.nadmm_hessvec_static(C.byref(head), None, fake, fake, None) == nadmm.NADMM_EINVAL
    assert lib.nadmm_hessvec_static(C.byref(head), fake, fake, None, None) == nadmm.NADMM_EINVAL
    big = fake_problem(n=500000, p=2000, Cc=20)                                     # 50.9 MB of scratch
    assert lib.nadmm_hessvec_static_bytes(C.byref(big)) > cap
    assert lib.nadmm_hessvec_static(C.byref(big), fake, fake, fake, None) == nadmm.NADMM_ESCRATCH
    assert b"built-in" in lib.nadmm_status_string(nadmm.NADMM_ESCRATCH)
    bad = fake_problem(n=0, p=784, Cc=10)
    assert lib.nadmm_hessvec_static_bytes(C.byref(bad)) == 0
    assert lib.nadmm_hessvec_static(C.byref(bad), fake, fake, fake, None) == nadmm.NADMM_EINVAL


def test_scratch_sizes_in_the_header_are_the_library_s(lib):
    figures = re.findall(r"(\d+) x (\d+), C = (\d+) needs ([\d.]+) MB", re.sub(r"\n \*\s*", " ", open(HEADER).read()))
    assert len(figures) == 4
    for n, p, cls, mb in figures:
        got = lib.nadmm_hessvec_static_bytes(C.byref(fake_problem(n=int(n), p=int(p), Cc=int(cls))))
        assert round(got / 1e6, 1) == float(mb), (n, p, cls, got)


PENDING_UPDATES = r"""
#include <cstdio>
#include "nadmm_internal.h"
using namespace nadmm;
int main() {  // every one of these is refused before anything is launched: no device is touched
  static DevState st;
  static float v[4096];
  static double part[64];
  auto call = [&](bool narrow, int p, int NC, bool b0, bool b1, int kind, int ndot, int64_t dlen) {
    RowArgs a{};
    a.A = v; a.n = 100; a.p = p; a.lda = p; a.NC = NC; a.kind = kind; a.Pin = v; a.B0 = b0 ? v : nullptr; a.B1 = b1 ? v : nullptr;
    CgPend c{};
    c.st = &st; c.ndot = ndot; c.dlen = dlen; c.dot_part = part; c.q = v;
    std::printf("%d ", (int)(narrow ? launch_narrow(a, v, 1, nullptr, &c) : launch_fused(a, v, 1, nullptr, &c)));
  };
  for (int narrow = 0; narrow < 2; ++narrow) {
    call(narrow, 64, 5, true, true, kRowsHv, 2, 320);       // X given: the kernel would not look at the update
    call(narrow, 64, 5, false, false, kRowsHv, 2, 320);     // no operand that the update could become
    call(narrow, 64, 5, false, true, kRowsGrad, 2, 320);    // a sweep that takes none
    call(narrow, 64, 5, false, true, kRowsHv, 0, 320);      // no sums of <d, q>
    call(narrow, 64, 5, false, true, kRowsHv, 1000, 320);   // more of them than threads
    call(narrow, 64, 5, false, true, kRowsHv, 2, 319);      // a vector of another length
  }
  call(true, 64, 20, false, true, kRowsHv, 2, 1280);        // two blocks of classes: no kernel with an update
  std::printf("\n");
  return 0;
}
"""

# The driver of Algorithm 3 with stand-ins for the kernel launches, on host memory: every sweep, reduction and line search goes by the
# word that is set at its launch, and the head of iteration `stop` finds the gradient finished.
NEWTON_DRIVER = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "nadmm_internal.h"
namespace nadmm {
static int stop_at, grads, directions, steps, heads, shared;  // shared: heads that wrote a word their own kernel goes by
static double last_gg;
static bool on(const int32_t* flag) { return flag == nullptr || *flag != 0; }
static void head(const NewtonHeadArgs& h, const int32_t* flag) {
  const int32_t before = flag != nullptr ? *flag : 0;
  if (*newton_entered(h.st, h.iter) == 0) newton_head_skipped(h);
  else newton_head_scalars(h, h.iter == stop_at ? last_gg : 1.0, 2.0);
  if (flag != nullptr) {
    shared += *flag != before || flag != newton_entered(h.st, h.iter);
    ++heads;
  }
}
static const int32_t* swept_by;  // what the last product went by
static hipError_t rows(const RowArgs& a) {
  if (on(a.flag) && a.kind == kRowsGrad) ++grads;
  if (a.kind == kRowsHv) swept_by = a.flag;
  return hipSuccess;
}
hipError_t launch_state_init(DevState* st, const int32_t* outer, hipStream_t) {
  st->newton_even = st->newton_odd = outer != nullptr ? *outer : 1;
  return hipSuccess;
}
hipError_t launch_generic_rows(const RowArgs& a, hipStream_t) { return rows(a); }
hipError_t launch_generic_cols(const ColArgs&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_fused(const RowArgs& a, float*, int, hipStream_t, const CgPend*, const SearchArgs*) { return rows(a); }
hipError_t launch_narrow(const RowArgs& a, float*, int, hipStream_t, const CgPend*) { return rows(a); }
hipError_t launch_wide(const RowArgs& a, void*, bool, float*, int, hipStream_t) { return rows(a); }
// A CG update by several workgroups: up to 131072 unknowns the state's slots and the two residuals take turns, beginning with slot 0, and the
// product and its reduction before it went by the slot that it reads; beyond, everything stays in place.
static int updates, off_turn, turn;
static const float *residual, *next_residual, *summed;
static hipError_t update(const CgUpdateArgs& a) {
  ++updates;
  if (cg_one_step(a.d)) {
    if (turn == 0) residual = a.r;
    else off_turn += a.r != next_residual;
    off_turn += a.slot_in != (turn & 1) || a.r_out == nullptr || a.r_out == a.r || ((turn & 1) == 0) != (a.r == residual);
    off_turn += swept_by != &a.st->cgs[a.slot_in].active || summed != a.r || a.ndot != reduce_out_blocks(a.d);
    next_residual = a.r_out;
  } else {
    off_turn += a.r_out != nullptr || summed != nullptr || swept_by != &a.st->cg_active;
  }
  ++turn;
  return hipSuccess;
}
hipError_t launch_wide_direction(const CgUpdateArgs& a, const Shape&, void*, hipStream_t) { return update(a); }
hipError_t launch_sliced_logits(const RowArgs& a, hipStream_t) { return rows(a); }
hipError_t launch_sliced_cols(const RowArgs&, const float*, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_thin(const RowArgs& a, float*, int, hipStream_t, const CgPend* cg, const ReduceArgs*, const NewtonHeadArgs* h, const SearchArgs*) {
  rows(a);
  if (h != nullptr) head(*h, a.flag);
  if (cg != nullptr) {
    if (cg->st->cgs[cg->slot_in].active != 0 && cg->final_p == 0) ++directions;
    cg->st->cgs[cg->slot_in ^ 1] = cg->st->cgs[cg->slot_in];
  }
  return hipSuccess;
}
hipError_t launch_reduce_out(const ReduceArgs& r, hipStream_t) {
  if (r.kind == 0) {
    summed = r.r_dot;
    off_turn += r.dot_part != nullptr && r.has_head == 0 && r.cur == nullptr && r.flag != swept_by;
  }
  if (r.has_head != 0) head(r.head, r.flag);
  return hipSuccess;
}
hipError_t launch_newton_head(const NewtonHeadArgs& h, hipStream_t) {
  turn = 0;  // a CG solve begins
  head(h, nullptr);
  return hipSuccess;
}
hipError_t launch_cg_reduce_update(const ReduceArgs&, const CgUpdateArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_cg_update(const CgUpdateArgs& a, hipStream_t) { return update(a); }
hipError_t launch_sparse_plan(const SparseView&, const SparseWindows&, const SparseView&, const SparseWindows&, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_sparse_pack(const float*, const float*, int64_t, int, float*, const int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_spmm(const SpmmArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_logit_rows(const RowArgs& a, const float*, int, int, hipStream_t) { return rows(a); }
hipError_t launch_cg_pending_finish(const CgPend&, hipStream_t) { return hipSuccess; }
hipError_t launch_ls_eval(const LsEvalArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_ls_tail(const LsTailArgs& a, hipStream_t) { steps += on(a.flag); return hipSuccess; }
}  // namespace nadmm
using namespace nadmm;
int main() {
  struct Case { int64_t n; int32_t p, C, path; } cases[] = {{5000, 28, 2, 0}, {5000, 29, 3, 0}, {60000, 784, 10, 0}, {100000, 70, 7, 0},
                                                            {5000, 90, 20, 0}, {5000, 1100, 4, 0}, {5000, 28, 2, 1}, {5000, 3072, 10, 0}, {500, 4096, 33, 0},
                                                            {100, 4097, 33, 0}, {100, 5000, 3, 1}, {100, 2000, 21, 5}, {100, 131073, 2, 5}};
  nadmm_sparse sparse{};
  alignas(16) static float v[4];
  static int32_t labels[4];
  for (const Case& c : cases)
    for (int max_cg : {0, 1, 3})
      for (double gg : {0.0, 1e-12, std::nan("")})
        for (stop_at = 0; stop_at <= 4; ++stop_at) {  // 4: never
          nadmm_problem prob{};
          prob.d_A = v; prob.n = c.n; prob.p = c.p; prob.lda = c.p; prob.d_labels = labels; prob.C = c.C;
          prob.loss_scale = 1.f; prob.rho = 1.f;
          nadmm_params params{};
          params.max_newton = 4; params.max_cg = max_cg; params.max_ls = 10; params.grad_tol = 1e-3f;
          params.armijo_beta = 1e-4f; params.backtrack_gamma = 0.5f;
          if (c.path == 5) {
            static int64_t ptr[2];
            sparse.nnz = 1000; sparse.d_row_ptr = sparse.d_col_ptr = ptr; sparse.d_col_idx = sparse.d_row_idx = labels; sparse.d_val = sparse.d_val_t = v;
            prob.sparse = &sparse;
          }
          nadmm_set_kernel_path(c.path);
          const size_t bytes = nadmm_workspace_bytes(&prob, &params);
          void* ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
          grads = directions = steps = shared = updates = off_turn = 0;
          last_gg = gg;
          const int rc = nadmm_local_newton(&prob, v, &params, nullptr, ws, bytes, nullptr);
          std::free(ws);
          const bool thin = c.path == 0 && c.p <= 32;
          const bool several = c.p > 1000 || c.p == 90;  // these vectors are updated by several workgroups
          if (rc != 0 || shared != 0 || off_turn != 0 || updates != (several ? 4 * max_cg : 0) || steps != stop_at || grads != (stop_at < 4 ? stop_at + 1 : 4) ||
              (thin && max_cg == 3 && directions != 2 * stop_at)) {
            std::printf("n %ld p %d C %d path %d cg %d stop %d: rc %d shared %d steps %d grads %d directions %d updates %d, %d off their turn\n", (long)c.n, c.p, c.C,
                        c.path, max_cg, stop_at, rc, shared, steps, grads, directions, updates, off_turn);
            return 1;
          }
        }
  std::printf("heads %d\n", heads);  // made by a workgroup of another kernel
  return heads > 0 ? 0 : 1;
}
"""

# Which kernels a gradient launches, with stand-ins for the launches.  Arguments: n p lda C, path to force.
ROUTES = r"""
#include <cstdio>
#include <cstdlib>
#include "nadmm_internal.h"
namespace nadmm {
static const char* taken = "other";
hipError_t launch_thin(const RowArgs&, float*, int, hipStream_t, const CgPend*, const ReduceArgs*, const NewtonHeadArgs*, const SearchArgs*) {
  taken = "thin";
  return hipSuccess;
}
hipError_t launch_narrow(const RowArgs&, float*, int, hipStream_t, const CgPend*) { taken = "narrow"; return hipSuccess; }
hipError_t launch_fused(const RowArgs&, float*, int, hipStream_t, const CgPend*, const SearchArgs*) { taken = "fused"; return hipSuccess; }
hipError_t launch_reduce_out(const ReduceArgs&, hipStream_t) { return hipSuccess; }
}  // namespace nadmm
int main(int argc, char** argv) {
  alignas(16) static float v[4];
  static double loss;
  static int32_t labels[4];
  for (int i = 1; i + 4 < argc; i += 5) {
    nadmm_problem prob{};
    prob.d_A = v; prob.n = std::atoll(argv[i]); prob.p = std::atoi(argv[i + 1]); prob.lda = std::atoi(argv[i + 2]); prob.C = std::atoi(argv[i + 3]);
    prob.d_labels = labels; prob.loss_scale = 1.f; prob.rho = 1.f;
    nadmm_set_kernel_path(std::atoi(argv[i + 4]));
    const size_t bytes = nadmm_workspace_bytes(&prob, nullptr);
    void* ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    const int rc = nadmm_loss_grad(&prob, v, &loss, v, ws, bytes, nullptr);
    std::printf("%s%d ", nadmm::taken, rc != 0 ? rc : nadmm_query_kernel_path(&prob));
    std::free(ws);
  }
  return 0;
}
"""

PARTIALS = r"""
#include <cstdio>
#include "nadmm_internal.h"
int main() {  // workgroups of the kernel for narrow rows, one and two blocks of classes, at the edges of 2 to 9 rounds each
  for (int p : {9, 32, 33, 64, 65, 96})
    for (int NC : {3, 16, 17, 32})
      for (int rounds = 1; rounds <= 9; ++rounds)
        for (int past : {0, 1}) {
          const int64_t round = p <= 32 ? (NC > 16 ? 128 : 256) : (p <= 64 && NC <= 16 ? 128 : 64);
          nadmm::Shape s{};
          s.n = 512 * round * rounds + past; s.p = p; s.NC = NC; s.d = (int64_t)p * NC;
          const int per = rounds + past, total = 512 * rounds + past;
          const int want = per >= 3 && per <= 8 ? 512 : (total + per - 1) / per;  // else equally many rounds each
          if (nadmm::narrow_num_partials(s) != want) {
            std::printf("p %d NC %d n %lld: %d, not %d\n", p, NC, (long long)s.n, nadmm::narrow_num_partials(s), want);
            return 1;
          }
        }
  return 0;
}
"""

LDS_MASK = r"""
#include <thread>
#include <vector>
#include "nadmm_internal.h"
// stand-ins for the runtime: the function under test is the header's
static thread_local int device = 0;
hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
static nadmm::LdsLimitMask mask;
int main() {
  std::vector<std::thread> ts;
  for (int k = 0; k < 8; ++k) ts.emplace_back([k] { device = k; for (int i = 0; i < 1000; ++i) nadmm::ensure_lds_limit(nullptr, &mask); });
  for (auto& t : ts) t.join();
  return mask.load() == 0xff ? 0 : 1;
}
"""
GXX = ["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{os.path.join(ROOT, 'include')}",
       f"-I{os.path.join(ROOT, 'paper_1807_07132_amd', 'csrc')}", "-Wno-unused-result"]


def test_a_pending_cg_update_that_a_kernel_would_not_apply_is_refused(lib, tmp_path):
    src, exe = tmp_path / "pending.cpp", tmp_path / "pending"
    src.write_text(PENDING_UPDATES)
    subprocess.check_call([*GXX, str(src), nadmm.LIB_PATH, f"-Wl,-rpath,{os.path.dirname(nadmm.LIB_PATH)}", "-Wl,--allow-shlib-undefined",
                           "-o", str(exe)])
    assert subprocess.check_output([str(exe)], timeout=60).split() == [b"1"] * 13      # hipErrorInvalidValue


def test_no_kernel_writes_the_word_its_workgroups_go_by(lib, tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(NEWTON_DRIVER)
    subprocess.check_call([*GXX, "-O1", str(src), nadmm.LIB_PATH, f"-Wl,-rpath,{os.path.dirname(nadmm.LIB_PATH)}", "-Wl,--allow-shlib-undefined",
                           "-o", str(exe)])
    run = subprocess.run([str(exe)], timeout=60, capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_aligned_thin_rows_with_padding_take_the_thin_kernel_under_either_number(lib, tmp_path):
    src, exe = tmp_path / "routes.cpp", tmp_path / "routes"
    src.write_text(ROUTES)
    subprocess.check_call([*GXX, "-O1", str(src), nadmm.LIB_PATH, f"-Wl,-rpath,{os.path.dirname(nadmm.LIB_PATH)}", "-Wl,--allow-shlib-undefined",
                           "-o", str(exe)])
    cases, want = [], []
    for n, p, lda, cls, number in ((2048, 30, 32, 2, 3), (2049, 30, 32, 2, 2), (65535, 15, 16, 4, 2), (65536, 15, 16, 4, 3), (393215, 30, 32, 3, 2),
                                   (393216, 30, 32, 3, 3), (5000, 5, 8, 4, 2), (5000, 5, 8, 3, 3), (40000, 30, 32, 3, 2)):
        cases += [(n, p, lda, cls, path) for path in ((0, 2, 3) if number == 2 else (0, 3))]
        want += ["thin2", "thin2", "thin3"] if number == 2 else ["thin3", "thin3"]
    cases += [(2048, 30, 32, 2, 2), (65536, 15, 16, 4, 2), (5000, 32, 32, 2, 2)]      # the matrix-core kernels by force, as for dense rows
    want += ["fused2", "narrow2", "fused2"]
    got = subprocess.check_output([str(exe), *[str(v) for c in cases for v in c]], timeout=60, text=True).split()
    assert got == want, list(zip(cases, got, want))


def test_narrow_rows_workgroups_of_one_and_two_blocks_of_classes(lib, tmp_path):
    src, exe = tmp_path / "partials.cpp", tmp_path / "partials"
    src.write_text(PARTIALS)
    subprocess.check_call([*GXX, str(src), nadmm.LIB_PATH, f"-Wl,-rpath,{os.path.dirname(nadmm.LIB_PATH)}", "-Wl,--allow-shlib-undefined",
                           "-o", str(exe)])
    run = subprocess.run([str(exe)], timeout=60, capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_lds_limit_is_noted_without_a_race(tmp_path):
    src, exe = tmp_path / "mask.cpp", tmp_path / "mask"
    src.write_text(LDS_MASK)
    subprocess.check_call([*GXX, "-g", "-O1", "-fsanitize=thread", "-pthread", str(src), "-o", str(exe)])
    run = subprocess.run([str(exe)], timeout=60, capture_output=True, text=True)       # a reported race fails the program
    if "unexpected memory mapping" in run.stderr:
        pytest.skip("the thread sanitizer does not start on this kernel's address layout")
    assert run.returncode == 0, run.stderr


def test_traffic_figures_go_by_every_file_their_kernels_include(tmp_path):
    """The benchmark reports traffic measured with the sources as they are: a change of any file that a path's kernels include counts."""
    import importlib.util
    import shutil
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    csrc = tmp_path / "csrc"
    shutil.copytree(os.path.join(ROOT, "paper_1807_07132_amd", "csrc"), csrc)
    flags = [f if "csrc" not in f else f"-I{csrc}" for f in GXX]
    for path, sources in bench.PATH_SOURCES.items():
        deps = subprocess.check_output([*flags, "-MM", "-x", "c++", *[str(csrc / s) for s in sources], str(csrc / "nadmm_vec.hip")], text=True)
        files = {os.path.basename(f) for f in deps.replace("\\\n", " ").split() if os.path.dirname(f) == str(csrc)}
        assert "nadmm_internal.h" in files and set(sources) <= files
        before = bench.source_digest(path, str(csrc))
        assert before == bench.source_digest(path)
        for f in files:
            kept = (csrc / f).read_bytes()
            (csrc / f).write_bytes(kept + b"\n// changed\n")
            assert bench.source_digest(path, str(csrc)) != before, (path, f)
            (csrc / f).write_bytes(kept)


def test_product_path_does_not_import_the_oracle():
    code = ("import sys; sys.path.insert(0, %r); import paper_1807_07132_amd.nadmm, paper_1807_07132_amd.workloads;"
            "assert not any(m == 'oracle' or m.startswith('oracle.') for m in sys.modules)" % ROOT)
    subprocess.check_call([sys.executable, "-c", code])


def test_admm_host_validation(lib):
    params = nadmm.make_admm_params(3, nadmm.make_params(2, 5, 10))
    fake = C.c_void_p(0x4000)
    workers = (nadmm.nadmm_problem * 3)(*[fake_problem(n=500 + 10 * i) for i in range(3)])
    need = lib.nadmm_admm_workspace_bytes(workers, 3, C.byref(params))
    single = max(lib.nadmm_workspace_bytes(C.byref(workers[i]), None) for i in range(3))
    assert need > single
    assert lib.nadmm_admm_workspace_bytes(workers, 0, C.byref(params)) == 0
    assert lib.nadmm_admm_workspace_bytes(workers, nadmm.NADMM_MAX_WORKERS + 1, C.byref(params)) == 0
    call = lambda w, N, lam, prm, ws: lib.nadmm_admm_solve(w, N, lam, fake, fake, fake, C.byref(prm), None, fake, ws, None)
    assert call(workers, 3, 0.1, params, need - 1) == nadmm.NADMM_EWORKSPACE
    assert call(workers, 3, -0.1, params, need) == nadmm.NADMM_EINVAL
    bad = nadmm.make_admm_params(-1, nadmm.make_params(2, 5, 10))
    assert call(workers, 3, 0.1, bad, need) == nadmm.NADMM_EINVAL
    for kw in (dict(penalty_rule=2), dict(penalty_rule=1, rb_mu=0.5), dict(penalty_rule=1, rb_tau=1.0),
               dict(penalty_rule=1, rb_tau=float("nan"))):
        assert call(workers, 3, 0.1, nadmm.make_admm_params(3, nadmm.make_params(2, 5, 10), **kw), need) == nadmm.NADMM_EINVAL
    mixed = (nadmm.nadmm_problem * 2)(fake_problem(p=20), fake_problem(p=24))     # shards must agree in p and C
    assert lib.nadmm_admm_workspace_bytes(mixed, 2, C.byref(params)) == 0
    rho = (C.c_float * 2)(1.0, -1.0)
    assert lib.nadmm_admm_consensus(2, 40, fake, fake, fake, rho, 0.1, 0.0, 0.0, None, fake, 1 << 16, None) == nadmm.NADMM_EINVAL
    rho = (C.c_float * 2)(1.0, 1.0)
    assert lib.nadmm_admm_consensus(2, 40, fake, fake, fake, rho, 0.1, 0.0, 0.0, None, fake, 16, None) == nadmm.NADMM_EWORKSPACE


def test_kernel_path_switch_is_per_thread(lib):
    """The forced kernel path belongs to the calling host thread: another thread still sees the automatic choice."""
    import threading
    assert lib.nadmm_set_kernel_path(2) == 0
    try:
        seen = []
        t = threading.Thread(target=lambda: seen.append(lib.nadmm_set_kernel_path(1)))
        t.start()
        t.join()
        assert seen == [0]                                # the other thread's previous value: untouched by this one
        assert lib.nadmm_set_kernel_path(2) == 2          # and its own setting did not reach this thread
    finally:
        lib.nadmm_set_kernel_path(0)
