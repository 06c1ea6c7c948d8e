"""nadmm_hessvec_static: the Hessian-vector product on the library's built-in scratch buffer (for callers that cannot
allocate) against nadmm_hessvec with a caller-allocated workspace and against the float64 oracle.  Two calls in a row,
the second on a smaller problem, on every kernel path; this file is collected last so that the rest of the suite has
already run in the same process when it does, and it passes in a fresh process too."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

from oracle import nadmm_oracle as orc
from paper_1807_07132_amd import nadmm, workloads
from parity_utils import TOL_PRIMITIVE, oracle_problem, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_path():
    yield
    nadmm.nadmm_set_kernel_path(0)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


PAIRS = {
    # name: (larger problem, smaller problem run right after it on the same buffer, kernel path[, forced])
    "fused": (lambda: workloads.image_like(0, n=9000), lambda: workloads.generic(700, 100, 7, seed=12), 2),
    "thin": (lambda: workloads.tall_binary(0, n=60011), lambda: workloads.generic(300, 12, 4, seed=19), 3),
    "sliced": (lambda: workloads.wide(0, n=2100), lambda: workloads.generic(300, 1100, 4, seed=25, x_std=0.05), 4),
    # narrow rows that are not 16-byte aligned: the kernel for them and the thin-data kernel; the vector kernels by force
    "narrow": (lambda: workloads.generic(1237, 45, 5, seed=3), lambda: workloads.generic(65, 33, 3, seed=10), 2),
    "thin_odd": (lambda: workloads.generic(60011, 29, 2, seed=3), lambda: workloads.generic(300, 13, 4, seed=19), 3),
    "vector": (lambda: workloads.generic(1237, 45, 5, seed=3), lambda: workloads.generic(65, 33, 3, seed=10), 1, True),
    "sparse": (lambda: workloads.sparse_generic(800, 1500, 6, 25, seed=1), lambda: workloads.sparse_generic(200, 300, 4, 10, seed=2), 5),
}


@pytest.mark.parametrize("name", list(PAIRS))
def test_static_scratch_matches_the_workspace_call(name):
    big, small, path = PAIRS[name][:3]
    nadmm.nadmm_set_kernel_path(path if len(PAIRS[name]) > 3 else 0)
    outs = []
    for make in (big, small, big):         # larger, smaller, larger again: stale contents of the buffer must not matter
        w = make()
        gp = nadmm.Problem.from_workload(w)
        assert nadmm.nadmm_query_kernel_path(gp) == path
        assert 0 < nadmm.nadmm_hessvec_static_bytes(gp) <= nadmm.nadmm_static_scratch_bytes()
        X, V = dev(w.X0), dev(w.V)
        want = nadmm.nadmm_hessvec(gp, X, V)
        got = torch.full_like(want, float("nan"))
        nadmm.nadmm_hessvec_static(gp, X, V, got)
        torch.cuda.synchronize()
        assert torch.equal(got, want)       # same kernels in the same order: bit for bit
        assert rel_l2(got.cpu().numpy(), orc.hessvec(oracle_problem(w), w.X0, w.V)) <= TOL_PRIMITIVE
        outs.append(got)
    assert torch.equal(outs[0], outs[2])


def test_static_scratch_at_the_headline_shape_and_rejection_beyond_the_buffer():
    w = workloads.image_like(0)
    gp = nadmm.Problem.from_workload(w)
    nadmm.nadmm_set_kernel_path(0)
    assert nadmm.nadmm_hessvec_static_bytes(gp) < 20 << 20
    X, V = dev(w.X0), dev(w.V)
    want = nadmm.nadmm_hessvec(gp, X, V)
    got = torch.empty_like(want)
    before = torch.cuda.memory_allocated()
    for _ in range(3):
        nadmm.nadmm_hessvec_static(gp, X, V, got)
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == before
    assert torch.equal(got, want)
    # a share whose rows of D alone exceed the buffer: rejected on the host, nothing enqueued
    n_big = nadmm.nadmm_static_scratch_bytes() // (4 * 9) + 1
    fake = nadmm.Problem(gp.A, gp.labels, w.C, w.s, w.lam, w.rho, gp.z, gp.y)
    fake.c.n = n_big
    with pytest.raises(nadmm.NadmmError) as ei:
        nadmm.nadmm_hessvec_static(fake, X, V, got)
    assert ei.value.code == nadmm.NADMM_ESCRATCH


def test_static_scratch_where_only_two_sweeps_fit():
    """Wide rows whose 256 partial sums exceed the buffer: nadmm_hessvec makes one sweep, the static call two.  Products with V
    and with D carry 2^-16 per term in both, which bounds the difference by four times that."""
    w = workloads.generic(8192, 2048, 17, seed=8, x_std=0.5 / 2048 ** 0.5, mean=True)
    gp = nadmm.Problem.from_workload(w)
    need = nadmm.nadmm_hessvec_static_bytes(gp)
    assert need <= nadmm.nadmm_static_scratch_bytes() and need < 4 * 2048 * 16 * 256   # no room for the partial sums of the single pass
    X, V = dev(w.X0), dev(w.V)
    want = nadmm.nadmm_hessvec(gp, X, V)
    got = torch.full_like(want, float("nan"))
    nadmm.nadmm_hessvec_static(gp, X, V, got)
    again = torch.full_like(want, float("nan"))
    nadmm.nadmm_hessvec_static(gp, X, V, again)
    torch.cuda.synchronize()
    assert torch.equal(got, again)
    ref = orc.hessvec(oracle_problem(w), w.X0, w.V)
    assert rel_l2(got.cpu().numpy(), ref) <= TOL_PRIMITIVE and rel_l2(want.cpu().numpy(), ref) <= TOL_PRIMITIVE
    assert rel_l2(got.cpu().numpy(), want.cpu().numpy().astype("float64")) <= 4 * 2.0 ** -16


@pytest.mark.parametrize("n,C", [(86000, 33), (172000, 17), (244000, 10)])
def test_static_scratch_without_room_for_the_shares_of_long_rows(n, C):
    """Sparse storage where the sums that workgroups share do not fit the buffer and everything else does: rows and columns of several windows are
    then summed by one workgroup, in the same order.  Two operands in two passes (C-1 > 16) and in one; lengths around and far beyond a window."""
    p, NC = 3000, C - 1
    rng = np.random.default_rng(C)
    group = 4 * (8 if NC > 16 else 4)
    nnz = 12 * n
    cols = np.minimum((p * rng.random(nnz) ** 3).astype(np.int64), p - 1)     # columns of some hundred to tens of thousands of entries
    rows = rng.integers(0, n, size=nnz)
    full = np.concatenate([np.full(k, i) for i, k in zip((5, 6, 7, n - 2), (3000, 2048, 1024, 2999))])   # rows of several windows
    A = sp.csr_matrix((np.ones(nnz + len(full), np.float32), (np.concatenate([rows, full]), np.concatenate([cols, *[np.arange(k) for k in (3000, 2048, 1024, 2999)]]))),
                      shape=(n, p))
    A.data[:] = rng.standard_normal(A.nnz) * 0.2
    b = rng.integers(0, C, size=n).astype(np.int32)
    X = (rng.standard_normal((p, NC)) * 0.1).astype(np.float32)
    V = rng.standard_normal((p, NC)).astype(np.float32)
    gp = nadmm.Problem(nadmm.SparseA.from_scipy(A, A.tocsc()), dev(b), C, 1.0, 1e-3, 1.0, None, None)
    used = 4 * (2 * n * NC + group * max(n, 2 * p) + p * NC)
    need = nadmm.nadmm_hessvec_static_bytes(gp)
    windows = [(A.nnz + 8 * m) >> 11 for m in (n, p)]                         # there are no fewer
    assert need <= nadmm.nadmm_static_scratch_bytes() < need + 16 * NC * max(windows)
    assert need < used + 64 * max(windows)                                    # tables and no shares
    want = nadmm.nadmm_hessvec(gp, dev(X), dev(V))
    got = torch.full_like(want, float("nan"))
    for _ in range(2):
        nadmm.nadmm_hessvec_static(gp, dev(X), dev(V), got)
        torch.cuda.synchronize()
        assert torch.equal(got, want)       # the same additions in the same order
    op = orc.Problem(A, b, C, s=1.0, lam=1e-3, rho=1.0)
    assert rel_l2(got.cpu().numpy(), orc.hessvec(op, X, V)) <= TOL_PRIMITIVE
