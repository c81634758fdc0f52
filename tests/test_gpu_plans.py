"""SpMV plans: what the plan queries report is what is launched, and a plan
that was tuned or set is taken by every system of its class."""
import numpy as np
import pytest
import torch

from paper_1708_01773_amd import fe as F
from tests.gpu_util import Pair, rel, say

pytestmark = pytest.mark.gpu


def _timed_spmv(solve):
    """(solution, info, SpMV launches timed): every 16th iteration of the three-kernel form is timed."""
    F.set_timing(True)
    try:
        F.get_timing(reset=True)
        x, info = solve()
        torch.cuda.synchronize()
        return x, info, F.get_timing(reset=True)["spmv_calls"]
    finally:
        F.set_timing(False)


# A system small enough for the one-workgroup solver takes a plan that was set
# or tuned for its class, through the CSR and with the pattern evaluated.
@pytest.mark.parametrize("dim,n,k,prob", [(2, [33, 32], 1, "poisson"), (3, [4, 4, 5], 2, "poisson"),
                                          (3, [3, 3, 2], 2, "elasticity")])
@pytest.mark.parametrize("how", ["set", "tuned"])
def test_small_systems_take_the_plan_of_their_class(dim, n, k, prob, how):
    pair = Pair(dim, n, k, prob, seed=91)
    A = pair.gpu_assembly()
    say(f"[small plan] dim {dim} n {n} k {k} {prob} rows {A.n_rows} {how}")
    assert A.n_rows <= 4096
    ws = torch.empty(F.pcg_query(A.n_rows), dtype=torch.uint8, device="cuda")

    def csr():
        x = torch.zeros(A.n_rows, dtype=torch.float64, device="cuda")
        return x, F.pcg_solve(A.csr, A.rhs, x, 1e-11, 5000, ws)

    def mesh():
        x = torch.zeros(A.n_rows, dtype=torch.float64, device="cuda")
        return x, A.solve(x, 1e-11, 5000, ws)

    F.spmv_tuning_reset()
    try:
        for solve in (csr, mesh):
            x0, i0, calls = _timed_spmv(solve)
            assert i0["status"] == F.FE_OK and calls == 0
            if how == "tuned" and solve is csr:
                F.spmv_autotune(A.csr, reps=2)
            elif how == "tuned":
                F.spmv_autotune_mesh(pair.mesh, k, pair.coeff, A.csr, reps=2)
            elif solve is csr:
                F.spmv_plan_set(A.n_rows, A.nnz, 0, 4)
            else:
                F.spmv_plan_set_mesh(pair.mesh, k, pair.coeff, 2, 8)
            x1, i1, calls = _timed_spmv(solve)
            assert i1["status"] == F.FE_OK and calls == (i1["iters"] + 15) // 16
            assert abs(i1["iters"] - i0["iters"]) <= 1
            assert rel(x1.cpu().numpy(), x0.cpu().numpy()) <= 1e-8
    finally:
        F.spmv_tuning_reset()


def _abs_product(A, x):
    c = F.csr_struct(A.n_rows, A.nnz, A.rowptr, A.colind, A.values[: A.nnz].abs(), A.rhs, A.dinv)
    y = torch.empty_like(x)
    F.spmv(c, x.abs(), y)
    return y


# The reported plan is the launched one: setting it leaves the product as it
# is.  Rows of 9 to 290 entries; in 2D Q2, 2042 and 2054 tiles of 256 rows (below
# 2048 smaller tiles are taken); rows below and from 96 and 256 entries; at most
# 1024 rows (tiles by the row length alone) and more.  The product is that of one
# wave per row up to rounding.
@pytest.mark.parametrize("dim,n,k,prob,plan", [(2, [100, 90], 1, "poisson", (9, 256)), (2, [60, 50], 2, "poisson", (9, 128)),
                                               (2, [362, 362], 2, "poisson", (9, 128)), (2, [363, 363], 2, "poisson", (9, 256)),
                                               (3, [11, 11, 11], 1, "poisson", (9, 256)), (3, [12, 11, 11], 1, "poisson", (9, 64)),
                                               (3, [17, 17, 18], 1, "poisson", (9, 64)), (3, [9, 8, 10], 2, "poisson", (9, 32)),
                                               (3, [6, 5, 7], 3, "poisson", (9, 16)), (3, [9, 8, 9], 3, "poisson", (9, 16)),
                                               (3, [6, 5, 5], 2, "elasticity", (9, 16)), (3, [6, 6, 7], 2, "elasticity", (9, 16)),
                                               (3, [4, 5, 4], 3, "elasticity", (9, 8)), (3, [6, 5, 6], 3, "elasticity", (1, 1)),
                                               (2, [3, 3], 2, "poisson", (9, 256)), (2, [2, 2], 1, "poisson", (9, 256))])
def test_reported_csr_plan_is_the_launched_one(dim, n, k, prob, plan):
    pair = Pair(dim, n, k, prob, seed=92)
    A = pair.gpu_assembly()
    say(f"[csr plan] dim {dim} n {n} k {k} {prob} rows {A.n_rows} nnz {A.nnz}")
    x = torch.from_numpy(np.random.Generator(np.random.PCG64(93)).standard_normal(A.n_rows)).cuda()
    y0, y1, y2 = (torch.full_like(x, float("nan")) for _ in range(3))
    F.spmv_tuning_reset()
    try:
        mode, rpw, _ = F.spmv_plan_of(A.n_rows, A.nnz)
        assert (mode, rpw) == plan
        F.spmv(A.csr, x, y0)
        F.spmv_plan_set(A.n_rows, A.nnz, mode, rpw)
        F.spmv(A.csr, x, y1)
        F.spmv_plan_set(A.n_rows, A.nnz, 1, 1)
        F.spmv(A.csr, x, y2)
        scale = _abs_product(A, x)
        torch.cuda.synchronize()
    finally:
        F.spmv_tuning_reset()
    assert torch.equal(y0, y1)
    # a row of m entries, summed in two orders: each within m eps of the sum of magnitudes (m < 700)
    assert bool(torch.all((y0 - y2).abs() <= 2 * 700 * 2.0 ** -53 * scale))


# The same for the evaluated pattern.  Scalar order 2: two chunks a block (24^3,
# 5x60x60) and more (25^3, 6x64x64), values below and past what stays cached (38^3,
# 39^3); orders 3 and 4 below and past a chunk for each CU; vector and 2D classes.
# Plans (2, 8) and (6, 8) give the same products to the last bit.
@pytest.mark.parametrize("dim,n,k,prob,plan", [(3, [24, 24, 24], 2, "poisson", (6, 8)), (3, [25, 25, 25], 2, "poisson", (2, 8)),
                                               (3, [5, 60, 60], 2, "poisson", (6, 8)), (3, [6, 64, 64], 2, "poisson", (2, 8)),
                                               (3, [38, 38, 38], 2, "poisson", (2, 8)), (3, [39, 39, 39], 2, "poisson", (6, 8)),
                                               (3, [8, 8, 8], 3, "poisson", (2, 8)), (3, [9, 9, 9], 3, "poisson", (6, 8)),
                                               (3, [6, 6, 6], 4, "poisson", (2, 8)), (3, [7, 7, 7], 4, "poisson", (6, 8)),
                                               (3, [5, 6, 7], 2, "elasticity", (6, 4)), (2, [40, 30], 3, "poisson", (2, 8)),
                                               (3, [9, 8, 7], 1, "poisson", (4, 27))])
def test_reported_mesh_plan_is_the_launched_one(dim, n, k, prob, plan):
    pair = Pair(dim, n, k, prob, jitter=0.1, seed=94)
    A = pair.gpu_assembly()
    say(f"[mesh plan] dim {dim} n {n} k {k} {prob} rows {A.n_rows} nnz {A.nnz}")
    x = torch.from_numpy(np.random.Generator(np.random.PCG64(95)).standard_normal(A.n_rows)).cuda()
    ys = []
    F.spmv_tuning_reset()
    try:
        rep = F.spmv_plan_of_mesh(pair.mesh, k, pair.coeff)[:2]
        assert rep == plan
        plans = [None, rep] + ([(2, 8), (6, 8)] if plan[1] == 8 else [])
        for p in plans:
            if p:
                F.spmv_plan_set_mesh(pair.mesh, k, pair.coeff, *p)
                assert F.spmv_plan_of_mesh(pair.mesh, k, pair.coeff)[:2] == p
            y = torch.full_like(x, float("nan"))
            F.spmv_mesh(pair.mesh, k, pair.coeff, A.csr, x, y)
            ys.append(y)
        yc = torch.empty_like(x)
        F.spmv(A.csr, x, yc)
        scale = _abs_product(A, x)
        torch.cuda.synchronize()
    finally:
        F.spmv_tuning_reset()
    assert all(torch.equal(y, ys[0]) for y in ys[1:])
    assert bool(torch.all((ys[0] - yc).abs() <= 2 * 800 * 2.0 ** -53 * scale))  # rows of at most 729 entries
