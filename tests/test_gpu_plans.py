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
