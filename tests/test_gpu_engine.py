"""The PCG engine's loop: chunks of iterations, the stop counter, limits."""
import pytest
import torch

from paper_1708_01773_amd import fe as F
from tests.gpu_util import Pair, say

pytestmark = pytest.mark.gpu


def test_long_solves_stop_where_the_allocation_free_solve_does():
    """The counter of a long solve is read every 8 to 64 iterations, that of the
    allocation-free solve after chunks of 8 doubling to 128: the iterates must
    not depend on it, neither at convergence nor at an iteration limit inside,
    at the end of and past the chunks."""
    pair = Pair(2, [24, 22], 4, "elasticity", seed=111, source=(0.3, -1.0))
    A = pair.gpu_assembly()
    ws = torch.empty(F.pcg_query(A.n_rows), dtype=torch.uint8, device="cuda")
    x, y = (torch.zeros(A.n_rows, dtype=torch.float64, device="cuda") for _ in range(2))
    info = F.pcg_solve(A.csr, A.rhs, x, 1e-12, 50000, ws)
    say(f"[long solve] rows {A.n_rows} iters {info['iters']}")
    assert A.n_rows > 4096 and info["status"] == F.FE_OK and info["iters"] > 1024
    assert F.pcg_solve_noalloc(A.csr, A.rhs, y, 1e-12, 50000) == info and torch.equal(x, y)
    for maxit in (1, 8, 9, 600, 1025, info["iters"] - 1, info["iters"], info["iters"] + 1):
        x.zero_()
        y.zero_()
        i = F.pcg_solve(A.csr, A.rhs, x, 1e-12, maxit, ws, check=False)
        assert i["iters"] == min(maxit, info["iters"])
        assert i["status"] == (F.FE_OK if maxit >= info["iters"] else F.FE_ENOTCONV)
        assert F.pcg_solve_noalloc(A.csr, A.rhs, y, 1e-12, maxit, check=False) == i and torch.equal(x, y)
