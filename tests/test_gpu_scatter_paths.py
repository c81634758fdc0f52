"""Scatter of 3D vector problems of order >= 2: run by run and entry by entry,
on both sides of the lines between them."""
import numpy as np
import pytest
import torch

from paper_1708_01773_amd import fe as F
from tests.gpu_util import MATRIX_RTOL, Pair, rel, say

pytestmark = pytest.mark.gpu


# Blocks of four nodes: Q2 13x13x12 3594 and 14x14x13 4557 (the line lies at
# 4096), Q3 10x9x9 4901.
@pytest.mark.parametrize("n,k", [([13, 13, 12], 2), ([14, 14, 13], 2), ([10, 9, 9], 3)])
def test_scatter_beside_the_line_matches_oracle(n, k):
    pair = Pair(3, n, k, "elasticity", seed=121, source=(0.4, 1.0, -0.7))
    A = pair.gpu_assembly()
    S = pair.system
    say(f"[scatter] n={n} k={k} blocks {(A.n_rows // 3 + 3) // 4}")
    assert rel(A.values[: A.nnz].cpu().numpy(), S.values) <= MATRIX_RTOL
    assert rel(A.rhs[: A.n_rows].cpu().numpy(), S.rhs) <= MATRIX_RTOL
    assert rel(A.dinv[: A.n_rows].cpu().numpy(), 1.0 / S.scipy().diagonal()) <= MATRIX_RTOL


# Alone each system is small and goes run by run; in the batch they are many
# nodes, and the orders and precisions that take entries then do.  Same bits.
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n,k", [([9, 10, 11], 2), ([6, 7, 5], 3), ([4, 4, 5], 4)])
def test_batched_scatter_takes_either_path_to_the_same_bits(n, k, prec):
    pairs = [Pair(3, n, k, "elasticity", precision=prec, seed=122 + i) for i in range(4)]
    B = F.BatchAssembly([p.mesh for p in pairs], [k] * 4, [p.coeff for p in pairs])
    B.assemble()
    say(f"[scatter batch] n={n} k={k} {prec} blocks {(B.n_rows[0] // 3 + 3) // 4} x 4")
    for i, p in enumerate(pairs):
        A = p.gpu_assembly()
        assert torch.equal(A.values[: A.nnz], B.values[i][: A.nnz])
        assert torch.equal(A.rhs[: A.n_rows], B.rhs[i][: A.n_rows])
        assert torch.equal(A.dinv[: A.n_rows], B.dinv[i][: A.n_rows])
