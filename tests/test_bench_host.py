"""Host checks of the benchmark's accounting (no GPU needed)."""
import pytest

import bench as B


@pytest.mark.parametrize("dim,k,prob", [(3, 1, "elasticity"), (3, 2, "poisson"), (3, 3, "elasticity"), (3, 4, "elasticity"),
                                        (2, 2, "poisson"), (2, 4, "elasticity")])
def test_fp64_integration_flops_are_those_of_the_sums_by_factors(dim, k, prob):
    """The kernel's loops walked: a fused multiply-add is two flops, a product or a sum one."""
    m, el = k + 1, prob == "elasticity"
    flops = 0
    if dim == 3:
        for a2 in range(m):
            for _ in range(a2, m):                                 # b2
                flops += m * m * m * 9 * (2 + (4 if el else 0))     # q0, q1, q2; nine coefficients
                flops += m * m * m * m * 9 * 2                      # a1, b1, q0, q1: nine terms of V
                flops += m * m * m * m * 2 * 3                      # a1, b1, q0, b0: two products of V and b0
                flops += m * m * m * m * m * 2 * 2                  # and a0: two terms of an entry
    else:
        flops += m ** 4 * (4 + 8 + (16 if el else 0))               # a1, b1, q0, q1
        flops += m ** 4 * 2 * 3 + m ** 5 * 2 * 2
    flops *= dim * dim if el else 1
    wl = dict(dim=dim, k=k, problem=prob)
    assert B.k3_flops(wl, 7, "fp64") == 7 * flops
    assert B.k3_unit(wl, "fp64") == "vector"
    # the contraction over all points, which the 16-bit kernels do
    nn = m ** dim
    assert B.k3_flops(wl, 7, "bf16") == 7 * (18 * nn ** 3 if el else 2 * nn * nn * dim * nn)
