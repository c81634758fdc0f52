"""The one-workgroup PCG of small systems: its iterates against a CG on the
host, its forms, threads and launches."""
import threading

import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla
import torch

from paper_1708_01773_amd import fe as F
from tests.gpu_util import Pair, rel, say

pytestmark = pytest.mark.gpu


def test_threads_solve_small_systems_of_different_lds_sizes():
    """Systems that need 70 to 150 KB of LDS, each thread its own, at the same
    time: every solve launches with what its system needs and gives the bits
    of the solve alone."""
    pairs = [Pair(3, [8, 8, 8], 1, seed=101), Pair(2, [33, 33], 1, seed=102), Pair(2, [38, 38], 1, seed=103),
             Pair(3, [8, 9, 9], 1, seed=104)]
    systems = []
    for p in pairs:
        A = p.gpu_assembly()
        ws = torch.empty(F.pcg_query(A.n_rows), dtype=torch.uint8, device="cuda")
        x = torch.zeros(A.n_rows, dtype=torch.float64, device="cuda")
        info = F.pcg_solve(A.csr, A.rhs, x, 1e-10, 2000, ws)
        lds = 16 * A.n_rows + 4 * A.n_rows + 10 * A.nnz
        say(f"[threads] rows {A.n_rows} nnz {A.nnz} lds about {lds}")
        assert info["status"] == F.FE_OK and 64 * 1024 < lds < 156 * 1024
        systems.append((A, ws, x, info))
    torch.cuda.synchronize()
    bad = []

    def work(A, ws, ref, info):
        try:
            s = torch.cuda.Stream()
            x = torch.empty_like(ref)
            with torch.cuda.stream(s):
                for _ in range(40):
                    x.zero_()
                    i = F.pcg_solve(A.csr, A.rhs, x, 1e-10, 2000, ws, s)
                    if i != info or not torch.equal(x, ref):
                        bad.append((A.n_rows, i))
                        return
        except Exception as e:  # reported by the main thread
            bad.append((A.n_rows, repr(e)))

    ts = [threading.Thread(target=work, args=s) for s in systems]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def _bordered(n, every, seed):
    """Diagonally dominant tridiagonal matrix with one row and column of n / every entries."""
    g = np.random.Generator(np.random.PCG64(seed))
    S = sp.diags([2.6 + g.random(n)], [0]) + sp.diags([-g.random(n - 1)], [1])
    S = sp.lil_matrix(S + sp.triu(S, 1).T)
    S[n // 2, ::every] = S[::every, n // 2] = 0.5 / n * np.ones((1, len(range(0, n, every))))
    S[n // 2, n // 2] = 3.0
    S = S.tocsr()
    S.sort_indices()
    return S


def _device_csr(S):
    t = [torch.from_numpy(a).cuda() for a in (S.indptr.astype(np.int64), S.indices.astype(np.int32), S.data,
                                              np.ones(S.shape[0]), 1.0 / S.diagonal())]
    return F.csr_struct(S.shape[0], S.nnz, *t), t


# One long row among short ones: summed by its lane group up to 128 entries a
# lane, by a whole wave from there (n = 300: two lanes a row, the matrix would
# fit registers but for that row; 1000 and 4000: one lane a row).
@pytest.mark.parametrize("n,every", [(300, 1), (300, 2), (1000, 1), (1000, 8), (4000, 1), (4000, 32), (4096, 1)])
def test_small_system_with_a_long_row(n, every):
    say(f"[long row] n={n} every {every}")
    S = _bordered(n, every, 105)
    csr, t = _device_csr(S)
    ws = torch.empty(F.pcg_query(n), dtype=torch.uint8, device="cuda")
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    info = F.pcg_solve(csr, t[3], x, 1e-13, 500, ws)
    assert info["status"] == F.FE_OK and info["true_relres"] <= 1e-12
    # eigenvalues of A are above 1/2 (Gershgorin): the error is below 2e-12 ||b||
    xd = spla.spsolve(S.tocsc(), np.ones(n))
    assert np.linalg.norm(x.cpu().numpy() - xd) <= 2e-12 * np.sqrt(n)
    y = torch.zeros_like(x)
    again = F.pcg_solve(csr, t[3], y, 1e-13, 500, ws)
    assert again == info and torch.equal(x, y)  # the order of the sums is fixed
