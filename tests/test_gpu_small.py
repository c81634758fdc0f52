"""The one-workgroup PCG of small systems: its iterates against a CG on the
host, its forms, threads and launches."""
import threading

import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla
import torch

import oracle as O
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


def _forms(pair, A):
    """The solves of one system through every form of its matrix: (name, solve(x, rtol, maxit))."""
    ws = torch.empty(F.pcg_query(A.n_rows), dtype=torch.uint8, device="cuda")
    out = [("csr", lambda x, rtol, it: F.pcg_solve(A.csr, A.rhs, x, rtol, it, ws, check=False)),
           ("mesh", lambda x, rtol, it: F.pcg_solve_mesh(pair.mesh, pair.k, pair.coeff, A.csr, A.rhs, x, rtol, it, ws,
                                                         check=False)),
           ("noalloc", lambda x, rtol, it: F.pcg_solve_noalloc(A.csr, A.rhs, x, rtol, it, check=False))]
    if pair.k == 1 and pair.prob == "poisson":
        sym = torch.empty(F.sym_query(pair.mesh, 1, pair.coeff) // 8, dtype=torch.float64, device="cuda")
        F.sym_from_csr(pair.mesh, 1, pair.coeff, A.csr, sym)
        out.append(("sym", lambda x, rtol, it: F.pcg_solve_sym(pair.mesh, 1, pair.coeff, A.csr, sym, A.rhs, x, rtol, it,
                                                               ws, check=False)))
    return out


# Iterates after a given number of iterations are those of the oracle's CG.  The
# matrix in registers, in LDS, its values from L2; the pattern read, evaluated, and
# the symmetric storage.  The two sum in different orders: an iteration's two
# scalars differ by at most 2 n eps relative (sums of positive terms: r.r, p.Ap up
# to the cancellation within A p, a factor of |A||p| / |A p| below 100 here), and
# ten iterations multiply that by less than 10 each at worst in the first few; with
# n <= 4096: 10 * 2 * 4096 * 1.1e-16 * 100 = 9e-10.
@pytest.mark.parametrize("dim,n,k,prob", [(2, [31, 30], 1, "poisson"), (2, [36, 35], 1, "poisson"),
                                          (2, [64, 65], 1, "poisson"), (3, [5, 5, 5], 2, "poisson"),
                                          (2, [9, 8], 3, "elasticity")])
def test_truncated_iterates_are_those_of_the_oracle(dim, n, k, prob):
    pair = Pair(dim, n, k, prob, seed=106, source=(0.4, 1.0, -0.7))
    A = pair.gpu_assembly()
    S = pair.system
    for it in (1, 2, 3, 7, 10):
        o = O.pcg(S.rowptr, S.colind, S.values, S.rhs, 1e-14, it)
        assert o["iters"] == it
        for name, solve in _forms(pair, A):
            x = torch.zeros(A.n_rows, dtype=torch.float64, device="cuda")
            info = solve(x, 1e-14, it)
            say(f"[truncated] {dim}D n={n} k={k} {prob} rows {A.n_rows} {name} it {it}: {rel(x.cpu().numpy(), o['x']):.1e}")
            assert info["status"] == F.FE_ENOTCONV and info["iters"] == it
            assert abs(info["relres"] - o["relres"]) <= 1e-9 * o["relres"]
            assert rel(x.cpu().numpy(), o["x"]) <= 9e-10


# Strips fixed at one end need more iterations than one launch takes (1024), so
# the solve goes on from the state that a launch left; in a batch with a larger
# system the launches are 16 iterations long.  In registers, in LDS, from L2.
STRIPS = [([1, 480], 1), ([2, 560], 1), ([2, 600], 1)]


@pytest.mark.parametrize("n,k", STRIPS)
def test_solves_go_on_from_the_state_of_the_last_launch(n, k):
    pair = Pair(2, n, k, faces=0b0100, seed=107)
    A = pair.gpu_assembly()
    xd = spla.spsolve(pair.system.scipy().tocsc(), pair.system.rhs)
    x = {}
    for name, solve in _forms(pair, A):
        x[name] = torch.zeros(A.n_rows, dtype=torch.float64, device="cuda")
        info = solve(x[name], 1e-12, 20000)
        kappa = info["lambda_max_est"] / info["lambda_min_est"]
        say(f"[strip] n={n} rows {A.n_rows} {name}: {info['iters']} iterations, kappa {kappa:.1e}, "
            f"{rel(x[name].cpu().numpy(), xd):.1e}")
        assert info["status"] == F.FE_OK and info["iters"] > 1024
        # every iteration adds a rounding of x, which the matrix sees up to kappa
        assert rel(x[name].cpu().numpy(), xd) <= 2.0 ** -53 * kappa * info["iters"]
    assert torch.equal(x["csr"], x["noalloc"])
    big = Pair(3, [9, 9, 9], 2, seed=108)
    B = big.gpu_assembly()
    assert B.n_rows > 4096
    bws = torch.empty(F.pcg_batch_query([A.n_rows, B.n_rows]), dtype=torch.uint8, device="cuda")
    for name in ("csr", "mesh"):
        xs = [torch.zeros(m, dtype=torch.float64, device="cuda") for m in (A.n_rows, B.n_rows)]
        if name == "csr":
            st, _ = F.pcg_solve_batch([A.csr, B.csr], [A.rhs, B.rhs], xs, 1e-12, 20000, bws)
        else:
            st, _ = F.pcg_solve_batch_mesh([pair.mesh, big.mesh], [k, 2], [pair.coeff, big.coeff], [A.csr, B.csr],
                                           [A.rhs, B.rhs], xs, 1e-12, 20000, bws)
        assert st == F.FE_OK and torch.equal(xs[0], x[name]), name


@pytest.mark.parametrize("n,k", STRIPS)
def test_fp32_inner_solves_go_on_from_the_state_of_the_last_launch(n, k):
    """The FP32 forms: inner solves of a refinement, more than 1024 iterations
    each.  A correction reduces the error to that of the matrix rounded to FP32,
    2^-24 kappa, below a tenth here (kappa < 1.5e6): nine reach 1e-9."""
    pair = Pair(2, n, k, faces=0b0100, seed=107)
    A = pair.gpu_assembly()
    ws = torch.empty(F.refine_query(A.n_rows), dtype=torch.uint8, device="cuda")
    v32 = A.values[: A.nnz].float()
    sym32 = torch.empty(F.sym_query(pair.mesh, 1, pair.coeff) // 8, dtype=torch.float32, device="cuda")
    F.sym_fp32_from_csr(pair.mesh, 1, pair.coeff, A.csr, sym32)
    xd = spla.spsolve(pair.system.scipy().tocsc(), pair.system.rhs)
    runs = {"csr": lambda x: F.refine_solve(A.csr, A.csr, A.rhs, x, 1e-9, 1e-6, 30, 20000, ws, values32=v32),
            "mesh": lambda x: F.refine_solve_mesh(pair.mesh, k, pair.coeff, A.csr, A.csr, A.rhs, x, 1e-9, 1e-6, 30, 20000,
                                                  ws, values32=v32),
            "sym": lambda x: F.refine_solve_sym(pair.mesh, k, pair.coeff, A.csr, A.csr, sym32, A.rhs, x, 1e-9, 1e-6, 30,
                                                20000, ws)}
    kappa = F.pcg_solve(A.csr, A.rhs, torch.zeros_like(A.rhs), 1e-12, 20000, ws)
    kappa = kappa["lambda_max_est"] / kappa["lambda_min_est"]
    for name, run in runs.items():
        x = torch.zeros(A.n_rows, dtype=torch.float64, device="cuda")
        info = run(x)
        say(f"[strip fp32] n={n} rows {A.n_rows} {name}: {info} kappa {kappa:.1e} {rel(x.cpu().numpy(), xd):.1e}")
        assert info["status"] == F.FE_OK and info["relres"] <= 1e-9
        assert kappa < 1.5e6 and info["outer_iters"] <= 9 and info["inner_iters"] > 1024 * info["outer_iters"]
        assert rel(x.cpu().numpy(), xd) <= 10 * kappa * 1e-9
