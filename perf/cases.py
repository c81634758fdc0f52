"""Performance cases of the framework: what its users run, through its public entry points.

Every case is a dict of plain values with a "kind":

* ``assemble``: the numeric phase (element integration and scatter) of a structured system,
* ``step``: assembly and Jacobi-PCG solve of a structured system (Poisson, elasticity),
* ``spmv``: the product y = A x of an assembled structured system, its pattern evaluated from the mesh,
* ``refine``: both assemblies and the mixed-precision solve (FP32 inner operator, FP64 residuals),
* ``batch``: many uneven problems assembled and refined together,
* ``dg``: the assembly of an interior-penalty DG system,
* ``simplex``: assembly and PCG solve of a P_k system on a general simplicial mesh.

The set-up a program does once per mesh (numbering, sparsity pattern, workspaces) is in ``prepare``.
Meshes are bricks with interior vertices jittered by 0.15 h (below h / 6 no draw inverts a cell) and
lognormal cell coefficients.  Solves run to a relative residual of 1e-12, so that a solution is
determined to well below the distance at which two programs' solutions are told apart; refinement
runs to 1e-10, as its benchmark form does (each correction gains four to five digits).
``exact`` is the same finite element system written with plain torch operations in FP64.
"""
import itertools
import math

import numpy as np
import torch

MAXIT = 100000
RTOL = 1e-12
GAMMA = {1: 16.0, 2: 36.0, 3: 64.0, 4: 100.0}  # DG penalty 4 (k + 1)^2


def listed():
    return [
        # a small 2D problem, the teaching-size solve: latency and launches
        dict(name="poisson2d_q1_32_step", kind="step", dim=2, n0=32, n1=32, n2=1, order=1, problem="poisson",
             precision="fp64", via="csr"),
        # one small request of a serving stream (orders 1..4, sizes from 8 cells per axis)
        dict(name="poisson3d_q2_10_step", kind="step", dim=3, n0=10, n1=10, n2=10, order=2, problem="poisson",
             precision="fp64", via="mesh"),
        # the benchmark workload: 128^3 Q1, assembly + symmetric storage + PCG
        dict(name="poisson3d_q1_128_step", kind="step", dim=3, n0=128, n1=128, n2=128, order=1, problem="poisson",
             precision="fp64", via="sym"),
        # assembly alone on a ragged Q1 brick (time stepping, coefficient updates)
        dict(name="poisson3d_q1_odd_assemble", kind="assemble", dim=3, n0=193, n1=67, n2=129, order=1,
             problem="poisson", precision="fp64"),
        # mixed precision at an odd size: FP32 integration and storage inside, FP64 residuals outside
        dict(name="poisson3d_q1_odd_refine", kind="refine", dim=3, n0=61, n1=47, n2=53),
        # high-order elasticity assembly in FP64
        dict(name="elasticity_q4_24_assemble", kind="assemble", dim=3, n0=24, n1=24, n2=24, order=4,
             problem="elasticity", precision="fp64"),
        # the reduced-precision element GEMMs
        dict(name="elasticity_q3_32_assemble_bf16", kind="assemble", dim=3, n0=32, n1=32, n2=32, order=3,
             problem="elasticity", precision="bf16"),
        # the operator of a vector problem, as an outer Krylov or eigenvalue method applies it
        dict(name="elasticity_q2_48_spmv", kind="spmv", dim=3, n0=48, n1=48, n2=48, order=2, problem="elasticity"),
        # an elasticity solve on a ragged brick
        dict(name="elasticity_q2_odd_step", kind="step", dim=3, n0=19, n1=23, n2=17, order=2, problem="elasticity",
             precision="fp64", via="mesh"),
        # a batch of uneven problems, FP32 integration refined to FP64
        dict(name="batch_16_refine", kind="batch", count=16, nmin=8, nmax=20),
        # discontinuous Galerkin assembly
        dict(name="dg_q2_32_assemble", kind="dg", dim=3, n0=32, n1=32, n2=32, order=2),
        # quadratic tetrahedra on a general mesh, solved on the plain CSR
        dict(name="simplex_p2_20_step", kind="simplex", dim=3, n0=20, n1=20, n2=20, order=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _brick(rng, dim, order, ncomp, lo, hi):
    """Cells per axis, unequal and often odd, with lo..hi rows (about)."""
    rows = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    side = (rows / ncomp) ** (1.0 / dim) / order
    n = [max(2, int(round(side * math.exp(rng.uniform(-0.35, 0.35))))) for _ in range(dim)]
    return n + [1] * (3 - dim)


def draw(rng):
    kind = rng.choice(["assemble", "assemble", "assemble", "step", "step", "step", "spmv", "spmv", "refine", "batch",
                       "dg", "simplex"])
    dim = 2 if rng.random() < 0.2 else 3
    order = rng.choice([1, 2, 3, 4])
    problem = rng.choice(["poisson", "elasticity"])
    ncomp = dim if problem == "elasticity" else 1
    if kind == "assemble":
        top = {1: 3e6, 2: 2e6, 3: 1.2e6, 4: 8e5}[order]
        n = _brick(rng, dim, order, ncomp, 2e3, top)
        return dict(kind=kind, dim=dim, n0=n[0], n1=n[1], n2=n[2], order=order, problem=problem,
                    precision=rng.choice(["fp64", "fp64", "fp32", "fp16", "bf16"]) if dim == 3 else "fp64")
    if kind == "step":
        n = _brick(rng, dim, order, ncomp, 500, {1: 3e5, 2: 1e5, 3: 5e4, 4: 3e4}[order])
        via = rng.choice(["csr", "mesh"] + (["sym"] if order == 1 and problem == "poisson" else []))
        return dict(kind=kind, dim=dim, n0=n[0], n1=n[1], n2=n[2], order=order, problem=problem,
                    precision=rng.choice(["fp64", "fp64", "fp32"]) if dim == 3 else "fp64", via=via)
    if kind == "spmv":
        n = _brick(rng, dim, order, ncomp, 2e4, {1: 4e6, 2: 2e6, 3: 1.5e6, 4: 1e6}[order])
        return dict(kind=kind, dim=dim, n0=n[0], n1=n[1], n2=n[2], order=order, problem=problem)
    if kind == "refine":
        n = _brick(rng, 3, 1, 1, 5e3, 5e5)
        return dict(kind=kind, dim=3, n0=n[0], n1=n[1], n2=n[2])
    if kind == "batch":
        nmax = rng.randint(10, 18)
        return dict(kind=kind, count=rng.randint(4, 16), nmin=rng.randint(6, 9), nmax=nmax)
    if kind == "dg":
        order = rng.choice([1, 2, 3])
        n = _brick(rng, dim, 1, (order + 1) ** dim, 2e4, 9e5)
        return dict(kind=kind, dim=dim, n0=n[0], n1=n[1], n2=n[2], order=order)
    order = rng.choice([1, 2, 3])
    n = _brick(rng, dim, order, 1, 2e3, 9e4)
    return dict(kind="simplex", dim=dim, n0=n[0], n1=n[1], n2=n[2], order=order)


# ---------------------------------------------------------------------------
# Inputs (host arrays, drawn from the seed alone)
# ---------------------------------------------------------------------------
def _cells(case):
    return [case["n0"], case["n1"], case["n2"]][: case["dim"]]


def _mesh_arrays(dim, n, seed):
    """(vertices (nv, dim), x fastest; cell coefficients) of a jittered brick."""
    g = np.random.Generator(np.random.PCG64(seed))
    axes = [np.arange(m + 1, dtype=np.float64) / m for m in n]
    grids = np.meshgrid(*axes[::-1], indexing="ij")[::-1]  # x varies fastest
    v = np.stack([a.ravel() for a in grids], axis=1)
    inner = np.ones(v.shape[0], dtype=bool)
    for r in range(dim):
        inner &= (v[:, r] > 0.0) & (v[:, r] < 1.0)
    v[inner] += g.uniform(-0.15, 0.15, size=(int(inner.sum()), dim)) / np.array(n, dtype=np.float64)
    return np.ascontiguousarray(v), np.exp(g.standard_normal(int(np.prod(n))))


def _simplex_arrays(dim, n, seed):
    """A jittered brick cut into dim! simplices per cell, vertices, cells and local vertices shuffled."""
    v, _ = _mesh_arrays(dim, n, seed)
    stride = [1, n[0] + 1, (n[0] + 1) * (n[1] + 1)][:dim]
    idx = np.meshgrid(*[np.arange(m) for m in n[::-1]], indexing="ij")[::-1]
    base = sum(i.ravel() * s for i, s in zip(idx, stride))
    cells = []
    for perm in itertools.permutations(range(dim)):
        c = [base]
        for r in perm:
            c.append(c[-1] + stride[r])
        cells.append(np.stack(c, axis=1))
    cells = np.concatenate(cells)
    g = np.random.Generator(np.random.PCG64(seed + 1))
    relabel = g.permutation(v.shape[0])
    w = np.empty_like(v)
    w[relabel] = v
    cells = relabel[cells][g.permutation(cells.shape[0])]
    cells = np.take_along_axis(cells, np.argsort(g.random(cells.shape), axis=1), axis=1)
    return np.ascontiguousarray(w), np.ascontiguousarray(cells.astype(np.int32)), np.exp(
        g.standard_normal(cells.shape[0]))


def _batch_specs(case, seed):
    g = np.random.Generator(np.random.PCG64(case["count"] * 1000 + case["nmin"] * 100 + case["nmax"]))
    return [(int(n), int(k), seed * 1000 + i) for i, (n, k) in enumerate(
        zip(g.integers(case["nmin"], case["nmax"] + 1, case["count"]), g.integers(1, 4, case["count"])))]


def _source(problem, dim):
    return ((0.0, 0.0, -1.0) if dim == 3 else (0.0, -1.0)) if problem == "elasticity" else (1.0,)


def _spmv_input(n, seed):
    return torch.from_numpy(np.random.Generator(np.random.PCG64(seed + 2)).standard_normal(n))


# ---------------------------------------------------------------------------
# The framework
# ---------------------------------------------------------------------------
def prepare(case, seed):
    from paper_1708_01773_amd import fe as F
    kind = case["kind"]

    def coeff(precision="fp64", problem=None, dim=None):
        problem = problem or case.get("problem", "poisson")
        dim = dim or case["dim"]
        return F.make_coeff(problem, precision, source_kind=F.FE_SOURCE_CONST, source=_source(problem, dim), dim=dim)

    def bytes_(n):
        return torch.empty(max(int(n), 8), dtype=torch.uint8, device="cuda")

    if kind == "batch":
        specs = _batch_specs(case, seed)
        meshes = [F.create_mesh(3, [n] * 3, *_mesh_arrays(3, [n] * 3, s)) for n, _, s in specs]
        orders = [k for _, k, _ in specs]
        lo = F.BatchAssembly(meshes, orders, [coeff("fp32", "poisson", 3) for _ in specs])
        hi = F.BatchAssembly(meshes, orders, [coeff("fp64", "poisson", 3) for _ in specs])
        return dict(kind=kind, F=F, meshes=meshes, orders=orders, lo=lo, hi=hi, ws=bytes_(F.refine_batch_query(lo.n_rows)))
    n = _cells(case)
    if kind == "simplex":
        v, cells, k = _simplex_arrays(case["dim"], n, seed)
        G = F.Simplex(case["dim"], v, cells, case["order"], coeff(), cell_coeff=k)
        return dict(kind=kind, F=F, G=G, x=torch.zeros(G.n_rows, dtype=torch.float64, device="cuda"),
                    ws=bytes_(F.pcg_query(G.n_rows)))
    v, k = _mesh_arrays(case["dim"], n, seed)
    mesh = F.create_mesh(case["dim"], n, v, k)
    if kind == "dg":
        return dict(kind=kind, F=F, A=F.DGAssembly(mesh, case["order"], coeff(), GAMMA[case["order"]]))
    order = 1 if kind == "refine" else case["order"]
    A = F.Assembly(mesh, order, coeff(case.get("precision", "fp64")))
    A.pattern()
    s = dict(kind=kind, F=F, A=A, mesh=mesh, x=torch.zeros(A.n_rows, dtype=torch.float64, device="cuda"))
    if kind == "spmv":
        A.assemble()
        s["x"] = _spmv_input(A.n_rows, seed).cuda()
        s["y"] = torch.empty_like(s["x"])
    elif kind == "refine":
        s["lo"] = F.Assembly(mesh, order, coeff("fp32"))
        s["lo"].pattern()
        s["sym32"] = torch.empty(F.sym_query(mesh, order, A.coeff) // 8, dtype=torch.float32, device="cuda")
        s["ws"] = bytes_(F.refine_query(A.n_rows))
    elif kind == "step":
        s["via"] = case["via"]
        s["ws"] = bytes_(F.pcg_query(A.n_rows))
        if case["via"] == "sym":
            s["sym"] = torch.empty(F.sym_query(mesh, order, A.coeff) // 8, dtype=torch.float64, device="cuda")
    return s


def run(s):
    F, kind = s["F"], s["kind"]
    if kind == "batch":
        lo, hi = s["lo"], s["hi"]
        lo.assemble()
        hi.assemble()
        for x in hi.x:
            x.zero_()
        F.refine_solve_batch_mesh(s["meshes"], s["orders"], hi.coeffs, hi.csrs, lo.csrs, hi.rhs, hi.x, 1e-10, 1e-5, 50,
                                  MAXIT, s["ws"])
        return dict(x=[x[:n] for x, n in zip(hi.x, hi.n_rows)])
    if kind == "simplex":
        G = s["G"]
        G.assemble()
        s["x"].zero_()
        F.pcg_solve(G.csr, G.rhs, s["x"], RTOL, MAXIT, s["ws"])
        return dict(values=G.values[: G.nnz], rhs=G.rhs, dinv=G.dinv, x=s["x"])
    A = s["A"]
    if kind == "spmv":
        F.spmv_mesh(s["mesh"], A.order, A.coeff, A.csr, s["x"], s["y"])
        return dict(y=s["y"])
    A.assemble()
    if kind in ("assemble", "dg"):
        return dict(values=A.values[: A.nnz], rhs=A.rhs, dinv=A.dinv)
    x = s["x"]
    x.zero_()
    if kind == "refine":
        lo = s["lo"]
        lo.assemble()
        F.sym_fp32_from_csr(s["mesh"], 1, lo.coeff, lo.csr, s["sym32"])
        F.refine_solve_sym(s["mesh"], 1, lo.coeff, A.csr, lo.csr, s["sym32"], A.rhs, x, 1e-10, 1e-5, 50, MAXIT, s["ws"])
        return dict(x=x)
    if s["via"] == "csr":
        F.pcg_solve(A.csr, A.rhs, x, RTOL, MAXIT, s["ws"])
    elif s["via"] == "mesh":
        A.solve(x, RTOL, MAXIT, s["ws"])
    else:
        F.sym_from_csr(s["mesh"], 1, A.coeff, A.csr, s["sym"])
        F.pcg_solve_sym(s["mesh"], 1, A.coeff, A.csr, s["sym"], A.rhs, x, RTOL, MAXIT, s["ws"])
    return dict(values=A.values[: A.nnz], rhs=A.rhs, x=x)


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _sizes(dim, n, k, ncomp):
    """(rows, nonzeros) of the conforming system with every boundary node fixed."""
    rows, nnz = ncomp, ncomp * ncomp
    for m in n[:dim]:
        w = _axis(m, k)[1]
        rows *= len(w)
        nnz *= int(w.sum())
    return rows, nnz


def _integration_flops(dim, cells, k, ncomp):
    """Element matrices by one-dimensional contractions: the last one fills (k+1)^2d entries from (k+1) points for
    each of the four value / derivative pairs along its axis; the ones before are a (k+1)-th of that each.  Symmetric
    halves are counted once."""
    last = (k + 1) ** (2 * dim + 1) * 4 * 2 / 2
    return cells * (ncomp * (ncomp + 1) / 2) * last * (1 + 1 / (k + 1))


def _assembly_work(dim, n, k, ncomp, elem_flops=True):
    cells = int(np.prod(n[:dim]))
    rows, nnz = _sizes(dim, n, k, ncomp)
    verts = int(np.prod([m + 1 for m in n[:dim]]))
    return 8 * (nnz + 2 * rows + cells + dim * verts), _integration_flops(dim, cells, k, ncomp)


def _iterations(n, k, elasticity=False):
    """Jacobi-PCG iterations to 1e-12, about: proportional to the longest axis in cells, more with the order and for
    elasticity.  Fitted to the counts on the listed bricks (Q1 128: 531, Q2 10: 120, elasticity Q2 23: 519)."""
    return int(max(n) * {1: 4.2, 2: 12.0, 3: 34.0, 4: 55.0}[k] * (1.9 if elasticity else 1.0)) + 2


def work(case):
    kind = case["kind"]
    if kind == "batch":
        b = f = 0.0
        for n, k, _ in _batch_specs(case, 0):
            rows, nnz = _sizes(3, [n] * 3, k, 1)
            ab, af = _assembly_work(3, [n] * 3, k, 1)
            it = int(1.2 * _iterations([n], k))
            b += 2 * ab + it * (8 * nnz + 80 * rows)
            f += 2 * af + it * (2 * nnz + 10 * rows)
        return dict(bytes=b, flops=f)
    dim, n = case["dim"], _cells(case)
    if kind == "dg":
        k = case["order"]
        cells, nn = int(np.prod(n)), (k + 1) ** dim
        blocks = cells + 2 * sum(cells // m * (m - 1) for m in n)
        verts = int(np.prod([m + 1 for m in n]))
        return dict(bytes=8.0 * (blocks * nn * nn + 2 * cells * nn + dim * verts),
                    flops=_integration_flops(dim, cells, k, 1) + 12.0 * blocks * nn * nn)
    if kind == "simplex":
        k = case["order"]
        nloc = math.comb(k + dim, dim)
        cells = int(np.prod(n)) * math.factorial(dim)
        rows = int(np.prod([m * k - 1 for m in n]))
        nnz = rows * {2: {1: 7, 2: 11.5, 3: 17}, 3: {1: 15, 2: 28.5, 3: 48}}[dim][k]
        verts = int(np.prod([m + 1 for m in n]))
        it = int(1.4 * _iterations(n, k))
        # P_k stiffness is a fixed combination of dim (dim + 1) / 2 reference matrices
        return dict(bytes=8.0 * nnz + 16 * rows + 4 * cells * (dim + 1) + 8 * cells + 8 * dim * verts
                    + it * (12.0 * nnz + 88 * rows),
                    flops=cells * nloc * nloc * dim * (dim + 1) / 2 + it * (2.0 * nnz + 10 * rows))
    k = 1 if kind == "refine" else case["order"]
    el = case.get("problem") == "elasticity"
    ncomp = dim if el else 1
    rows, nnz = _sizes(dim, n, k, ncomp)
    if kind == "spmv":
        return dict(bytes=8.0 * nnz + 16 * rows, flops=2.0 * nnz)
    b, f = _assembly_work(dim, n, k, ncomp)
    if kind == "assemble":
        return dict(bytes=float(b), flops=float(f))
    it = _iterations(n, k, el)
    if kind == "refine":  # two assemblies; inner iterations on the FP32 upper triangle
        it = int(1.35 * it)
        return dict(bytes=2 * b + it * (4.0 * (nnz + rows) / 2 + 80 * rows), flops=2 * f + it * (2.0 * nnz + 10 * rows))
    mat = {"csr": 12.0 * nnz + 8 * rows, "mesh": 8.0 * nnz, "sym": 8.0 * (nnz + rows) / 2}[case["via"]]
    return dict(bytes=b + it * (mat + 80.0 * rows), flops=f + it * (2.0 * nnz + 10 * rows))


# ---------------------------------------------------------------------------
# The same systems in plain torch, FP64
# ---------------------------------------------------------------------------
def _dev():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.asarray(a), dtype=dtype, device=_dev())


def _gauss(m):
    x, w = np.polynomial.legendre.leggauss(m)
    return 0.5 * (x + 1.0), 0.5 * w


def _basis_1d(k, x):
    """Values and derivatives (len(x), k + 1) of the equidistant Lagrange basis on [0, 1]."""
    nodes = np.arange(k + 1) / k
    V, D = np.ones((len(x), k + 1)), np.zeros((len(x), k + 1))
    for i in range(k + 1):
        others = [j for j in range(k + 1) if j != i]
        for j in others:
            V[:, i] *= (x - nodes[j]) / (nodes[i] - nodes[j])
        for s in others:
            t = np.ones(len(x)) / (nodes[i] - nodes[s])
            for j in others:
                if j != s:
                    t = t * (x - nodes[j]) / (nodes[i] - nodes[j])
            D[:, i] += t
    return V, D


def _basis(dim, k, pts):
    """Values (nq, nn) and reference gradients (nq, nn, dim) of the tensor basis, first axis fastest."""
    one = [_basis_1d(k, pts[:, r]) for r in range(dim)]
    phi, grad = [], []
    for a in itertools.product(range(k + 1), repeat=dim):
        a = a[::-1]
        phi.append(np.prod([one[r][0][:, a[r]] for r in range(dim)], axis=0))
        grad.append(np.stack([np.prod([one[r][1 if r == s else 0][:, a[r]] for r in range(dim)], axis=0)
                              for s in range(dim)], axis=1))
    return np.stack(phi, axis=1), np.stack(grad, axis=1)


def _tensor_points(dim, m):
    x, w = _gauss(m)
    pts, wts = [], []
    for q in itertools.product(range(m), repeat=dim):
        q = q[::-1]
        pts.append([x[i] for i in q])
        wts.append(np.prod([w[i] for i in q]))
    return np.array(pts).reshape(-1, dim), np.array(wts)


def _cell_vertices(dim, n, v):
    """(ncells, 2^dim, dim) coordinates of the cells' vertices, cells x fastest."""
    stride = [1, n[0] + 1, (n[0] + 1) * (n[1] + 1) if dim == 3 else 0]
    idx = np.meshgrid(*[np.arange(m) for m in n[::-1]], indexing="ij")[::-1]
    base = sum(i.ravel() * s for i, s in zip(idx, stride))
    loc = np.array([sum(((c >> r) & 1) * stride[r] for r in range(dim)) for c in range(1 << dim)])
    return _t(v)[_t(base[:, None] + loc[None, :], torch.int64)]


def _geometry(X, pts):
    """J^-1 (c, q, s, r) and det J (c, q) of the multilinear map at reference points."""
    _, dN = _basis(X.shape[2], 1, pts)
    J = torch.einsum("cvr,qvs->cqrs", X, _t(dN))
    return torch.linalg.inv(J), torch.linalg.det(J)


def _axis(m, k):
    """(first column, width) of every free node 1 .. m k - 1 of an axis."""
    i = np.arange(1, m * k)
    lo = np.where(i % k == 0, i - k, i // k * k)
    hi = np.where(i % k == 0, i + k, i // k * k + k)
    lo, hi = np.maximum(lo, 1), np.minimum(hi, m * k - 1)
    return lo, hi - lo + 1


def _hex_system(dim, n, k, problem, v, coef):
    """rowptr, colind, values, rhs of the free system with plain torch."""
    ncomp = dim if problem == "elasticity" else 1
    dev = _dev()
    n = list(n)
    cl, w = zip(*[_axis(m, k) for m in n])
    f = [len(a) for a in cl]
    nf = int(np.prod(f))
    T = lambda a: torch.as_tensor(a, dtype=torch.int64, device=dev)  # noqa: E731
    cl, w = [T(a) for a in cl], [T(a) for a in w]
    # row lengths in the order (.., y, x, component)
    length = w[0]
    for r in range(1, dim):
        length = (w[r][:, None] * length[None, :]).reshape(-1)
    length = (length * ncomp).repeat_interleave(ncomp)
    rowptr = torch.zeros(nf * ncomp + 1, dtype=torch.int64, device=dev)
    torch.cumsum(length, 0, out=rowptr[1:])
    nnz = int(rowptr[-1])
    values = torch.zeros(nnz, dtype=torch.float64, device=dev)
    rhs = torch.zeros(nf * ncomp, dtype=torch.float64, device=dev)
    pts, wq = _tensor_points(dim, k + 1)
    phi, dphi = (_t(a) for a in _basis(dim, k, pts))
    wq = _t(wq)
    X = _cell_vertices(dim, n, v)
    coef = _t(coef)
    nn, nq = phi.shape[1], phi.shape[0]
    nloc = nn * ncomp
    src = _source(problem, dim)
    lam, mu = 0.3 / (1.3 * 0.4), 1.0 / 2.6
    local = np.array([a[::-1] for a in itertools.product(range(k + 1), repeat=dim)])
    ncells = X.shape[0]
    chunk = max(1, min(ncells, int(2e8 / 8 / max(nloc * nloc, nq * nn * dim))))
    eye = torch.eye(ncomp, dtype=torch.float64, device=dev)
    for c0 in range(0, ncells, chunk):
        c = torch.arange(c0, min(c0 + chunk, ncells), device=dev)
        Ji, det = _geometry(X[c], pts)
        wd = wq[None, :] * det.abs()
        G = torch.einsum("cqsr,qas->crqa", Ji, dphi)
        # the cell coefficient scales the whole form, Poisson and elasticity alike
        WG = G * (wd * coef[c][:, None])[:, None, :, None]
        if ncomp == 1:
            A = torch.matmul(G.reshape(len(c), -1, nn).transpose(1, 2).contiguous(), WG.reshape(len(c), -1, nn))
        else:
            M = torch.matmul(G.transpose(2, 3).contiguous()[:, :, None], WG[:, None])  # c, i, j, a, b
            tr = sum(M[:, l, l] for l in range(dim))
            A = lam * M + mu * M.transpose(1, 2) + mu * eye[None, :, :, None, None] * tr[:, None, None]
            A = A.permute(0, 3, 1, 4, 2).reshape(len(c), nloc, nloc)
        F = torch.einsum("cq,qa->ca", wd, phi)
        # node indices along each axis, positions of the entries
        e = [c % n[0], c // n[0] % n[1]] + ([c // (n[0] * n[1])] if dim == 3 else [])
        I = [e[r][:, None] * k + T(local[:, r])[None, :] for r in range(dim)]
        free = torch.ones_like(I[0], dtype=torch.bool)
        for r in range(dim):
            free &= (I[r] > 0) & (I[r] < n[r] * k)
        t = [(I[r] - 1).clamp(0, f[r] - 1) for r in range(dim)]
        rank = t[0]
        for r in range(1, dim):
            rank = rank + int(np.prod(f[:r])) * t[r]
        pos, scale = torch.zeros((len(c), nn, nn), dtype=torch.int64, device=dev), ncomp
        for r in range(dim):
            pos += (I[r][:, None, :] - cl[r][t[r]][:, :, None]) * (
                scale if isinstance(scale, int) else scale[:, :, None])
            scale = w[r][t[r]] * scale
        both = free[:, :, None] & free[:, None, :]
        for i in range(ncomp):
            start = rowptr[rank * ncomp + i][:, :, None]
            rhs.index_add_(0, (rank * ncomp + i)[free], (F * src[i])[free])
            for j in range(ncomp):
                block = A.reshape(len(c), nn, ncomp, nn, ncomp)[:, :, i, :, j]
                values.index_add_(0, (start + pos + j)[both], block[both])
    return rowptr, cl, w, f, ncomp, values, rhs


def _hex_colind(rowptr, cl, w, f, ncomp):
    """Column indices of the structured pattern (the free node boxes, lexicographic)."""
    dim = len(f)
    nf = int(np.prod(f))
    node = torch.arange(nf, device=rowptr.device)
    t, rest = [], node
    for r in range(dim):
        t.append(rest % f[r])
        rest = rest // f[r]
    row = torch.repeat_interleave(torch.arange(nf * ncomp, device=rowptr.device), rowptr[1:] - rowptr[:-1])
    p = torch.arange(int(rowptr[-1]), device=rowptr.device) - rowptr[row]
    nd = row // ncomp
    comp, p = p % ncomp, p // ncomp
    col, step = torch.zeros_like(p), 1
    for r in range(dim):
        wr = w[r][t[r]][nd]
        col += (p % wr + cl[r][t[r]][nd] - 1) * step
        p = p // wr
        step *= f[r]
    return col * ncomp + comp


def _diagonal(rowptr, colind, values):
    row = torch.repeat_interleave(torch.arange(rowptr.numel() - 1, device=rowptr.device), rowptr[1:] - rowptr[:-1])
    at = torch.nonzero(row == colind).reshape(-1)
    return values[at]


def _solve(rowptr, colind, values, b, rtol=1e-14):
    """Jacobi-PCG to the accuracy FP64 allows."""
    n = b.numel()
    A = torch.sparse_csr_tensor(rowptr, colind, values, size=(n, n))
    dinv = 1.0 / _diagonal(rowptr, colind, values)
    x = torch.zeros_like(b)
    for _ in range(2):  # restarted once from the true residual
        r = b - A @ x
        z = dinv * r
        p, rz = z.clone(), torch.dot(r, z)
        for it in range(20000):
            q = A @ p
            a = rz / torch.dot(p, q)
            x += a * p
            r -= a * q
            z = dinv * r
            new = torch.dot(r, z)
            p = z + (new / rz) * p
            rz = new
            if it % 25 == 24 and float(torch.linalg.vector_norm(r)) <= rtol * float(torch.linalg.vector_norm(b)):
                break
    return x


def _dg_system(dim, n, k, v):
    """values (the library's row order), rhs and diagonal of the interior-penalty form, tau = 1, coefficient 1."""
    nn = (k + 1) ** dim
    ncells = int(np.prod(n))
    X = _cell_vertices(dim, n, v)
    pts, wq = _tensor_points(dim, k + 1)
    phi, dphi = (_t(a) for a in _basis(dim, k, pts))
    Ji, det = _geometry(X, pts)
    wd = _t(wq)[None, :] * det.abs()
    G = torch.einsum("cqsr,qas->cqar", Ji, dphi)
    D = torch.einsum("cqar,cq,cqbr->cab", G, wd, G)
    rhs = torch.einsum("cq,qa->ca", wd, phi)
    del G, Ji
    cell = torch.arange(ncells, device=X.device)
    stride = [1, n[0], n[0] * n[1] if dim == 3 else 0]
    coord = [cell // stride[r] % n[r] for r in range(dim)]
    off = {}  # (axis, side) -> (cells, blocks)

    def side(K, r, at):
        """phi (q, nn), n-normal vector with measure (c, q, dim), gradients (c, q, nn, dim) on xi_r = at."""
        p2, w2 = _tensor_points(dim - 1, k + 1)
        full = np.insert(p2, r, float(at), axis=1)
        ph, dp = (_t(a) for a in _basis(dim, k, full))
        ji, dt = _geometry(X[K], full)
        return ph, _t(w2), ji[:, :, r, :] * dt[:, :, None], torch.einsum("cqsr,qas->cqar", ji, dp)

    for r in range(dim):
        K = cell[coord[r] < n[r] - 1]
        L = K + stride[r]
        pK, w2, nv, gK = side(K, r, 1)
        pL, _, _, gL = side(L, r, 0)
        dS = torch.linalg.vector_norm(nv, dim=2)
        area = (w2 * dS).sum(1)
        sigma = GAMMA[k] / (area.sqrt() if dim == 3 else area)
        unit = nv / dS[:, :, None]
        W = w2 * dS
        dK, dL = (torch.einsum("cqar,cqr->cqa", g, unit) for g in (gK, gL))
        ph, dn, sg = (pK, pL), (dK, dL), (1.0, -1.0)

        def block(i, j):
            cons = torch.einsum("cq,qa,cqb->cab", W, ph[i], dn[j]) * (-0.5 * sg[i])
            sym = torch.einsum("cq,cqa,qb->cab", W, dn[i], ph[j]) * (-0.5 * sg[j])
            pen = torch.einsum("cq,c,qa,qb->cab", W, sigma, ph[i], ph[j]) * (sg[i] * sg[j])
            return cons + sym + pen

        D.index_add_(0, K, block(0, 0))
        D.index_add_(0, L, block(1, 1))
        off[(r, 1)] = (K, block(0, 1))
        off[(r, 0)] = (L, block(1, 0))
        for at in (0, 1):
            B = cell[coord[r] == (n[r] - 1 if at else 0)]
            ph1, w2, nv, g = side(B, r, at)
            nv = nv if at else -nv
            dS = torch.linalg.vector_norm(nv, dim=2)
            area = (w2 * dS).sum(1)
            sigma = GAMMA[k] / (area.sqrt() if dim == 3 else area)
            d = torch.einsum("cqar,cqr->cqa", g, nv / dS[:, :, None])
            W = w2 * dS
            c1 = torch.einsum("cq,qa,cqb->cab", W, ph1, d)
            D.index_add_(0, B, -c1 - c1.transpose(1, 2) + torch.einsum("cq,c,qa,qb->cab", W, sigma, ph1, ph1))
    # row blocks: cells ascending
    count = torch.ones(ncells, dtype=torch.int64, device=X.device)
    for K, _ in off.values():
        count[K] += 1
    start = torch.cumsum(count, 0) - count
    values = torch.zeros(int(count.sum()) * nn * nn, dtype=torch.float64, device=X.device)
    slot = torch.zeros_like(count)
    order = [(r, 0) for r in reversed(range(dim))] + [None] + [(r, 1) for r in range(dim)]
    a = torch.arange(nn, device=X.device)
    for key in order:
        K, blk = (cell, D) if key is None else off[key]
        pos = (start[K] * nn * nn)[:, None, None] + a[None, :, None] * (count[K] * nn)[:, None, None] + (
            slot[K] * nn)[:, None, None] + a[None, None, :]
        values[pos.reshape(-1)] = blk.reshape(-1)
        slot[K] += 1
    return values, rhs.reshape(-1), 1.0 / torch.diagonal(D, dim1=1, dim2=2).reshape(-1)


def _simplex_system(dim, k, v, cells, coef):
    """rowptr, colind, values, rhs of P_k on a simplicial mesh, zero data on the whole boundary."""
    lat = np.array([a[::-1] for a in itertools.product(range(k + 1), repeat=dim) if sum(a) <= k])
    nloc = len(lat)
    bary = np.concatenate([k - lat.sum(1, keepdims=True), lat], axis=1)  # weights of the dim + 1 vertices
    # nodes: equal where the vertices of nonzero weight and the weights agree, numbered by first appearance
    ids = np.where(bary[None] > 0, cells[:, None, :].astype(np.int64), -1)
    key = np.sort(np.where(ids >= 0, ids * (k + 1) + bary[None], -1), axis=2)
    code = np.zeros(key.shape[:2], dtype=np.int64)
    uniq = [np.unique(key[:, :, r], return_inverse=True)[1].reshape(key.shape[:2]) for r in range(dim + 1)]
    for u in uniq:
        code = np.unique(code * (int(u.max()) + 1) + u, return_inverse=True)[1].reshape(code.shape)
    _, first, inv = np.unique(code.reshape(-1), return_index=True, return_inverse=True)
    rank = np.empty(len(first), dtype=np.int64)
    rank[np.argsort(first)] = np.arange(len(first))
    node = rank[inv.reshape(-1)].reshape(code.shape)
    # boundary: nodes of the facets of one cell only
    fixed = np.zeros(len(first), dtype=bool)
    facets = np.concatenate([np.sort(np.delete(cells, j, axis=1), axis=1) for j in range(dim + 1)]).astype(np.int64)
    _, fi, cnt = np.unique(facets @ (len(v) ** np.arange(dim)), return_inverse=True, return_counts=True)
    lone = (cnt[fi.reshape(-1)] == 1).reshape(dim + 1, len(cells))
    for j in range(dim + 1):
        fixed[node[lone[j]][:, bary[:, j] == 0]] = True
    number = np.where(fixed, -1, np.cumsum(~fixed) - 1)
    dof = _t(number[node], torch.int64)
    nfree = int((~fixed).sum())
    # reference basis by the change of basis from monomials; collapsed Gauss points
    expo = lat.astype(np.float64)
    mono = lambda p: np.prod(p[:, None, :] ** expo[None], axis=2)  # noqa: E731
    C = np.linalg.inv(mono(lat / k))
    u, w = _tensor_points(dim, k + 2)
    p, jac = u.copy(), w.copy()
    p[:, 1] *= 1 - u[:, 0]
    jac *= 1 - u[:, 0]
    if dim == 3:
        p[:, 2] *= (1 - u[:, 0]) * (1 - u[:, 1])
        jac *= (1 - u[:, 0]) * (1 - u[:, 1])
    phi = mono(p) @ C
    dphi = []
    for s in range(dim):
        low = expo.copy()
        low[:, s] = np.maximum(low[:, s] - 1, 0)
        dphi.append((expo[:, s] * np.prod(p[:, None, :] ** low[None], axis=2)) @ C)
    dphi = _t(np.stack(dphi, axis=2))
    Xc = _t(v)[_t(cells, torch.int64)]
    J = (Xc[:, 1:] - Xc[:, :1]).transpose(1, 2)
    det = torch.linalg.det(J).abs()
    Ji = torch.linalg.inv(J)
    R = torch.einsum("q,qas,qbt->stab", _t(jac), dphi, dphi)
    K = torch.einsum("csr,ctr,c->cst", Ji, Ji, det * _t(coef))
    A = torch.einsum("cst,stab->cab", K, R)
    F = det[:, None] * _t(jac @ phi)[None, :]
    free = dof >= 0
    rhs = torch.zeros(nfree, dtype=torch.float64, device=A.device)
    rhs.index_add_(0, dof[free], F[free])
    both = free[:, :, None] & free[:, None, :]
    flat = (dof[:, :, None] * nfree + dof[:, None, :])[both]
    keys, inv = torch.unique(flat, return_inverse=True)
    values = torch.zeros(keys.numel(), dtype=torch.float64, device=A.device)
    values.index_add_(0, inv, A[both])
    rowptr = torch.zeros(nfree + 1, dtype=torch.int64, device=A.device)
    torch.cumsum(torch.bincount(keys // nfree, minlength=nfree), 0, out=rowptr[1:])
    return rowptr, keys % nfree, values, rhs


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for n, k, s in _batch_specs(case, seed):
            rowptr, cl, w, f, nc, values, rhs = _hex_system(3, [n] * 3, k, "poisson", *_mesh_arrays(3, [n] * 3, s))
            out.append(_solve(rowptr, _hex_colind(rowptr, cl, w, f, nc), values, rhs))
        return dict(x=out)
    dim, n = case["dim"], _cells(case)
    if kind == "simplex":
        rowptr, colind, values, rhs = _simplex_system(dim, case["order"], *_simplex_arrays(dim, n, seed))
        return dict(values=values, rhs=rhs, dinv=1.0 / _diagonal(rowptr, colind, values),
                    x=_solve(rowptr, colind, values, rhs))
    v, coef = _mesh_arrays(dim, n, seed)
    if kind == "dg":
        values, rhs, dinv = _dg_system(dim, n, case["order"], v)
        return dict(values=values, rhs=rhs, dinv=dinv)
    order, problem = (1, "poisson") if kind == "refine" else (case["order"], case["problem"])
    rowptr, cl, w, f, nc, values, rhs = _hex_system(dim, n, order, problem, v, coef)
    if kind == "assemble":
        # the diagonal: the row node's own box position, its own component
        nf = rhs.numel() // nc
        node, pos, scale = torch.arange(nf, device=rhs.device), 0, nc
        for r in range(dim):
            t = node % f[r]
            node = node // f[r]
            pos = pos + (t + 1 - cl[r][t]) * scale
            scale = scale * w[r][t]
        at = rowptr[:-1].reshape(nf, nc) + pos[:, None] + torch.arange(nc, device=rhs.device)[None, :]
        return dict(values=values, rhs=rhs, dinv=1.0 / values[at.reshape(-1)])
    colind = _hex_colind(rowptr, cl, w, f, nc)
    if kind == "spmv":
        A = torch.sparse_csr_tensor(rowptr, colind, values, size=(rhs.numel(),) * 2)
        return dict(y=A @ _spmv_input(rhs.numel(), seed).to(rhs.device))
    x = _solve(rowptr, colind, values, rhs)
    return dict(x=x) if kind == "refine" else dict(values=values, rhs=rhs, x=x)
