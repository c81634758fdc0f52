// fe_dg.hip -- interior-penalty discontinuous Galerkin for -Laplace(u) = f on
// the brick (Sect. 3.12 eq. ip_dg_formulations; the facet matrices of eq.
// local_to_face_matrix; facet integration of Sect. 3.13).
//
// Space: Q_k on every cell with no DOF shared between cells, DOF(K, a) =
// K nn + a (local node order of the conforming space).  The CSR row of
// DOF(K, a) holds the nn columns of K and of each facet neighbour of K, cells
// in ascending order, so the pattern is a closed form of the cell index.
//
// Assembly is a gather over cells, with no atomics: one workgroup per few cells
// writes every entry of the nn rows of its cells.
//  - The volume block is the Poisson element matrix with coefficient 1 (the
//    integration kernels of fe_integrate*.hip).
//  - Each of the 2d facets of K adds its two facet matrices with K as the row
//    side: A^F_KK into the diagonal block and A^F_KL into the block of the
//    neighbour L.  The neighbour writes the other two, A^F_LL and A^F_LK, from
//    its own side.
//  - The facet form is unchanged when the two sides and the normal are
//    swapped, so every cell uses its own outward normal.
//  - The facet's measure, normal and penalty always come from the cell below
//    the facet (the lower index along the facet's axis).  Both cells then see
//    the same numbers, and for tau = 1 the blocks A^F_KL and A^F_LK are
//    transposes of each other to the last bit.
//  - The two sides of a brick facet carry the same quadrature points in the
//    same order: the point permutation between the sides is the identity.
//
// Trace structure used by the facet kernel.  The trace of the Lagrange basis
// on a facet is nonzero only for the (k+1)^(d-1) nodes on it.  Its value at
// a facet point is a product of 1D Lagrange values, the same on both sides.
// With
//   A[t][b] = sum_q W_q phi_t(q) (n . grad phi_b^K)(q)   (K's normal derivatives)
//   B[t][b] = sum_q W_q phi_t(q) (n . grad phi_b^L)(q)   (the neighbour's)
//   M[t][u] = sum_q W_q phi_t(q) phi_u(q)                 (facet mass)
// for facet nodes t and u, cell nodes b, K's outward unit normal n and W_q =
// Gauss weight x facet measure, every facet entry is a signed combination of
// at most three of these values.  For b with index j along the facet's axis
// and tangential index u they are D_end(j) X0[t][u], plus X1[t][u] if b is on
// the facet: the kernel sums X0, X1 and M once for each (t, u).
#include <algorithm>
#include <cmath>

#include "fe_geom.h"
#include "fe_internal.h"

namespace fe {

struct DgArgs {
    int32_t dim, k;
    int32_t n[3];
    int64_t st[3];  // cell id strides 1, n0, n0 n1
    int64_t ncells, n_rows, nnz;
    double gamma, tau;
    // 1D tables: Gauss points and weights on [0,1]; Lagrange values and
    // derivatives at the Gauss points [i (k+1) + q] and at the ends [2 i + e]
    double gx[kMaxQ1], gw[kMaxQ1];
    double L[kMaxQ1 * kMaxQ1], D[kMaxQ1 * kMaxQ1];
    double Le[2 * kMaxQ1], De[2 * kMaxQ1];
};

__host__ __device__ __forceinline__ int64_t dg_prefix(const DgArgs &d, int64_t K)
{
    return dg_prefix_n(d.dim, d.n[0], d.n[1], d.n[2], K);
}

// Facet neighbours of K and their column slots (the loops unrolled, so that the
// arrays stay in registers: placed in LDS by the compiler they cost a read of
// the dispatch packet, 12 us a launch).  Facet f = 2 r + side
// (side 1: x_r grows); nb[f] = -1 on the boundary.  Slots number the cells
// of K's row block in ascending id order: lower neighbours (far axis first),
// K itself, upper neighbours.
__host__ __device__ __forceinline__ void dg_cell_faces(const DgArgs &d, int64_t K, int64_t nb[6], int slot[6],
                                                       int &self, int &nc)
{
    const int64_t c[3] = {K % d.n[0], (K / d.n[0]) % d.n[1], d.dim == 3 ? K / (int64_t(d.n[0]) * d.n[1]) : 0};
    int s = 0;
#pragma unroll
    for (int r = 2; r >= 0; r--) {
        if (r >= d.dim) continue;
        const bool has = c[r] > 0;
        nb[2 * r] = has ? K - d.st[r] : -1;
        slot[2 * r] = has ? s++ : -1;
    }
    self = s++;
#pragma unroll
    for (int r = 0; r < 3; r++) {
        if (r >= d.dim) continue;
        const bool has = c[r] < d.n[r] - 1;
        nb[2 * r + 1] = has ? K + d.st[r] : -1;
        slot[2 * r + 1] = has ? s++ : -1;
    }
    nc = s;
}

// ---------------------------------------------------------------------------
// Pattern: one workgroup per cell writes the row pointers and columns of its
// nn rows (row a of K: nc nn columns, the nn DOFs of each cell of the block).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dg_pattern_kernel(DgArgs d, int32_t nn, int64_t *__restrict__ rowptr,
                                                         int32_t *__restrict__ colind)
{
    __shared__ int64_t sCells[7];
    __shared__ int sNc;
    const int64_t K = xcd_block(blockIdx.x, gridDim.x);
    if (threadIdx.x == 0) {
        int64_t nb[6];
        int slot[6], self, nc;
        dg_cell_faces(d, K, nb, slot, self, nc);
        for (int f = 0; f < 2 * d.dim; f++)
            if (slot[f] >= 0) sCells[slot[f]] = nb[f];
        sCells[self] = K;
        sNc = nc;
    }
    __syncthreads();
    const int nc = sNc;
    const int64_t base = int64_t(nn) * nn * dg_prefix(d, K);
    const int rlen = nc * nn;
    for (int a = threadIdx.x; a < nn; a += blockDim.x) rowptr[K * nn + a] = base + int64_t(a) * rlen;
    if (K == d.ncells - 1 && threadIdx.x == 0) rowptr[d.n_rows] = d.nnz;
    for (int e = threadIdx.x; e < nn * rlen; e += blockDim.x) {
        const int pos = e % rlen;
        colind[base + e] = int32_t(sCells[pos / nn] * nn + pos % nn);
    }
}

// ---------------------------------------------------------------------------
// Facet kernel
// ---------------------------------------------------------------------------
template <int DIM, int KO>
struct DgShape {
    static constexpr int K1 = KO + 1;
    static constexpr int NN = DIM == 3 ? K1 * K1 * K1 : K1 * K1;  // nodes per cell
    static constexpr int NF = DIM == 3 ? K1 * K1 : K1;           // nodes per facet
    static constexpr int NP = NF;                                // facet points (k + 1 per direction)
    static constexpr int NFACE = 2 * DIM;
    static constexpr int NT = NF * NF;  // threads of a cell: one per pair (t, u) of tangential indices
    // 3D Q2: three cells (243 of 256 threads) beat one in 128 threads (896 us
    // against 857) and two in 192 (848 against 815)
    static constexpr int BS = NT > 256 ? 640 : (DIM == 3 && KO >= 2 ? 256 : 64);
    static constexpr int CB = BS / NT;  // most cells per workgroup
    // waves per SIMD asked of the register allocator: 3D Q2 takes 128 registers
    // instead of 136 and a fourth wave (857 -> 815 us at 32^3 with the element
    // matrices; a fifth spills, 1055)
    static constexpr int MINW = DIM == 3 && KO == 2 ? 4 : 1;
    static_assert(CB >= 1 && CB * NN <= BS, "a thread per row of the workgroup's cells");
};

// First node (index 0 along axis R) of tangential index t: its digits have the
// strides of the other axes.
template <int DIM, int KO, int R>
__device__ __forceinline__ int dg_tangent(int t)
{
    constexpr int K1 = KO + 1;
    if (DIM == 2) return R == 0 ? t * K1 : t;
    if (R == 0) return t * K1;
    if (R == 2) return t;
    return t % K1 + (t / K1) * (K1 * K1);
}

// One thread's (t, u) of its cell, and its 1D products at the Gauss points of
// the two tangential directions: phi_t phi_u, phi_t phi_u' and phi_t' phi_u.
struct DgPair {
    int t, u;
    const double *m0, *g0, *h0, *m1, *g1, *h1;
};

// Both facets of axis R for one pair (t, u): their entries (a, b) with a =
// (ar, t), b = (br, u), for all ar and br.  sS holds, for each facet point, W,
// W J^-1 n on K's side and on the neighbour's (along r, t0, t1).
template <int DIM, int KO, int R>
__device__ __forceinline__ void dg_axis(const DgArgs &d, const DgPair &P, const double *__restrict__ sS,
                                        const double *__restrict__ sSig, const int *__restrict__ sSlot,
                                        double *__restrict__ diag, double *__restrict__ out, int rlen)
{
    using S = DgShape<DIM, KO>;
    constexpr int K1 = S::K1, NN = S::NN, NP = S::NP;
    constexpr int UQ = KO <= 1 ? KO + 1 : 1;
    constexpr int SR = R == 0 ? 1 : (R == 1 ? K1 : K1 * K1);  // node stride along R
    const int a0 = dg_tangent<DIM, KO, R>(P.t), b0 = dg_tangent<DIM, KO, R>(P.u);
    double dg[K1][K1];
#pragma unroll
    for (int i = 0; i < K1; i++)
#pragma unroll
        for (int j = 0; j < K1; j++) dg[i][j] = 0.0;
#pragma unroll
    for (int side = 0; side < 2; side++) {
        const int f = 2 * R + side;
        const int slot = sSlot[f];
        const bool interior = slot >= 0;
        // X0 = sum_q W (J^-1 n)_r phi_t phi_u on either side, X1 = sum_q W
        // phi_t ((J^-1 n)_t0 d0 phi_u + (J^-1 n)_t1 d1 phi_u), T1 the same with
        // t and u exchanged, M = sum_q W phi_t phi_u
        double M = 0.0, X0 = 0.0, X1 = 0.0, T1 = 0.0, Y0 = 0.0, Y1 = 0.0;
        const double *__restrict__ q = sS + f * NP * 8;
        if (DIM == 2) {
#pragma unroll
            for (int q0 = 0; q0 < K1; q0++, q += 8) {
                M += q[0] * P.m0[q0];
                X0 += q[1] * P.m0[q0];
                X1 += q[2] * P.g0[q0];
                T1 += q[2] * P.h0[q0];
                Y0 += q[4] * P.m0[q0];
                Y1 += q[5] * P.g0[q0];
            }
        } else {
            double m1[K1], g1[K1], h1[K1];
#pragma unroll
            for (int q1 = 0; q1 < K1; q1++) {
                m1[q1] = P.m1[q1];
                g1[q1] = P.g1[q1];
                h1[q1] = P.h1[q1];
            }
#pragma unroll UQ
            for (int q0 = 0; q0 < K1; q0++) {
                double wM = 0.0, wX = 0.0, wY = 0.0, a = 0.0, ga = 0.0, ha = 0.0, b = 0.0, gb = 0.0;
#pragma unroll
                for (int q1 = 0; q1 < K1; q1++) {
                    const double *__restrict__ v = q + (q0 + q1 * K1) * 8;
                    wM += v[0] * m1[q1];
                    wX += v[1] * m1[q1];
                    a += v[2] * m1[q1];
                    ga += v[3] * g1[q1];
                    ha += v[3] * h1[q1];
                    wY += v[4] * m1[q1];
                    b += v[5] * m1[q1];
                    gb += v[6] * g1[q1];
                }
                M += wM * P.m0[q0];
                X0 += wX * P.m0[q0];
                X1 = fma(ga, P.m0[q0], fma(a, P.g0[q0], X1));
                T1 = fma(ha, P.m0[q0], fma(a, P.h0[q0], T1));
                Y0 += wY * P.m0[q0];
                Y1 = fma(gb, P.m0[q0], fma(b, P.g0[q0], Y1));
            }
        }
        // normal derivatives: A of K's basis functions, B of the neighbour's
        // (whose reference coordinate along R is 1 - side); index on the facet
        // along R on K's side is e, on the neighbour's side o.  The roundings are
        // spelled out where the two cells of a facet compute the same number in
        // different roles: their blocks are transposes to the last bit at tau 1.
        constexpr int ends[2] = {0, KO};
        const int e = ends[side], o = ends[1 - side];
        const double cc = interior ? 0.5 : 1.0;
        double A[K1], At[K1], B[K1];
#pragma unroll
        for (int i = 0; i < K1; i++) {
            const double de = d.De[2 * i + side], dn = d.De[2 * i + 1 - side];
            A[i] = i == e ? fma(de, X0, X1) : de * X0;
            At[i] = i == e ? fma(de, X0, T1) : de * X0;
            B[i] = i == o ? fma(dn, Y0, Y1) : dn * Y0;
        }
#pragma unroll
        for (int i = 0; i < K1; i++) {
            dg[e][i] -= cc * A[i];
            dg[i][e] -= cc * d.tau * At[i];
        }
        dg[e][e] = fma(sSig[f], M, dg[e][e]);
        if (interior) {
            double *__restrict__ w = out + (int64_t(a0) * rlen + slot * NN + b0);
#pragma unroll
            for (int i = 0; i < K1; i++)
#pragma unroll
                for (int j = 0; j < K1; j++) {
                    double v = 0.0;
                    if (i == e) v = -0.5 * B[j];
                    if (j == o) v = fma(0.5 * d.tau, At[i], v);
                    if (i == e && j == o) v = fma(-sSig[f], M, v);
                    w[int64_t(i) * SR * rlen + j * SR] = v;
                }
        }
    }
#pragma unroll
    for (int i = 0; i < K1; i++)
#pragma unroll
        for (int j = 0; j < K1; j++)
            if (i == 0 || i == KO || j == 0 || j == KO) diag[(a0 + i * SR) * NN + b0 + j * SR] += dg[i][j];
}

// One workgroup per CB cells, one thread per cell and pair (t, u) of
// tangential indices.  Phases:
//  0. neighbours, vertices of the cells and their neighbours, and the element
//     matrices into LDS; the 1D products of a pair into registers;
//  1. the geometry of every (cell, facet, point) by one thread: the facet
//     normal from the cell below the facet, then weight times J^-1 n on each
//     side, Dirichlet data; 2. penalties;
//  3. per axis, from the sums over the points of both facets, a pair's
//     (k + 1)^2 entries of the diagonal block and of each neighbour's.
// What bounds it: waiting, for the barriers of a cell and the stores.  The basis is a
// tensor product, so along the axis of a facet only the ends differ: a pair's
// entries come from six sums over the points (phi_t phi_u with W and with the
// normal parts of either side, phi_t grad phi_u likewise), each separable in
// the two tangential directions, instead of a table of normal derivatives per
// (facet node, basis function), built facet by facet by one workgroup per cell
// and read back seven values an entry: kernel 1063 -> 556 us at 32^3 Q2 (1.30 GB of
// entries, 1.51 GB written: 2.7 TB/s; 2690 vector instructions a cell, waves waiting
// for 61% of their cycles).
// With the element matrices (of the contraction kernels, before they were
// summed by factors) 1209 -> 815, 3D Q1 33x29x35 151 -> 78, Q3 20x21x19 1360 ->
// 785, Q4 14x13x12 2500 -> 1092, 2D Q1 300x280 129 -> 55, Q4 90x100 243 -> 208;
// of the 815, 250 go into storing the neighbours' blocks: runs of 24 to 72
// bytes of 216-byte pieces.  Passing the blocks through LDS makes the pieces
// whole and costs two barriers a facet: 857 -> 839 at Q2, 780 -> 859 at Q3.
template <int DIM, int KO>
__global__ __launch_bounds__((DgShape<DIM, KO>::BS), (DgShape<DIM, KO>::MINW)) void dg_cell_kernel(
    DgArgs d, MeshArgs m, ProblemArgs p, ElemLayout el, const double *__restrict__ E, const double *__restrict__ F,
    const int64_t *__restrict__ rowptr, double *__restrict__ values, double *__restrict__ rhs,
    double *__restrict__ dinv, int cells)
{
    using S = DgShape<DIM, KO>;
    constexpr int K1 = S::K1, NN = S::NN, NF = S::NF, NP = S::NP, NFACE = S::NFACE, BS = S::BS, CB = S::CB;
    constexpr int NT = S::NT, NV = 1 << DIM;
    __shared__ double sDiag[CB][NN * NN];
    // per facet point: W, W J^-1 n on K's side (along r, t0, t1) and on the
    // neighbour's, n = K's outward normal, and the Dirichlet value
    __shared__ __attribute__((aligned(16))) double sS[CB][NFACE * NP * 8];
    __shared__ double sV[CB][1 + NFACE][NV][3];  // vertices of K (slot 0) and of the neighbour across facet f (1 + f)
    __shared__ double sPr[2][K1 * K1 * K1];      // phi_t phi_u and phi_t phi_u' at a 1D Gauss point, [(t K1 + u) K1 + q]
    __shared__ double sL[K1 * K1], sD[K1 * K1], sG[2][K1];  // 1D tables: read by lane, so not from the arguments
    __shared__ double sSig[CB][NFACE];
    __shared__ int sSlot[CB][NFACE], sSelf[CB], sNc[CB];

    const int64_t Kb = xcd_block(blockIdx.x, gridDim.x) * cells;
    const int tid = threadIdx.x;
    const int ncb = d.ncells - Kb < cells ? int(d.ncells - Kb) : cells;  // cells of this workgroup
    if (tid < ncb) {
        int64_t nb[6];
        int slot[6], self, nc;
        dg_cell_faces(d, Kb + tid, nb, slot, self, nc);
#pragma unroll
        for (int f = 0; f < NFACE; f++) sSlot[tid][f] = slot[f];
        sSelf[tid] = self;
        sNc[tid] = nc;
    }
    for (int e = tid; e < ncb * ((1 + NFACE) * NV); e += BS) {
        const int ci = e / ((1 + NFACE) * NV), i = e - ci * ((1 + NFACE) * NV), sl = i / NV, v = i % NV;
        const int32_t cell = int32_t(Kb) + ci;  // rows, so cells, are below 2^31
        const int32_t cy = cell / d.n[0], cz = DIM == 3 ? cy / d.n[1] : 0;
        const int r = sl > 0 ? (sl - 1) >> 1 : 3, step = (sl - 1) & 1 ? 1 : -1;
        const int32_t c0 = cell - cy * d.n[0] + (r == 0 ? step : 0);
        const int32_t c1 = (DIM == 3 ? cy - cz * d.n[1] : cy) + (r == 1 ? step : 0);
        const int32_t c2 = cz + (r == 2 ? step : 0);
        if (c0 < 0 || c0 >= d.n[0] || c1 < 0 || c1 >= d.n[1] || c2 < 0 || (DIM == 3 && c2 >= d.n[2])) continue;
        const int64_t vid = (c0 + (v & 1)) + int64_t(m.n0 + 1) * ((c1 + ((v >> 1) & 1)) +
                                                                  int64_t(m.n1 + 1) * (DIM == 3 ? c2 + ((v >> 2) & 1) : 0));
        sV[ci][sl][v][0] = m.x[vid];
        sV[ci][sl][v][1] = m.y[vid];
        sV[ci][sl][v][2] = DIM == 3 ? m.z[vid] : 0.0;
    }
    if (tid < K1 * K1) {
        sL[tid] = d.L[tid];
        sD[tid] = d.D[tid];
    }
    if (tid < K1) {
        sG[0][tid] = d.gx[tid];
        sG[1][tid] = d.gw[tid];
    }
    // the diagonal blocks start from the element matrices
    for (int e = tid; e < ncb * (NN * NN); e += BS) {
        const int ci = e / (NN * NN), i = e - ci * (NN * NN);
        sDiag[ci][i] = E[elem_index(Kb + ci, i / NN, i % NN, NN, el.cb, el.packed, el.ne)];
    }
    const int rc = tid / NN, rb = tid - rc * NN;  // row of the workgroup that this thread holds the rhs of
    double racc = rc < ncb ? F[(Kb + rc) * NN + rb] : 0.0;
    DgPair P;
    const int ci = CB == 1 ? 0 : tid / NT;  // one cell: what depends on it stays uniform
    const bool on = CB == 1 ? tid < NT : ci < ncb;
    {
        const int pr = min(tid - ci * NT, NT - 1);
        P.t = pr / NF;
        P.u = pr - P.t * NF;
        const int t0 = P.t % K1, t1 = P.t / K1 % K1, u0 = P.u % K1, u1 = P.u / K1 % K1;
        P.m0 = sPr[0] + (t0 * K1 + u0) * K1;
        P.g0 = sPr[1] + (t0 * K1 + u0) * K1;
        P.h0 = sPr[1] + (u0 * K1 + t0) * K1;
        P.m1 = sPr[0] + (t1 * K1 + u1) * K1;
        P.g1 = sPr[1] + (t1 * K1 + u1) * K1;
        P.h1 = sPr[1] + (u1 * K1 + t1) * K1;
    }
    __syncthreads();

    for (int e = tid; e < K1 * K1 * K1; e += BS) {
        const int t = e / (K1 * K1), u = e / K1 % K1, q = e % K1;
        sPr[0][e] = sL[t * K1 + q] * sL[u * K1 + q];
        sPr[1][e] = sL[t * K1 + q] * sD[u * K1 + q];
    }
    // 1. the facet normal from the cell below the facet (K on its upper facets
    // and on the boundary), then J^-1 n there and on the other side
    for (int i = tid; i < ncb * (NFACE * NP); i += BS) {
        const int cj = i / (NFACE * NP), fq = i - cj * (NFACE * NP), f = fq / NP, q = fq - f * NP;
        const int r = f >> 1, side = f & 1;
        const bool interior = sSlot[cj][f] >= 0;
        const int t0 = DIM == 2 ? 1 - r : (r == 0 ? 1 : 0), t1 = DIM == 2 ? -1 : (r == 2 ? 1 : 2);
        const int q0 = q % K1, q1 = q / K1;
        double *__restrict__ o = sS[cj] + fq * 8;
        double n[3] = {0.0, 0.0, 0.0}, w = 0.0;
#pragma unroll 1
        for (int gs = 0; gs < 2; gs++) {
            const bool mine = gs == 0 ? side == 1 || !interior : !(side == 1 || !interior);  // K's own side
            if (gs == 1 && !interior) break;
            const double er = mine == (side == 1) ? 1.0 : 0.0;  // reference coordinate along r
            double xi[3];
#pragma unroll
            for (int sx = 0; sx < 3; sx++) xi[sx] = sx == r ? er : (sx == t0 ? sG[0][q0] : (sx == t1 ? sG[0][q1] : 0.0));
            double X[NV][3], J[9], Ji[9], xq[3];
#pragma unroll
            for (int v = 0; v < NV; v++)
#pragma unroll
                for (int c = 0; c < 3; c++) X[v][c] = sV[cj][mine ? 0 : 1 + f][v][c];
            const double det = geometry<DIM>(X, xi, J, Ji, xq);
            if (!(det > 0.0)) atomicOr(m.status, 1);
            if (gs == 0) {
                double nn2 = 0.0;
#pragma unroll
                for (int rr = 0; rr < DIM; rr++)
                    if (rr == r) {
#pragma unroll
                        for (int c = 0; c < DIM; c++) n[c] = det * Ji[rr * DIM + c];
                    }
#pragma unroll
                for (int c = 0; c < DIM; c++) nn2 += n[c] * n[c];
                const double dS = sqrt(nn2);
                const double sgn = side ? 1.0 : -1.0;
#pragma unroll
                for (int c = 0; c < DIM; c++) n[c] = sgn * (n[c] / dS);
                w = (sG[1][q0] * (DIM == 3 ? sG[1][q1] : 1.0)) * dS;
                o[0] = w;
            }
#pragma unroll
            for (int sx = 0; sx < DIM; sx++) {
                double mv = 0.0;
#pragma unroll
                for (int c = 0; c < DIM; c++) mv += Ji[sx * DIM + c] * n[c];
                o[(mine ? 1 : 4) + (sx == r ? 0 : (sx == t0 ? 1 : 2))] = w * mv;
            }
            if (mine) {
                double u = 0.0;
                if (!interior && p.dirichlet_kind == FE_DIRICHLET_AFFINE) {
                    u = p.aff[0];
#pragma unroll
                    for (int c = 0; c < DIM; c++) u += p.aff[1 + c] * xq[c];
                }
                o[7] = u;
            }
        }
    }
    __syncthreads();
    if (tid < ncb * NFACE) {
        const int cj = tid / NFACE, f = tid - cj * NFACE;
        double area = 0.0;
#pragma unroll
        for (int q = 0; q < NP; q++) area += sS[cj][(f * NP + q) * 8];
        sSig[cj][f] = d.gamma / (DIM == 3 ? sqrt(area) : area);
    }
    __syncthreads();

    // weak Dirichlet data of row b on its cell's boundary facets:
    // sum_q W u_D (-tau n.grad phi_b + sigma phi_b)
    if (rc < ncb && p.dirichlet_kind == FE_DIRICHLET_AFFINE) {
        const int b0 = rb % K1, b1 = rb / K1 % K1, b2 = DIM == 3 ? rb / (K1 * K1) : 0;
        for (int f = 0; f < NFACE; f++) {
            if (sSlot[rc][f] >= 0) continue;
            const int r = f >> 1, side = f & 1;
            const int br = r == 0 ? b0 : (r == 1 ? b1 : b2), bt0 = r == 0 ? b1 : b0, bt1 = r == 2 ? b1 : b2;
            const double le = d.Le[2 * br + side], de = d.De[2 * br + side], sig = sSig[rc][f];
            double sr = 0.0;
            for (int q = 0; q < NP; q++) {
                const int i0 = bt0 * K1 + q % K1, i1 = bt1 * K1 + q / K1;
                const double l0 = sL[i0], l1 = DIM == 3 ? sL[i1] : 1.0;
                const double *__restrict__ v = sS[rc] + (f * NP + q) * 8;
                double dn = v[1] * (de * l0 * l1) + v[2] * (le * sD[i0] * l1);
                if (DIM == 3) dn += v[3] * (le * l0 * sD[i1]);
                double t = -d.tau * dn;
                if (br == (side ? KO : 0)) t += sig * (v[0] * (l0 * l1));
                sr += v[7] * t;
            }
            racc += sr;
        }
    }
    if (rc < ncb) rhs[(Kb + rc) * NN + rb] = racc;

    const int cs = CB > 1 && on ? ci : 0;
    const int64_t row0 = rowptr[(Kb + cs) * NN];
    const int rlen = sNc[cs] * NN;
    if (on) dg_axis<DIM, KO, 0>(d, P, sS[ci], sSig[ci], sSlot[ci], sDiag[ci], values + row0, rlen);
    __syncthreads();
    if (on) dg_axis<DIM, KO, 1>(d, P, sS[ci], sSig[ci], sSlot[ci], sDiag[ci], values + row0, rlen);
    __syncthreads();
    if constexpr (DIM == 3) {
        if (on) dg_axis<DIM, KO, 2>(d, P, sS[ci], sSig[ci], sSlot[ci], sDiag[ci], values + row0, rlen);
        __syncthreads();
    }
    // the diagonal blocks, and 1 / their diagonals; the cell's threads are a
    // multiple of nn, so a thread keeps its column
    if (on) {
        constexpr int NR = NT / NN;  // rows at a time
        const int lane = tid - ci * NT;
        double *__restrict__ out = values + (row0 + sSelf[ci] * NN + int64_t(lane / NN) * rlen + lane % NN);
#pragma unroll
        for (int i = 0; i < NN / NR; i++) out[int64_t(i) * NR * rlen] = sDiag[ci][lane + i * NT];
    }
    if (rc < ncb) dinv[(Kb + rc) * NN + rb] = 1.0 / sDiag[rc][rb * NN + rb];
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static DgArgs make_dg(int dim, const int32_t *n, int k, double gamma, double tau)
{
    DgArgs d{};
    d.dim = dim;
    d.k = k;
    d.n[0] = n[0];
    d.n[1] = n[1];
    d.n[2] = dim == 3 ? n[2] : 1;
    d.st[0] = 1;
    d.st[1] = d.n[0];
    d.st[2] = int64_t(d.n[0]) * d.n[1];
    d.ncells = d.st[2] * d.n[2];
    int nn = 1;
    for (int r = 0; r < dim; r++) nn *= k + 1;
    d.n_rows = d.ncells * nn;
    d.nnz = int64_t(nn) * nn * dg_prefix(d, d.ncells);
    d.gamma = gamma;
    d.tau = tau;
    RefTables rt;
    ref_tables(k, rt);
    for (int i = 0; i <= k; i++) {
        d.gx[i] = rt.gx[i];
        d.gw[i] = rt.gw[i];
        lagrange_1d(k, i, 0.0, d.Le[2 * i], d.De[2 * i]);
        lagrange_1d(k, i, 1.0, d.Le[2 * i + 1], d.De[2 * i + 1]);
    }
    for (int t = 0; t < (k + 1) * (k + 1); t++) {
        d.L[t] = rt.L[t];
        d.D[t] = rt.D[t];
    }
    return d;
}

void dg_sizes(int dim, const int32_t *n, int k, int64_t &n_rows, int64_t &nnz)
{
    const DgArgs d = make_dg(dim, n, k, 1.0, 1.0);
    n_rows = d.n_rows;
    nnz = d.nnz;
}

SpaceArgs dg_space(int dim, const int32_t *n, int k)
{
    const DgArgs d = make_dg(dim, n, k, 1.0, 1.0);
    SpaceArgs sa{};
    sa.dim = dim;
    sa.k = k;
    sa.ncomp = 1;
    sa.nn = int32_t(d.n_rows / (d.ncells > 0 ? d.ncells : 1));
    sa.nloc = sa.nn;
    for (int r = 0; r < 3; r++) sa.ax[r].n = d.n[r];
    sa.ncells = d.ncells;
    sa.n_rows = d.n_rows;
    sa.nnz = d.nnz;
    return sa;
}

fe_status launch_dg_pattern(int dim, const int32_t *n, int k, int64_t *rowptr, int32_t *colind, hipStream_t s)
{
    const DgArgs d = make_dg(dim, n, k, 1.0, 1.0);
    if (d.ncells == 0) return FE_OK;
    const int32_t nn = int32_t(d.n_rows / d.ncells);
    hipLaunchKernelGGL(dg_pattern_kernel, dim3(d.ncells), dim3(256), 0, s, d, nn, rowptr, colind);
    FE_HIP(hipGetLastError());
    return FE_OK;
}

fe_status launch_dg_facets(int dim, const int32_t *n, int k, double gamma, double tau, const MeshArgs &ma,
                           const ProblemArgs &pa, const ElemLayout &el, const void *ws, const int64_t *rowptr,
                           double *values, double *rhs, double *dinv, hipStream_t s)
{
    const DgArgs d = make_dg(dim, n, k, gamma, tau);
    if (d.ncells == 0) return FE_OK;
    const double *E = static_cast<const double *>(ws);
    const double *F = reinterpret_cast<const double *>(static_cast<const char *>(ws) + el.f_offset);
    // Few cells: a workgroup takes fewer of them, so that four workgroups a CU
    // share the chain of phases (with the element matrices, 3D Q2 6x7x5 22.7 ->
    // 19.9 us)
#define FE_DGK(D, KO)                                                                                          \
    {                                                                                                          \
        const int cells = int(std::min<int64_t>(DgShape<D, KO>::CB, (d.ncells + 1023) / 1024));                \
        hipLaunchKernelGGL((dg_cell_kernel<D, KO>), dim3((d.ncells + cells - 1) / cells),                      \
                           dim3((DgShape<D, KO>::BS)), 0, s, d, ma, pa, el, E, F, rowptr, values, rhs, dinv,   \
                           cells);                                                                             \
    }
    if (dim == 3) {
        switch (k) {
            case 1: FE_DGK(3, 1); break;
            case 2: FE_DGK(3, 2); break;
            case 3: FE_DGK(3, 3); break;
            default: FE_DGK(3, 4); break;
        }
    } else {
        switch (k) {
            case 1: FE_DGK(2, 1); break;
            case 2: FE_DGK(2, 2); break;
            case 3: FE_DGK(2, 3); break;
            default: FE_DGK(2, 4); break;
        }
    }
#undef FE_DGK
    FE_HIP(hipGetLastError());
    return FE_OK;
}

}  // namespace fe
