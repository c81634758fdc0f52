// fe_integrate_tensor.hip -- K3 in FP64 on quadrilaterals and hexahedra of order
// 2..4 (and Q1 elasticity): element matrices by sum factorization (Sect. 3.7 eq. fematrix;
// the Poisson element loop of Sect. 8.5 for a tensor-product basis).
//
// With a = (a0, a1, a2), q = (q0, q1, q2), phi_a = prod_d phi_{a_d}(xi_d) and
// J^-1 at q, the block of components (i, j) is
//   A_ij[a][b] = sum_rs sum_q D_rs^ij(q) d_r phi_a(q) d_s phi_b(q),
//   Poisson     D_rs    = w k sum_l Ji_rl Ji_sl
//   elasticity  D_rs^ij = w k (lambda Ji_ri Ji_sj + mu (Ji_rj Ji_si + delta_ij sum_l Ji_rl Ji_sl))
// and every d_r phi_a d_s phi_b separates into three 1D factors.  Per pair of
// planes (a2, b2) the sum runs one direction at a time:
//   U_rs(q0, q1)          = sum_q2 D_rs(q) T(a2, b2, q2)        9 arrays
//   V_xy(q0; a1, b1)      = sum_q1 sum U_rs(q0, q1) T(a1, b1, q1)   x, y: derivative along axis 0 on a, on b
//   A(a0, b0; a1, b1)     = sum_q0 V_xy(q0) T(a0, b0, q0)
// with T a product of values or derivatives: at Q4 some 30 operations per
// entry and component pair where the contraction over the 125 points has 125.
// In 2D the first sum falls away.  The FP64 matrix instructions run at the rate of the vector unit (64 cycles
// for a 16 x 16 x 4 product), so they gain nothing for the longer sum.
#include <algorithm>
#include <cmath>

#include "fe_geom.h"
#include "fe_internal.h"

namespace fe {

template <int K1, int PROB>
struct TensorShape {
    static constexpr int NC = PROB == 1 ? 3 : 1;
    static constexpr int NIJ = NC * NC;
    static constexpr int NN = K1 * K1 * K1, NLOC = NN * NC;  // nodes = points; rows
    static constexpr int T = K1 * K1 * NC;                   // rows of a plane of nodes
    static constexpr int TP = T | 1;                         // pitch of a staged tile: odd, so its columns are in distinct banks
    static constexpr int NPAIR = K1 * (K1 + 1) / 2;          // pairs of planes a2 <= b2
    // Pairs at a time.  Poisson: all (Q4: five of fifteen, for the tile's LDS).
    // Elasticity: one (Q3: two measured 3.59 ms against 2.54 at 32^3; Q1: all
    // three 0.80 against 0.48 at 60^3), but Q2 three, one cell a workgroup
    // (1.96 ms at 48^3; one pair and three cells 2.31, six pairs 2.30).
    static constexpr int PG = PROB == 1 ? (K1 == 3 ? 3 : 1) : (K1 == 5 ? 5 : NPAIR);
    static constexpr int NPASS = NPAIR / PG;
    static constexpr int LP = NIJ * K1 * K1;  // threads of a pair: (i, j) and (q0, q1), later (a1, b1)
    static constexpr int LN = PG * LP;        // threads of a cell
    static constexpr int BS = PROB == 1 ? (K1 == 4 ? 192 : 256) : (K1 == 3 ? 256 : (K1 == 4 ? 192 : 128));
    // Cells per workgroup.  Small systems fill their workgroup with cells: Q1
    // elasticity with seven 0.48 ms, three 0.52, one in 64 threads 0.72.
    static constexpr int CB = BS / LN;
    // Least workgroups a cell's passes are split over.  Part p takes passes p,
    // p + parts, ..., so neighbouring tiles are stored at about the same time,
    // by workgroups of one XCD, and the cache lines that two pieces of a row
    // share are completed before they are evicted.  Q4 elasticity (1.1 MB a
    // cell): 5.5 ms with one part, 4.9 with three, 4.4 with five (4.7 when a
    // part takes consecutive passes), 4.8 with fifteen, as every part repeats
    // the geometry; below Q4 that costs more than it gives (Q3 2.6 / 2.8 with
    // three, Q2 2.0 / 2.2).
    static constexpr int PARTS = PROB == 1 && K1 == 5 ? 5 : 1;
    static constexpr int MINW = K1 == 5 ? 2 : (K1 == 3 ? 4 : 3);  // waves per SIMD: as many as the LDS lets run
    static constexpr int NG = PROB == 1 ? 17 : 7;  // doubles per point (odd: distinct banks)
    static_assert(NPAIR % PG == 0 && CB >= 1 && LP == NC * T, "thread layout");
};

// One workgroup = CB cells, or a part of their passes over the plane pairs.
// One thread per pair, components (i, j) and (q0, q1) in the first sum,
// (a1, b1) in the second and third, which it does for one q0 after the other,
// the K1^2 entries (a0, b0) in registers.  The tile of a pair (T x T entries)
// is staged in LDS and stored along the rows of the matrix, as the pair's
// block and as its mirror; on a2 = b2 only the upper triangle is taken, so the
// element matrix is symmetric to the last bit.
// What bounds it: the sums and their LDS round trips (without the stores Q4
// elasticity 3.4 ms, Q3 2.2, Q2 1.7, Poisson Q2 0.23), at Q4 then the stores of
// the mirror (15.6 GB in 4.4 ms, 3.5 TB/s; without the mirror's 6.2 GB 3.6 ms),
// whose row pieces of 600 bytes begin and end inside cache lines; non-temporal
// stores made that worse (6.5 ms).  Measured
// (contraction on the matrix cores, for Q1 elasticity on the vector unit / this
// kernel, ms): elasticity Q1 60^3 3.47 / 0.48, Q2 48^3 2.34 / 1.96, Q3 32^3
// 3.29 / 2.58, Q4 24^3 8.99 / 4.40; Poisson Q2 48^3 0.72 / 0.27, Q3 40^3 1.63 /
// 0.68, Q4 30^3 4.21 / 1.16.
template <int K1, int PROB>
__device__ __forceinline__ void k3_tensor_body(const MeshArgs &m, const ProblemArgs &p, const RefTables &rt,
                                               int64_t ncells, int parts, double *__restrict__ E,
                                               double *__restrict__ F, int64_t bid)
{
    using S = TensorShape<K1, PROB>;
    constexpr int NC = S::NC, NN = S::NN, NLOC = S::NLOC, T = S::T, TP = S::TP, PG = S::PG, CB = S::CB, BS = S::BS;
    constexpr int KK = K1 * K1, NG = S::NG, UQ = PROB == 1 ? 1 : K1;
    __shared__ double sX[CB][8][3];
    __shared__ double sL[KK], sD[KK];
    // per point: w k Ji Ji^T (upper triangle by rows, times mu for elasticity); elasticity also w k and J^-1
    __shared__ double sQ[CB][NN][NG];
    __shared__ double sU[CB][PG][S::NIJ][9 * KK];
    __shared__ double sT[CB][PG][T * TP];  // first the loads w |det J| f_c of the points
    double *const sF = &sT[0][0][0];
    static_assert(NN * NC <= PG * T * TP, "the loads fit where the tiles come later");

    const int tid = threadIdx.x;
    const int part = int(bid % parts);
    const int64_t c0 = (bid / parts) * CB;
    const int ncb = ncells - c0 < CB ? int(ncells - c0) : CB;
    for (int e = tid; e < ncb * 8; e += BS) {
        const int v = e % 8;
        const int64_t cell = c0 + e / 8;
        const int64_t e0 = cell % m.n0, e1 = (cell / m.n0) % m.n1, e2 = cell / (int64_t(m.n0) * m.n1);
        const int64_t vid = (e0 + (v & 1)) + int64_t(m.n0 + 1) * ((e1 + ((v >> 1) & 1)) + int64_t(m.n1 + 1) * (e2 + ((v >> 2) & 1)));
        sX[e / 8][v][0] = m.x[vid];
        sX[e / 8][v][1] = m.y[vid];
        sX[e / 8][v][2] = m.z[vid];
    }
    for (int e = tid; e < KK; e += BS) {
        sL[e] = rt.L[e];
        sD[e] = rt.D[e];
    }
    __syncthreads();
    // geometry of every point
    for (int e = tid; e < ncb * NN; e += BS) {
        const int ci = e / NN, q = e - ci * NN;
        const int q0 = q % K1, q1 = (q / K1) % K1, q2 = q / KK;
        const double xi[3] = {rt.gx[q0], rt.gx[q1], rt.gx[q2]};
        double J[9], Ji[9], xq[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < 9; t++) J[t] = 0.0;
#pragma unroll
        for (int v = 0; v < 8; v++) {
            double f[3];
#pragma unroll
            for (int r = 0; r < 3; r++) f[r] = ((v >> r) & 1) ? xi[r] : 1.0 - xi[r];
            const double s0 = v & 1 ? 1.0 : -1.0, s1 = v & 2 ? 1.0 : -1.0, s2 = v & 4 ? 1.0 : -1.0;
            const double n = f[0] * f[1] * f[2], d0 = s0 * (f[1] * f[2]), d1 = s1 * (f[0] * f[2]), d2 = s2 * (f[0] * f[1]);
#pragma unroll
            for (int r = 0; r < 3; r++) {
                const double x = sX[ci][v][r];
                xq[r] += x * n;
                J[r * 3 + 0] += x * d0;
                J[r * 3 + 1] += x * d1;
                J[r * 3 + 2] += x * d2;
            }
        }
        const double c00 = J[4] * J[8] - J[5] * J[7];
        const double c01 = J[5] * J[6] - J[3] * J[8];
        const double c02 = J[3] * J[7] - J[4] * J[6];
        const double det = J[0] * c00 + J[1] * c01 + J[2] * c02;
        if (!(det > 0.0)) atomicOr(m.status, 1);
        const double id = 1.0 / det;
        Ji[0] = c00 * id;
        Ji[1] = (J[2] * J[7] - J[1] * J[8]) * id;
        Ji[2] = (J[1] * J[5] - J[2] * J[4]) * id;
        Ji[3] = c01 * id;
        Ji[4] = (J[0] * J[8] - J[2] * J[6]) * id;
        Ji[5] = (J[2] * J[3] - J[0] * J[5]) * id;
        Ji[6] = c02 * id;
        Ji[7] = (J[1] * J[6] - J[0] * J[7]) * id;
        Ji[8] = (J[0] * J[4] - J[1] * J[3]) * id;
        const double wd = rt.gw[q0] * rt.gw[q1] * rt.gw[q2] * fabs(det);
        const double w = wd * (m.coef ? m.coef[c0 + ci] : 1.0);
        const double wm = PROB == 1 ? p.mu * w : w;
        double *__restrict__ o = sQ[ci][q];
        int u = 0;
#pragma unroll
        for (int r = 0; r < 3; r++)
#pragma unroll
            for (int s = r; s < 3; s++) {
                double t = Ji[r * 3] * Ji[s * 3];
                t = fma(Ji[r * 3 + 1], Ji[s * 3 + 1], t);
                t = fma(Ji[r * 3 + 2], Ji[s * 3 + 2], t);
                o[u++] = wm * t;
            }
        if (PROB == 1) {
            o[6] = w;
#pragma unroll
            for (int t = 0; t < 9; t++) o[7 + t] = Ji[t];
        }
        for (int c = 0; c < NC; c++) sF[e * NC + c] = wd * source_value(p, 3, xq, c);
    }
    __syncthreads();
    // load vector, one direction after the other
    if (part == 0) {
        for (int e = tid; e < ncb * NLOC; e += BS) {
            const int ci = e / NLOC, row = e - ci * NLOC, a = row / NC, c = row - a * NC;
            const int a0 = a % K1, a1 = (a / K1) % K1, a2 = a / KK;
            const double *__restrict__ g = sF + ci * NN * NC + c;
            double f2 = 0.0;
            for (int q2 = 0; q2 < K1; q2++) {
                double f1 = 0.0;
#pragma unroll 1
                for (int q1 = 0; q1 < K1; q1++) {
                    double f0 = 0.0;
#pragma unroll
                    for (int q0 = 0; q0 < K1; q0++) f0 = fma(sL[a0 * K1 + q0], g[((q2 * K1 + q1) * K1 + q0) * NC], f0);
                    f1 = fma(sL[a1 * K1 + q1], f0, f1);
                }
                f2 = fma(sL[a2 * K1 + q2], f1, f2);
            }
            F[(c0 + ci) * NLOC + row] = f2;
        }
    }

    const int ci = tid / S::LN, ln = tid - ci * S::LN;
    const bool on = ci < ncb;
    const int cs = on ? ci : 0;
    const int x01 = ln % KK, x0 = x01 % K1, x1 = x01 / K1;
    const int ij = ln / KK % S::NIJ, i = ij / NC, j = ij - i * NC, pg = on ? ln / S::LP : 0;
    // 1D factors of (a1, b1) = (x1, x0), kept for all passes
    double vv[K1], dv[K1], vd[K1], dd[K1];
#pragma unroll
    for (int q = 0; q < K1; q++) {
        const double la = sL[x1 * K1 + q], da = sD[x1 * K1 + q], lb = sL[x0 * K1 + q], db = sD[x0 * K1 + q];
        vv[q] = la * lb;
        dv[q] = da * lb;
        vd[q] = la * db;
        dd[q] = da * db;
    }
    const double lam = p.lambda, mu = p.mu;
#pragma unroll 1
    for (int pass = part; pass < S::NPASS; pass += parts) {
        int a2 = 0, b2 = pass * PG + pg;  // pair number -> (a2, b2), a2 <= b2
#pragma unroll
        for (int r = 0; r < K1 - 1; r++)
            if (b2 >= K1 - a2) {
                b2 -= K1 - a2;
                a2++;
            }
        b2 += a2;
        double *__restrict__ U = sU[cs][pg][ij];
        if (on) {
            double u[9];
#pragma unroll
            for (int t = 0; t < 9; t++) u[t] = 0.0;
#pragma unroll UQ
            for (int q2 = 0; q2 < K1; q2++) {
                const double la = sL[a2 * K1 + q2], da = sD[a2 * K1 + q2], lb = sL[b2 * K1 + q2], db = sD[b2 * K1 + q2];
                const double t00 = la * lb, t10 = da * lb, t01 = la * db, t11 = da * db;  // derivative on a, on b
                const double *__restrict__ o = sQ[cs][x01 + KK * q2];
                const double tr[9] = {o[0], o[1], o[2], o[1], o[3], o[4], o[2], o[4], o[5]};
                double A[3], B[3], C[3], G[3];
                if (PROB == 1) {
                    const double wl = lam * o[6], wm = mu * o[6];
#pragma unroll
                    for (int r = 0; r < 3; r++) {
                        G[r] = o[7 + r * 3 + i];
                        C[r] = o[7 + r * 3 + j];
                        A[r] = wl * G[r];
                        B[r] = wm * C[r];
                    }
                }
#pragma unroll
                for (int r = 0; r < 3; r++)
#pragma unroll
                    for (int s = 0; s < 3; s++) {
                        double D = tr[r * 3 + s];
                        if (PROB == 1) D = fma(A[r], C[s], fma(B[r], G[s], i == j ? D : 0.0));
                        u[r * 3 + s] = fma(D, r == 2 ? (s == 2 ? t11 : t10) : (s == 2 ? t01 : t00), u[r * 3 + s]);
                    }
            }
#pragma unroll
            for (int t = 0; t < 9; t++) U[t * KK + x0 * K1 + x1] = u[t];  // (q0, q1) = (x0, x1)
        }
        __syncthreads();
        double *__restrict__ tile = sT[cs][pg];
        if (on) {
            double out[K1][K1];
#pragma unroll
            for (int a = 0; a < K1; a++)
#pragma unroll
                for (int b = 0; b < K1; b++) out[a][b] = 0.0;
#pragma unroll 1
            for (int q0 = 0; q0 < K1; q0++) {
                double Vdd = 0.0, Vdv = 0.0, Vvd = 0.0, Vvv = 0.0;
                const double *__restrict__ W = U + q0 * K1;
#pragma unroll
                for (int q = 0; q < K1; q++) {
                    Vdd = fma(W[0 * KK + q], vv[q], Vdd);
                    Vdv = fma(W[1 * KK + q], vd[q], fma(W[2 * KK + q], vv[q], Vdv));
                }
                if (K1 == 5) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < K1; q++) {
                    Vvd = fma(W[3 * KK + q], dv[q], fma(W[6 * KK + q], vv[q], Vvd));
                    Vvv = fma(W[4 * KK + q], dd[q], fma(W[5 * KK + q], dv[q], Vvv));
                    Vvv = fma(W[7 * KK + q], vd[q], fma(W[8 * KK + q], vv[q], Vvv));
                }
#pragma unroll
                for (int b = 0; b < K1; b++) {
                    const double lb = rt.L[b * K1 + q0], db = rt.D[b * K1 + q0];
                    const double yd = fma(Vdd, db, Vdv * lb), yv = fma(Vvd, db, Vvv * lb);
#pragma unroll
                    for (int a = 0; a < K1; a++)
                        out[a][b] = fma(rt.D[a * K1 + q0], yd, fma(rt.L[a * K1 + q0], yv, out[a][b]));
                }
            }
            double *__restrict__ w = tile + (x1 * K1 * NC + i) * TP + x0 * K1 * NC + j;
#pragma unroll
            for (int a = 0; a < K1; a++)
#pragma unroll
                for (int b = 0; b < K1; b++) w[a * NC * TP + b * NC] = out[a][b];
        }
        __syncthreads();
        if (on) {
            // LP = NC T: NC rows at a time, a thread keeps its column
            const int l = ln - pg * S::LP, sub = l / T, col = l - sub * T;
            double *__restrict__ Ec = E + (c0 + ci) * (int64_t(NLOC) * NLOC);
            double *__restrict__ blk = Ec + ((a2 * T + sub) * NLOC + b2 * T + col);
            double *__restrict__ mir = Ec + ((b2 * T + sub) * NLOC + a2 * T + col);
            const bool diag = a2 == b2;
            // K1 rows of the tile in flight at a time
#pragma unroll 1
            for (int i0 = 0; i0 < KK; i0 += K1) {
                double t[K1], u[K1];
#pragma unroll
                for (int e = 0; e < K1; e++) {
                    const int row = (i0 + e) * NC + sub;
                    t[e] = tile[row * TP + col];
                    u[e] = tile[col * TP + row];
                }
#pragma unroll
                for (int e = 0; e < K1; e++) {
                    const int row = (i0 + e) * NC;
                    if (!diag || row + sub <= col) blk[row * NLOC] = t[e];
                    if (!diag || row + sub > col) mir[row * NLOC] = u[e];
                }
            }
        }
    }
}

template <int K1, int PROB>
__global__ __launch_bounds__((TensorShape<K1, PROB>::BS), (TensorShape<K1, PROB>::MINW)) void k3_tensor_kernel(MeshArgs m, ProblemArgs p, RefTables rt,
                                                                                 int64_t ncells, int parts,
                                                                                 double *__restrict__ E,
                                                                                 double *__restrict__ F)
{
    k3_tensor_body<K1, PROB>(m, p, rt, ncells, parts, E, F, xcd_block(blockIdx.x, gridDim.x));
}

template <int K1, int PROB>
__global__ __launch_bounds__((TensorShape<K1, PROB>::BS), (TensorShape<K1, PROB>::MINW)) void k3_tensor_batch_kernel(const AsmJob *__restrict__ jobs,
                                                                                       const int32_t *__restrict__ boff,
                                                                                       int njobs)
{
    int64_t lb, nb;
    const AsmJob &J = jobs[find_job(boff, njobs, lb, nb)];
    k3_tensor_body<K1, PROB>(J.m, J.p, J.rt, J.s.ncells, J.parts, static_cast<double *>(J.E), J.F, lb);
}

// 2D: one workgroup = CB cells, one thread per cell, components (i, j) and
// (a1, b1), which sums over q1 for one q0 after the other, the K1^2 entries
// (a0, b0) in registers.  The matrices of the cells are put together in LDS,
// the lower triangle as the mirror of the upper, and leave as one contiguous
// range.  What bounds it: instructions and the LDS round trips (Q2 2.8 TB/s,
// Q4 elasticity 5.3).  Against one workgroup per cell with an outer product
// over slabs of points, us: Poisson Q2 400x300 809 -> 28, elasticity Q1 400x300
// 629 -> 32, Q4 150x150 3035 -> 213; one Q4 elasticity cell 52 -> 9.4.
template <int K1, int PROB>
struct PlaneShape {
    static constexpr int NC = PROB == 1 ? 2 : 1;
    static constexpr int NN = K1 * K1, NLOC = NN * NC;
    static constexpr int LN = NC * NC * NN;  // threads of a cell
    static constexpr int BS = 256, CB = BS / LN;
    static constexpr int NG = PROB == 1 ? 9 : 3;  // doubles per point (odd: distinct banks)
};

template <int K1, int PROB>
__global__ __launch_bounds__((PlaneShape<K1, PROB>::BS)) void k3_plane_kernel(MeshArgs m, ProblemArgs p, RefTables rt,
                                                                               int64_t ncells, double *__restrict__ E,
                                                                               double *__restrict__ F)
{
    using S = PlaneShape<K1, PROB>;
    constexpr int NC = S::NC, NN = S::NN, NLOC = S::NLOC, CB = S::CB, BS = S::BS, NG = S::NG;
    __shared__ double sL[NN], sD[NN];
    // per point: w k Ji Ji^T (00, 01, 11; times mu for elasticity); elasticity also w k and J^-1
    __shared__ double sQ[CB][NN][NG];
    __shared__ double sE[CB * NLOC * NLOC];
    __shared__ double sF[CB][NN * NC];
    const int tid = threadIdx.x;
    const int64_t c0 = xcd_block(blockIdx.x, gridDim.x) * CB;
    const int ncb = ncells - c0 < CB ? int(ncells - c0) : CB;
    for (int e = tid; e < NN; e += BS) {
        sL[e] = rt.L[e];
        sD[e] = rt.D[e];
    }
    for (int e = tid; e < ncb * NN; e += BS) {
        const int ci = e / NN, q = e - ci * NN, q0 = q % K1, q1 = q / K1;
        const double xi[3] = {rt.gx[q0], rt.gx[q1], 0.0};
        double X[4][3], J[9], Ji[9], xq[3];
        load_vertices<2>(m, c0 + ci, X);
        const double det = geometry<2>(X, xi, J, Ji, xq);
        if (!(det > 0.0)) atomicOr(m.status, 1);
        const double wd = rt.gw[q0] * rt.gw[q1] * fabs(det);
        const double w = wd * (m.coef ? m.coef[c0 + ci] : 1.0);
        const double wm = PROB == 1 ? p.mu * w : w;
        double *__restrict__ o = sQ[ci][q];
        o[0] = wm * fma(Ji[1], Ji[1], Ji[0] * Ji[0]);
        o[1] = wm * fma(Ji[1], Ji[3], Ji[0] * Ji[2]);
        o[2] = wm * fma(Ji[3], Ji[3], Ji[2] * Ji[2]);
        if (PROB == 1) {
            o[3] = w;
#pragma unroll
            for (int t = 0; t < 4; t++) o[4 + t] = Ji[t];
        }
        for (int c = 0; c < NC; c++) sF[ci][q * NC + c] = wd * source_value(p, 2, xq, c);
    }
    __syncthreads();
    for (int e = tid; e < ncb * NLOC; e += BS) {
        const int ci = e / NLOC, row = e - ci * NLOC, a = row / NC, c = row - a * NC, a0 = a % K1, a1 = a / K1;
        double f1 = 0.0;
        for (int q1 = 0; q1 < K1; q1++) {
            double f0 = 0.0;
#pragma unroll
            for (int q0 = 0; q0 < K1; q0++) f0 = fma(sL[a0 * K1 + q0], sF[ci][(q1 * K1 + q0) * NC + c], f0);
            f1 = fma(sL[a1 * K1 + q1], f0, f1);
        }
        F[c0 * NLOC + e] = f1;
    }
    const int ci = tid / S::LN, ln = tid - ci * S::LN;
    if (ci < ncb) {
        const int b1 = ln % K1, a1 = ln / K1 % K1, ij = ln / NN, i = ij / NC, j = ij - i * NC;
        const double lam = p.lambda, mu = p.mu;
        double out[K1][K1];
#pragma unroll
        for (int a = 0; a < K1; a++)
#pragma unroll
            for (int b = 0; b < K1; b++) out[a][b] = 0.0;
#pragma unroll 1
        for (int q0 = 0; q0 < K1; q0++) {
            double Vdd = 0.0, Vdv = 0.0, Vvd = 0.0, Vvv = 0.0;
#pragma unroll
            for (int q1 = 0; q1 < K1; q1++) {
                const double la = sL[a1 * K1 + q1], da = sD[a1 * K1 + q1], lb = sL[b1 * K1 + q1], db = sD[b1 * K1 + q1];
                const double *__restrict__ o = sQ[ci][q1 * K1 + q0];
                double D[4] = {o[0], o[1], o[1], o[2]};  // r s
                if (PROB == 1) {
                    const double wl = lam * o[3], wm = mu * o[3];
#pragma unroll
                    for (int r = 0; r < 2; r++)
#pragma unroll
                        for (int t = 0; t < 2; t++)
                            D[2 * r + t] = fma(wl * o[4 + 2 * r + i], o[4 + 2 * t + j],
                                               fma(wm * o[4 + 2 * r + j], o[4 + 2 * t + i], i == j ? D[2 * r + t] : 0.0));
                }
                Vdd = fma(D[0], la * lb, Vdd);
                Vdv = fma(D[1], la * db, Vdv);
                Vvd = fma(D[2], da * lb, Vvd);
                Vvv = fma(D[3], da * db, Vvv);
            }
#pragma unroll
            for (int b = 0; b < K1; b++) {
                const double lb = rt.L[b * K1 + q0], db = rt.D[b * K1 + q0];
                const double yd = fma(Vdd, db, Vdv * lb), yv = fma(Vvd, db, Vvv * lb);
#pragma unroll
                for (int a = 0; a < K1; a++)
                    out[a][b] = fma(rt.D[a * K1 + q0], yd, fma(rt.L[a * K1 + q0], yv, out[a][b]));
            }
        }
        double *__restrict__ t = sE + ci * (NLOC * NLOC);
#pragma unroll
        for (int a = 0; a < K1; a++)
#pragma unroll
            for (int b = 0; b < K1; b++) {
                const int I = (a1 * K1 + a) * NC + i, J = (b1 * K1 + b) * NC + j;
                if (I <= J) t[I * NLOC + J] = out[a][b];
                if (I < J) t[J * NLOC + I] = out[a][b];
            }
    }
    __syncthreads();
    double *__restrict__ Ec = E + c0 * (NLOC * NLOC);
    for (int e = tid; e < ncb * (NLOC * NLOC); e += BS) Ec[e] = sE[e];
}

// Calls body.template operator()<K1, PROB>() for (order, problem).
template <class Body>
static fe_status with_tensor(int k, bool el, Body body)
{
    switch (k * 2 + (el ? 1 : 0)) {
        case 3: return body.template operator()<2, 1>();
        case 4: return body.template operator()<3, 0>();
        case 5: return body.template operator()<3, 1>();
        case 6: return body.template operator()<4, 0>();
        case 7: return body.template operator()<4, 1>();
        case 8: return body.template operator()<5, 0>();
        case 9: return body.template operator()<5, 1>();
        default: return set_error(FE_EINVAL, "no sum-factorized kernel for this space");
    }
}

struct TensorBlocks {
    int64_t ncells;
    int64_t &blocks;
    int32_t &parts;
    template <int K1, int PROB>
    fe_status operator()() const
    {
        using S = TensorShape<K1, PROB>;
        // few cells: the passes of a workgroup are split over several, up to
        // four workgroups per CU
        const int64_t groups = (ncells + S::CB - 1) / S::CB;
        parts = int32_t(std::min<int64_t>(S::NPASS, std::max<int64_t>(S::PARTS, 1024 / std::max<int64_t>(1, groups))));
        blocks = groups * parts;
        return FE_OK;
    }
};

int64_t tensor_blocks(const SpaceArgs &sa, const ProblemArgs &pa, int32_t &parts)
{
    int64_t blocks = 0;
    parts = 1;
    with_tensor(sa.k, pa.problem == FE_ELASTICITY, TensorBlocks{sa.ncells, blocks, parts});
    return blocks;
}

struct TensorSingle {
    const SpaceArgs &sa;
    const MeshArgs &ma;
    const ProblemArgs &pa;
    const RefTables &rt;
    double *E, *F;
    hipStream_t s;
    template <int K1, int PROB>
    fe_status operator()() const
    {
        int32_t parts = 1;
        const int64_t grid = tensor_blocks(sa, pa, parts);
        if (grid == 0) return FE_OK;
        hipLaunchKernelGGL((k3_tensor_kernel<K1, PROB>), dim3(grid), dim3((TensorShape<K1, PROB>::BS)), 0, s, ma, pa, rt,
                           sa.ncells, parts, E, F);
        FE_HIP(hipGetLastError());
        return FE_OK;
    }
};

struct TensorBatch {
    const AsmJob *jobs;
    const int32_t *boff;
    int njobs, grid;
    hipStream_t s;
    template <int K1, int PROB>
    fe_status operator()() const
    {
        hipLaunchKernelGGL((k3_tensor_batch_kernel<K1, PROB>), dim3(grid), dim3((TensorShape<K1, PROB>::BS)), 0, s, jobs,
                           boff, njobs);
        FE_HIP(hipGetLastError());
        return FE_OK;
    }
};

template <int K1, int PROB>
static fe_status launch_plane(const MeshArgs &ma, const ProblemArgs &pa, const RefTables &rt, int64_t ncells, double *E,
                              double *F, hipStream_t s)
{
    constexpr int CB = PlaneShape<K1, PROB>::CB;
    hipLaunchKernelGGL((k3_plane_kernel<K1, PROB>), dim3((ncells + CB - 1) / CB), dim3((PlaneShape<K1, PROB>::BS)), 0, s,
                       ma, pa, rt, ncells, E, F);
    FE_HIP(hipGetLastError());
    return FE_OK;
}

fe_status launch_integrate_plane(const SpaceArgs &sa, const MeshArgs &ma, const ProblemArgs &pa, const RefTables &rt,
                                 double *E, double *F, hipStream_t s)
{
    if (sa.ncells == 0) return FE_OK;
    switch (sa.k * 2 + (pa.problem == FE_ELASTICITY ? 1 : 0)) {
        case 3: return launch_plane<2, 1>(ma, pa, rt, sa.ncells, E, F, s);
        case 4: return launch_plane<3, 0>(ma, pa, rt, sa.ncells, E, F, s);
        case 5: return launch_plane<3, 1>(ma, pa, rt, sa.ncells, E, F, s);
        case 6: return launch_plane<4, 0>(ma, pa, rt, sa.ncells, E, F, s);
        case 7: return launch_plane<4, 1>(ma, pa, rt, sa.ncells, E, F, s);
        case 8: return launch_plane<5, 0>(ma, pa, rt, sa.ncells, E, F, s);
        case 9: return launch_plane<5, 1>(ma, pa, rt, sa.ncells, E, F, s);
        default: return set_error(FE_EINVAL, "unsupported element size");
    }
}

fe_status launch_integrate_tensor(const SpaceArgs &sa, const MeshArgs &ma, const ProblemArgs &pa, const RefTables &rt,
                                  double *E, double *F, hipStream_t s)
{
    return with_tensor(sa.k, pa.problem == FE_ELASTICITY, TensorSingle{sa, ma, pa, rt, E, F, s});
}

fe_status launch_tensor_batch(const AsmJob &h, const AsmJob *jobs, const int32_t *boff, int njobs, int grid,
                              hipStream_t s)
{
    return with_tensor(h.s.k, h.p.problem == FE_ELASTICITY, TensorBatch{jobs, boff, njobs, grid, s});
}

}  // namespace fe
