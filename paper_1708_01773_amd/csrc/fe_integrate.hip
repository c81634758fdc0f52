// fe_integrate.hip -- K3: cell-wise numerical integration of the Galerkin
// element matrices and loads (Sect. 3.7 eq. fematrix, the element loop of the
// Poisson example in Sect. 8.5), on the reference cell [0,1]^d with the
// order-1 geometry map and tensor Gauss-Legendre quadrature of k+1 points per
// direction.  Geometry (J, det J, J^-1) is always FP64.
//
// Poisson:    A_ab = sum_q w_q k_K |det J_q| grad phi_a . grad phi_b
// Elasticity: A_(a,i),(b,j) = sum_q w_q k_K |det J_q|
//               [lambda d_i phi_a d_j phi_b + mu (delta_ij grad phi_a . grad phi_b + d_j phi_a d_i phi_b)]
// Load:       F_(a,c) = sum_q w_q |det J_q| f_c(x_q) phi_a(xi_q)
// Lifting:    F_a -= sum_{b fixed} A_ab u_D(b)   (Sect. 10.4)
#include <cmath>
#include <type_traits>

#include "fe_geom.h"
#include "fe_internal.h"

namespace fe {

ElemLayout elem_layout(const SpaceArgs &sa, int precision)
{
    ElemLayout el{};
    const bool q1_scalar = sa.k == 1 && sa.ncomp == 1;
    el.cb = q1_scalar ? 64 : 1;
    el.packed = q1_scalar ? 1 : 0;
    el.ne = q1_scalar ? sa.nloc * (sa.nloc + 1) / 2 : sa.nloc * sa.nloc;
    el.elem_bytes = precision == FE_FP64 ? 8 : 4;
    const int64_t cells_pad = (sa.ncells + el.cb - 1) / el.cb * el.cb;
    el.e_bytes = (size_t(cells_pad) * el.ne * el.elem_bytes + 255) / 256 * 256;
    el.f_offset = el.e_bytes;
    el.total = el.f_offset + (size_t(sa.ncells) * sa.nloc * sizeof(double) + 255) / 256 * 256;
    return el;
}

// ---------------------------------------------------------------------------
// Q1 scalar kernel: one thread per cell, element matrix in registers (the 36
// upper-triangle entries in 3D), written in the blocked layout
// E[(c/64)][a*8+b][c%64] so that a wave's stores of one entry are 512
// contiguous bytes.  Q1 is HBM-bound (6 flop per byte of E) and its 8 x 8 x 24
// product would fill a quarter of a 16 x 16 matrix tile, so it runs on the
// vector units in every precision.  PREC > 0: the two GEMM operands (the
// gradients, and the gradients times w_q k |det J_q|) are rounded to FP32 /
// FP16 / BF16 and accumulated in FP32, the result stored as FP32; for FP16 /
// BF16 they are first scaled by per-cell powers of two (undone exactly).
// ---------------------------------------------------------------------------
template <int PREC>
__device__ __forceinline__ float round_in(double v)
{
    if (PREC == FE_FP16) return float(_Float16(float(v)));
    if (PREC == FE_BF16) return float(__bf16(float(v)));
    return float(v);
}

template <int DIM, int PREC>
__device__ __forceinline__ void k3_q1_body(const SpaceArgs &s, const MeshArgs &m, const ProblemArgs &p,
                                           const RefTables &rt, void *__restrict__ Ev, double *__restrict__ F,
                                           int64_t bid)
{
    constexpr int NN = 1 << DIM;
    constexpr int NT = NN * (NN + 1) / 2;
    using Acc = typename std::conditional<PREC == FE_FP64, double, float>::type;
    const int64_t cell = bid * blockDim.x + threadIdx.x;
    if (cell >= s.ncells) return;
    double X[NN][3];
    load_vertices<DIM>(m, cell, X);
    const double coef = m.coef ? m.coef[cell] : 1.0;
    // per-cell operand scaling for FP16 / BF16
    double alpha = 1.0, beta = 1.0;
    if (PREC == FE_FP16 || PREC == FE_BF16) {
        double wmax = 0.0, det0 = 0.0;
#pragma unroll
        for (int q = 0; q < NN; q++) {
            const int q0 = q & 1, q1 = (q >> 1) & 1, q2 = (q >> 2) & 1;
            const double xi[3] = {rt.gx[q0], rt.gx[q1], DIM == 3 ? rt.gx[q2] : 0.0};
            double J[9], Ji[9], xq[3];
            const double det = geometry<DIM>(X, xi, J, Ji, xq);
            if (q == 0) det0 = det;
            wmax = fmax(wmax, rt.gw[q0] * rt.gw[q1] * (DIM == 3 ? rt.gw[q2] : 1.0) * fabs(det) * coef);
        }
        const double h = DIM == 3 ? cbrt(fabs(det0)) : sqrt(fabs(det0));
        alpha = exp2(floor(log2(h > 0.0 ? h : 1.0)));
        beta = alpha * (wmax > 0.0 ? exp2(-floor(log2(wmax))) : 1.0);
    }
    Acc acc[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) acc[t] = Acc(0);
    double fl[NN];
#pragma unroll
    for (int a = 0; a < NN; a++) fl[a] = 0.0;
    bool bad = false;
    // the points one at a time: unrolled, every point's operands stayed live
    // at once (366 VGPRs, one wave per SIMD; 224 and two waves this way)
#pragma unroll 1
    for (int q = 0; q < NN; q++) {
        const int q0 = q & 1, q1 = (q >> 1) & 1, q2 = (q >> 2) & 1;
        const double xi[3] = {rt.gx[q0], rt.gx[q1], DIM == 3 ? rt.gx[q2] : 0.0};
        const double w = rt.gw[q0] * rt.gw[q1] * (DIM == 3 ? rt.gw[q2] : 1.0);
        double J[9], Ji[9], xq[3];
        const double det = geometry<DIM>(X, xi, J, Ji, xq);
        bad |= !(det > 0.0);
        const double wdet = w * fabs(det);
        const double wd = wdet * coef;
        const double fq = source_value(p, DIM, xq, 0);
        // physical gradients of the 2^d shape functions (Sect. 3.7 eq. shape_grad)
        double g[NN][DIM];
#pragma unroll
        for (int a = 0; a < NN; a++) {
            const int a0 = a & 1, a1 = (a >> 1) & 1, a2 = (a >> 2) & 1;
            double gr[3];
            const double L0 = rt.L[a0 * 2 + q0], L1 = rt.L[a1 * 2 + q1];
            const double D0 = rt.D[a0 * 2 + q0], D1 = rt.D[a1 * 2 + q1];
            if (DIM == 3) {
                const double L2 = rt.L[a2 * 2 + q2], D2 = rt.D[a2 * 2 + q2];
                gr[0] = D0 * L1 * L2;
                gr[1] = L0 * D1 * L2;
                gr[2] = L0 * L1 * D2;
                fl[a] += wdet * fq * (L0 * L1 * L2);
            } else {
                gr[0] = D0 * L1;
                gr[1] = L0 * D1;
                fl[a] += wdet * fq * (L0 * L1);
            }
#pragma unroll
            for (int i = 0; i < DIM; i++) {
                double v = 0.0;
#pragma unroll
                for (int sd = 0; sd < DIM; sd++) v += Ji[sd * DIM + i] * gr[sd];
                g[a][i] = v;
            }
        }
        if (PREC == FE_FP64) {
            int t = 0;
#pragma unroll
            for (int a = 0; a < NN; a++)
#pragma unroll
                for (int b = a; b < NN; b++, t++) {
                    double dot = 0.0;
#pragma unroll
                    for (int i = 0; i < DIM; i++) dot += g[a][i] * g[b][i];
                    acc[t] += Acc(wd * dot);
                }
        } else {
            float ga[NN][DIM], hb[NN][DIM];
#pragma unroll
            for (int a = 0; a < NN; a++)
#pragma unroll
                for (int i = 0; i < DIM; i++) {
                    ga[a][i] = round_in<PREC>(g[a][i] * alpha);
                    hb[a][i] = round_in<PREC>(g[a][i] * wd * beta);
                }
            int t = 0;
#pragma unroll
            for (int a = 0; a < NN; a++)
#pragma unroll
                for (int b = a; b < NN; b++, t++)
#pragma unroll
                    for (int i = 0; i < DIM; i++) acc[t] = fmaf(ga[a][i], hb[b][i], float(acc[t]));
        }
    }
    if (bad) atomicOr(m.status, 1);
    const double unscale = 1.0 / (alpha * beta);
    const int64_t blk = cell / 64, lane = cell % 64;
    using Out = Acc;
    // packed upper triangle, entry t = (a, b), a <= b, in row-major order
    Out *Eb = static_cast<Out *>(Ev) + blk * (NT * 64) + lane;
#pragma unroll
    for (int t = 0; t < NT; t++) Eb[t * 64] = PREC == FE_FP64 ? acc[t] : Out(double(acc[t]) * unscale);
#pragma unroll
    for (int a = 0; a < NN; a++) F[cell * NN + a] = fl[a];
}

template <int DIM, int PREC>
__global__ __launch_bounds__(256) void k3_q1_kernel(SpaceArgs s, MeshArgs m, ProblemArgs p, RefTables rt,
                                                     void *__restrict__ Ev, double *__restrict__ F)
{
    k3_q1_body<DIM, PREC>(s, m, p, rt, Ev, F, xcd_block(blockIdx.x, gridDim.x));
}

template <int DIM, int PREC>
__global__ __launch_bounds__(256) void k3_q1_batch_kernel(const AsmJob *__restrict__ jobs,
                                                           const int32_t *__restrict__ boff, int njobs)
{
    int64_t lb, nb;
    const AsmJob &J = jobs[find_job(boff, njobs, lb, nb)];
    k3_q1_body<DIM, PREC>(J.s, J.m, J.p, J.rt, J.E, J.F, lb);
}

// ---------------------------------------------------------------------------
// Dirichlet lifting for non-zero (affine) data: F_a -= sum_{b fixed} A_ab u_D(b)
// on every cell that has fixed DOFs (one wave per cell).
// ---------------------------------------------------------------------------
template <int DIM, typename ET>
__global__ __launch_bounds__(64) void k3_lift_kernel(SpaceArgs s, MeshArgs m, ProblemArgs p, const int32_t *cell_dofs,
                                                     int cb, int packed, int ne, const ET *__restrict__ E,
                                                     double *__restrict__ F)
{
    const int64_t cell = blockIdx.x;
    const int nloc = s.nloc, k = s.k, k1 = k + 1, nc = s.ncomp;
    const int32_t *g = cell_dofs + cell * nloc;
    bool any = false;
    for (int t = 0; t < nloc; t++) any |= g[t] < 0;
    if (!any) return;
    double X[1 << DIM][3];
    load_vertices<DIM>(m, cell, X);
    for (int a = threadIdx.x; a < nloc; a += blockDim.x) {
        if (g[a] < 0) continue;
        double lift = 0.0;
        for (int b = 0; b < nloc; b++) {
            if (g[b] >= 0) continue;
            const int node = b / nc, c = b % nc;
            const double xi[3] = {double(node % k1) / k, double((node / k1) % k1) / k,
                                  DIM == 3 ? double(node / (k1 * k1)) / k : 0.0};
            double J[9], Ji[9], xb[3];
            geometry<DIM>(X, xi, J, Ji, xb);
            double u = p.aff[4 * c];
            for (int r = 0; r < DIM; r++) u += p.aff[4 * c + 1 + r] * xb[r];
            lift += double(E[elem_index(cell, a, b, nloc, cb, packed, ne)]) * u;
        }
        F[cell * nloc + a] -= lift;
    }
}

// ---------------------------------------------------------------------------
// Launch
// ---------------------------------------------------------------------------
fe_status launch_integrate(const SpaceArgs &sa, const MeshArgs &ma, const ProblemArgs &pa, const RefTables &rt,
                           const ElemLayout &el, void *ws, hipStream_t s)
{
    double *E = static_cast<double *>(ws);
    double *F = reinterpret_cast<double *>(static_cast<char *>(ws) + el.f_offset);
    if (sa.ncells == 0) return FE_OK;
    if (tensor_integrated(sa, pa)) return launch_integrate_tensor(sa, ma, pa, rt, E, F, s);
    if (sa.dim == 3 && sa.k >= 2) return launch_integrate_mfma(sa, ma, pa, rt, ws, F, s);
    fe_status st = FE_OK;
    if (sa.k == 1 && sa.ncomp == 1) {
        const int64_t grid = (sa.ncells + 255) / 256;
#define FE_Q1(D, P) hipLaunchKernelGGL((k3_q1_kernel<D, P>), dim3(grid), dim3(256), 0, s, sa, ma, pa, rt, ws, F)
        if (sa.dim == 3) {
            switch (pa.precision) {
                case FE_FP64: FE_Q1(3, FE_FP64); break;
                case FE_FP32: FE_Q1(3, FE_FP32); break;
                case FE_FP16: FE_Q1(3, FE_FP16); break;
                default: FE_Q1(3, FE_BF16); break;
            }
        } else {
            switch (pa.precision) {
                case FE_FP64: FE_Q1(2, FE_FP64); break;
                case FE_FP32: FE_Q1(2, FE_FP32); break;
                case FE_FP16: FE_Q1(2, FE_FP16); break;
                default: FE_Q1(2, FE_BF16); break;
            }
        }
#undef FE_Q1
        FE_HIP(hipGetLastError());
    } else if (pa.precision != FE_FP64) {
        return set_error(FE_EINVAL, "reduced-precision integration needs 3D hexahedra (any order) or scalar Q1");
    } else {
        st = launch_integrate_plane(sa, ma, pa, rt, E, F, s);
    }
    return st;
}

fe_status launch_lift(const SpaceArgs &sa, const MeshArgs &ma, const ProblemArgs &pa, const int32_t *cell_dofs,
                      const ElemLayout &el, void *ws, hipStream_t s)
{
    if (pa.dirichlet_kind != FE_DIRICHLET_AFFINE || sa.ncells == 0) return FE_OK;
    double *F = reinterpret_cast<double *>(static_cast<char *>(ws) + el.f_offset);
    if (el.elem_bytes == 8) {
        const double *E = static_cast<const double *>(ws);
        if (sa.dim == 3)
            hipLaunchKernelGGL((k3_lift_kernel<3, double>), dim3(sa.ncells), dim3(64), 0, s, sa, ma, pa, cell_dofs,
                               el.cb, el.packed, el.ne, E, F);
        else
            hipLaunchKernelGGL((k3_lift_kernel<2, double>), dim3(sa.ncells), dim3(64), 0, s, sa, ma, pa, cell_dofs,
                               el.cb, el.packed, el.ne, E, F);
    } else {
        const float *E = static_cast<const float *>(ws);
        if (sa.dim == 3)
            hipLaunchKernelGGL((k3_lift_kernel<3, float>), dim3(sa.ncells), dim3(64), 0, s, sa, ma, pa, cell_dofs,
                               el.cb, el.packed, el.ne, E, F);
        else
            hipLaunchKernelGGL((k3_lift_kernel<2, float>), dim3(sa.ncells), dim3(64), 0, s, sa, ma, pa, cell_dofs,
                               el.cb, el.packed, el.ne, E, F);
    }
    FE_HIP(hipGetLastError());
    return FE_OK;
}

// ---------------------------------------------------------------------------
// Batched launches (one launch per kernel class, jobs in a device table)
// ---------------------------------------------------------------------------
bool integrate_batchable(const SpaceArgs &sa, const ProblemArgs &pa)
{
    return (sa.k == 1 && sa.ncomp == 1) || (sa.dim == 3 && sa.k >= 2);
}

int64_t integrate_blocks(const SpaceArgs &sa, const ProblemArgs &pa, int32_t &parts)
{
    parts = 1;
    if (tensor_integrated(sa, pa)) return tensor_blocks(sa, pa, parts);
    if (sa.dim == 3 && sa.k >= 2) return mfma_blocks(sa, pa, parts);
    return (sa.ncells + 255) / 256;
}

fe_status launch_integrate_batch(const AsmJob &h, const AsmJob *jobs, const int32_t *boff, int njobs, int grid,
                                 hipStream_t s)
{
    if (grid == 0) return FE_OK;
    const SpaceArgs &sa = h.s;
    if (tensor_integrated(sa, h.p)) return launch_tensor_batch(h, jobs, boff, njobs, grid, s);
    if (sa.dim == 3 && sa.k >= 2) return launch_mfma_batch(h, jobs, boff, njobs, grid, s);
    if (!(sa.k == 1 && sa.ncomp == 1)) return set_error(FE_EINVAL, "no batched kernel for this class");
#define FE_Q1B(D, P) hipLaunchKernelGGL((k3_q1_batch_kernel<D, P>), dim3(grid), dim3(256), 0, s, jobs, boff, njobs)
    if (sa.dim == 3) {
        switch (h.p.precision) {
            case FE_FP64: FE_Q1B(3, FE_FP64); break;
            case FE_FP32: FE_Q1B(3, FE_FP32); break;
            case FE_FP16: FE_Q1B(3, FE_FP16); break;
            default: FE_Q1B(3, FE_BF16); break;
        }
    } else {
        switch (h.p.precision) {
            case FE_FP64: FE_Q1B(2, FE_FP64); break;
            case FE_FP32: FE_Q1B(2, FE_FP32); break;
            case FE_FP16: FE_Q1B(2, FE_FP16); break;
            default: FE_Q1B(2, FE_BF16); break;
        }
    }
#undef FE_Q1B
    FE_HIP(hipGetLastError());
    return FE_OK;
}

}  // namespace fe
