// fe_xblock.h -- how the block-staged SpMV (plan mode 6) cuts a system assembled
// on a brick into chunks of rows, and the box of unknowns a chunk stages.  On the
// host as well as on the device, so that the sizes can be checked without one.
#pragma once

#include <algorithm>

#include "fe_internal.h"

namespace fe {

constexpr int kXbBlock = 256;  // threads of a block

// How the block-staged traversal (plan mode 6) cuts a system into chunks.
struct XbShape {
    int32_t rc = 1, m = 1, pcs = 1, yb = 1;  // groups per line stretch, lines per chunk, stretches per line, y blocks
    int32_t nchunks = 0;
    int32_t lds = 0;  // bytes of the staged box
};

constexpr int xb_lanes(int shape) { return shape == 8 ? 4 : 16; }
constexpr int xb_group_rows(int shape, int nc) { return shape == 8 ? 1 : nc; }

// The cut with the least work: every chunk streams up to G groups whatever it
// holds (idle lanes cost what busy ones do) and stages its box, so short lines
// of nodes are taken several to a chunk and long ones in equal stretches.
inline XbShape xb_shape(const SpaceArgs &sa, int shape)
{
    const int nc = sa.ncomp, k = sa.k, G = kXbBlock / xb_lanes(shape), gr = xb_group_rows(shape, nc);
    const int64_t f0 = sa.ax[0].f, f1 = sa.ax[1].f, f2 = sa.ax[2].f;
    XbShape best{};
    if (f0 == 0 || f1 == 0 || f2 == 0) return best;
    const int64_t gpl = f0 * nc / gr;  // groups per line
    double row = nc;                   // values per row, average over the vertex and interior nodes of an axis
    for (int r = 0; r < sa.dim; r++) row *= double(2 * k + 1 + (k - 1) * (k + 1)) / k;
    double cost = 0.0;
    const int64_t p0 = (gpl + G - 1) / G;
    for (int64_t pcs = p0; pcs < p0 + 4 && pcs <= gpl; pcs++) {
        const int64_t rc = (gpl + pcs - 1) / pcs;
        const int64_t m = std::max<int64_t>(1, std::min<int64_t>(f1, G / rc));
        const int64_t yb = (f1 + m - 1) / m;
        const int64_t nodes = std::min<int64_t>(f0, (rc * gr - 1) / nc + 2 + 2 * k);
        const int64_t wy = std::min<int64_t>(f1, m + 2 * k), wz = sa.dim == 3 ? std::min<int64_t>(f2, 2 * k + 1) : 1;
        const int64_t staged = nc * nodes * wy * wz;
        const double c = double(yb * pcs) * (G * gr * row + 2.0 * double(staged));
        if (best.nchunks == 0 || c < cost) {
            cost = c;
            best = XbShape{int32_t(rc), int32_t(m), int32_t((gpl + rc - 1) / rc), int32_t(yb), 0, int32_t(8 * staged)};
            best.nchunks = int32_t(f2 * yb * best.pcs);
        }
    }
    return best;
}

// A chunk: lines ya .. ya + ny - 1 of plane t2, the rows [lr0, lr1) of each; and
// the union of the rows' column boxes: run unknowns along x from node cla, W1
// lines from cya, w2 planes from cl2 (P2: the prefix of the plane's rows).
struct XbBox {
    int32_t t2, ya, ny, lr0, lr1, cla, run, cya, W1, cl2, w2, P2;
};

__host__ __device__ __forceinline__ XbBox xb_box(const AxisClosed (&A)[3], const XbShape &xb, int32_t k, int32_t nc,
                                                 int32_t gr, int32_t f1, int32_t rpl, int32_t ch)
{
    XbBox b;
    const int32_t q = ch / xb.pcs, pc = ch - q * xb.pcs;
    b.t2 = q / xb.yb;
    b.ya = (q - b.t2 * xb.yb) * xb.m;
    b.ny = b.ya + xb.m < f1 ? xb.m : f1 - b.ya;
    b.lr0 = pc * xb.rc * gr;
    b.lr1 = b.lr0 + xb.rc * gr < rpl ? b.lr0 + xb.rc * gr : rpl;
    int32_t wa, Pa, wb, clb, Pb, wya, Pya, wyb, cyb, Pyb;
    axis_row(A[0], k, A[0].lo + b.lr0 / nc, wa, b.cla, Pa);
    axis_row(A[0], k, A[0].lo + (b.lr1 - 1) / nc, wb, clb, Pb);
    axis_row(A[1], k, A[1].lo + b.ya, wya, b.cya, Pya);
    axis_row(A[1], k, A[1].lo + b.ya + b.ny - 1, wyb, cyb, Pyb);
    axis_row(A[2], k, A[2].lo + b.t2, b.w2, b.cl2, b.P2);
    b.run = nc * (clb + wb - b.cla);
    b.W1 = cyb + wyb - b.cya;
    return b;
}

}  // namespace fe
