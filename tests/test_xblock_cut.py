"""Host check of the block-staged SpMV's cut into chunks (no GPU needed).

A small program, compiled from the header that the kernel uses, walks every
chunk of many systems: both shapes, one to three components, orders 1 to 4,
short, long, ragged and one-cell-thin bricks in 2D and 3D, every choice of
fixed faces.  For every chunk it computes the staged box as the kernel does and
checks it against the LDS that the launch asks for and the buffer limit; that
the box holds the columns of every row of the chunk; and that every row of the
system belongs to exactly one thread group of one chunk."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1708_01773_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "fe_xblock.h"
using namespace fe;

static long long checked = 0, worst = 0;

static bool walk(int dim, const int *n, int k, int nc, unsigned faces, int shape, long long cap)
{
    SpaceArgs sa{};
    sa.dim = dim;
    sa.k = k;
    sa.ncomp = nc;
    AxisClosed A[3];
    for (int r = 0; r < 3; r++) {
        const int N = r < dim ? n[r] * k : 0;
        const int lo = r < dim && (faces >> (2 * r) & 1) ? 1 : 0, hi = r < dim && (faces >> (2 * r + 1) & 1) ? N - 1 : N;
        if (hi < lo) return true;  // no free node
        sa.ax[r].lo = lo;
        sa.ax[r].f = hi - lo + 1;
        sa.ax[r].N = N;
        sa.ax[r].n = r < dim ? n[r] : 1;
        A[r] = AxisClosed{lo, hi, N, lo * (k + 1) + k * ((lo + k - 1) / k)};
    }
    const int f0 = int(sa.ax[0].f), f1 = int(sa.ax[1].f), f2 = int(sa.ax[2].f);
    const int gr = xb_group_rows(shape, nc), L = xb_lanes(shape), G = kXbBlock / L, rpl = nc * f0;
    const XbShape xb = xb_shape(sa, shape);
    worst = std::max<long long>(worst, xb.lds);
    if (xb.lds > 8 * cap || xb.nchunks < 1 || xb.rc < 1 || xb.rc * xb.m > G) return false;
    std::vector<int> seen(size_t(rpl) * f1 * f2, 0);
    for (int ch = 0; ch < xb.nchunks; ch++) {
        const XbBox b = xb_box(A, xb, k, nc, gr, f1, rpl, ch);
        checked++;
        if (8LL * b.run * b.W1 * b.w2 > xb.lds || b.ny < 1 || b.t2 >= f2 || b.ya + b.ny > f1) return false;
        for (int g = 0; g < G; g++) {
            const int gj = g / xb.rc, lrow = b.lr0 + (g - gj * xb.rc) * gr;
            if (int((unsigned(g) * (65536u / unsigned(xb.rc) + 1u)) >> 16) != gj) return false;  // the kernel's division
            if (gj >= b.ny || lrow >= b.lr1) continue;
            int w0, cl0, P0, w1, cl1, P1;
            axis_row(A[0], k, A[0].lo + lrow / nc, w0, cl0, P0);
            axis_row(A[1], k, A[1].lo + b.ya + gj, w1, cl1, P1);
            const int x0 = nc * (cl0 - b.cla), y0 = cl1 - b.cya;
            if (x0 < 0 || x0 + nc * w0 > b.run || y0 < 0 || y0 + w1 > b.W1) return false;
            for (int c = 0; c < gr; c++) seen[(size_t(b.t2) * f1 + b.ya + gj) * rpl + lrow + c]++;
        }
    }
    for (int s : seen)
        if (s != 1) return false;
    return true;
}

int main()
{
    const int bricks[][3] = {{1, 1, 1}, {2, 1, 3}, {3, 2, 2}, {4, 5, 3}, {7, 3, 2}, {9, 1, 2}, {16, 2, 2}, {17, 3, 1},
                             {33, 2, 1}, {40, 1, 1}, {1, 40, 1}, {1, 1, 40}, {2, 13, 3}, {5, 6, 11}, {64, 1, 2}, {12, 12, 2},
                             {65, 2, 2}, {130, 1, 1}, {23, 19, 2}};
    for (const auto &n : bricks)
        for (int dim = 2; dim <= 3; dim++)
            for (int k = 1; k <= 4; k++)
                for (unsigned faces = 0; faces < (1u << (2 * dim)); faces++)
                    for (int nc = 1; nc <= 3; nc++)
                        for (int shape = 8; shape >= (nc > 1 ? 4 : 8); shape -= 4)
                            if (!walk(dim, n, k, nc, faces, shape, CAP)) {
                                std::printf("dim %d n %d %d %d k %d nc %d faces %u shape %d\n", dim, n[0], n[1], n[2], k, nc,
                                            faces, shape);
                                return 1;
                            }
    std::printf("%lld chunks, largest box %lld bytes\n", checked, worst);
    return 0;
}
"""


def test_every_chunk_fits_its_lds_and_covers_its_rows(tmp_path):
    cap = int(re.search(r"constexpr int kXbCap = (\d+);", open(os.path.join(CSRC, "fe_solve.hip")).read()).group(1))
    src, exe = tmp_path / "cut.hip", tmp_path / "cut"
    src.write_text(PROGRAM)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", f"-DCAP={cap}LL",
                        "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
