// route_dump.cpp -- which kernel each component of a coarse-to-fine transfer
// takes, and whether the marching kernel's tap selection gives the stencils
// (ch_route.h and ch_plan.h, test infrastructure).
//
// stdin:  lines "ncz ncy ncx nz ny nx esize rmax"
// stdout: per line, for u, v, w: "rm taken taps-right piped", rm 0: the marching
//         kernel does not apply (taps-right 1)
#include <cstdio>
#include <vector>

#include "../../paper_2105_01865_amd/csrc/ch_plan.h"
#include "../../paper_2105_01865_amd/csrc/ch_route.h"

static std::vector<double> pts(int n, double off)
{
    std::vector<double> t(n);
    for (int i = 0; i < n; ++i) t[i] = (i + off) / n;
    return t;
}

// first tap of target q of a group, from the group's first
static int tap(int pattern, int q) { return pattern == chk::MARCH_FACE ? q / 2 : (q + 1) / 2; }

int main()
{
    int ncz, ncy, ncx, nz, ny, nx, es, rmax;
    while (scanf("%d %d %d %d %d %d %d %d", &ncz, &ncy, &ncx, &nz, &ny, &nx, &es, &rmax) == 8) {
        for (int c = 0; c < 3; ++c) {
            const double ox = c == 0 ? 0.0 : 0.5, oy = c == 1 ? 0.0 : 0.5;
            const chp::SrcAxis ax{pts(ncx, ox), chp::AXIS_PERIODIC}, ay{pts(ncy, oy), chp::AXIS_PERIODIC};
            std::vector<int> ix, iy;
            std::vector<double> w;
            if (!chp::hermite_stencils(ax, pts(nx, ox), &ix, &w) ||
                !chp::hermite_stencils(ay, pts(ny, oy), &iy, &w))
                return 3;
            const int xwin = chp::interp_xwin(ix, nx, ncx);
            const int rm = chp::interp_march_rows(iy, nx, ny, ncx, ncy, xwin);
            const int64_t tn[3] = {nx, ny, nz + (c == 2)};
            const int xp = chp::interp_pattern(ix, nx, ncx, 4);
            const int yp = chp::interp_pattern(iy, ny, ncy, chk::MARCH_BAND);
            const chp::MarchShape m = chp::march_shape(es, ncx, tn);
            const bool piped = chp::interp_piped(es, rmax, ncx);
            const bool taken = chp::march_taken(es, rm, xp, yp, m, ncx, tn, piped);
            // the kernel: known patterns only in the pairs it is built for
            const bool known = (xp == chk::MARCH_FACE && yp == chk::MARCH_CENTRE) ||
                               (xp == chk::MARCH_CENTRE && yp != chk::MARCH_ANY);
            const int rows = !known ? rm : yp == chk::MARCH_FACE ? 7 : 8;
            bool right = true;
            for (int i = 0; i < nx && rm; ++i)
                for (int t = 0; t < 4; ++t) {
                    const int ws = ix[4 * (i / 4 * 4)];
                    const int d = known ? tap(xp, i % 4) + t : (ix[4 * i + t] - ws + ncx) % ncx;
                    right = right && d < 6 && (ws + d) % ncx == ix[4 * i + t];
                }
            for (int j = 0; j < ny && rm; ++j)
                for (int t = 0; t < 4; ++t) {
                    const int jj = j % chk::MARCH_BAND, base = iy[4 * (j - jj)];
                    const int l = known ? tap(yp, jj) : (iy[4 * j] - base + ncy) % ncy;
                    right = right && l <= jj && l + 4 <= rows && (base + l + t) % ncy == iy[4 * j + t];
                }
            // the launch covers every target: bands of rows, chunks of planes,
            // a thread for every coarse column and every 4 targets of a row
            right = right && (!rm || (m.sxw >= ncx && m.sxw * m.nsub <= 256 && (nx + 3) / 4 <= 256 &&
                                      (int64_t)m.nband * m.nsub * chk::MARCH_BAND >= ny &&
                                      (int64_t)m.nchunk * m.kc >= tn[2]));
            printf("%d %d %d %d%s", rm, taken ? 1 : 0, right ? 1 : 0, piped ? 1 : 0, c < 2 ? " " : "\n");
        }
    }
    return 0;
}
