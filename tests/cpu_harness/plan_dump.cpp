// plan_dump.cpp -- prints the launch plan of boxes as the library reports it
// (test infrastructure).
//
// stdin:  "nbox prec x_rows z_chunk seg_len dt", then per box "nx ny nz h bcx bcy bcz"
//         (Cn = h, Pe = 0.9 / h)
// stdout: "x_rows z_chunk seg_option longest-segment", or "FAIL message"
#include <cstdio>
#include <vector>

#include "../../paper_2105_01865_amd/csrc/ch_plan.h"

int main()
{
    int nbox, prec, x_rows, zc, seg;
    double dt;
    if (scanf("%d %d %d %d %d %lf", &nbox, &prec, &x_rows, &zc, &seg, &dt) != 6) return 2;
    std::vector<ch_grid> g(nbox);
    std::vector<double> Cn(nbox), Pe(nbox);
    std::vector<ch_bc> bc(nbox);
    for (int b = 0; b < nbox; ++b) {
        long long nx, ny, nz;
        if (scanf("%lld %lld %lld %lf %d %d %d", &nx, &ny, &nz, &g[b].h, &bc[b].x, &bc[b].y,
                  &bc[b].z) != 7)
            return 2;
        g[b].nx = nx;
        g[b].ny = ny;
        g[b].nz = nz;
        Cn[b] = g[b].h;
        Pe[b] = 0.9 / g[b].h;
    }
    ch_opts o;
    chp::default_opts(&o);
    o.precision = prec;
    o.x_rows = x_rows;
    o.z_chunk = zc;
    o.seg_len = seg;
    chp::Plan P;
    if (chp::plan_init(P, nbox, g.data(), Cn.data(), Pe.data(), nullptr, bc.data(), &o) != CH_OK ||
        chp::plan_dt(P, dt) != CH_OK) {
        printf("FAIL %s\n", P.err.c_str());
        return 0;
    }
    printf("%d %d %d %d\n", P.x_rows, P.zc, chp::seg_option(P), P.seg_cap);
    return 0;
}
