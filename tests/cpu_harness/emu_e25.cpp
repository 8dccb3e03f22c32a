// emu_e25.cpp -- CPU harness of the explicit scheme's row program (test
// infrastructure): the steps of emu.cpp's explicit mode with
// pass_x_e25_row_program in place of the general x program, under the
// library's launch plan.  The same PARAMS, IN_DIR and OUT_DIR: its result
// goes to OUT_DIR/C_row.bin, then emu.cpp's own run follows; exits with 4 where
// the plan does not take the row program.
#define main emu_main
#include "emu.cpp"
#undef main

template <typename T>
static int go_row(chp::Plan& P, const std::string& in, const std::string& out, int nsteps)
{
    if (!P.e25_row) return 4;
    const std::vector<double> zero(P.tot[0], 0.0);
    T* C = dev_copy<T>(read_bin(in + "/C.bin", P.tot[0]));
    T* E = dev_copy<T>(zero);
    T* qa = dev_copy<T>(zero);
    T* u = dev_copy<T>(read_bin(in + "/u.bin", P.tot[1]));
    T* v = dev_copy<T>(read_bin(in + "/v.bin", P.tot[2]));
    T* w = dev_copy<T>(read_bin(in + "/w.bin", P.tot[3]));
    chd::CpuExec ex{P.x_threads};
    std::vector<chd::XE25State<T>> st(ex.nth);
    for (int s = 0; s < nsteps; ++s)
        for (int k = 0; k < 3; ++k) {
            const chd::PassArgs pa = chp::pass_args(P, k, 0);
            for (int task = 0; task < P.ntask[0]; ++task) {
                unsigned char* lds = (unsigned char*)malloc(P.e25_lds);
                memset(lds, 0xff, P.e25_lds);
                chd::pass_x_e25_row_program<T>(ex, st.data(), P.boxes[0], pa, task, C, u, v, w, E,
                                               qa, lds);
                free(lds);
            }
            std::swap(C, qa);
        }
    std::vector<double> res(P.tot[0]);
    for (int64_t i = 0; i < P.tot[0]; ++i) res[i] = double(C[i]);
    FILE* f = fopen((out + "/C_row.bin").c_str(), "wb");
    fwrite(res.data(), sizeof(double), res.size(), f);
    fclose(f);
    free(C); free(E); free(qa); free(u); free(v); free(w);
    return 0;
}

int main(int argc, char** argv)
{
    if (argc != 4) return 2;
    FILE* f = fopen(argv[1], "r");
    int nbox, prec, solve, x_rows, seg, waves, zchunk, nsteps, mode, xgen;
    double kappa, eps, dt;
    ch_grid g;
    ch_bc bc;
    double Cn, Pe;
    long long nx, ny, nz;
    if (!f || fscanf(f, "%d %d %lf %lf %d %d %d %d %d %lf %d %d %d", &nbox, &prec, &kappa, &eps,
                     &solve, &x_rows, &seg, &waves, &zchunk, &dt, &nsteps, &mode, &xgen) != 13 ||
        fscanf(f, "%lld %lld %lld %lf %lf %lf %d %d %d", &nx, &ny, &nz, &g.h, &Cn, &Pe, &bc.x,
               &bc.y, &bc.z) != 9)
        return 2;
    fclose(f);
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    ch_opts o;
    chp::default_opts(&o);
    o.precision = prec;
    o.weno_eps = eps;
    o.z_chunk = zchunk;
    chp::Plan P;
    P.e25 = true;
    if (chp::plan_init(P, 1, &g, &Cn, &Pe, nullptr, &bc, &o) != CH_OK ||
        chp::plan_dt(P, dt) != CH_OK)
        return 3;
    const int rc = prec == CH_FP64 ? go_row<double>(P, argv[2], argv[3], nsteps)
                                   : go_row<float>(P, argv[2], argv[3], nsteps);
    // then the general program, into OUT_DIR/C.bin (which may be the input)
    return rc ? rc : emu_main(argc, argv);
}
