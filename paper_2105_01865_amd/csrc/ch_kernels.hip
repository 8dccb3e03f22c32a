// ch_kernels.hip -- HIP kernels of libch for gfx950 (CDNA4).
//
// One RK3 substage of the Cahn-Hilliard update is three launches
// (arXiv 2105.01865, eq-fac-1 .. eq-fac-3):
//   k_pass_x : explicit terms, RHS and the x-line solve; one work-group owns
//              complete x-lines, so the RHS goes straight into LDS and the
//              solve never leaves the chip
//   k_pass_y : y-line solve, x-columns across the lanes of a wave
//   k_pass_z : z-line solve and C += dC
// The path is stencil- and bandwidth-bound: no MFMA.  Work-group ids are
// remapped so that consecutive tasks (neighbouring lines that share stencil
// halos) land on the same XCD and its L2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ch_device.h"
#include "ch_kernels.h"

namespace chk {

// Waves per SIMD the single-precision, one-cell-per-thread x kernel of the
// implicit scheme is compiled for (its register budget); the other variants
// keep the compiler's choice (forcing them spills).
#ifndef X_WAVES_F32_HINT
#define X_WAVES_F32_HINT 5
#endif

// Work-groups are dispatched round-robin over the 8 XCDs of the chip; give
// each XCD a contiguous range of tasks.
__device__ __forceinline__ int xcd_task(int wg, int nwg)
{
    const int nxcd = 8;
    const int per = nwg / nxcd, rem = nwg % nxcd;
    const int x = wg % nxcd, l = wg / nxcd;
    return (x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per) + l;
}

// NT bounds the work-group size and so the registers per lane: 512 VGPRs per
// SIMD lane over the group's waves per SIMD (256 for 512 threads, 170 for
// 768, 128 for 1024).  E25 selects the explicit 25-point scheme (no solve,
// the new C is written to Q).
template <typename T, typename A, int MI, int NT, bool E25>
__global__ void __launch_bounds__(NT)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && MI == 1 && !E25 ? X_WAVES_F32_HINT : 1)))
k_pass_x(const chd::BoxDesc* __restrict__ boxes, int nbox, chd::PassArgs pa,
         const T* __restrict__ C, const T* __restrict__ U, const T* __restrict__ V,
         const T* __restrict__ W, T* __restrict__ E, T* __restrict__ Q)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int task = xcd_task(blockIdx.x, gridDim.x);
    const int b = chd::find_box(boxes, nbox, chd::PASS_X, task);
    chd::GpuExec ex{(int)threadIdx.x, (int)blockDim.x};
    chd::XState<T, A, MI> st;
    // double precision with registers to spare: uniform constants in lane registers
    constexpr bool VCONST = sizeof(T) == 8 && MI == 1 && NT <= 512 && !E25;
    chd::pass_x_program<T, A, MI, E25, chd::GpuExec, VCONST>(ex, &st, boxes[b], pa, task, C, U, V,
                                                             W, E, Q, smem);
}

// The row x-pass program (pass_x_row_program); NT bounds the group size, RM
// is the row mode (one row per task, several with per-thread row offsets, or
// several of whole waves).  Single precision with one row of a 512-cell line:
// at most 64 VGPRs (none spilled), so that four groups of 8 waves share a CU
// rather than three (the 512^3 x pass 941-955 -> 919-927 us; at 256 threads
// the same bound adds instructions and gains nothing).
template <typename T, typename A, int NT, int RM>
__global__ void __launch_bounds__(NT)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && RM == chd::XR_ONE && NT == 512 ? 8 : 1)))
k_pass_x_row(const chd::BoxDesc* __restrict__ boxes, int nbox, chd::PassArgs pa,
             const T* __restrict__ C, const T* __restrict__ U, const T* __restrict__ V,
             const T* __restrict__ W, T* __restrict__ E, T* __restrict__ Q)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int task = xcd_task(blockIdx.x, gridDim.x);
    const int b = chd::find_box(boxes, nbox, chd::PASS_X, task);
    chd::GpuExec ex{(int)threadIdx.x, (int)blockDim.x};
    chd::XRowState<T, A> st;
    chd::pass_x_row_program<T, A, RM, chd::GpuExec>(ex, &st, boxes[b], pa, task, C, U, V, W, E,
                                                    Q, smem);
}

// The segmented x-pass program (pass_x_seg_program): E read from Ein, the
// new one written to Eout.
template <typename T, typename A>
__global__ void __launch_bounds__(256)
k_pass_x_seg(const chd::BoxDesc* __restrict__ boxes, int nbox, chd::PassArgs pa,
             const T* __restrict__ C, const T* __restrict__ U, const T* __restrict__ V,
             const T* __restrict__ W, const T* __restrict__ Ein, T* __restrict__ Eout,
             T* __restrict__ Q)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int task = xcd_task(blockIdx.x, gridDim.x);
    const int b = chd::find_box(boxes, nbox, chd::PASS_X, task);
    chd::GpuExec ex{(int)threadIdx.x, (int)blockDim.x};
    chd::XSegState<T, A> st;
    chd::pass_x_seg_program<T, A, chd::GpuExec>(ex, &st, boxes[b], pa, task, C, U, V, W, Ein,
                                                Eout, Q, smem);
}

// The explicit 25-point scheme's row program (pass_x_e25_row_program).
template <typename T, int NT>
__global__ void __launch_bounds__(NT)
k_pass_x_e25(const chd::BoxDesc* __restrict__ boxes, chd::PassArgs pa, const T* __restrict__ C,
             const T* __restrict__ U, const T* __restrict__ V, const T* __restrict__ W,
             T* __restrict__ E, T* __restrict__ Q)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int task = xcd_task(blockIdx.x, gridDim.x);
    chd::GpuExec ex{(int)threadIdx.x, (int)blockDim.x};
    chd::XE25State<T> st;
    chd::pass_x_e25_row_program<T, chd::GpuExec>(ex, &st, boxes[0], pa, task, C, U, V, W, E, Q,
                                                 smem);
}

template <typename T, typename A, int PASS, int SPLIT>
__global__ void __launch_bounds__(512)
k_pass_line(const chd::BoxDesc* __restrict__ boxes, int nbox, chd::PassArgs pa,
            const T* __restrict__ Qin, T* __restrict__ Qout)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int task = xcd_task(blockIdx.x, gridDim.x);
    const int b = chd::find_box(boxes, nbox, PASS, task);
    chd::GpuExec ex{(int)threadIdx.x, (int)blockDim.x};
    chd::LineState<A> st;
    chd::pass_line_program<T, A, chd::GpuExec, SPLIT>(ex, &st, boxes[b], pa, PASS, task, Qin, Qout,
                                                      smem);
}

// Mass, stage 1 body: block `blk` of box bd (MASS_BLOCK elements of C),
// summed in double in a fixed order, written to *partial.
template <typename T>
__device__ void mass_partial_body(const chd::BoxDesc& bd, int blk, const T* __restrict__ C,
                                  double* __restrict__ partial)
{
    __shared__ double sh[chd::MASS_THREADS];
    const int tid = threadIdx.x;
    sh[tid] = chd::mass_thread_sum<T>(tid, bd, blk, C);
    __syncthreads();
    for (int s = chd::MASS_THREADS / 2; s > 0; s >>= 1) {
        if (tid < s) sh[tid] += sh[tid + s];
        __syncthreads();
    }
    if (tid == 0) *partial = sh[0];
}

// Mass, stage 2 body: a box's nmblk partials summed in a fixed order and
// scaled by h^3.
__device__ void mass_final_body(const double* __restrict__ partial, int nmblk, double h3,
                                double* __restrict__ out)
{
    __shared__ double sh[chd::MASS_THREADS];
    const int tid = threadIdx.x;
    double s = 0.0;
    for (int i = tid; i < nmblk; i += chd::MASS_THREADS) s += partial[i];
    sh[tid] = s;
    __syncthreads();
    for (int st = chd::MASS_THREADS / 2; st > 0; st >>= 1) {
        if (tid < st) sh[tid] += sh[tid + st];
        __syncthreads();
    }
    if (tid == 0) *out = sh[0] * h3;
}

// Mass, stage 1: one fixed block of C per work-group (the box found from the
// block index).
template <typename T>
__global__ void __launch_bounds__(chd::MASS_THREADS)
k_mass_partial(const chd::BoxDesc* __restrict__ boxes, int nbox, const T* __restrict__ C,
               double* __restrict__ partial)
{
    const int blk = blockIdx.x;
    int lo = 0, hi = nbox - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (boxes[mid].mblk0 <= blk) lo = mid;
        else hi = mid - 1;
    }
    const chd::BoxDesc& bd = boxes[lo];
    mass_partial_body<T>(bd, blk - bd.mblk0, C, partial + blk);
}

// Mass, stage 2: one work-group per box.
__global__ void __launch_bounds__(chd::MASS_THREADS)
k_mass_final(const chd::BoxDesc* __restrict__ boxes, const double* __restrict__ partial,
             const double* __restrict__ h3, double* __restrict__ out)
{
    const chd::BoxDesc& bd = boxes[blockIdx.x];
    mass_final_body(partial + bd.mblk0, bd.nmblk, h3[blockIdx.x], out + blockIdx.x);
}

// The same two stages for one field described by value (no box table in
// device memory): the allocation-free mass.
template <typename T>
__global__ void __launch_bounds__(chd::MASS_THREADS)
k_mass_partial_one(chd::BoxDesc bd, const T* __restrict__ C, double* __restrict__ partial)
{
    mass_partial_body<T>(bd, blockIdx.x, C, partial + blockIdx.x);
}

__global__ void __launch_bounds__(chd::MASS_THREADS)
k_mass_final_one(int nmblk, const double* __restrict__ partial, double h3,
                 double* __restrict__ out)
{
    mass_final_body(partial, nmblk, h3, out);
}

// Velocity check: non-finite values anywhere, non-zero normal velocity on a
// no-flux wall.  Each work-group writes its two counts to flags[2 * wg].
template <typename T>
__global__ void __launch_bounds__(256)
k_check_velocity(const chd::BoxDesc* __restrict__ boxes, int nbox, const T* __restrict__ U,
                 const T* __restrict__ V, const T* __restrict__ W, int* __restrict__ flags)
{
    __shared__ int sh[2][256];
    int bad = 0, wall = 0;
    for (int b = 0; b < nbox; ++b) {
        const chd::BoxDesc& bd = boxes[b];
        const int nx = bd.n[0], ny = bd.n[1], nz = bd.n[2];
        const int64_t cnt[3] = {(int64_t)nz * ny * bd.nf[0], (int64_t)nz * bd.nf[1] * nx,
                                (int64_t)bd.nf[2] * ny * nx};
        const T* arr[3] = {U + bd.u_off, V + bd.v_off, W + bd.w_off};
        for (int d = 0; d < 3; ++d) {
            for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < cnt[d];
                 e += (int64_t)gridDim.x * blockDim.x) {
                const T val = arr[d][e];
                if (!(val == val) || val - val != T(0)) ++bad;
                if (bd.bc[d] == 1) {
                    int64_t f;
                    if (d == 0) f = e % bd.nf[0];
                    else if (d == 1) f = (e / nx) % bd.nf[1];
                    else f = e / ((int64_t)ny * nx);
                    if ((f == 0 || f == bd.nf[d] - 1) && val != T(0)) ++wall;
                }
            }
        }
    }
    const int tid = threadIdx.x;
    sh[0][tid] = bad;
    sh[1][tid] = wall;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) {
            sh[0][tid] += sh[0][tid + s];
            sh[1][tid] += sh[1][tid + s];
        }
        __syncthreads();
    }
    if (tid == 0) {
        flags[2 * blockIdx.x] = sh[0][0];
        flags[2 * blockIdx.x + 1] = sh[1][0];
    }
}

// Coarse-to-fine velocity transfer, the separable tensor-product
// interpolation of sec. 3.4.  Work item = (band of JB target rows, target
// plane k), k fastest; each work-group takes a contiguous run of items
// (XCD-contiguous runs), so consecutive items are neighbouring target planes
// of one band, whose z stencils share most of their coarse planes: those
// rows come from L2 (at 512^3 from 256^2 coarse rows, which the marching kernel
// takes now, 234 -> 201 us per FP32 component inside a step against the
// plane-major order):
//   A. the band's coarse rows, each combined over the 4 source planes of k's
//      z stencil, into LDS (coalesced along x; MA rows' loads in flight per
//      thread, through buffer resources on the 4 planes);
//   B. each target row of the band combines 4 of those rows (its y stencil)
//      into a second LDS row;
//   C. x stencil.  With the 6-point window property each thread owns 4
//      consecutive targets: it reads the 6 window points once and applies a
//      4 x 6 weight matrix built at start-up (4-wide stores); otherwise every
//      target reads its 4 taps.
// Band, z and y stencil entries are uniform per item and row, so they are
// read into scalar registers.  Every target element is written once, with
// non-temporal stores (nothing reads it back while it is in the caches, and
// streaming it out leaves them to the coarse rows, which are read again);
// the coarse data is read through the caches about (rows per band / band
// height) times per target plane.
// PIPE: an item's rows are loaded while the targets of the one before are
// stored, where one batch of loads covers them (512^3 from 256^2 coarse rows,
// before the marching kernel below took that shape: 241 -> 234 us FP32; 256 to
// 320 columns 252 us without, 222 with; 256 to 256 81 and 70).
template <typename T, int JB, int MA, bool PIPE>
__global__ void __launch_bounds__(256)
k_interp(InterpArgs a, const T* __restrict__ src, T* __restrict__ dst,
         const int* __restrict__ band, const int* __restrict__ izt, const T* __restrict__ wzt,
         const int* __restrict__ lyt, const T* __restrict__ wyt, const int* __restrict__ ixt,
         const double* __restrict__ wxt)
{
    typedef T T4 __attribute__((ext_vector_type(4)));
    constexpr int XQ = 4, NW = 6;
    extern __shared__ __align__(16) unsigned char smem[];
    const int sx = a.sx;
    T* zr = reinterpret_cast<T*>(smem);           // rmax x sx
    T* yr = zr + (size_t)a.rmax * sx;             // JB x sx
    const int tid = threadIdx.x, nt = blockDim.x;
    const int nb = (a.tny + JB - 1) / JB;
    const int items = nb * a.tnz;
    const uint32_t pbytes = (uint32_t)(a.plane * sizeof(T));

    // x: thread -> targets xi0 .. xi0 + 3 of rows jj = rg0 (mod rgs)
    const int tc = (a.tnx + XQ - 1) / XQ;
    const bool win = a.xwin && tc <= nt;
    const int rgs = win ? nt / tc : 1;
    const int rg0 = win ? tid / tc : 0;
    const int xi0 = win ? XQ * (tid - rg0 * tc) : 0;
    const bool xact = win && rg0 < rgs;
    const bool vec = (a.tnx % XQ) == 0 && (reinterpret_cast<uintptr_t>(dst) % sizeof(T4)) == 0;
    int ws = 0;
    if (xact) ws = ixt[4 * xi0];
    int woff[NW];   // window points ws .. ws + NW - 1, cyclic in x
#pragma unroll
    for (int n = 0; n < NW; ++n) woff[n] = ws + n < sx ? ws + n : (ws + n) % sx;
    T M[XQ][NW];
#pragma unroll
    for (int q = 0; q < XQ; ++q)
#pragma unroll
        for (int n = 0; n < NW; ++n) M[q][n] = T(0);
    if (xact) {
#pragma unroll
        for (int q = 0; q < XQ; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool ok = xi0 + q < a.tnx;
                int d = ok ? ixt[4 * (xi0 + q) + t] - ws : 0;
                if (d < 0) d += sx;
                const T w = ok ? T(wxt[4 * (xi0 + q) + t]) : T(0);
#pragma unroll
                for (int n = 0; n < NW; ++n) M[q][n] += d == n ? w : T(0);
            }
    }

    const int per = (items + a.nwg - 1) / a.nwg;
    const int it0 = xcd_task(blockIdx.x, a.nwg) * per;
    const int it1 = it0 + per < items ? it0 + per : items;
    // PIPE (one batch of loads covers an item: the coarse row fits the group
    // and no band is taller than the rows in flight): the next item's coarse
    // rows are loaded while this item's targets are stored, issued before
    // phase C and combined into LDS at the top of the next item.
    constexpr bool pipe = PIPE;
    T vp[PIPE ? MA : 1][4];
    auto issue = [&](int item) {   // the item's coarse rows at column tid
        if constexpr (!PIPE) return;
        const int b = item / a.tnz, k = item - b * a.tnz;
        const int base = band[2 * b], span = band[2 * b + 1];
        const chd::PlaneRef<T> p0(src + (int64_t)izt[4 * k] * a.plane, pbytes);
        const chd::PlaneRef<T> p1(src + (int64_t)izt[4 * k + 1] * a.plane, pbytes);
        const chd::PlaneRef<T> p2(src + (int64_t)izt[4 * k + 2] * a.plane, pbytes);
        const chd::PlaneRef<T> p3(src + (int64_t)izt[4 * k + 3] * a.plane, pbytes);
        const int cx = tid < sx ? tid : 0;
#pragma unroll
        for (int m = 0; m < (PIPE ? MA : 1); ++m) {
            int rr = base + m;
            if (rr >= a.sy) rr -= a.sy;
            const uint32_t boff = (uint32_t)((m < span ? rr * sx + cx : cx) * (int)sizeof(T));
            vp[m][0] = p0(boff);
            vp[m][1] = p1(boff);
            vp[m][2] = p2(boff);
            vp[m][3] = p3(boff);
        }
    };
    if (pipe && it0 < it1) issue(it0);
    for (int item = it0; item < it1; ++item) {
        const int b = item / a.tnz, k = item - b * a.tnz;
        const int j0 = b * JB;
        const int nj = a.tny - j0 < JB ? a.tny - j0 : JB;
        const int base = band[2 * b], span = band[2 * b + 1];
        __syncthreads();   // the previous item's readers are done with the LDS
        // A: coarse rows base .. base + span - 1 (cyclic), z stencil applied
        if constexpr (PIPE) {
            const T w0 = wzt[4 * k], w1 = wzt[4 * k + 1], w2 = wzt[4 * k + 2], w3 = wzt[4 * k + 3];
            if (tid < sx)
#pragma unroll
                for (int m = 0; m < (PIPE ? MA : 1); ++m)
                    if (m < span)
                        zr[m * sx + tid] =
                            ((w0 * vp[m][0] + w1 * vp[m][1]) + w2 * vp[m][2]) + w3 * vp[m][3];
        } else {
            const chd::PlaneRef<T> p0(src + (int64_t)izt[4 * k] * a.plane, pbytes);
            const chd::PlaneRef<T> p1(src + (int64_t)izt[4 * k + 1] * a.plane, pbytes);
            const chd::PlaneRef<T> p2(src + (int64_t)izt[4 * k + 2] * a.plane, pbytes);
            const chd::PlaneRef<T> p3(src + (int64_t)izt[4 * k + 3] * a.plane, pbytes);
            const T w0 = wzt[4 * k], w1 = wzt[4 * k + 1], w2 = wzt[4 * k + 2], w3 = wzt[4 * k + 3];
            for (int r0 = 0; r0 < span; r0 += MA)
                for (int cx = tid; cx < sx; cx += nt) {
                    T v[MA][4];
#pragma unroll
                    for (int m = 0; m < MA; ++m) {
                        int rr = base + r0 + m;
                        if (rr >= a.sy) rr -= a.sy;
                        const uint32_t boff =
                            (uint32_t)((r0 + m < span ? rr * sx + cx : cx) * (int)sizeof(T));
                        v[m][0] = p0(boff);
                        v[m][1] = p1(boff);
                        v[m][2] = p2(boff);
                        v[m][3] = p3(boff);
                    }
#pragma unroll
                    for (int m = 0; m < MA; ++m)
                        if (r0 + m < span)
                            zr[(r0 + m) * sx + cx] =
                                ((w0 * v[m][0] + w1 * v[m][1]) + w2 * v[m][2]) + w3 * v[m][3];
                }
        }
        __syncthreads();
        // B: the band's target rows, y stencil applied
        for (int cx = tid; cx < sx; cx += nt) {
#pragma unroll
            for (int jj = 0; jj < JB; ++jj) {
                if (jj < nj) {
                    const int* l = lyt + 4 * (j0 + jj);
                    const T* y = wyt + 4 * (j0 + jj);
                    yr[jj * sx + cx] = ((y[0] * zr[l[0] + cx] + y[1] * zr[l[1] + cx])
                                        + y[2] * zr[l[2] + cx]) + y[3] * zr[l[3] + cx];
                }
            }
        }
        __syncthreads();
        if (pipe && item + 1 < it1) issue(item + 1);
        // C: x stencil, every target point written once
        T* out = dst + ((int64_t)k * a.tny + j0) * a.tnx;
        if (win) {
            if (xact)
                for (int jj = rg0; jj < nj; jj += rgs) {
                    const T* row = yr + jj * sx;
                    T p[NW];
#pragma unroll
                    for (int n = 0; n < NW; ++n) p[n] = row[woff[n]];
                    T y[XQ];
#pragma unroll
                    for (int q = 0; q < XQ; ++q) {
                        T acc = M[q][0] * p[0];
#pragma unroll
                        for (int n = 1; n < NW; ++n) acc += M[q][n] * p[n];
                        y[q] = acc;
                    }
                    T* o = out + (int64_t)jj * a.tnx + xi0;
                    if (vec) {
                        __builtin_nontemporal_store(T4{y[0], y[1], y[2], y[3]},
                                                    reinterpret_cast<T4*>(o));
                    } else {
#pragma unroll
                        for (int q = 0; q < XQ; ++q)
                            if (xi0 + q < a.tnx) __builtin_nontemporal_store(y[q], o + q);
                    }
                }
        } else {
            for (int jj = 0; jj < nj; ++jj)
                for (int i = tid; i < a.tnx; i += nt) {
                    const T* row = yr + jj * sx;
                    T acc = T(0);
                    for (int t = 0; t < 4; ++t) acc += T(wxt[4 * i + t]) * row[ixt[4 * i + t]];
                    __builtin_nontemporal_store(acc, out + (int64_t)jj * a.tnx + i);
                }
        }
    }
}

// The same transfer for upsampling in y with coarse rows of at most 256 points
// (MARCH_ROWS consecutive target rows span at most RM coarse rows, whose taps
// are consecutive; the x taps of 4 targets lie in 6 points).  A work-group
// takes a band of target rows and marches up through kc target planes.  Its
// waves are split into sub-bands of MARCH_ROWS rows; a thread owns one coarse
// column of its sub-band and keeps the RM rows of the item's four coarse planes
// in registers: the z stencil, then the y stencil are formed there, so only the
// target rows on the coarse columns go through LDS (two buffers, one barrier
// per plane).  The next plane's loads go out before this plane's x stencil, and
// not at all where it reads the same four coarse planes.
//
// XP and YP say where the taps of neighbouring targets start: at two fine cells
// per coarse one the first taps of consecutive targets are 0 0 1 1 (MARCH_FACE:
// faces on faces) or 0 1 1 2 (MARCH_CENTRE: centres on centres) in every group,
// so each target takes its four taps with no selection; MARCH_ANY selects (a
// 4 x 6 matrix in x, the row among RM - 3 in y).
//
// What bounds it: the stencils' VALU work and the groups' chains of loads,
// barrier and stores; the stores alone take 90 us at 512^3 FP32.  Per component,
// caches cold, against the general kernel (three barriers and scalar loads of
// the y stencil per item, the z stencil's rows through LDS): 512^3 FP32 169-182
// against 202 us, FP64 331-340 against 379-383, 256^3 FP32 34 against 76, FP64
// 54 against 114.  With selected taps and 11 rows it takes 256 registers in double
// precision, one wave per SIMD; march_taken has what it is measured to gain where.
constexpr int MARCH_ROWS = MARCH_BAND;
// first tap of target q in its group
template <int P>
constexpr int march_tap(int q)
{
    return P == MARCH_FACE ? q / 2 : (q + 1) / 2;
}

template <typename T, int RM, int XP, int YP>
__global__ void __launch_bounds__(256)
k_interp_march(InterpArgs a, MarchArgs m, const T* __restrict__ src, T* __restrict__ dst,
               const int* __restrict__ iy0, const int* __restrict__ izt,
               const T* __restrict__ wzt, const T* __restrict__ wyt,
               const int* __restrict__ ixt, const double* __restrict__ wxt)
{
    typedef T T4 __attribute__((ext_vector_type(4)));
    constexpr int XQ = 4, MR = MARCH_ROWS;
    constexpr int NW = XP == MARCH_ANY ? 6 : march_tap<XP>(XQ - 1) + 4;   // points of 4 targets
    constexpr int NX = XP == MARCH_ANY ? NW : 4;                          // weights of a target
    extern __shared__ __align__(16) unsigned char smem[];
    T* yr = reinterpret_cast<T*>(smem);   // 2 x (nsub MR) x sx
    constexpr uint32_t sT = sizeof(T);
    const int sx = a.sx, nsub = m.nsub, nt = 256;
    const int tid = threadIdx.x;
    const uint32_t pbytes = (uint32_t)(a.plane * sizeof(T));
    const int wg = xcd_task(blockIdx.x, gridDim.x);
    const int bandi = wg / m.nchunk, chunk = wg - bandi * m.nchunk;
    const int k0 = chunk * m.kc, k1 = k0 + m.kc < a.tnz ? k0 + m.kc : a.tnz;
    const int j0 = bandi * MR * nsub;                          // the group's target rows
    const int njw = a.tny - j0 < MR * nsub ? a.tny - j0 : MR * nsub;
    const int bufsz = MR * nsub * sx;

    // y stencil of this wave's sub-band: coarse rows base, base + 1, ... (cyclic),
    // the taps of target row jj from row l[jj] of them on
    const int sub = chd::uniform_i(tid / m.sxw);
    const int js = j0 + MR * sub;
    const bool wact = sub < nsub && js < a.tny;
    const int cx = tid - sub * m.sxw;
    const bool cact = wact && cx < sx;
    const int jb = wact ? js : 0;
    const int base = iy0[jb];
    uint32_t roff[RM];   // byte offset of coarse row base + r
#pragma unroll
    for (int r = 0; r < RM; ++r) roff[r] = (uint32_t)((base + r) % a.sy * sx) * sT;
    const uint32_t xb = (uint32_t)(cact ? cx : 0) * sT;

    T vp[RM][4];
    auto issue = [&](int k) {
        const chd::PlaneRef<T> p0(src + (int64_t)izt[4 * k] * a.plane, pbytes);
        const chd::PlaneRef<T> p1(src + (int64_t)izt[4 * k + 1] * a.plane, pbytes);
        const chd::PlaneRef<T> p2(src + (int64_t)izt[4 * k + 2] * a.plane, pbytes);
        const chd::PlaneRef<T> p3(src + (int64_t)izt[4 * k + 3] * a.plane, pbytes);
#pragma unroll
        for (int r = 0; r < RM; ++r) {
            vp[r][0] = p0(xb, roff[r]);
            vp[r][1] = p1(xb, roff[r]);
            vp[r][2] = p2(xb, roff[r]);
            vp[r][3] = p3(xb, roff[r]);
        }
    };
    issue(k0);

    int l[MR];
    T wy[MR][4];
#pragma unroll
    for (int jj = 0; jj < MR; ++jj) {
        const int j = jb + jj < a.tny ? jb + jj : a.tny - 1;
        if constexpr (YP == MARCH_ANY) {
            int d = iy0[j] - base;
            if (d < 0) d += a.sy;
            l[jj] = d;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) wy[jj][t] = wyt[4 * j + t];
    }

    // x stencil of this thread: targets xi0 .. xi0 + 3 of rows rg0 (mod rgs) from
    // the NW points from ws on.  The table reads are unconditional (a target
    // past the end repeats the last one), so that they go out together.
    const int tc = (a.tnx + XQ - 1) / XQ;
    const int rgs = nt / tc, rg0 = tid / tc;
    const int xi0 = XQ * (tid - rg0 * tc);
    const bool xact = rg0 < rgs;
    const bool vec = (a.tnx % XQ) == 0 && (reinterpret_cast<uintptr_t>(dst) % sizeof(T4)) == 0;
    const int ws = ixt[4 * xi0];
    int woff[NW];
#pragma unroll
    for (int n = 0; n < NW; ++n) woff[n] = (ws + n) % sx;
    T M[XQ][NX];
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
        const int i = xi0 + q < a.tnx ? xi0 + q : a.tnx - 1;
        if constexpr (XP == MARCH_ANY) {
#pragma unroll
            for (int n = 0; n < NX; ++n) M[q][n] = T(0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                int d = ixt[4 * i + t] - ws;
                if (d < 0) d += sx;
                const T w = T(wxt[4 * i + t]);
#pragma unroll
                for (int n = 0; n < NX; ++n) M[q][n] += d == n ? w : T(0);
            }
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) M[q][t] = T(wxt[4 * i + t]);
        }
    }

    for (int k = k0; k < k1; ++k) {
        T* buf = yr + ((k - k0) & 1) * bufsz;
        {
            const T w0 = wzt[4 * k], w1 = wzt[4 * k + 1], w2 = wzt[4 * k + 2], w3 = wzt[4 * k + 3];
            T zc[RM];
#pragma unroll
            for (int r = 0; r < RM; ++r)
                zc[r] = ((w0 * vp[r][0] + w1 * vp[r][1]) + w2 * vp[r][2]) + w3 * vp[r][3];
            T* out = buf + MR * sub * sx + cx;
#pragma unroll
            for (int jj = 0; jj < MR; ++jj) {
                auto comb = [&](int c) {
                    return ((wy[jj][0] * zc[c] + wy[jj][1] * zc[c + 1]) + wy[jj][2] * zc[c + 2]) +
                           wy[jj][3] * zc[c + 3];
                };
                T o = T(0);
                if constexpr (YP == MARCH_ANY) {
                    // the taps start at most one row later per target row
#pragma unroll
                    for (int c = 0; c <= (jj < RM - 4 ? jj : RM - 4); ++c)
                        if (l[jj] == c) o = comb(c);
                } else {
                    o = comb(march_tap<YP>(jj));
                }
                if (cact && js + jj < a.tny) out[jj * sx] = o;
            }
        }
        __syncthreads();
        if (k + 1 < k1) {
            const int* z0 = izt + 4 * k;
            if (z0[4] != z0[0] || z0[5] != z0[1] || z0[6] != z0[2] || z0[7] != z0[3]) issue(k + 1);
        }
        // x stencil, every target point written once
        if (xact) {
            T* out = dst + ((int64_t)k * a.tny + j0) * a.tnx + xi0;
            for (int jj = rg0; jj < njw; jj += rgs) {
                const T* row = buf + jj * sx;
                T p[NW];
#pragma unroll
                for (int n = 0; n < NW; ++n) p[n] = row[woff[n]];
                T y[XQ];
#pragma unroll
                for (int q = 0; q < XQ; ++q) {
                    const int c = XP == MARCH_ANY ? 0 : march_tap<XP>(q);
                    T acc = M[q][0] * p[c];
#pragma unroll
                    for (int n = 1; n < NX; ++n) acc += M[q][n] * p[c + n];
                    y[q] = acc;
                }
                T* o = out + (int64_t)jj * a.tnx;
                if (vec) {
                    if (m.nt)
                        __builtin_nontemporal_store(T4{y[0], y[1], y[2], y[3]},
                                                    reinterpret_cast<T4*>(o));
                    else
                        *reinterpret_cast<T4*>(o) = T4{y[0], y[1], y[2], y[3]};
                } else {
#pragma unroll
                    for (int q = 0; q < XQ; ++q)
                        if (xi0 + q < a.tnx) o[q] = y[q];
                }
            }
        }
    }
}

// Solenoidal transfer, pieces other than the interpolation itself.
//
// Coarse normal gradient at the coarse cell centres, one row (k, j) per
// work-group: comp 0 differences u along x, 1 differences v along y, 2
// differences w along z (sz + 1 planes of w, cell heights 1 / dzinv[k]).
template <typename T>
__global__ void __launch_bounds__(256)
k_grad(const T* __restrict__ src, int comp, int sx, int sy, int sz,
       const double* __restrict__ dzinv, T* __restrict__ out)
{
    const int64_t plane = (int64_t)sx * sy;
    for (int64_t row = blockIdx.x; row < (int64_t)sy * sz; row += gridDim.x) {
        const int k = (int)(row / sy), j = (int)(row - (int64_t)k * sy);
        const T* p = src + row * sx;
        T* o = out + row * sx;
        if (comp == 0) {
            for (int i = threadIdx.x; i < sx; i += blockDim.x)
                o[i] = (p[i + 1 < sx ? i + 1 : 0] - p[i]) * T(sx);
        } else if (comp == 1) {
            const T* q = src + ((int64_t)k * sy + (j + 1 < sy ? j + 1 : 0)) * sx;
            for (int i = threadIdx.x; i < sx; i += blockDim.x) o[i] = (q[i] - p[i]) * T(sy);
        } else {
            const T s = T(dzinv[k]);
            for (int i = threadIdx.x; i < sx; i += blockDim.x) o[i] = (p[i + plane] - p[i]) * s;
        }
    }
}

// Largest closure magnitude of a work-group into part[blockIdx.x].
__device__ __forceinline__ void group_max(double v, double* __restrict__ part)
{
    __shared__ double red[4];
    for (int d = 32; d > 0; d >>= 1) v = fmax(v, __shfl_xor(v, d));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = red[0];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, red[w]);
        part[blockIdx.x] = m;
    }
}

// Integration along x, one wavefront per row (in place): the row holds the
// interpolated gradient at the fine cell centres on entry and
//   u[i] = ref[row] + h sum_{i' < i} G[i']
// on exit.  Each lane takes CH consecutive points (32 bytes, two 16-byte
// vector accesses when the row allows), forms their prefix sums, and one
// wave-wide scan of the lane totals joins them.  The |h sum G| of the whole
// row is the closure left at the periodic seam.
template <typename T>
__global__ void __launch_bounds__(256)
k_scan_x(T* __restrict__ buf, const T* __restrict__ ref, int nx, int64_t nrows, T h,
         double* __restrict__ part)
{
    constexpr int CH = 32 / sizeof(T);
    typedef T TV __attribute__((ext_vector_type(CH / 2)));
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const bool vec = nx % (64 * CH) == 0 && reinterpret_cast<uintptr_t>(buf) % 16 == 0;
    double mx = 0.0;
    for (int64_t row = (int64_t)blockIdx.x * 4 + wv; row < nrows; row += (int64_t)gridDim.x * 4) {
        T* p = buf + row * nx;
        const T r = ref[row];
        T acc = T(0);
        for (int i0 = 0; i0 < nx; i0 += 64 * CH) {
            const int b0 = i0 + lane * CH;
            T g[CH];
            if (vec) {
                const TV lo = *reinterpret_cast<const TV*>(p + b0);
                const TV hi = *reinterpret_cast<const TV*>(p + b0 + CH / 2);
#pragma unroll
                for (int m = 0; m < CH / 2; ++m) {
                    g[m] = lo[m];
                    g[m + CH / 2] = hi[m];
                }
            } else {
#pragma unroll
                for (int m = 0; m < CH; ++m) g[m] = b0 + m < nx ? p[b0 + m] : T(0);
            }
            T loc[CH];
            T run = T(0);
#pragma unroll
            for (int m = 0; m < CH; ++m) {
                loc[m] = run;
                run += g[m];
            }
            T s = run;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const T t = __shfl_up(s, d);
                if (lane >= d) s += t;
            }
            const T ex = acc + (s - run);
            T o[CH];
#pragma unroll
            for (int m = 0; m < CH; ++m) o[m] = r + h * (ex + loc[m]);
            if (vec) {
                TV lo, hi;
#pragma unroll
                for (int m = 0; m < CH / 2; ++m) {
                    lo[m] = o[m];
                    hi[m] = o[m + CH / 2];
                }
                *reinterpret_cast<TV*>(p + b0) = lo;
                *reinterpret_cast<TV*>(p + b0 + CH / 2) = hi;
            } else {
#pragma unroll
                for (int m = 0; m < CH; ++m)
                    if (b0 + m < nx) p[b0 + m] = o[m];
            }
            acc += __shfl(s, 63);
        }
        mx = fmax(mx, (double)fabs(h * acc));
    }
    group_max(mx, part);
}

// Integration along y (in place), one thread per (k, i) column:
//   v[j] = ref[k][i] + h sum_{j' < j} G[j'].
template <typename T>
__global__ void __launch_bounds__(256)
k_scan_y(T* __restrict__ buf, const T* __restrict__ ref, int nx, int ny, int nz, T h,
         double* __restrict__ part)
{
    double mx = 0.0;
    const int64_t ncol = (int64_t)nz * nx;
    for (int64_t col = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; col < ncol;
         col += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = col / nx, i = col - k * nx;
        T* p = buf + k * ny * nx + i;
        const T r = ref[col];
        T acc = T(0);
        int j = 0;
        for (; j + 8 <= ny; j += 8) {
            T g[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) g[q] = p[(int64_t)(j + q) * nx];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                p[(int64_t)(j + q) * nx] = r + h * acc;
                acc += g[q];
            }
        }
        for (; j < ny; ++j) {
            const T g = p[(int64_t)j * nx];
            p[(int64_t)j * nx] = r + h * acc;
            acc += g;
        }
        mx = fmax(mx, (double)fabs(h * acc));
    }
    group_max(mx, part);
}

// Integration along z (in place), one thread per (j, i) column: planes
// 0 .. nz-1 hold G on entry; w[k] = h sum_{k' < k} G[k'] (w = 0 on the
// bottom wall) and the top wall plane nz is set to 0.
template <typename T>
__global__ void __launch_bounds__(256)
k_scan_z(T* __restrict__ buf, int64_t plane, int nz, T h, double* __restrict__ part)
{
    double mx = 0.0;
    for (int64_t col = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; col < plane;
         col += (int64_t)gridDim.x * blockDim.x) {
        T* p = buf + col;
        T acc = T(0);
        int k = 0;
        for (; k + 8 <= nz; k += 8) {
            T g[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) g[q] = p[(int64_t)(k + q) * plane];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                p[(int64_t)(k + q) * plane] = h * acc;
                acc += g[q];
            }
        }
        for (; k < nz; ++k) {
            const T g = p[(int64_t)k * plane];
            p[(int64_t)k * plane] = h * acc;
            acc += g;
        }
        p[(int64_t)nz * plane] = T(0);
        mx = fmax(mx, (double)fabs(h * acc));
    }
    group_max(mx, part);
}

// Drop labelling (the drop-size diagnostics of sec. 4): cells with
// C >= threshold, joined through faces (periodic axes wrap), by union-find.
// A label points to a smaller linear index of the same drop or to itself (a
// root); unions link the larger root under the smaller with atomicMin, so
// every drop ends with its smallest index as its root.
//
// The box is cut into tiles of CCL_TX x CCL_TY x CCL_TZ cells.  Four launches:
//   k_ccl_tile   labels each tile on its own in LDS; the tile's roots (one per
//                drop and tile) go to a list, with their cells in cnt[root]
//   k_ccl_merge  joins labels across the faces between tiles
//   k_ccl_sum    adds each tile root's cells to its drop's root
//   k_ccl_drops  lists the roots that are left, with their cells
// Only cells on a tile's faces and roots have a label in memory: nothing else
// is read again.  So C is read once, the label array is written for 45 % of the
// cells and read for the faces between tiles, and the global union-find chains
// run over tile roots instead of cells.  256^3, 64 drops, FP32: 70 us for the
// four (37 + 21 + 5 + 5) against 440 us with labels for every cell (per-cell
// unions 300, flattening 47, counting 41, listing 20, start labels 29).
// What bounds it: the tile pass streams C, the merge pass waits on the latency
// of its label chains.
constexpr int CCL_TX = 64, CCL_TY = 8, CCL_TZ = 8;   // a tile row is one wave
constexpr int CCL_ROWS = CCL_TY * CCL_TZ;
constexpr int CCL_WROWS = CCL_ROWS / 4;              // rows of each of the group's four waves
constexpr int64_t CCL_MAX_WG = 1 << 20;              // groups of a launch at most (they loop)

// Labels that other threads may be changing: the loads go to the level where
// the atomics act (LDS of the work-group, or the device's coherent level).
template <int SCOPE>
__device__ __forceinline__ int ccl_load(const int* lab, int a)
{
    return __hip_atomic_load(lab + a, __ATOMIC_RELAXED, SCOPE);
}

template <int SCOPE>
__device__ __forceinline__ int ccl_find(const int* lab, int a)
{
    int b = ccl_load<SCOPE>(lab, a);
    while (b != a) {   // labels only decrease along the chain: it ends
        a = b;
        b = ccl_load<SCOPE>(lab, a);
    }
    return a;
}

template <int SCOPE>
__device__ __forceinline__ void ccl_union(int* lab, int a, int b)
{
    // each retry lowers max(a, b) strictly, so the loop ends
    for (;;) {
        a = ccl_find<SCOPE>(lab, a);
        b = ccl_find<SCOPE>(lab, b);
        if (a == b) return;
        if (a > b) {
            const int t = a;
            a = b;
            b = t;
        }
        const int old = __hip_atomic_fetch_min(lab + b, a, __ATOMIC_RELAXED, SCOPE);
        if (old == b) return;
        b = old;   // b had been linked meanwhile: join a with b's parent
    }
}

// One tile per work-group.  A row's drop cells are one wave's ballot, kept as
// a 64-bit mask, so the runs along x need no union.  The union-find works on
// runs: run k of a row that starts at bit b has the number row * 32 + b / 2
// (starts are at least two bits apart, and the numbers rise with the cells'
// linear indices).  Each thread takes a quarter of a row's bits, so all rows'
// unions go in parallel; two rows are joined once per stretch of bits they
// share.  A tile without drop cells only writes its faces.  meta[0] counts the
// tile roots of the box (also those past the list's end at cap).
template <typename T>
__global__ void __launch_bounds__(256)
k_ccl_tile(const T* __restrict__ C, int nx, int ny, int nz, T thr, int* __restrict__ lab,
           int* __restrict__ cnt, int* __restrict__ meta, int* __restrict__ list, int cap)
{
    typedef unsigned long long u64;
    __shared__ int L[CCL_ROWS * 32];  // labels of the runs
    __shared__ int S[CCL_ROWS * 32];  // cells, at the roots
    __shared__ u64 mask[CCL_ROWS];    // drop cells of each row
    __shared__ int nroot, base;
    const int tx = (nx + CCL_TX - 1) / CCL_TX, ty = (ny + CCL_TY - 1) / CCL_TY;
    const int ntile = tx * ty * ((nz + CCL_TZ - 1) / CCL_TZ);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    constexpr int WG = __HIP_MEMORY_SCOPE_WORKGROUP;
    static_assert(CCL_WROWS == 2 * CCL_TY && CCL_ROWS == 64, "a wave holds two planes of rows");
    // the run that holds bit b of row r with mask m
    auto run_of = [](int r, u64 m, int b) {
        const u64 gap = ~m & ((u64(1) << b) - 1);
        return r * 32 + (gap ? 64 - __clzll((long long)gap) : 0) / 2;
    };
    // this thread's row and bits in the passes over the runs
    const int row = threadIdx.x >> 2;
    const u64 quarter = u64(0xffff) << (16 * (threadIdx.x & 3));
    // f(b) at each set bit b of the thread's quarter
    auto each = [&](u64 bits, auto&& f) {
        for (bits &= quarter; bits; bits &= bits - 1) f(__ffsll((long long)bits) - 1);
    };
    for (int tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const int x0 = tile % tx * CCL_TX, y0 = tile / tx % ty * CCL_TY,
                  z0 = tile / tx / ty * CCL_TZ;
        const bool xin = x0 + lane < nx;
        const bool xface = lane == 0 || lane == CCL_TX - 1 || x0 + lane == nx - 1;
        // linear index of the first cell of the tile's row r (fewer than 2^31 cells)
        auto row_off = [&](int r) {
            return (uint32_t)(z0 + r / CCL_TY) * plane + (uint32_t)(y0 + r % CCL_TY) * nx + x0;
        };
        // the wave's rows: 16 wv + i
        const int rw = wv * CCL_WROWS;
        auto row_in = [&](int i) {
            return y0 + i % CCL_TY < ny && z0 + (rw + i) / CCL_TY < nz;
        };
        if (threadIdx.x == 0) nroot = 0;
        T v[CCL_WROWS];
#pragma unroll
        for (int i = 0; i < CCL_WROWS; ++i) {
            v[i] = T(0);
            if (row_in(i) && xin) v[i] = C[row_off(rw + i) + lane];
        }
        u64 m[CCL_WROWS];
        u64 any = 0;
#pragma unroll
        for (int i = 0; i < CCL_WROWS; ++i) {
            m[i] = __ballot(row_in(i) && xin && v[i] >= thr);
            any |= m[i];
            if (lane == 0) mask[rw + i] = m[i];
        }
        const bool drops = __syncthreads_or(any != 0);
        const u64 mr = drops ? mask[row] : 0, starts = mr & ~(mr << 1);
        if (drops) {
            each(starts, [&](int b) {
                L[row * 32 + b / 2] = row * 32 + b / 2;
                S[row * 32 + b / 2] = 0;
            });
            __syncthreads();
            if (row % CCL_TY > 0) {
                const u64 mn = mask[row - 1], both = mr & mn;
                each(both & ~(both << 1), [&](int b) {
                    ccl_union<WG>(L, run_of(row, mr, b), run_of(row - 1, mn, b));
                });
            }
            if (row >= CCL_TY) {
                const u64 mn = mask[row - CCL_TY], both = mr & mn;
                each(both & ~(both << 1), [&](int b) {
                    ccl_union<WG>(L, run_of(row, mr, b), run_of(row - CCL_TY, mn, b));
                });
            }
            __syncthreads();
            // each run's root, and the cells of the run added to it
            each(starts, [&](int b) {
                const u64 end = ~mr & ~((u64(2) << b) - 1);   // gaps above the start
                const int len = (end ? __ffsll((long long)end) - 1 : 64) - b;
                const int k = row * 32 + b / 2, root = ccl_find<WG>(L, k);
                __hip_atomic_store(L + k, root, __ATOMIC_RELAXED, WG);
                atomicAdd(S + root, len);
                if (root == k) atomicAdd(&nroot, 1);
            });
            __syncthreads();
            // room for the tile's roots in the list, claimed while the labels
            // are written
            if (threadIdx.x == 0) base = nroot > 0 ? atomicAdd(meta, nroot) : 0;
        }
        // labels of the faces' cells
#pragma unroll
        for (int i = 0; i < CCL_WROWS; ++i) {
            if (!row_in(i)) continue;
            const int y = y0 + i % CCL_TY, z = z0 + (rw + i) / CCL_TY;
            const bool rface = i % CCL_TY == 0 || i % CCL_TY == CCL_TY - 1 || y == ny - 1 ||
                               z == z0 || z == z0 + CCL_TZ - 1 || z == nz - 1;
            if (!xin || !(rface || xface)) continue;
            int label = -1;
            if ((m[i] >> lane) & 1) {
                const int root = L[run_of(rw + i, m[i], lane)], rr = root >> 5;
                const u64 mq = mask[rr];
                const int b = 2 * (root & 31);   // the root's run starts at b or b + 1
                label = (int)(row_off(rr) + b + (((mq & ~(mq << 1)) >> b) & 1 ? 0 : 1));
            }
            lab[row_off(rw + i) + lane] = label;
        }
        if (!drops) continue;
        __syncthreads();
        // the roots: label, cells, place in the list
        each(starts, [&](int b) {
            const int k = row * 32 + b / 2;
            if (L[k] != k) return;
            const int g = (int)(row_off(row) + b);
            lab[g] = g;
            cnt[g] = S[k];
            const int e = base + atomicAdd(&nroot, -1) - 1;
            if (e < cap) list[e] = g;
        });
        __syncthreads();   // the group's LDS is free for its next tile
    }
}

// Faces between tiles (work-groups [0, gx) the x faces, [gx, gx + gy) the y
// faces, the rest the z faces): a drop cell on a tile's low face is joined with
// its neighbour below the face (wrapping on periodic axes).  Neighbouring lanes
// hold neighbouring cells along the face; where the lane below joins the same
// two tiles through cells next to both of this lane's, the join is already
// made.
__global__ void __launch_bounds__(256)
k_ccl_merge(int* lab, int nx, int ny, int nz, int px, int py, int pz, int gx, int gy)
{
    constexpr int DEV = __HIP_MEMORY_SCOPE_AGENT;
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    const int blk = blockIdx.x;
    // cell a and its neighbour b (fewer than 2^31 cells); f: the lane's position
    // along the face (neighbouring lanes differ by one in it), with tile edges
    // every ft
    uint32_t a = 0, b = 0;
    int f = 0, ft = 1;
    bool on = false;
    if (blk < gx) {
        const uint32_t t = (uint32_t)blk * 256 + threadIdx.x;
        const uint32_t tx = (nx + CCL_TX - 1) / CCL_TX;
        const uint32_t q = t / ny, y = t - q * ny;
        const uint32_t z = q / tx, x = (q - z * tx) * CCL_TX;
        on = z < (uint32_t)nz && (x > 0 || px);
        a = z * plane + y * nx + x;
        b = x > 0 ? a - 1 : a + nx - 1;
        f = (int)y;
        ft = CCL_TY;
    } else {
        const bool yface = blk < gx + gy;
        const uint32_t t = (uint32_t)(blk - (yface ? gx : gx + gy)) * 256 + threadIdx.x;
        const uint32_t q = t / nx, x = t - q * nx;
        f = (int)x;
        ft = CCL_TX;
        if (yface) {
            const uint32_t tyn = (ny + CCL_TY - 1) / CCL_TY;
            const uint32_t z = q / tyn, y = (q - z * tyn) * CCL_TY;
            on = z < (uint32_t)nz && (y > 0 || py);
            a = z * plane + y * nx + x;
            b = y > 0 ? a - nx : a + (uint32_t)(ny - 1) * nx;
        } else {
            const uint32_t zt = q / ny, y = q - zt * ny, z = zt * CCL_TZ;
            on = z < (uint32_t)nz && (z > 0 || pz);
            a = z * plane + y * nx + x;
            b = z > 0 ? a - plane : a + (uint32_t)(nz - 1) * plane;
        }
    }
    // the labels' signs (drop or background) never change here: plain loads
    const bool both = on && lab[a] >= 0 && lab[b] >= 0;
    const unsigned long long m = __ballot(both);
    const int lane = threadIdx.x & 63;
    const bool done = lane > 0 && f % ft != 0 && ((m >> (lane - 1)) & 1);
    if (both && !done) ccl_union<DEV>(lab, (int)a, (int)b);
}

// The cells of every tile root that has been linked under another root go to
// that root (only final roots are added to).  Each thread shortens its own
// label's chain as it climbs (its label's label takes the label's place), so
// that the threads of one long drop climb in strides that double: with plain
// climbing a line of 10^6 cells in one drop, a chain of 15625 tile roots, took
// 220-440 us.
__global__ void __launch_bounds__(256)
k_ccl_sum(int* __restrict__ lab, int* __restrict__ cnt, const int* __restrict__ meta,
          const int* __restrict__ list, int cap)
{
    constexpr int DEV = __HIP_MEMORY_SCOPE_AGENT;
    const int n = meta[0] < cap ? meta[0] : cap;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const int r = list[e];
        int root = lab[r], up = lab[root];   // most chains end here
        // labels only decrease along the chain, and a label read while its
        // owner shortens it is an ancestor either way: it ends at the root
        while (up != root) {
            root = up;
            __hip_atomic_store(lab + r, root, __ATOMIC_RELAXED, DEV);
            up = ccl_load<DEV>(lab, root);
        }
        if (root != r) atomicAdd(cnt + root, cnt[r]);
    }
}

// Final roots and their cells (in no particular order) as pairs into out;
// meta[1] receives the number of drops.
__global__ void __launch_bounds__(256)
k_ccl_drops(const int* __restrict__ lab, const int* __restrict__ cnt, int* __restrict__ meta,
            const int* __restrict__ list, int cap, int* __restrict__ out)
{
    const int n = meta[0] < cap ? meta[0] : cap;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const int r = list[e];
        if (lab[r] == r) {
            const int k = atomicAdd(meta + 1, 1);
            out[2 * k] = r;
            out[2 * k + 1] = cnt[r];
        }
    }
}

// Split-density pressure step (sec. 3.2: eq-split, eq-newpoi, eq-u) on the
// staggered mesh: P and C at the cells, u / v / w on the low faces of the
// cells (w has nz + 1 planes between walls, zero on both).  The density is
// rho2 + (rho1 - rho2) clamp(C, 0, 1); a face takes the mean of its two
// cells, and 1/rho on a face is the refined hardware reciprocal (fast_rcp).
template <typename T>
__device__ __forceinline__ T press_rho(const PressArgs& a, T c)
{
    const T cc = c < T(0) ? T(0) : (c > T(1) ? T(1) : c);
    return T(a.rho2) + T(a.rho1 - a.rho2) * cc;
}

// Phat = 2 P - Pold, then Pold <- P (the next step's history).
template <typename T>
__global__ void __launch_bounds__(256)
k_press_prep(const T* __restrict__ P, T* __restrict__ Pold, T* __restrict__ phat, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const T p = P[i];
        phat[i] = T(2) * p - Pold[i];
        Pold[i] = p;
    }
}

// The cell kernels of the pressure step take tiles of tx (2^lx) x-columns by ty
// rows and march each column up tz planes, carrying the plane below in
// registers, so no plane is fetched twice for its z neighbours.  Planes are
// addressed through 32-bit byte offsets from a per-plane base (a plane is
// under 4 GiB).  Work-groups of rhs_threads and UPD_THREADS.
struct PressTile {
    int lx, tx, ty, tz;
};
template <typename T>
constexpr int rhs_threads() { return sizeof(T) == 8 ? 256 : 512; }
constexpr int UPD_THREADS = 256;

__host__ __device__ __forceinline__ int64_t press_tiles(PressTile p, int nx, int ny, int nz)
{
    return (int64_t)((nx + p.tx - 1) / p.tx) * ((ny + p.ty - 1) / p.ty) * ((nz + p.tz - 1) / p.tz);
}

// Tile of a work-group of `threads`: of the widths `widest` down to 64 (FP64) or
// 128 columns (FP32: 512 bytes a row; 256 bytes cost more in lines fetched twice
// than they save in padding, 180 x 240 x 100: the step 195 us against 184) the
// one that pads a row of nx least, the widest of equals, and marches of up to
// `longest` planes, halved down to `shortest` while there are under 2048 tiles
// (eight groups per CU).  Against 256 columns and the longest march everywhere (us
// per pressure step): 300^3 FP32 1057 -> 909, FP64 1669 -> 1477, 320 x 200 x 150
// FP32 357 -> 326, 64^3 FP64 92 -> 76, 90 x 300 x 40 FP64 148 -> 131; 512^3 FP32,
// where nothing changes, 3922 / 3913.
template <typename T>
inline PressTile press_tile(int threads, int widest, int longest, int shortest, int nx, int ny,
                            int nz)
{
    PressTile p{0, widest, threads / widest, longest};
    for (int w = widest; w >= (sizeof(T) == 8 ? 64 : 128); w /= 2)
        if ((nx + w - 1) / w * w < (nx + p.tx - 1) / p.tx * p.tx) p.tx = w;
    p.ty = threads / p.tx;
    while ((1 << p.lx) < p.tx) ++p.lx;
    while (p.tz / 2 >= shortest && press_tiles(p, nx, ny, nz) < 2048) p.tz /= 2;
    return p;
}

// Column of thread t in task `task`: x, y and the march z0 .. z1 - 1; false
// for a thread past the mesh.
__device__ __forceinline__ bool press_column(PressTile p, int64_t task, int t, int nx, int ny,
                                             int nz, int* x, int* y, int* z0, int* z1)
{
    const int tx = (nx + p.tx - 1) / p.tx, ty = (ny + p.ty - 1) / p.ty;
    const int bx = (int)(task % tx);
    const int64_t rest = task / tx;
    const int by = (int)(rest % ty), bz = (int)(rest / ty);
    *x = bx * p.tx + (t & (p.tx - 1));
    *y = by * p.ty + (t >> p.lx);
    *z0 = bz * p.tz;
    *z1 = *z0 + p.tz < nz ? *z0 + p.tz : nz;
    return *x < nx && *y < ny;
}

// Right-hand side of eq-newpoi at every cell:
// div[(1 - rho2/rho_f) grad Phat] + (rho2/dt) div u*.
template <typename T>
__global__ void __launch_bounds__(rhs_threads<T>())
k_press_rhs(PressTile tile, PressArgs a, const T* __restrict__ C, const T* __restrict__ ph,
            const T* __restrict__ u, const T* __restrict__ v, const T* __restrict__ w,
            T* __restrict__ rhs)
{
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t plane = (int64_t)nx * ny;
    constexpr uint32_t sT = sizeof(T);
    const uint32_t pbytes = (uint32_t)(plane * sT);
    const T ih = T(1.0 / a.h), r2 = T(a.rho2), sdiv = T(a.rho2 / a.dt);
    auto at = [&](const T* f, int z) { return chd::PlaneRef<T>(f + (int64_t)z * plane, pbytes); };
    const int64_t ntask = press_tiles(tile, nx, ny, nz);
    for (int64_t task = blockIdx.x; task < ntask; task += gridDim.x) {
        int x, y, z0, z1;
        if (!press_column(tile, task, (int)threadIdx.x, nx, ny, nz, &x, &y, &z0, &z1)) continue;
        const int xm = x > 0 ? x - 1 : nx - 1, xp = x + 1 < nx ? x + 1 : 0;
        const int ym = y > 0 ? y - 1 : ny - 1, yp = y + 1 < ny ? y + 1 : 0;
        const uint32_t oc = (uint32_t)(y * nx + x) * sT, oxm = (uint32_t)(y * nx + xm) * sT,
                       oxp = (uint32_t)(y * nx + xp) * sT, oym = (uint32_t)(ym * nx + x) * sT,
                       oyp = (uint32_t)(yp * nx + x) * sT;
        // rho and Phat of the column below the march (periodic wrap; not used
        // at the bottom wall) and at its first plane, and w on its low face
        T rlo = T(0), plo = T(0);
        if (z0 > 0 || !a.zwalls) {
            const int zb = z0 > 0 ? z0 - 1 : nz - 1;
            rlo = press_rho(a, at(C, zb)(oc));
            plo = at(ph, zb)(oc);
        }
        T rc = press_rho(a, at(C, z0)(oc)), pc = at(ph, z0)(oc);
        T wlo = at(w, z0)(oc);
        for (int z = z0; z < z1; ++z) {
            const int zp = z + 1 < nz ? z + 1 : 0;
            const bool up = !a.zwalls || z + 1 < nz;
            T rhi = T(0), phi = T(0);
            if (up) {
                rhi = press_rho(a, at(C, zp)(oc));
                phi = at(ph, zp)(oc);
            }
            const T whi = at(w, a.zwalls ? z + 1 : zp)(oc);
            const chd::PlaneRef<T> Cz = at(C, z), Pz = at(ph, z), Uz = at(u, z), Vz = at(v, z);
            // flux through the face between the cell and a neighbour (on the +
            // side when s = 1): (1 - rho2/rho_f) (Phat[hi] - Phat[lo]) / h
            auto flux = [&](T rn, T pn, int s) {
                const T rf = T(0.5) * (rc + rn);
                const T g = s > 0 ? pn - pc : pc - pn;
                return (T(1) - r2 * chd::fast_rcp(rf)) * g * ih;
            };
            T d = flux(press_rho(a, Cz(oxp)), Pz(oxp), 1) - flux(press_rho(a, Cz(oxm)), Pz(oxm), -1)
                + flux(press_rho(a, Cz(oyp)), Pz(oyp), 1) - flux(press_rho(a, Cz(oym)), Pz(oym), -1);
            if (up) d += flux(rhi, phi, 1);
            if (!a.zwalls || z > 0) d -= flux(rlo, plo, -1);
            const T du = Uz(oxp) - Uz(oc);
            const T dv = Vz(oyp) - Vz(oc);
            const T dw = whi - wlo;
            at(rhs, z).store(oc, d * ih + sdiv * (du + dv + dw) * ih);
            rlo = rc;
            plo = pc;
            rc = rhi;
            pc = phi;
            wlo = whi;
        }
    }
}

// Solve along z per (ky, kx) mode after the 2-D transforms in x and y
// (between walls): (1/h^2)(p[k+1] - 2 p[k] + p[k-1]) + lxy p[k] = f[k] with
// p[-1] = p[0], p[nz] = p[nz-1] (dP/dz = 0).  The rows are diagonally
// dominant for lxy < 0 and are eliminated from both ends at once: lane l
// (l < 32) of a wave takes mode g*32 + l from row 0 up to row M - 1 (M = nz/2),
// lane l + 32 the same mode from row nz - 1 down to M + 1; row M then
// couples the two eliminated halves,
//   (b_M - c_{M-1}/h^2 - e_{M+1}/h^2) p_M = f_M - (d_{M-1} + g_{M+1})/h^2,
// and each lane substitutes back over its half.  This halves the serial chain
// and doubles the threads of the plain Thomas sweep.  Spectra are [nz][ny][nxp]
// complex (re, im interleaved, nxp >= nx/2 + 1); cp holds nz x ny x nxp reals of
// scratch, of which one per block of PK rows is used.  The result is scaled by
// `scale` (the inverse transform's 1 / (nx ny)).
//
// What bounds it: each wave's chain of blocks of PK rows, so the next block's
// loads go out before this block's rows are eliminated; on large planes the
// bytes.  The mean mode is one serial chain over all of z, its loads behind its
// stores; it has a work-group of its own (press_mean) that stages z through LDS.
// 512^3 FP32: 433 us against 677-706 with the mean mode in a lane of a wave and
// each block's loads after the one before (the spectrum read and written twice at
// a copy's rate: 440), FP64 983 against 1183.  Two forms, one arithmetic: LONG
// forms the rows' addresses in 64 bits (236 VGPRs in single, 179 in double
// precision, 2 waves per SIMD); the other counts elements in 32 bits (127 and
// 117, 4 waves), which planes of many modes and few rows need (launch_press_solve).
template <typename T>
struct Cplx;
template <>
struct Cplx<float> {
    typedef float2 V;
};
template <>
struct Cplx<double> {
    typedef double2 V;
};

// The mean mode (lxy = 0) of that solve is singular: its mean over z is removed
// from f, then p[0] = 0 and the rows 0 .. nz-2 give p[1 .. nz-1] by
// p[k+1] = 2 p[k] - p[k-1] + h^2 f[k] (p[-1] = p[0]), and the mean of p is
// removed.  One work-group: z goes through LDS in chunks of MEAN_CHUNK rows,
// thread 0 runs the real parts and thread 1 the imaginary ones.
constexpr int MEAN_CHUNK = 1024;

template <typename T>
__device__ void press_mean(T* __restrict__ fs, int64_t s2, int nz, T h2, T sc)
{
    __shared__ T sh[2][MEAN_CHUNK];
    __shared__ T mean[2];
    const int tid = threadIdx.x, nt = blockDim.x;
    // f (p) of the chunk's rows into (out of) LDS
    auto load = [&](int k0, int n) {
        __syncthreads();
        for (int e = tid; e < 2 * n; e += nt) sh[e & 1][e >> 1] = fs[(k0 + (e >> 1)) * s2 + (e & 1)];
        __syncthreads();
    };
    constexpr int B = 8;   // rows read ahead of the chain
    T acc = T(0);
    for (int k0 = 0; k0 < nz; k0 += MEAN_CHUNK) {
        const int n = nz - k0 < MEAN_CHUNK ? nz - k0 : MEAN_CHUNK;
        load(k0, n);
        if (tid < 2) {
            int k = 0;
            for (; k + B <= n; k += B) {
                T v[B];
#pragma unroll
                for (int q = 0; q < B; ++q) v[q] = sh[tid][k + q];
#pragma unroll
                for (int q = 0; q < B; ++q) acc += v[q];
            }
            for (; k < n; ++k) acc += sh[tid][k];
        }
    }
    const T m = acc / T(nz);
    T pr = T(0), qr = T(0), sr = T(0);   // p[k-1], p[k], sum of p
    for (int k0 = 0; k0 < nz; k0 += MEAN_CHUNK) {
        const int n = nz - k0 < MEAN_CHUNK ? nz - k0 : MEAN_CHUNK;
        load(k0, n);
        if (tid < 2) {
            auto row = [&](int k, T f) {
                const T fr = f - m;
                sh[tid][k] = qr;
                sr += qr;
                const T lr = k0 + k == 0 ? qr : pr;
                const T nr = T(2) * qr - lr + h2 * fr;
                pr = qr;
                qr = nr;
            };
            int k = 0;
            for (; k + B <= n; k += B) {
                T v[B];
#pragma unroll
                for (int q = 0; q < B; ++q) v[q] = sh[tid][k + q];
#pragma unroll
                for (int q = 0; q < B; ++q) row(k + q, v[q]);
            }
            for (; k < n; ++k) row(k, sh[tid][k]);
            if (k0 + n == nz) mean[tid] = sr / T(nz);
        }
        __syncthreads();
        for (int e = tid; e < 2 * n; e += nt) fs[(k0 + (e >> 1)) * s2 + (e & 1)] = sh[e & 1][e >> 1];
    }
    __syncthreads();
    for (int64_t e = tid; e < 2 * (int64_t)nz; e += nt) {
        T* p = fs + (e >> 1) * s2 + (e & 1);
        *p = (*p - mean[e & 1]) * sc;
    }
}

template <typename T, bool LONG>
__global__ void __launch_bounds__(256, LONG ? 1 : 4)
k_press_tri(T* __restrict__ spec, T* __restrict__ cp, int nx, int ny, int nz, int nxp, double h,
            double scale)
{
    typedef typename Cplx<T>::V V;
    const int nxh = nx / 2 + 1;
    const int64_t nm = (int64_t)ny * nxp;           // complex elements between planes
    const T sc = T(scale);
    if (blockIdx.x == 0) {
        press_mean<T>(spec, 2 * nm, nz, T(h * h), sc);
        return;
    }
    const int nmi = (int)nm;                        // (fewer than 2^31 elements in all)
    const int ngroups = (nmi + 31) / 32;
    const double PI = 3.14159265358979323846;
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5;
    const int M = nz / 2;
    const int len = half == 0 ? M : nz - 1 - M;     // rows eliminated by this lane
    const int lmin = nz - 1 - M;                    // ... by the lane with fewer (M or M - 1)
    const T ih2 = T(1.0 / (h * h));
    constexpr int PK = sizeof(T) == 4 ? 8 : 4;      // rows per block
    const int wave0 = (int)((blockIdx.x - 1) * (blockDim.x >> 6) + (threadIdx.x >> 6));
    const int nwaves = (int)((gridDim.x - 1) * (blockDim.x >> 6));
    // the group loop is uniform over a wave: every lane reaches the exchange
    for (int g = wave0; g < ngroups; g += nwaves) {
        const uint32_t m = (uint32_t)g * 32 + (lane & 31);
        const int j = (int)(m / (uint32_t)nxp), i = (int)(m - (uint32_t)j * nxp);
        const bool on = m < (uint32_t)nmi && i < nxh && m != 0;   // m = 0 is the mean mode
        const int mm = on ? (int)m : 0;
        const double sx = sin(PI * i / nx), sy = sin(PI * j / ny);
        const T lxy = T(-4.0 / (h * h) * (sx * sx + sy * sy));
        // row s of the lane's half in spec and cp: LONG, at strides of its own from
        // the half's end; else by 32-bit element numbers, with half the registers
        const int64_t st = half == 0 ? nm : -nm;
        const int e0 = mm + (half == 0 ? 0 : (nz - 1) * nmi), de = half == 0 ? nmi : -nmi;
        V* const f = reinterpret_cast<V*>(spec);
        V* const fl = f + mm + (half == 0 ? 0 : (nz - 1) * nm);
        T* const cl = cp + mm + (half == 0 ? 0 : (nz - 1) * nm);
        auto fat = [&](int s) -> V& { return LONG ? fl[s * st] : f[(uint32_t)(e0 + s * de)]; };
        auto cat = [&](int s) -> T& { return LONG ? cl[s * st] : cp[(uint32_t)(e0 + s * de)]; };
        auto diag = [&](int s) { return lxy - (s == 0 ? ih2 : T(2) * ih2); };   // a half's row s
        // a block's rows (past the half's end its last row again)
        auto load = [&](int s0, V* v) {
            if (LONG && s0 + PK <= lmin) {
                const V* p = fl + s0 * st;
#pragma unroll
                for (int q = 0; q < PK; ++q) v[q] = p[q * st];
            } else {
#pragma unroll
                for (int q = 0; q < PK; ++q) v[q] = fat(s0 + q < len ? s0 + q : len - 1);
            }
        };
        // elimination towards row M in blocks of PK rows: d into f, and into
        // cp at each block's first row the c entering the block (the block's
        // c are formed again from it on the way back)
        T c = T(0), dr = T(0), di = T(0);
        if (on && len > 0) {
            V nv[PK];
            load(0, nv);
            for (int s0 = 0; s0 < len; s0 += PK) {
                cat(s0) = c;
                V fv[PK];
#pragma unroll
                for (int q = 0; q < PK; ++q) fv[q] = nv[q];
                if (s0 + PK < len) load(s0 + PK, nv);
#pragma unroll
                for (int q = 0; q < PK; ++q) {
                    const int sq = s0 + q;
                    if (sq >= len) break;
                    const T den = diag(sq) - ih2 * c;
                    c = ih2 / den;
                    dr = (fv[q].x - ih2 * dr) / den;
                    di = (fv[q].y - ih2 * di) / den;
                    V o;
                    o.x = dr;
                    o.y = di;
                    fat(sq) = o;
                }
            }
        }
        // row M, read by the lower lane only, and the other half's last
        // coefficients (zero for an empty half), across the wave
        T fmr = T(0), fmi = T(0);
        if (on && half == 0) {
            const V v = f[mm + M * nmi];
            fmr = v.x;
            fmi = v.y;
        }
        const T oc = __shfl_xor(c, 32), odr = __shfl_xor(dr, 32), odi = __shfl_xor(di, 32);
        const T ofr = __shfl_xor(fmr, 32), ofi = __shfl_xor(fmi, 32);
        if (on) {
            if (half == 1) {
                fmr = ofr;
                fmi = ofi;
            }
            const T dM = lxy - (M == nz - 1 ? ih2 : T(2) * ih2);   // (M > 0 always)
            const T den = dM - ih2 * (c + oc);
            T xr = (fmr - ih2 * (dr + odr)) / den;
            T xi = (fmi - ih2 * (di + odi)) / den;
            if (half == 0) {
                V o;
                o.x = xr * sc;
                o.y = xi * sc;
                f[mm + M * nmi] = o;
            }
            // back substitution from row M outwards, block by block: the
            // block's c again from its checkpoint (the same operations as on
            // the way up, so the same values), then its rows in reverse
            if (len > 0) {
                V nv[PK];
                int s0 = (len - 1) / PK * PK;
                load(s0, nv);
                T cnext = cat(s0);
                for (; s0 >= 0; s0 -= PK) {
                    V fv[PK];
                    T cc[PK];
                    T cin = cnext;
#pragma unroll
                    for (int q = 0; q < PK; ++q) fv[q] = nv[q];
                    if (s0 >= PK) {
                        load(s0 - PK, nv);
                        cnext = cat(s0 - PK);
                    }
#pragma unroll
                    for (int q = 0; q < PK; ++q) {
                        cc[q] = T(0);
                        if (s0 + q >= len) break;
                        const T dn = diag(s0 + q) - ih2 * cin;
                        cin = ih2 / dn;
                        cc[q] = cin;
                    }
#pragma unroll
                    for (int q = PK - 1; q >= 0; --q) {
                        const int sq = s0 + q;
                        if (sq >= len) continue;
                        xr = fv[q].x - cc[q] * xr;
                        xi = fv[q].y - cc[q] * xi;
                        V o;
                        o.x = xr * sc;
                        o.y = xi * sc;
                        fat(sq) = o;
                    }
                }
            }
        }
    }
}

// sin(pi i / n), i < count: the eigenvalue tables of the periodic solve, made
// once per mesh.
__global__ void __launch_bounds__(256) k_press_sines(double* __restrict__ out, int n, int count)
{
    const double PI = 3.14159265358979323846;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) out[i] = sin(PI * i / n);
}

// Periodic z: divide the 3-D spectrum [nz][ny][nxp] by the eigenvalue of the
// 7-point Laplacian, zero mode to 0, scaled by 1 / (nx ny nz).  The sines come
// from the tables tx, ty, tz: with three double-precision sines per element the
// pass was compute-bound (240 x 180 x 160 FP64: 21 us now, 40 then).
template <typename T>
__global__ void __launch_bounds__(256)
k_press_div(T* __restrict__ spec, int nx, int ny, int nz, int nxp, double h, double scale,
            const double* __restrict__ tx, const double* __restrict__ ty,
            const double* __restrict__ tz)
{
    typedef typename Cplx<T>::V V;
    const uint32_t nxh = nx / 2 + 1;
    const uint32_t n = (uint32_t)nz * ny * nxh;   // fewer than 2^31 cells
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x) {
        const uint32_t r = e / nxh, i = e - r * nxh, k = r / ny, j = r - k * ny;
        const double sx = tx[i], sy = ty[j], sz = tz[k];
        const double lam = -4.0 / (h * h) * (sx * sx + sy * sy + sz * sz);
        const T f = (e == 0) ? T(0) : T(scale / lam);
        V* p = reinterpret_cast<V*>(spec) + ((int64_t)r * nxp + i);
        V v = *p;
        v.x *= f;
        v.y *= f;
        *p = v;
    }
}

// eq-u on the low faces of every cell (the wall faces of z stay as they are),
// z-marching tiles as for the right-hand side.
template <typename T>
__global__ void __launch_bounds__(UPD_THREADS)
k_press_update(PressTile tile, PressArgs a, const T* __restrict__ C, const T* __restrict__ P,
               const T* __restrict__ ph, T* __restrict__ u, T* __restrict__ v, T* __restrict__ w)
{
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t plane = (int64_t)nx * ny;
    constexpr uint32_t sT = sizeof(T);
    const uint32_t pbytes = (uint32_t)(plane * sT);
    const T ih = T(1.0 / a.h), ir2 = T(1.0 / a.rho2), dt = T(a.dt);
    auto at = [&](const T* f, int z) { return chd::PlaneRef<T>(f + (int64_t)z * plane, pbytes); };
    const int64_t ntask = press_tiles(tile, nx, ny, nz);
    for (int64_t task = blockIdx.x; task < ntask; task += gridDim.x) {
        int x, y, z0, z1;
        if (!press_column(tile, task, (int)threadIdx.x, nx, ny, nz, &x, &y, &z0, &z1)) continue;
        const int xm = x > 0 ? x - 1 : nx - 1, ym = y > 0 ? y - 1 : ny - 1;
        const uint32_t oc = (uint32_t)(y * nx + x) * sT, oxm = (uint32_t)(y * nx + xm) * sT,
                       oym = (uint32_t)(ym * nx + x) * sT;
        // rho, P and Phat of the column below the march (periodic wrap; not
        // used at the bottom wall)
        T rlo = T(0), qlo = T(0), hlo = T(0);
        if (z0 > 0 || !a.zwalls) {
            const int zb = z0 > 0 ? z0 - 1 : nz - 1;
            rlo = press_rho(a, at(C, zb)(oc));
            qlo = at(P, zb)(oc);
            hlo = at(ph, zb)(oc);
        }
        for (int z = z0; z < z1; ++z) {
            const chd::PlaneRef<T> Cz = at(C, z), Pz = at(P, z), Hz = at(ph, z);
            const T rc = press_rho(a, Cz(oc)), pc = Pz(oc), hc = Hz(oc);
            auto corr = [&](T rn, T qn, T hn) {   // face between a low neighbour and the cell
                const T rf = T(0.5) * (rc + rn);
                return dt * ((pc - qn) * ih * ir2 + (chd::fast_rcp(rf) - ir2) * (hc - hn) * ih);
            };
            const chd::PlaneRef<T> Uz = at(u, z), Vz = at(v, z), Wz = at(w, z);
            Uz.store(oc, Uz(oc) - corr(press_rho(a, Cz(oxm)), Pz(oxm), Hz(oxm)));
            Vz.store(oc, Vz(oc) - corr(press_rho(a, Cz(oym)), Pz(oym), Hz(oym)));
            if (!a.zwalls || z > 0) Wz.store(oc, Wz(oc) - corr(rlo, qlo, hlo));
            rlo = rc;
            qlo = pc;
            hlo = hc;
        }
    }
}

// ---------------------------------------------------------------------------
// host-side launchers (declared in ch_kernels.h)
// ---------------------------------------------------------------------------
template <typename T, typename A, int MI, int NT, bool E25>
static hipError_t launch_x(int nwg, int nth, size_t lds, hipStream_t st, const chd::BoxDesc* boxes,
                           int nbox, const chd::PassArgs& pa, const void* C, const void* U,
                           const void* V, const void* W, void* E, void* Q)
{
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)&k_pass_x<T, A, MI, NT, E25>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_pass_x<T, A, MI, NT, E25>), dim3(nwg), dim3(nth), lds, st, boxes, nbox, pa,
                       (const T*)C, (const T*)U, (const T*)V, (const T*)W, (T*)E, (T*)Q);
    return hipGetLastError();
}

template <typename T, typename A, bool E25>
static hipError_t launch_x_mode(int mi, int nwg, int nth, size_t lds, hipStream_t st,
                                const chd::BoxDesc* boxes, int nbox, const chd::PassArgs& pa,
                                const void* C, const void* U, const void* V, const void* W,
                                void* E, void* Q)
{
    if (mi == 1 && nth <= 512)
        return launch_x<T, A, 1, 512, E25>(nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W, E, Q);
    if (mi == 1)
        return launch_x<T, A, 1, 1024, E25>(nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W, E, Q);
    if (nth <= 768)
        return launch_x<T, A, 2, 768, E25>(nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W, E, Q);
    return launch_x<T, A, 2, 1024, E25>(nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W, E, Q);
}

template <typename T, typename A, int NT, int RM>
static hipError_t launch_x_row(int nwg, int nth, size_t lds, hipStream_t st,
                               const chd::BoxDesc* boxes, int nbox, const chd::PassArgs& pa,
                               const void* C, const void* U, const void* V, const void* W,
                               void* E, void* Q)
{
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)&k_pass_x_row<T, A, NT, RM>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_pass_x_row<T, A, NT, RM>), dim3(nwg), dim3(nth), lds, st, boxes, nbox,
                       pa, (const T*)C, (const T*)U, (const T*)V, (const T*)W, (T*)E, (T*)Q);
    return hipGetLastError();
}

template <typename T, typename A, int RM>
static hipError_t launch_x_row_nt(int nwg, int nth, size_t lds, hipStream_t st,
                                  const chd::BoxDesc* boxes, int nbox, const chd::PassArgs& pa,
                                  const void* C, const void* U, const void* V, const void* W,
                                  void* E, void* Q)
{
    if (nth <= 256)
        return launch_x_row<T, A, 256, RM>(nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W, E, Q);
    if (nth <= 512)
        return launch_x_row<T, A, 512, RM>(nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W, E, Q);
    return launch_x_row<T, A, 1024, RM>(nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W, E, Q);
}

template <typename T, typename A>
hipError_t launch_pass_x(int mi, int nwg, int nth, size_t lds, hipStream_t st,
                         const chd::BoxDesc* boxes, int nbox, const chd::PassArgs& pa,
                         const void* C, const void* U, const void* V, const void* W, void* E,
                         void* Q, bool e25, bool xrow, int xrm)
{
    if (xrow && !e25 && mi == 1) {
        if (xrm == chd::XR_WAVE)
            return launch_x_row_nt<T, A, chd::XR_WAVE>(nwg, nth, lds, st, boxes, nbox, pa, C, U,
                                                       V, W, E, Q);
        if (xrm == chd::XR_THREAD)
            return launch_x_row_nt<T, A, chd::XR_THREAD>(nwg, nth, lds, st, boxes, nbox, pa, C,
                                                         U, V, W, E, Q);
        return launch_x_row_nt<T, A, chd::XR_ONE>(nwg, nth, lds, st, boxes, nbox, pa, C, U, V,
                                                  W, E, Q);
    }
    if constexpr (std::is_same<T, A>::value) {
        if (e25)
            return launch_x_mode<T, A, true>(mi, nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W,
                                             E, Q);
    } else {
        if (e25) return hipErrorInvalidValue;   // the explicit mode has no solve precision
    }
    return launch_x_mode<T, A, false>(mi, nwg, nth, lds, st, boxes, nbox, pa, C, U, V, W, E, Q);
}

template <typename T, typename A>
hipError_t launch_pass_x_seg(int nwg, int nth, size_t lds, hipStream_t st,
                             const chd::BoxDesc* boxes, int nbox, const chd::PassArgs& pa,
                             const void* C, const void* U, const void* V, const void* W,
                             const void* Ein, void* Eout, void* Q)
{
    if (nth > 256) return hipErrorInvalidValue;
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)&k_pass_x_seg<T, A>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_pass_x_seg<T, A>), dim3(nwg), dim3(nth), lds, st, boxes, nbox, pa,
                       (const T*)C, (const T*)U, (const T*)V, (const T*)W, (const T*)Ein, (T*)Eout,
                       (T*)Q);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_pass_x_e25(int nwg, int nth, size_t lds, hipStream_t st,
                             const chd::BoxDesc* boxes, const chd::PassArgs& pa, const void* C,
                             const void* U, const void* V, const void* W, void* E, void* Q)
{
    auto go = [&](auto nt) {
        hipLaunchKernelGGL((k_pass_x_e25<T, decltype(nt)::value>), dim3(nwg), dim3(nth), lds, st,
                           boxes, pa, (const T*)C, (const T*)U, (const T*)V, (const T*)W, (T*)E,
                           (T*)Q);
        return hipGetLastError();
    };
    if (nth <= 256) return go(chd::IC<256>{});
    if (nth <= 512) return go(chd::IC<512>{});
    return go(chd::IC<1024>{});
}

template <typename T, typename A>
hipError_t launch_pass_line(int pass, int nwg, int nthreads, size_t lds, hipStream_t st,
                            const chd::BoxDesc* boxes, int nbox, const chd::PassArgs& pa,
                            const void* Qin, void* Qout, bool split)
{
    const auto fn = pass == chd::PASS_Y
        ? (split ? k_pass_line<T, A, chd::PASS_Y, 1> : k_pass_line<T, A, chd::PASS_Y, 0>)
        : (split ? k_pass_line<T, A, chd::PASS_Z, 1> : k_pass_line<T, A, chd::PASS_Z, 0>);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)fn,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fn, dim3(nwg), dim3(nthreads), lds, st, boxes, nbox, pa, (const T*)Qin,
                       (T*)Qout);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_mass(int nblk, int nbox, hipStream_t st, const chd::BoxDesc* boxes,
                       const void* C, double* partial, const double* h3, double* out)
{
    hipLaunchKernelGGL((k_mass_partial<T>), dim3(nblk), dim3(chd::MASS_THREADS), 0, st, boxes,
                       nbox, (const T*)C, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mass_final, dim3(nbox), dim3(chd::MASS_THREADS), 0, st, boxes, partial,
                       h3, out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_mass_one(hipStream_t st, const chd::BoxDesc& bd, const void* C,
                           double* partial, double h3, double* out)
{
    hipLaunchKernelGGL((k_mass_partial_one<T>), dim3(bd.nmblk), dim3(chd::MASS_THREADS), 0, st,
                       bd, (const T*)C, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mass_final_one, dim3(1), dim3(chd::MASS_THREADS), 0, st, bd.nmblk,
                       (const double*)partial, h3, out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_check_velocity(hipStream_t st, const chd::BoxDesc* boxes, int nbox,
                                 const void* U, const void* V, const void* W, int* flags)
{
    hipLaunchKernelGGL((k_check_velocity<T>), dim3(CHECK_WGS), dim3(256), 0, st, boxes, nbox,
                       (const T*)U, (const T*)V, (const T*)W, flags);
    return hipGetLastError();
}

template <typename T, int JB, int MA, bool PIPE>
static hipError_t launch_interp_k(hipStream_t st, const InterpArgs& a)
{
    if (a.lds > 65536) {
        hipError_t e = hipFuncSetAttribute((const void*)&k_interp<T, JB, MA, PIPE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)a.lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_interp<T, JB, MA, PIPE>), dim3((unsigned)a.nwg), dim3(256), a.lds, st,
                       a, (const T*)a.src, (T*)a.dst, a.band, a.iz, (const T*)a.wz, a.ly,
                       (const T*)a.wy, a.ix, a.wx);
    return hipGetLastError();
}

template <typename T, int JB>
static hipError_t launch_interp_jb(hipStream_t st, const InterpArgs& a)
{
    constexpr int MA = chp::interp_rows_ahead(sizeof(T));
    if (chp::interp_piped(sizeof(T), a.rmax, a.sx)) return launch_interp_k<T, JB, MA, true>(st, a);
    return launch_interp_k<T, JB, MA, false>(st, a);
}

template <typename T>
hipError_t launch_interp(hipStream_t st, const InterpArgs& a, const MarchArgs& m)
{
    if (m.rm) {
        const dim3 grid((unsigned)(m.nband * m.nchunk));
        const size_t lds = (size_t)2 * MARCH_ROWS * m.nsub * a.sx * sizeof(T);
        auto go = [&](auto rm, auto xp, auto yp) {
            hipLaunchKernelGGL((k_interp_march<T, decltype(rm)::value, decltype(xp)::value,
                                               decltype(yp)::value>),
                               grid, dim3(256), lds, st, a, m, (const T*)a.src, (T*)a.dst, m.iy0, a.iz,
                               (const T*)a.wz, (const T*)a.wy, a.ix, a.wx);
            return hipGetLastError();
        };
        using chd::IC;
        constexpr IC<MARCH_ANY> any{};
        constexpr IC<MARCH_FACE> face{};
        constexpr IC<MARCH_CENTRE> centre{};
        if (m.xp == MARCH_FACE && m.yp == MARCH_CENTRE) return go(IC<8>{}, face, centre);
        if (m.xp == MARCH_CENTRE && m.yp == MARCH_FACE) return go(IC<7>{}, centre, face);
        if (m.xp == MARCH_CENTRE && m.yp == MARCH_CENTRE) return go(IC<8>{}, centre, centre);
        if (m.rm == 8) return go(IC<8>{}, any, any);
        if (m.rm == 11) return go(IC<11>{}, any, any);
        return hipErrorInvalidValue;
    }
    switch (a.jb) {
    case 32: return launch_interp_jb<T, 32>(st, a);
    case 16: return launch_interp_jb<T, 16>(st, a);
    case 8: return launch_interp_jb<T, 8>(st, a);
    case 4: return launch_interp_jb<T, 4>(st, a);
    case 2: return launch_interp_jb<T, 2>(st, a);
    case 1: return launch_interp_jb<T, 1>(st, a);
    default: return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_grad(hipStream_t st, const void* src, int comp, int sx, int sy, int sz,
                       const double* dzinv, void* out)
{
    const int64_t rows = (int64_t)sy * sz;
    const int64_t nwg = rows < 262144 ? rows : 262144;
    hipLaunchKernelGGL((k_grad<T>), dim3((unsigned)nwg), dim3(256), 0, st, (const T*)src, comp,
                       sx, sy, sz, dzinv, (T*)out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_scan(hipStream_t st, int dir, void* buf, const void* ref, int nx, int ny,
                       int nz, double h, double* part)
{
    const int nwg = scan_groups(dir, nx, ny, nz);
    if (dir == 0)
        hipLaunchKernelGGL((k_scan_x<T>), dim3(nwg), dim3(256), 0, st, (T*)buf, (const T*)ref,
                           nx, (int64_t)ny * nz, T(h), part);
    else if (dir == 1)
        hipLaunchKernelGGL((k_scan_y<T>), dim3(nwg), dim3(256), 0, st, (T*)buf, (const T*)ref,
                           nx, ny, nz, T(h), part);
    else
        hipLaunchKernelGGL((k_scan_z<T>), dim3(nwg), dim3(256), 0, st, (T*)buf,
                           (int64_t)nx * ny, nz, T(h), part);
    return hipGetLastError();
}

static unsigned grid_for(int64_t n)
{
    const int64_t g = (n + 255) / 256;
    return (unsigned)(g < 65536 ? (g > 0 ? g : 1) : 65536);
}

template <typename T>
hipError_t launch_drops(hipStream_t st, const void* C, int nx, int ny, int nz, const int bc[3],
                        double thr, int* lab, int* cnt, int* meta, int* list, int cap, int* out)
{
    const int64_t tx = (nx + CCL_TX - 1) / CCL_TX, ty = (ny + CCL_TY - 1) / CCL_TY,
                  tz = (nz + CCL_TZ - 1) / CCL_TZ;
    hipLaunchKernelGGL((k_ccl_tile<T>),
                       dim3((unsigned)std::min<int64_t>(tx * ty * tz, CCL_MAX_WG)), dim3(256), 0,
                       st, (const T*)C, nx, ny, nz, T(thr), lab, cnt, meta, list, cap);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    auto groups = [](int64_t threads) { return (int)((threads + 255) / 256); };
    const int gx = groups(tx * ny * nz), gy = groups(nx * ty * nz), gz = groups((int64_t)nx * ny * tz);
    hipLaunchKernelGGL(k_ccl_merge, dim3((unsigned)(gx + gy + gz)), dim3(256), 0, st, lab, nx, ny,
                       nz, bc[0] == 0, bc[1] == 0, bc[2] == 0, gx, gy);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const unsigned nwg = (unsigned)std::min(256, (cap + 255) / 256);
    hipLaunchKernelGGL(k_ccl_sum, dim3(nwg), dim3(256), 0, st, lab, cnt, meta, list, cap);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ccl_drops, dim3(nwg), dim3(256), 0, st, lab, cnt, meta, list, cap, out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_press_prep(hipStream_t st, const void* P, void* Pold, void* phat, int64_t n)
{
    hipLaunchKernelGGL((k_press_prep<T>), dim3(grid_for(n)), dim3(256), 0, st, (const T*)P,
                       (T*)Pold, (T*)phat, n);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_press_rhs(hipStream_t st, const PressArgs& a, const void* C, const void* phat,
                            const void* u, const void* v, const void* w, void* rhs)
{
    const PressTile tl = press_tile<T>(rhs_threads<T>(), sizeof(T) == 8 ? 64 : 256,
                                    sizeof(T) == 8 ? 16 : 8, 4, a.nx, a.ny, a.nz);
    const int64_t tiles = press_tiles(tl, a.nx, a.ny, a.nz);
    hipLaunchKernelGGL((k_press_rhs<T>), dim3((unsigned)(tiles < 1048576 ? tiles : 1048576)),
                       dim3(rhs_threads<T>()), 0, st, tl, a, (const T*)C, (const T*)phat,
                       (const T*)u, (const T*)v, (const T*)w, (T*)rhs);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_press_solve(hipStream_t st, int zwalls, void* spec, void* cp, int nx, int ny,
                              int nz, int nxp, double h, const double* sines)
{
    if (zwalls) {
        // one work-group for the mean mode, one wave per 32 modes (two lanes per mode)
        const int64_t nm = (int64_t)ny * nxp;
        // The form by the rows (us, one of 2 waves per SIMD first): FP32 1024^2
        // planes of 8 rows 44 / 28 (before either 28), 16 rows 55 / 41 (43), 64
        // rows 190 / 179; 512^2 of 16 19 / 14, 32 28 / 22, 128 93 / 92, 256 203 /
        // 219, 512 434 / 452.  FP64 1024^2 of 8 42 / 35, 32 183 / 184; 512^2 of 32
        // 39.5 / 44.6, 64 87 / 89, 256 414 / 459.
        const auto k = (sizeof(T) == 8 ? nz >= 32 : nz >= 192) ? k_press_tri<T, true>
                                                               : k_press_tri<T, false>;
        hipLaunchKernelGGL(k, dim3(grid_for((nm + 31) / 32 * 64) + 1), dim3(256), 0, st, (T*)spec,
                           (T*)cp, nx, ny, nz, nxp, h, 1.0 / ((double)nx * ny));
    } else {
        const int64_t n = (int64_t)nz * ny * (nx / 2 + 1);
        const double* sy = sines + (nx / 2 + 1);
        hipLaunchKernelGGL((k_press_div<T>), dim3(grid_for(n)), dim3(256), 0, st, (T*)spec, nx,
                           ny, nz, nxp, h, 1.0 / ((double)nx * ny * nz), sines, sy, sy + ny);
    }
    return hipGetLastError();
}

hipError_t launch_press_sines(hipStream_t st, double* out, int nx, int ny, int nz)
{
    const int n[3] = {nx, ny, nz}, count[3] = {nx / 2 + 1, ny, nz};
    for (int d = 0; d < 3; ++d) {
        hipLaunchKernelGGL(k_press_sines, dim3(grid_for(count[d])), dim3(256), 0, st, out, n[d],
                           count[d]);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        out += count[d];
    }
    return hipSuccess;
}

template <typename T>
hipError_t launch_press_update(hipStream_t st, const PressArgs& a, const void* C, const void* P,
                               const void* phat, void* u, void* v, void* w)
{
    const PressTile tl = press_tile<T>(UPD_THREADS, 256, 2, 2, a.nx, a.ny, a.nz);
    const int64_t tiles = press_tiles(tl, a.nx, a.ny, a.nz);
    hipLaunchKernelGGL((k_press_update<T>), dim3((unsigned)(tiles < 1048576 ? tiles : 1048576)),
                       dim3(UPD_THREADS), 0, st, tl, a, (const T*)C, (const T*)P, (const T*)phat,
                       (T*)u, (T*)v, (T*)w);
    return hipGetLastError();
}

#define CH_INSTANTIATE(T, A)                                                                    \
    template hipError_t launch_pass_x<T, A>(int, int, int, size_t, hipStream_t,                 \
                                            const chd::BoxDesc*, int,                           \
                                            const chd::PassArgs&, const void*, const void*,     \
                                            const void*, const void*, void*, void*, bool,       \
                                            bool, int);                                         \
    template hipError_t launch_pass_x_seg<T, A>(int, int, size_t, hipStream_t,                  \
                                                const chd::BoxDesc*, int, const chd::PassArgs&, \
                                                const void*, const void*, const void*,          \
                                                const void*, const void*, void*, void*);        \
    template hipError_t launch_pass_line<T, A>(int, int, int, size_t, hipStream_t,              \
                                               const chd::BoxDesc*, int, const chd::PassArgs&,  \
                                               const void*, void*, bool);

CH_INSTANTIATE(double, double)
CH_INSTANTIATE(float, float)
CH_INSTANTIATE(float, double)

template hipError_t launch_pass_x_e25<double>(int, int, size_t, hipStream_t, const chd::BoxDesc*,
                                              const chd::PassArgs&, const void*, const void*,
                                              const void*, const void*, void*, void*);
template hipError_t launch_pass_x_e25<float>(int, int, size_t, hipStream_t, const chd::BoxDesc*,
                                             const chd::PassArgs&, const void*, const void*,
                                             const void*, const void*, void*, void*);
template hipError_t launch_mass<double>(int, int, hipStream_t, const chd::BoxDesc*, const void*,
                                        double*, const double*, double*);
template hipError_t launch_mass<float>(int, int, hipStream_t, const chd::BoxDesc*, const void*,
                                       double*, const double*, double*);
template hipError_t launch_mass_one<double>(hipStream_t, const chd::BoxDesc&, const void*, double*,
                                            double, double*);
template hipError_t launch_mass_one<float>(hipStream_t, const chd::BoxDesc&, const void*, double*,
                                           double, double*);
template hipError_t launch_check_velocity<double>(hipStream_t, const chd::BoxDesc*, int,
                                                  const void*, const void*, const void*, int*);
template hipError_t launch_check_velocity<float>(hipStream_t, const chd::BoxDesc*, int,
                                                 const void*, const void*, const void*, int*);
template hipError_t launch_interp<double>(hipStream_t, const InterpArgs&, const MarchArgs&);
template hipError_t launch_interp<float>(hipStream_t, const InterpArgs&, const MarchArgs&);
template hipError_t launch_drops<double>(hipStream_t, const void*, int, int, int, const int*,
                                         double, int*, int*, int*, int*, int, int*);
template hipError_t launch_drops<float>(hipStream_t, const void*, int, int, int, const int*,
                                        double, int*, int*, int*, int*, int, int*);
template hipError_t launch_grad<double>(hipStream_t, const void*, int, int, int, int,
                                        const double*, void*);
template hipError_t launch_grad<float>(hipStream_t, const void*, int, int, int, int,
                                       const double*, void*);
template hipError_t launch_scan<double>(hipStream_t, int, void*, const void*, int, int, int,
                                        double, double*);
template hipError_t launch_scan<float>(hipStream_t, int, void*, const void*, int, int, int,
                                       double, double*);

template hipError_t launch_press_prep<double>(hipStream_t, const void*, void*, void*, int64_t);
template hipError_t launch_press_rhs<double>(hipStream_t, const PressArgs&, const void*, const void*,
                                          const void*, const void*, const void*, void*);
template hipError_t launch_press_solve<double>(hipStream_t, int, void*, void*, int, int, int, int,
                                               double, const double*);
template hipError_t launch_press_update<double>(hipStream_t, const PressArgs&, const void*,
                                             const void*, const void*, void*, void*, void*);
template hipError_t launch_press_prep<float>(hipStream_t, const void*, void*, void*, int64_t);
template hipError_t launch_press_rhs<float>(hipStream_t, const PressArgs&, const void*, const void*,
                                          const void*, const void*, const void*, void*);
template hipError_t launch_press_solve<float>(hipStream_t, int, void*, void*, int, int, int, int,
                                              double, const double*);
template hipError_t launch_press_update<float>(hipStream_t, const PressArgs&, const void*,
                                             const void*, const void*, void*, void*, void*);

}  // namespace chk
