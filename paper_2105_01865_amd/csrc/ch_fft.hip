// ch_fft.hip -- the transforms of the fast Poisson solve (sec. 3.2) for gfx950.
//
// Real-to-complex transforms along x, complex ones along y and (periodic z)
// along z, of the spectrum [nz][ny][nxp].  Each is one pass over memory: a
// work-group brings a tile of whole lines into LDS, transforms them there and
// writes them back.
//   rows     2 CW rows of reals as CW complex lines (one row in the real, the
//            next in the imaginary parts), separated on the way out; in single
//            precision rows of odd length one by one
//   columns  CW neighbouring columns, in place: 8 (64 bytes in single, 128 in
//            double precision), or 4 on single-precision lines over 512 points
//   z solve  the same along z, forward, divided by the Laplacian's eigenvalues,
//            and back: the spectrum is read and written once for what would be
//            three passes
// Lengths are products of 2, 3 and 5 up to FFT_MAX (fft_radices); other meshes
// and those that are not better off here use the FFT library (own_lines).
//
// A line of n points goes through passes of radix 8, 6, 5, 4, 3 and 2 (Stockham's
// self-sorting order): butterfly j of a pass takes the points j + r n/R, times
// the twiddles exp(-2 pi i k r / (s R)) with k = j mod s (s the product of the
// radices before), and writes the points (j div s) s R + k + r s.  One LDS
// buffer: every thread reads all its butterflies, then, behind a barrier,
// writes them.  The inverse transform is the forward one of the conjugate,
// conjugated.
//
// What bounds it: memory, where two or more groups share a CU so that one group's
// loads run under another's passes: lines of up to 512 points (two groups, LDS and
// four waves per SIMD); in double precision beyond 512 one group takes up to 147 KB
// of LDS.  512^3 FP32 (537 MB in, 539 MB out a pass; copy 222 us): rows 209 us,
// columns 237; the z solve 447, planes 1.1 MB apart, where two groups on two XCDs
// share each line of 128 bytes (before, two transforms and a division); the
// whole periodic solve 2619 -> 1305 us.
// 240 x 180 x 160 FP64: rows 25 us, columns 28, z 42, against 23, 44 and 79
// (three passes) before.  Lengths that are powers of two have kernels without the
// radices 3, 5 and 6, whose registers cost the others occupancy (512^3 FP32,
// periodic: a solve 1496 -> 1305 us).
#include <hip/hip_runtime.h>

#include "ch_device.h"
#include "ch_kernels.h"

namespace chk {

template <typename T>
struct alignas(2 * sizeof(T)) CV {
    T x, y;
};

template <typename T>
__device__ __forceinline__ CV<T> operator+(CV<T> a, CV<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ CV<T> operator-(CV<T> a, CV<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ CV<T> operator*(T s, CV<T> a) { return {s * a.x, s * a.y}; }
template <typename T>
__device__ __forceinline__ CV<T> cmul(CV<T> a, CV<T> b)
{
    return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
// c x (+ c2 x2), the constants in single precision as two floats: rounded to one,
// their error is the same in every butterfly and adds up (27^3 FP32 periodic, rms
// error of a solve 2.0e-7 of the rms with one, 1.84e-7 with two; the library's
// transforms 1.86e-7).
__device__ __forceinline__ double cprod(double c, double x) { return c * x; }
__device__ __forceinline__ float cprod(double c, float x)
{
    const float hi = (float)c, lo = (float)(c - hi);
    return fmaf(hi, x, lo * x);
}
__device__ __forceinline__ double cprod(double c, double x, double c2, double x2)
{
    return c * x + c2 * x2;
}
__device__ __forceinline__ float cprod(double c, float x, double c2, float x2)
{
    const float hi = (float)c, lo = (float)(c - hi);
    const float hi2 = (float)c2, lo2 = (float)(c2 - hi2);
    return fmaf(hi, x, fmaf(hi2, x2, fmaf(lo, x, lo2 * x2)));
}
template <typename T>
__device__ __forceinline__ CV<T> cprod(double c, CV<T> a) { return {cprod(c, a.x), cprod(c, a.y)}; }
template <typename T>
__device__ __forceinline__ CV<T> cprod(double c, CV<T> a, double c2, CV<T> b)
{
    return {cprod(c, a.x, c2, b.x), cprod(c, a.y, c2, b.y)};
}
template <typename T>
__device__ __forceinline__ CV<T> times_mi(CV<T> a) { return {a.y, -a.x}; }   // -i a

// Forward discrete Fourier transform of R values in place.
template <int R, typename T>
__device__ __forceinline__ void dft(CV<T>* v)
{
    if constexpr (R == 2) {
        const CV<T> a = v[0], b = v[1];
        v[0] = a + b;
        v[1] = a - b;
    } else if constexpr (R == 3) {
        constexpr double c = 0.86602540378443864676;   // sin(pi/3)
        const CV<T> s = v[1] + v[2], d = times_mi(cprod(c, v[1] - v[2]));
        const CV<T> t = v[0] - T(0.5) * s;
        v[0] = v[0] + s;
        v[1] = t + d;
        v[2] = t - d;
    } else if constexpr (R == 4) {
        const CV<T> a = v[0] + v[2], b = v[0] - v[2], c = v[1] + v[3], d = times_mi(v[1] - v[3]);
        v[0] = a + c;
        v[1] = b + d;
        v[2] = a - c;
        v[3] = b - d;
    } else if constexpr (R == 5) {
        // cosines and sines of 2 pi/5 and 4 pi/5
        constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;
        constexpr double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;
        const CV<T> t1 = v[1] + v[4], t2 = v[2] + v[3], t3 = v[1] - v[4], t4 = v[2] - v[3];
        const CV<T> m1 = v[0] + cprod(c1, t1, c2, t2), m2 = v[0] + cprod(c2, t1, c1, t2);
        const CV<T> n1 = times_mi(cprod(s1, t3, s2, t4)), n2 = times_mi(cprod(s2, t3, -s1, t4));
        v[0] = v[0] + (t1 + t2);
        v[1] = m1 + n1;
        v[4] = m1 - n1;
        v[2] = m2 + n2;
        v[3] = m2 - n2;
    } else if constexpr (R == 6) {
        // two transforms of R / 2, then R / 2 of two: in the Good-Thomas order
        // (R / 2 is odd) no twiddles stand between them
        constexpr int H = R / 2;
        CV<T> e[H], o[H];
#pragma unroll
        for (int k = 0; k < H; ++k) {
            e[k] = v[2 * k];
            o[k] = v[(2 * k + H) % R];
        }
        dft<H>(e);
        dft<H>(o);
#pragma unroll
        for (int k = 0; k < H; ++k) {
            // output q with q = k mod H: even q the sum, odd q the difference
            const int a = k % 2 == 0 ? k : k + H, b = k % 2 == 0 ? k + H : k;
            v[a] = e[k] + o[k];
            v[b] = e[k] - o[k];
        }
    } else {
        static_assert(R == 8, "radix");
        const T h = T(0.70710678118654752440);   // sqrt(1/2)
        CV<T> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft<4>(e);
        dft<4>(o);
        o[1] = h * CV<T>{o[1].x + o[1].y, o[1].y - o[1].x};
        o[2] = times_mi(o[2]);
        o[3] = h * CV<T>{o[3].y - o[3].x, -o[3].y - o[3].x};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = e[k] + o[k];
            v[k + 4] = e[k] - o[k];
        }
    }
}

// One pass of radix R over the CW lines of a tile (point p of line c at
// L[p RP + c]); VPT bounds the points per thread.
template <int R, typename T, int CW, int RP, int VPT, int NT>
__device__ __forceinline__ void fft_pass(CV<T>* L, const CV<T>* tw, int n, int s, int tid)
{
    constexpr int NB = (VPT + R - 1) / R;
    const int nb = n / R, total = nb * CW, step = n / (s * R);
    const uint32_t inv = ((1u << 20) + s - 1) / s;   // j div s for j s < 2^20
    CV<T> v[NB][R];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int idx = tid + b * NT;
        if (idx >= total) break;
        const int c = idx % CW, j = idx / CW;
        const int k = j - (int)(((uint32_t)j * inv) >> 20) * s;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[b][r] = L[(j + r * nb) * RP + c];
            if (r > 0) v[b][r] = cmul(v[b][r], tw[k * r * step]);
        }
        dft<R>(v[b]);
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int idx = tid + b * NT;
        if (idx >= total) break;
        const int c = idx % CW, j = idx / CW;
        const int q = (int)(((uint32_t)j * inv) >> 20), k = j - q * s;
#pragma unroll
        for (int r = 0; r < R; ++r) L[(q * s * R + k + r * s) * RP + c] = v[b][r];
    }
    __syncthreads();
}

// The forward transform of a tile's lines in place; starts behind a barrier
// after the tile is filled, ends with one.
template <bool P2, typename T, int CW, int RP, int VPT, int NT>
__device__ __forceinline__ void fft_tile(CV<T>* L, const CV<T>* tw, const FftLine& f, int tid)
{
    __syncthreads();
    int s = 1;
    for (int p = 0; p < f.passes; ++p) {
        const int R = f.radix[p];
        switch (R) {
        case 8: fft_pass<8, T, CW, RP, VPT, NT>(L, tw, f.n, s, tid); break;
        case 4: fft_pass<4, T, CW, RP, VPT, NT>(L, tw, f.n, s, tid); break;
        case 2: fft_pass<2, T, CW, RP, VPT, NT>(L, tw, f.n, s, tid); break;
        default:
            if constexpr (!P2) {
                if (R == 3) fft_pass<3, T, CW, RP, VPT, NT>(L, tw, f.n, s, tid);
                if (R == 5) fft_pass<5, T, CW, RP, VPT, NT>(L, tw, f.n, s, tid);
                if constexpr (sizeof(T) == 4)
                    if (R == 6) fft_pass<6, T, CW, RP, VPT, NT>(L, tw, f.n, s, tid);
            }
        }
        s *= R;
    }
}

// Twiddles of the line on their way into LDS: loaded ahead of the tile, stored
// after its loads are issued (NT >= n / 2).
template <typename T, int NT>
struct Twiddles {
    CV<T> w[2];
    __device__ __forceinline__ void load(const FftLine& f, int tid)
    {
        const CV<T>* g = reinterpret_cast<const CV<T>*>(f.tw);
        w[0] = w[1] = CV<T>{T(0), T(0)};
        if (tid < f.n) w[0] = g[tid];
        if (tid + NT < f.n) w[1] = g[tid + NT];
    }
    __device__ __forceinline__ void store(CV<T>* tw, const FftLine& f, int tid) const
    {
        if (tid < f.n) tw[tid] = w[0];
        if (tid + NT < f.n) tw[tid + NT] = w[1];
    }
};

// Lines of a tile: CW columns; for rows, CW pairs of rows (each point's lines
// padded by one against bank conflicts of lanes along x).

// Columns of nplane planes [n][pitch], in place: column tile by column tile
// (neighbouring tiles of a plane on one XCD, where their shared cache lines
// meet).  inverse: conjugated in and out.
template <bool P2, typename T, int CW, int VPT, int NT>
__global__ void __launch_bounds__(NT, 4)
k_fft_cols(FftLine f, CV<T>* __restrict__ spec, int pitch, int ncol, int nplane, int inverse)
{
    extern __shared__ __align__(16) unsigned char smem[];
    CV<T>* tw = reinterpret_cast<CV<T>*>(smem);
    CV<T>* L = tw + f.n;
    const int tid = threadIdx.x, n = f.n;
    const int tiles = (ncol + CW - 1) / CW;
    const int per = (int)gridDim.x / 8, rem = (int)gridDim.x % 8;
    const int xcd = (int)blockIdx.x % 8, loc = (int)blockIdx.x / 8;
    const int wg = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + loc;
    const int c = tid % CW, c0 = wg % tiles * CW;
    const bool on = c0 + c < ncol;
    CV<T>* g = spec + (int64_t)(wg / tiles) * n * pitch + c0 + c;
    const T sg = inverse ? T(-1) : T(1);
    Twiddles<T, NT> wt;
    wt.load(f, tid);
    constexpr int RS = NT / CW;   // rows between a thread's points
    {
        CV<T> v[VPT];
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            const int row = tid / CW + q * RS;
            v[q] = CV<T>{T(0), T(0)};
            if (row < n && on) v[q] = g[(int64_t)row * pitch];
        }
        wt.store(tw, f, tid);
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            const int row = tid / CW + q * RS;
            if (row < n) L[row * CW + c] = CV<T>{v[q].x, sg * v[q].y};
        }
    }
    fft_tile<P2, T, CW, CW, VPT, NT>(L, tw, f, tid);
    if (!on) return;
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
        const int row = tid / CW + q * RS;
        if (row >= n) break;
        const CV<T> v = L[row * CW + c];
        g[(int64_t)row * pitch] = CV<T>{v.x, sg * v.y};
    }
}

// Periodic z: the lines along z of the spectrum [n][ny][nxp] (x and y already
// transformed), divided by the eigenvalues of the 7-point Laplacian (zero mode
// to 0) and scaled, then transformed back.  tx, ty, tz: the sines of
// launch_press_sines.
template <bool P2, typename T, int CW, int VPT, int NT>
__global__ void __launch_bounds__(NT, 4)
k_fft_zsolve(FftLine f, CV<T>* __restrict__ spec, int ny, int nxh, int nxp, double h, double scale,
             const double* __restrict__ tx, const double* __restrict__ ty,
             const double* __restrict__ tz)
{
    extern __shared__ __align__(16) unsigned char smem[];
    CV<T>* tw = reinterpret_cast<CV<T>*>(smem);
    CV<T>* L = tw + f.n;
    const int tid = threadIdx.x, n = f.n;
    const int64_t plane = (int64_t)ny * nxp;
    const int c = tid % CW;
    const int64_t col = (int64_t)blockIdx.x * CW + c;
    const int j = (int)(col / nxp), i = (int)(col - (int64_t)j * nxp);
    const bool on = j < ny && i < nxh;
    CV<T>* g = spec + col;
    Twiddles<T, NT> wt;
    wt.load(f, tid);
    constexpr int RS = NT / CW;
    {
        CV<T> v[VPT];
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            const int row = tid / CW + q * RS;
            v[q] = CV<T>{T(0), T(0)};
            if (row < n && on) v[q] = g[row * plane];
        }
        wt.store(tw, f, tid);
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            const int row = tid / CW + q * RS;
            if (row < n) L[row * CW + c] = v[q];
        }
    }
    const double sx = on ? tx[i] : 0.0, sy = on ? ty[j] : 1.0;
    const double sxy = sx * sx + sy * sy;
    for (int pass = 0; pass < 2; ++pass) {
        fft_tile<P2, T, CW, CW, VPT, NT>(L, tw, f, tid);
        if (pass == 1) break;
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            const int row = tid / CW + q * RS;
            if (row >= n) break;
            const double sz = tz[row];
            const double lam = -4.0 / (h * h) * (sxy + sz * sz);
            const T s = (col == 0 && row == 0) ? T(0) : T(scale / lam);
            const CV<T> v = L[row * CW + c];
            L[row * CW + c] = CV<T>{s * v.x, -(s * v.y)};
        }
    }
    if (!on) return;
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
        const int row = tid / CW + q * RS;
        if (row >= n) break;
        const CV<T> v = L[row * CW + c];
        g[row * plane] = CV<T>{v.x, -v.y};
    }
}

// Rows of reals to the half spectrum.  PAIR: 2 CW rows per group, two in a line;
// else CW rows, each a line's real parts (launch_fft_rows).
template <bool P2, bool PAIR, typename T, int CW, int VPT, int NT>
__global__ void __launch_bounds__(NT, 4)
k_fft_rows(FftLine f, const T* __restrict__ in, CV<T>* __restrict__ out, int nxp, int64_t nrows)
{
    constexpr int RP = CW + 1, ROWS = PAIR ? 2 * CW : CW;
    extern __shared__ __align__(16) unsigned char smem[];
    CV<T>* tw = reinterpret_cast<CV<T>*>(smem);
    CV<T>* L = tw + f.n;
    const int tid = threadIdx.x, n = f.n;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int nr = nrows - row0 < ROWS ? (int)(nrows - row0) : ROWS;
    Twiddles<T, NT> wt;
    wt.load(f, tid);
    for (int x = tid; x < n; x += NT) {
        T v[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) v[r] = r < nr ? in[(row0 + r) * n + x] : T(0);
#pragma unroll
        for (int p = 0; p < CW; ++p) {
            if constexpr (PAIR) L[x * RP + p] = CV<T>{v[2 * p], v[2 * p + 1]};
            else L[x * RP + p] = CV<T>{v[p], T(0)};
        }
    }
    wt.store(tw, f, tid);
    fft_tile<P2, T, CW, RP, VPT, NT>(L, tw, f, tid);
    // Z = A + i B: A[k] = (Z[k] + conj Z[n-k]) / 2, B[k] = (Z[k] - conj Z[n-k]) / (2 i)
    for (int k = tid; k <= n / 2; k += NT) {
        const int m = k == 0 ? 0 : n - k;
#pragma unroll
        for (int p = 0; p < CW; ++p) {
            if constexpr (PAIR) {
                if (2 * p >= nr) break;
                const CV<T> a = L[k * RP + p], b = L[m * RP + p];
                CV<T>* o = out + (row0 + 2 * p) * nxp + k;
                o[0] = CV<T>{T(0.5) * (a.x + b.x), T(0.5) * (a.y - b.y)};
                if (2 * p + 1 < nr) o[nxp] = CV<T>{T(0.5) * (a.y + b.y), T(0.5) * (b.x - a.x)};
            } else {
                if (p >= nr) break;
                out[(row0 + p) * nxp + k] = L[k * RP + p];
            }
        }
    }
}

// The half spectrum back to rows of reals (unscaled); the imaginary parts of
// the mean and of the highest wave of an even row do not count.
template <bool P2, bool PAIR, typename T, int CW, int VPT, int NT>
__global__ void __launch_bounds__(NT, 4)
k_fft_rows_back(FftLine f, const CV<T>* __restrict__ in, T* __restrict__ out, int nxp,
                int64_t nrows)
{
    constexpr int RP = CW + 1, ROWS = PAIR ? 2 * CW : CW;
    extern __shared__ __align__(16) unsigned char smem[];
    CV<T>* tw = reinterpret_cast<CV<T>*>(smem);
    CV<T>* L = tw + f.n;
    const int tid = threadIdx.x, n = f.n;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int nr = nrows - row0 < ROWS ? (int)(nrows - row0) : ROWS;
    Twiddles<T, NT> wt;
    wt.load(f, tid);
    // conj of Z = A + i B (PAIR; else of A) at k and n - k
    for (int k = tid; k <= n / 2; k += NT) {
        const bool real = k == 0 || 2 * k == n;
        CV<T> v[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            v[r] = CV<T>{T(0), T(0)};
            if (r < nr) v[r] = in[(row0 + r) * nxp + k];
            if (real) v[r].y = T(0);
        }
#pragma unroll
        for (int p = 0; p < CW; ++p) {
            if constexpr (PAIR) {
                const CV<T> a = v[2 * p], b = v[2 * p + 1];
                L[k * RP + p] = CV<T>{a.x - b.y, -(a.y + b.x)};
                if (!real) L[(n - k) * RP + p] = CV<T>{a.x + b.y, a.y - b.x};
            } else {
                L[k * RP + p] = CV<T>{v[p].x, -v[p].y};
                if (!real) L[(n - k) * RP + p] = v[p];
            }
        }
    }
    wt.store(tw, f, tid);
    fft_tile<P2, T, CW, RP, VPT, NT>(L, tw, f, tid);
    for (int x = tid; x < n; x += NT) {
#pragma unroll
        for (int p = 0; p < CW; ++p) {
            const CV<T> v = L[x * RP + p];
            if constexpr (PAIR) {
                if (2 * p < nr) out[(row0 + 2 * p) * n + x] = v.x;
                if (2 * p + 1 < nr) out[(row0 + 2 * p + 1) * n + x] = -v.y;
            } else if (p < nr) {
                out[(row0 + p) * n + x] = v.x;
            }
        }
    }
}

// ---- launchers --------------------------------------------------------------
// Column shapes (columns, threads) by a line's points.  Eight points per thread
// (sixteen spill; of these only the z solve of double-precision lines of over 512
// points that are no power of two does, 36 bytes a lane: 64 x 64 x 1000 124 us
// a solve against 186 in the library).  Tiles of 64 bytes in FP32, so that two groups share a CU
// (512^3: the transforms and the solve along walls 1623 us with 128-byte tiles of
// 1024 threads, 1468 with these).  No more threads than eight points each ask
// for: short lines leave the rest idle (640 x 30 x 32 FP64: 52 -> 48 us).
template <typename T, typename Go>
static hipError_t fft_shape(int n, Go&& go)
{
    using chd::IC;
    if (n <= 128) return go(IC<8>{}, IC<128>{});
    if (n <= 256) return go(IC<8>{}, IC<256>{});
    if (n <= 512) return go(IC<8>{}, IC<512>{});
    if constexpr (sizeof(T) == 8) return go(IC<8>{}, IC<1024>{});
    else return go(IC<4>{}, IC<512>{});
}
// Row shapes (pairs of rows, points per thread, threads).  Four pairs of FP32
// (eight: 1468 us for the same work, four: 1389), and of FP64, there with half
// the points per thread up to 256, where more threads hide the loads (256^3
// periodic: two pairs 282 us, four of eight points per thread 279, these 267).
template <typename T, typename Go>
static hipError_t fft_row_shape(int n, Go&& go)
{
    using chd::IC;
    if constexpr (sizeof(T) == 8) {
        if (n <= 64) return go(IC<4>{}, IC<4>{}, IC<64>{});
        if (n <= 128) return go(IC<4>{}, IC<4>{}, IC<128>{});
        if (n <= 256) return go(IC<4>{}, IC<4>{}, IC<256>{});
        if (n <= 512) return go(IC<4>{}, IC<8>{}, IC<256>{});
        return go(IC<2>{}, IC<4>{}, IC<512>{});
    } else {
        if (n <= 128) return go(IC<4>{}, IC<8>{}, IC<64>{});
        if (n <= 256) return go(IC<4>{}, IC<8>{}, IC<128>{});
        if (n <= 512) return go(IC<4>{}, IC<8>{}, IC<256>{});
        return go(IC<4>{}, IC<8>{}, IC<512>{});
    }
}

template <typename K>
static hipError_t fft_lds(K kernel, size_t lds)
{
    if (lds <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds);
}

template <typename T>
hipError_t launch_fft_cols(hipStream_t st, const FftLine& f, void* spec, int pitch, int ncol,
                           int nplane, bool inverse)
{
    return fft_shape<T>(f.n, [&](auto cw, auto nt) {
        constexpr int CW = decltype(cw)::value, NT = decltype(nt)::value;
        const size_t lds = (size_t)f.n * (CW + 1) * sizeof(CV<T>);
        const auto k = f.p2 ? k_fft_cols<true, T, CW, 8, NT> : k_fft_cols<false, T, CW, 8, NT>;
        hipError_t e = fft_lds(k, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3((unsigned)((ncol + CW - 1) / CW * nplane)),
                           dim3(NT), lds, st, f, (CV<T>*)spec, pitch, ncol, nplane,
                           inverse ? 1 : 0);
        return hipGetLastError();
    });
}

template <typename T>
hipError_t launch_fft_zsolve(hipStream_t st, const FftLine& f, void* spec, int nx, int ny, int nxp,
                             double h, const double* sines)
{
    const int nxh = nx / 2 + 1;
    const int64_t cols = (int64_t)ny * nxp;
    return fft_shape<T>(f.n, [&](auto cw, auto nt) {
        constexpr int CW = decltype(cw)::value, NT = decltype(nt)::value;
        const size_t lds = (size_t)f.n * (CW + 1) * sizeof(CV<T>);
        const auto k = f.p2 ? k_fft_zsolve<true, T, CW, 8, NT> : k_fft_zsolve<false, T, CW, 8, NT>;
        hipError_t e = fft_lds(k, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3((unsigned)((cols + CW - 1) / CW)), dim3(NT), lds, st,
                           f, (CV<T>*)spec, ny, nxh, nxp, h, 1.0 / ((double)nx * ny * f.n), sines, sines + nxh, sines + nxh + ny);
        return hipGetLastError();
    });
}

template <typename T>
hipError_t launch_fft_rows(hipStream_t st, const FftLine& f, const void* in, void* out, int nxp,
                           int64_t nrows, bool inverse)
{
    return fft_row_shape<T>(f.n, [&](auto cw, auto vpt, auto nt) {
        constexpr int CW = decltype(cw)::value, V = decltype(vpt)::value, NT = decltype(nt)::value;
        const size_t lds = (size_t)f.n * (CW + 2) * sizeof(CV<T>);
        // Two rows in a line cost a rounding each way, which in single precision and
        // on rows of odd length the library's transforms do not have (they halve
        // even ones): those go one by one.  RMS error of a solve, before the own
        // transforms, with rows in pairs, one by one: 81 x 75 x 60 1.95, 2.06, 1.95
        // (1e-7 of the rms), 25 x 15 x 9 1.58, 1.66, 1.53; 243^3 takes 251 us for
        // 215, 125^3 67 for 66 (894 and 128 in the library).
        const bool pair = sizeof(T) == 8 || f.n % 2 == 0;
        const int rows = pair ? 2 * CW : CW;
        const unsigned nwg = (unsigned)((nrows + rows - 1) / rows);
        auto back = f.p2 ? k_fft_rows_back<true, true, T, CW, V, NT>
                         : k_fft_rows_back<false, true, T, CW, V, NT>;
        auto forth = f.p2 ? k_fft_rows<true, true, T, CW, V, NT> : k_fft_rows<false, true, T, CW, V, NT>;
        if constexpr (sizeof(T) == 4)
            if (!pair) {
                back = k_fft_rows_back<false, false, T, CW, V, NT>;
                forth = k_fft_rows<false, false, T, CW, V, NT>;
            }
        const hipError_t e = inverse ? fft_lds(back, lds) : fft_lds(forth, lds);
        if (e != hipSuccess) return e;
        if (inverse)
            hipLaunchKernelGGL(back, dim3(nwg), dim3(NT), lds, st, f, (const CV<T>*)in, (T*)out, nxp,
                               nrows);
        else
            hipLaunchKernelGGL(forth, dim3(nwg), dim3(NT), lds, st, f, (const T*)in, (CV<T>*)out, nxp,
                               nrows);
        return hipGetLastError();
    });
}

#define FFT_INSTANTIATE(T)                                                                        \
    template hipError_t launch_fft_cols<T>(hipStream_t, const FftLine&, void*, int, int, int,     \
                                           bool);                                                 \
    template hipError_t launch_fft_zsolve<T>(hipStream_t, const FftLine&, void*, int, int, int,   \
                                             double, const double*);                              \
    template hipError_t launch_fft_rows<T>(hipStream_t, const FftLine&, const void*, void*, int,  \
                                           int64_t, bool);
FFT_INSTANTIATE(double)
FFT_INSTANTIATE(float)

}  // namespace chk
