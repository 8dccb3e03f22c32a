// ch_route.h -- which kernel a transfer or a transform takes, and the shapes of
// their launches: host rules without HIP, so that they can be checked on a CPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "../../include/ch.h"

namespace chk {

constexpr int MARCH_BAND = 8;   // target rows of a sub-band of the marching kernel
// Where the taps of consecutive targets start, within groups of 4 in x and
// MARCH_BAND in y: anywhere, at 0 0 1 1 .., or at 0 1 1 2 ..
enum { MARCH_ANY = 0, MARCH_FACE = 1, MARCH_CENTRE = 2 };

// Lines of the library's own transforms (ch_fft.hip): n points, a product of 2,
// 3 and 5 up to FFT_MAX, their passes' radices, and the twiddles
// exp(-2 pi i m / n), m < n, in the working precision (device memory).
constexpr int FFT_MAX = 1024;
struct FftLine {
    int n, passes, p2;   // p2: n is a power of two
    int radix[10];
    const void* tw;
};
// Radices of n's passes, as few as possible and then of the least sum (six:
// also 6, which FP32 has the registers for); false where the transforms do not
// take n.
inline bool fft_radices(int n, bool six, FftLine* f)
{
    f->n = n;
    f->passes = 0;
    f->p2 = (n & (n - 1)) == 0;
    f->tw = nullptr;
    if (n < 2 || n > FFT_MAX) return false;
    FftLine best = *f;
    int least = 0;
    auto search = [&](auto&& self, const FftLine& l, int rest, int top, int cost) -> void {
        if (rest == 1 && (least == 0 || cost < least)) {
            best = l;
            least = cost;
        }
        if (rest == 1 || l.passes == 10) return;
        for (int r : {8, 6, 5, 4, 3, 2}) {
            if (r > top || rest % r != 0 || (r == 6 && !six)) continue;
            FftLine m = l;
            m.radix[m.passes++] = r;
            self(self, m, rest / r, r, cost + 100 + r);
        }
    };
    search(search, *f, n, 8, 0);
    *f = best;
    return least > 0;
}

}  // namespace chk

namespace chp {

// The box that drops are labelled on: axes of one cell folded away (the cells
// keep their linear indices, and such an axis joins nothing), so that the
// others fill the labelling's tiles of 64 x 8 x 8 cells.  10^6 x 1 x 1 cells
// [z][y][x]: 5.4 ms a call in tiles of 1 x 1 x 8.
inline void drop_axes(const int n[3], const int bc[3], int m[3], int mbc[3])
{
    int k = 0;
    for (int d = 0; d < 3; ++d)
        if (n[d] > 1) {
            m[k] = n[d];
            mbc[k++] = bc[d];
        }
    for (; k < 3; ++k) {
        m[k] = 1;
        mbc[k] = CH_NOFLUX;
    }
}

// Whether the x taps of every 4 consecutive targets 4t .. 4t+3 lie within
// the 6 cyclically consecutive source points from target 4t's first tap.
inline bool interp_xwin(const std::vector<int>& ix, int64_t tnx, int sx)
{
    for (int64_t i0 = 0; i0 < tnx; i0 += 4) {
        const int ws = ix[4 * i0];
        for (int64_t i = i0; i < std::min<int64_t>(tnx, i0 + 4); ++i)
            for (int q = 0; q < 4; ++q)
                if ((ix[4 * i + q] - ws + sx) % sx >= 6) return false;
    }
    return true;
}

// Most work-groups of a marching transfer (beyond, its groups march further):
// whole rounds of those resident (6 per CU in single precision, 3 in double),
// two and eight.  512^3, us per component: FP32 1024 groups 199, 2048 181, 3008
// 169, 3328 182, 8192 184; FP64 2048 423, 4096 345, 6144 331, 8192 328.
constexpr int64_t march_wg(size_t esize) { return esize == 4 ? 3072 : 6144; }
// Single-precision targets from this size on are stored non-temporally: they
// are out of the caches before anything reads them (512^3 181 against 187 us).
// Below, the step or the integration that follows reads them from the caches,
// and in double precision a lane's 32 bytes are two half-line stores that only
// a cache joins (256^3 FP64 54 against 63 us, with the integration 112 against
// 140).
constexpr int64_t MARCH_NT_BYTES = 256ll << 20;

// Coarse rows a thread of the marching transfer holds (8 or 11), or 0 where it
// does not apply: coarse rows of at most 256 points, at most 1024 targets in x
// whose taps lie in 6-point windows, and in every 8 target rows from a multiple
// of 8 on consecutive y taps that start at most one coarse row later per row.
inline int interp_march_rows(const std::vector<int>& iy, int64_t tnx, int64_t tny, int sx, int sy, int xwin)
{
    if (sx > 256 || tnx > 1024 || !xwin || sy < 4) return 0;
    int span = 0;
    for (int64_t j = 0; j < tny; ++j) {
        const int64_t jb = j / chk::MARCH_BAND * chk::MARCH_BAND;
        for (int q = 1; q < 4; ++q)
            if (iy[4 * j + q] != (iy[4 * j] + q) % sy) return 0;
        const int l = (iy[4 * j] - iy[4 * jb] + sy) % sy;
        const int prev = j == jb ? 0 : (iy[4 * (j - 1)] - iy[4 * jb] + sy) % sy;
        if (l < prev || l > prev + 1) return 0;
        span = std::max(span, l + 4);
    }
    return span <= 8 ? 8 : span <= 11 ? 11 : 0;
}

// The pattern (chk::MARCH_*) of the targets' first taps in groups of `group`,
// each target's taps consecutive.
inline int interp_pattern(const std::vector<int>& ix, int64_t tn, int n, int group)
{
    bool face = true, centre = true;
    for (int64_t i = 0; i < tn; ++i) {
        for (int q = 1; q < 4; ++q)
            if (ix[4 * i + q] != (ix[4 * i] + q) % n) return chk::MARCH_ANY;
        const int g = (int)(i % group);
        const int d = (ix[4 * i] - ix[4 * (i - g)] + n) % n;
        face = face && d == g / 2;
        centre = centre && d == (g + 1) / 2;
    }
    return face ? chk::MARCH_FACE : centre ? chk::MARCH_CENTRE : chk::MARCH_ANY;
}

// Launch of a marching transfer: columns of a sub-band's threads (whole waves, so
// that a wave's columns belong to one sub-band), sub-bands per group, bands of
// groups, planes per group and the chunks of them, non-temporal stores.
struct MarchShape {
    int sxw, nsub, nband, kc, nchunk, nt;
};
// Planes per group so that the chip has a few groups per CU, at least 4 to
// reuse the stencils.
inline MarchShape march_shape(size_t esize, int64_t sx, const int64_t tn[3])
{
    MarchShape m;
    m.sxw = (int)((sx + 63) / 64 * 64);
    m.nsub = std::max(1, 256 / m.sxw);
    const int rows = chk::MARCH_BAND * m.nsub;
    m.nband = (int)((tn[1] + rows - 1) / rows);
    m.kc = std::max(4, (int)((tn[2] * m.nband + march_wg(esize) - 1) / march_wg(esize)));
    m.kc = (int)std::min<int64_t>(m.kc, tn[2]);
    m.nchunk = (int)((tn[2] + m.kc - 1) / m.kc);
    m.nt = esize == 4 && tn[0] * tn[1] * tn[2] * (int64_t)esize >= MARCH_NT_BYTES;
    return m;
}

// Whether the general kernel loads an item's coarse rows a whole item ahead: one
// batch of loads covers them (rmax: the tallest band).
constexpr int interp_rows_ahead(size_t esize) { return esize == 4 ? 20 : 12; }
inline bool interp_piped(size_t esize, int rmax, int64_t sx)
{
    return rmax <= interp_rows_ahead(esize) && sx <= 256;
}

// Whether a transfer with the marching kernel's properties (rm rows, patterns xp
// and yp) takes it; piped: the general kernel's variant it is measured against.
// With both patterns known (two fine cells per coarse one), always: 8^3 to 16^3
// FP32 37 -> 28 us, FP64 38 -> 35 (three components), and more at every size up
// to 512^3.  With selected taps where
//   - its groups occupy three quarters of the CUs: the general kernel's are
//     smaller (64 x 64 x 24 to 192 x 192 x 32, 54 groups, FP32 48 -> 54 us, FP64
//     55 -> 63; 240 x 120 x 16 to 360 x 180 x 24, 138 groups, FP32 50 -> 52; from
//     192 groups on FP32 gains 1.1 to 2.3 times, single shapes 0.98);
//   - in double precision not with 11 rows on coarse rows over 128 points, where
//     256 registers leave one wave per SIMD and up to half of the lanes idle and
//     the general kernel stores 4 targets at once (256 to 384 columns 477 -> 615
//     us, 132 to 220 75 -> 96); where it cannot, this one gains (435 columns 1409
//     -> 844).  One of its groups fills a CU, so neither where the last round of
//     256 leaves a third of the CUs idle (96 x 96 x 64 to 152 x 152 x 96, 240
//     groups, 70 -> 59 us; to 152 x 152 x 128, 320 groups, 80 -> 99);
//   - in single precision not with 11 rows on large meshes where the general one
//     is piped and stores 4 targets at once (256 x 256 x 160 to 384 x 384 x 240
//     238 -> 252 us, to 436 x 436 x 272 286 -> 308; from 256 x 256 x 96 to 384 x
//     384 x 144 189 -> 158, to 432 x 432 x 163 240 -> 198).
inline bool march_taken(size_t esize, int rm, int xp, int yp, const MarchShape& m, int64_t sx,
                        const int64_t tn[3], bool piped)
{
    if (rm == 0) return false;
    const bool known = (xp == chk::MARCH_FACE && yp == chk::MARCH_CENTRE) ||
                       (xp == chk::MARCH_CENTRE && yp != chk::MARCH_ANY);
    if (known) return true;
    const int64_t groups = (int64_t)m.nband * m.nchunk;
    if (groups < 192) return false;
    if (rm == 11 && esize == 8 && 3 * groups < 2 * ((groups + 255) / 256 * 256)) return false;
    if (rm == 8 || tn[0] % 4 != 0) return true;
    return esize == 4 ? !piped || tn[0] * tn[1] * tn[2] < (1 << 25) : sx <= 128;
}

// Row pitch of the pressure solve's spectrum in complex elements, at least nx/2 +
// 1.  Rounded up to a multiple of 8 rows start on 64 bytes (128 in double); with
// the bare nx/2 + 1 (257 at nx = 512) every row starts elsewhere in a cache line,
// which costs the column transforms: the library's 512^3 FP32 forward 807 -> 622
// us (FP64 1084 -> 873), a solve between walls at 128^3 FP64 77 -> 71, 100^3 67 ->
// 60.  Our own transforms take it from 16 elements on.  For the library's, rows of
// 96 to 1024 points between walls or of more than 2^20 cells: small periodic
// meshes and short rows lose its plans for them (periodic 32 x 64 x 64 FP32 26 us
// bare, 40 padded; walls 32 x 16 x 16 20.5 and 25.5), longer rows gain nothing and
// lose along z (2048 x 2048 x 32 walls FP32 2180 bare, 2380 padded, FP64 3860 and
// 4110).
inline int spectrum_pitch(int nx, int ny, int nz, bool walls, bool own)
{
    const int bare = nx / 2 + 1, padded = (bare + 7) / 8 * 8;
    const bool pad = own ? bare >= 16
                         : nx >= 96 && nx <= 1024 &&
                               (walls || (int64_t)nx * ny * nz > (1 << 20));
    return pad && (double)padded * ny * nz < 2147483647.0 ? padded : bare;
}

// Where the own transforms take the place of hipFFT's (times of a solve, hipFFT's
// first).  Periodic z: everywhere (512^3 FP32 2619 -> 1296 us, 300^3 FP64 1144 ->
// 525, 240 x 180 x 160 FP64 205 -> 145, 32^3 FP32 35 -> 31) but for short rows
// over many lines (32 x 128 x 128 FP64 46 -> 49 us, 30 x 128 x 100 FP32 36 -> 40:
// threads and column tiles mostly masked) and for small meshes of powers of two
// with few rows along y and long lines along z (16 x 16 x 256 FP32 26 -> 33, 128 x
// 16 x 128 FP32 29 -> 36.5, FP64 32 -> 37, 256 x 16 x 256 59 -> 63; 256 x 32 x 256
// 84 -> 78: few work-groups, and the library's shortest plans).  Walls in FP64: large planes
// (1024 x 1024 x 16 509 -> 402 us, 384 x 384 x 64 251 -> 193, 256^3 301 -> 293);
// smaller ones are better off with hipFFT's fewer launches (128^3 71 -> 80,
// 180 x 240 x 100 92 -> 105, 256 x 256 x 64 95 -> 98).  Walls in FP32 stay with
// hipFFT (512^3: 1880 against 1290 us): after a step the mean mode of the next
// right-hand side is what rounding left, which the solve along z amplifies by up
// to nz^2, and other sums, no further from the truth, move a second step's P by
// up to 4e-5 of it.
inline bool own_transforms(int nx, int ny, int nz, bool walls, int precision)
{
    const int64_t plane = (int64_t)nx * ny;
    if (walls) return precision == CH_FP64 && plane >= 65536 && plane * nz >= 4194304;
    const bool p2 = ((nx & (nx - 1)) | (ny & (ny - 1)) | (nz & (nz - 1))) == 0;
    if (p2 && ny <= 32 && nz >= 64 && plane * nz <= (1 << 20)) return false;
    return nx >= 36 || ny < 64;
}

// Whether a solve takes the own transforms, and the passes of their lines (two
// axes between walls).
inline bool own_lines(const int n[3], bool walls, int precision, chk::FftLine line[3])
{
    bool own = own_transforms(n[0], n[1], n[2], walls, precision);
    for (int d = 0; d < (walls ? 2 : 3); ++d)
        own = chk::fft_radices(n[d], precision == CH_FP32, &line[d]) && own;
    return own;
}

// Twiddles exp(-2 pi i m / n), m < n, as (re, im) pairs: formed in extended
// precision and rounded once.  From an angle rounded to double they are off by up
// to 4 units in the last place, which lines of 1000 points show (40 x 30 x 1000
// periodic FP64, rms error of a solve 8.8e-16 instead of 5.5e-16 of the rms).
inline std::vector<double> fft_twiddles(int n)
{
    const long double two_pi = 6.283185307179586476925286766559L;
    std::vector<double> w(2 * (size_t)n);
    for (int m = 0; m < n; ++m) {
        w[2 * m] = (double)std::cos(two_pi * m / n);
        w[2 * m + 1] = (double)-std::sin(two_pi * m / n);
    }
    return w;
}

}  // namespace chp
