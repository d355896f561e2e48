// bins_fft.h -- fast cosine and sine transforms of the bin scheme (bins_fft.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "common.h"

namespace pp {

// Epilogue factor of the binned coefficients (eqs. disa-a..d) for row u, column p; su = sin(u pi / 2m), sp likewise.
__device__ __forceinline__ double disa_factor(int u, int p, double su, double sp, double W, double H, int m) {
    const double pi = kPi;
    if (u == 0 && p == 0) return 0.0;
    if (u == 0) return 4.0 * H * H / ((double)p * p * p * pi * pi * pi * m) * sp;
    if (p == 0) return 4.0 * W * W / ((double)u * u * u * pi * pi * pi * m) * su;
    return 16.0 * W * W * H * H / ((double)u * p * ((double)u * u * H * H + (double)p * p * W * W) * pi * pi * pi * pi) *
           su * sp;
}

// Transform length m (bins per axis) as complex transforms of length L, a power of two:
//   m itself a power of two in [64, 8192]: L = m;
//   any other m up to 4096: L the power of two from max(8, 2 m - 1) on (the convolution length of
//   Bluestein's chirp transform).
// Larger m (and 4096 < m < 16384 other than 8192) have L = 0: no complex transform of 8192 points
// (144 KB of LDS) holds them, and the matrix products of bins.hip serve.
struct BinFft {
    int m, L;
    bool chirp;          // Bluestein's form
};

inline BinFft bin_fft_plan(int m) {
    BinFft f{m, 0, false};
    if (m >= 64 && m <= 8192 && (m & (m - 1)) == 0) {
        f.L = m;
    } else if (m <= 4096) {
        f.chirp = true;
        f.L = 8;
        while (f.L < 2 * m - 1) f.L *= 2;
    }
    return f;
}

// Doubles of the device tables.  L = m: m phases and m twiddles, complex.  Bluestein's form: m phases, L / 4 twiddles and L / 2 + 1
// points of the chirp's transform, at most 8 m doubles from m = 3 on (L <= 4 m - 4), 16 and 18 at m = 1 and 2 (L = 8).
inline size_t bin_fft_table_doubles(const BinFft &f) {
    if (!f.chirp) return 4 * (size_t)f.m;
    return 2 * ((size_t)f.m + (size_t)f.L / 4 + (size_t)f.L / 2 + 1);
}

// Points per workgroup: row passes 2048 (36 KB of LDS: four workgroups per CU) or one transform; column passes four
// transforms, eight columns, so that a row of them fills half a cache line, up to 8192 points.
inline int bin_fft_points(const BinFft &f, bool col) {
    const int pts = col ? 4 * f.L : f.L;
    return pts < 2048 ? 2048 : pts > 8192 ? 8192 : pts;
}

// Workgroups of one pass over `count` rows or columns (a transform is a pair of them).
inline int bin_fft_workgroups(const BinFft &f, bool col, int count) {
    const int G = bin_fft_points(f, col) / f.L;
    return ((count + 1) / 2 + G - 1) / G;
}

// Whether the fast transforms are the faster route for the coefficients; with a chirp, its table, made by one workgroup in each
// call, is most of a short call, and the products of m <= 32 are one chunk (both routes, us: m = 3 17.6 products, 15.5 fast; 8
// 18.0 and 22; 32, 1 x 1 17.7 and 24.3, 32 x 32 22.9 and 26.9; 48, 8 x 48 29.5 and 31.8, 24 x 24 32.4 and 31.9, 48 x 8 33.6 and 31.5; 65, 1 x 1 38.1 and 30.7).
inline bool bin_fft_for_coeffs(const BinFft &f, int Mu, int Mp) {
    if (f.L == 0) return false;
    return !f.chirp || f.m <= 4 || f.m >= 64 || (f.m > 32 && Mu > 16 && Mp > (Mu > 32 ? 4 : 16));
}

// Estimated time in us of a field with its three outputs: two transforms of Mu rows, three of m columns.  Fitted to 2,900 calls,
// m = 65 to 8192, 1 to 1024 frequencies (root mean square of the error 7 %): launches and tables, then the passes at the rate
// of 256 CUs; a workgroup of one pair of columns (L = 8192) loads and stores 16 bytes of a cache line.
inline double bin_fft_field_us(const BinFft &f, int Mu) {
    int lg = 0;
    while ((1 << lg) < f.L) ++lg;
    const double stages = (lg + 2) / 3 * (f.chirp ? 2 : 1);
    double us = 20.0 + (f.chirp ? 11.0 + 56.0 * f.L / 8192 : 0.0);
    for (const bool col : {false, true}) {
        const int pts = bin_fft_points(f, col), wgs = bin_fft_workgroups(f, col, col ? f.m : Mu) * (col ? 3 : 2);
        us += wgs / 256.0 * (pts / 8192.0 * (20.0 + 0.9 * stages) + (col && pts == f.L ? 15.0 : 0.0));
    }
    return us;
}

// Fills the device tables (bin_fft_table_doubles: phases, twiddles, the chirp's transform) that the transforms read.
hipError_t launch_bin_fft_tables(const BinFft &f, double *tab, hipStream_t s);

// Coefficients: Q[l][p] = sum_j P[l][j] C_p(j) (Q: m x Mp scratch), then
// a[u][p] = disa(u, p) sum_l C_u(l) Q[l][p].
hipError_t launch_bin_fft_coeffs(const BinFft &f, const double *tab, const double *P, double *Q, double *a, int Mu,
                                 int Mp, double W, double H, hipStream_t s);

// Field: R[u][j] = sum_p a_up C_p(j) and Rs[u][j] = sum_p (p pi / H) a_up S_p(j) (Mu x m scratch each), then psi, xi_x
// and xi_y at the bin centres; a NULL output is not written.
hipError_t launch_bin_fft_field(const BinFft &f, const double *tab, const double *a, double *R, double *Rs, double *psi,
                                double *xix, double *xiy, int Mu, int Mp, double W, double H, hipStream_t s);

}  // namespace pp
