// bins_fft.h -- fast cosine and sine transforms of the bin scheme (bins_fft.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace pp {

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
