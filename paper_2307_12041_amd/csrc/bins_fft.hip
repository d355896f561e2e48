// bins_fft.hip -- the separable cosine and sine transforms of the bin scheme (Sec. III-D, eqs. disa-a..d, dis-psi1,
// dis-ksi) as FP64 fast Fourier transforms in LDS.
//
// With N = m bins per axis and C_k(s) = cos(k (2s+1) pi / 2N), S_k(s) = sin(k (2s+1) pi / 2N):
//   forward   X_k = sum_s x_s C_k(s):  V = DFT of v, v_n = x_2n, v_{N-1-n} = x_{2n+1};  X_k = Re(e^{-i pi k / 2N} V_k);
//   inverse   y_s = sum_k c_k C_k(s):  v = inverse DFT of h, h_k = e^{i pi k / 2N} (c_k - i c_{N-k}) / 2, h_0 = c_0;
//             y_2n = v_n, y_{2n+1} = v_{N-1-n};
//   sine      sum_k c_k S_k(s) = (-1)^s sum_k c_{N-k} C_k(s).
// (The even-odd reordering is Makhoul's form of the cosine transform.)  One complex DFT carries two real transforms, as
// its real and imaginary part: the same transform of two neighbouring rows or columns.  (Rounding errors of one leak into
// the other in proportion to its size, so quantities of different magnitude, as psi and xi of one column, are not paired.)
//
// A length that is not a power of two takes Bluestein's form, V_k = b*_k sum_n (v_n b*_n) b_{k-n} with
// b_n = e^{i pi n^2 / N}: a cyclic convolution of length L >= 2N - 1 with the transform of b from a table.  Inverse
// transforms are forward ones with real and imaginary parts exchanged on the way in and out.
//
// An infinite or NaN element leaves every output of its pair of rows or columns without a finite value (a sum, a rotation or a
// product with a twiddle keeps one component of it so).  Each thread looks at its first output and, if it is not finite, sums all
// of its outputs directly instead: an infinity or NaN where the plain sum has one, a finite value for the pair's other member.
//
// Each pass reads and writes its arrays once; at m = 2048 a pass over one array moves 64 MiB that the memory-side cache
// holds.  Measured at m = 2048 (512): coefficients 21 + 31 us (11 + 9), field 47 + 93 us (10 + 13, two and three arrays),
// against 0.39-0.41 ms (0.09) for each of the seven transforms as a matrix product of 2 m^3 flops on the FP64 matrix cores
// (52 % of their peak at m = 2048; 16 workgroups in all at m = 512).  What is left is latency: a workgroup of a column pass
// loads, exchanges through LDS four times and stores with nothing of another workgroup to overlap (144 KB of LDS).
#include <math.h>

#include "bins_fft.h"
#include "common.h"

namespace pp {
namespace {

typedef double2 cplx;

__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return cplx{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return cplx{a.x - b.x, a.y - b.y}; }
__device__ __forceinline__ cplx cmul(cplx a, cplx b) { return cplx{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ cplx swapped(cplx a) { return cplx{a.y, a.x}; }
__device__ __forceinline__ cplx times_minus_i(cplx a) { return cplx{a.y, -a.x}; }

// Device tables (bin_fft_table_doubles of them):
//   T[k] = e^{i pi k / 2N}, k < N;
//   W[k] = e^{-2 pi i k / L}: k < L where L = N, one quadrant (k < L / 4) in Bluestein's form, which also has
//   Bh[k] = DFT_L(b) / L, k <= L / 2 (b is even, so Bh[L - k] = Bh[k]).
struct Tables {
    const cplx *T, *W, *Bh;
};

Tables tables(const BinFft &f, const double *tab) {
    Tables t;
    t.T = (const cplx *)tab;
    t.W = t.T + f.m;
    t.Bh = t.W + f.L / 4;
    return t;
}

// z times i^q (q modulo 4).
__device__ __forceinline__ cplx times_i_power(cplx z, int q) {
    const cplx t = (q & 1) ? cplx{-z.y, z.x} : z;
    return (q & 2) ? cplx{-t.x, -t.y} : t;
}

// e^{-2 pi i k / 2^lg} for 0 <= k < 2^lg.
template <bool CHIRP>
__device__ __forceinline__ cplx twiddle(const cplx *__restrict__ W, int k, int lg) {
    if constexpr (!CHIRP) return W[k];
    else return times_i_power(W[k & ((1 << (lg - 2)) - 1)], -(k >> (lg - 2)));
}

// b*_n = e^{-i pi n^2 / N}: the point 2 n^2 mod 4N of the circle that T holds a quadrant of.  n < N <= 4096: n^2 is exact in
// FP32, and its quotient by 2N (below 2048, inv = 1 / 2N) is at most one off.  (An integer division and a remainder here, in 24
// places of a thread, made the four passes of a 200 x 200 scheme 1.5 us longer together.)
__device__ __forceinline__ cplx chirp_conj(const cplx *__restrict__ T, int n, int N, float inv) {
    const int n2 = n * n;
    int r = n2 - (int)((float)n2 * inv) * 2 * N;   // n^2 mod 2N, give or take 2N
    r += r < 0 ? 2 * N : 0;
    r -= r >= 2 * N ? 2 * N : 0;
    const int q = 2 * r, quad = (q >= N) + (q >= 2 * N) + (q >= 3 * N);
    const cplx z = times_i_power(T[q - quad * N], quad);
    return cplx{z.x, -z.y};
}

// LDS: one complex of padding after every eight, so that the 16 lanes of a b128 access phase fall on different banks in
// every stage's writes (8 j + r becomes 9 j + r).
__device__ __forceinline__ int lpos(int i) { return i + (i >> 3); }
constexpr int lds_len(int n) { return n + n / 8; }

__device__ __forceinline__ void fft4(cplx &a, cplx &b, cplx &c, cplx &d) {   // natural order in and out
    const cplx y0 = cadd(a, c), y2 = csub(a, c), y1 = cadd(b, d), y3 = times_minus_i(csub(b, d));
    a = cadd(y0, y1); c = csub(y0, y1); b = cadd(y2, y3); d = csub(y2, y3);
}

__device__ __forceinline__ void fft8(cplx (&v)[8]) {
    const double q = 0.70710678118654752440;
    cplx s[4], d[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) { s[r] = cadd(v[r], v[r + 4]); d[r] = csub(v[r], v[r + 4]); }
    d[1] = cplx{q * (d[1].x + d[1].y), q * (d[1].y - d[1].x)};
    d[2] = times_minus_i(d[2]);
    d[3] = cplx{q * (d[3].y - d[3].x), -q * (d[3].x + d[3].y)};
    fft4(s[0], s[1], s[2], s[3]);
    fft4(d[0], d[1], d[2], d[3]);
#pragma unroll
    for (int r = 0; r < 4; ++r) { v[2 * r] = s[r]; v[2 * r + 1] = d[r]; }
}

// In-place Stockham DFTs of length L = 2^lg (lg >= 3) of all transforms of the workgroup: the thread with index j of its
// transform's L / 8 threads holds eight points per stage.  x: the transform's base in LDS (padded); W: twiddles in global
// memory (they stay in the caches).  Radix 8, after one radix 2 or 4 stage where 3 does not divide lg.  Every stage reads
// its points, meets at a barrier and writes them; the caller's data has to be complete, and the result is when it returns.
template <bool CHIRP>
__device__ __forceinline__ void dft(cplx *x, int j, int lg, const cplx *__restrict__ W) {
    const int E = 1 << (lg - 3);
    const int rem = lg % 3;
    cplx v[8];
    int ns = 1;
    if (rem) {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = x[lpos(j + r * E)];
        __syncthreads();
        if (rem == 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int o = 2 * (j + q * E);
                x[lpos(o)] = cadd(v[q], v[q + 4]);
                x[lpos(o + 1)] = csub(v[q], v[q + 4]);
            }
            ns = 2;
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                fft4(v[q], v[q + 2], v[q + 4], v[q + 6]);
                const int o = 4 * (j + q * E);
#pragma unroll
                for (int r = 0; r < 4; ++r) x[lpos(o + r)] = v[q + 2 * r];
            }
            ns = 4;
        }
        __syncthreads();
    }
    for (int sh = lg - 3 - rem; sh >= 0; sh -= 3, ns <<= 3) {   // ns = 2^(lg - 3 - sh)
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = x[lpos(j + r * E)];
        __syncthreads();
        const int jm = j & (ns - 1);
        if (ns > 1) {
            const int step = jm << sh;
#pragma unroll
            for (int r = 1; r < 8; ++r) v[r] = cmul(v[r], twiddle<CHIRP>(W, r * step, lg));
        }
        fft8(v);
        const int o = ((j - jm) << 3) + jm;
#pragma unroll
        for (int r = 0; r < 8; ++r) x[lpos(o + r * ns)] = v[r];
        __syncthreads();
    }
}

// T and W where L = N.
__global__ void k_fft_tables(int N, cplx *__restrict__ T, cplx *__restrict__ W) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N) return;
    double s, c;
    sincospi((double)k / (2.0 * N), &s, &c);
    T[k] = cplx{c, s};
    sincospi(2.0 * (double)k / (double)N, &s, &c);
    W[k] = cplx{c, -s};
}

// Bluestein's tables: one workgroup of L / 8 threads (Bh needs the others).
__global__ __launch_bounds__(1024) void k_fft_tables_chirp(int N, int lg, cplx *T, cplx *W, cplx *__restrict__ Bh) {
    __shared__ cplx lds[lds_len(8192)];
    const int L = 1 << lg, tid = threadIdx.x, nt = blockDim.x;
    const float inv = 1.0f / (float)(2 * N);
    double s, c;
    for (int k = tid; k < L / 4; k += nt) {
        sincospi(2.0 * (double)k / (double)L, &s, &c);
        W[k] = cplx{c, -s};
    }
    for (int k = tid; k < L; k += nt) lds[lpos(k)] = cplx{0.0, 0.0};
    for (int k = tid; k < N; k += nt) {
        sincospi((double)k / (2.0 * N), &s, &c);
        T[k] = cplx{c, s};
    }
    __syncthreads();
    for (int k = tid; k < N; k += nt) {
        const cplx b = chirp_conj(T, k, N, inv);
        lds[lpos(k)] = cplx{b.x, -b.y};
        if (k) lds[lpos(L - k)] = cplx{b.x, -b.y};
    }
    __syncthreads();
    dft<true>(lds, tid, lg, W);
    const double scale = 1.0 / (double)L;
    for (int k = tid; k <= L / 2; k += nt) {
        const cplx v = lds[lpos(k)];
        Bh[k] = cplx{v.x * scale, v.y * scale};
    }
}

enum Pass { ROW_FWD, COL_FWD, ROW_INV, COL_INV };

// One transform of a pass: input and output arrays, and for inverse passes cosine or sine of k scale c_k.
struct FftJob {
    const double *in;
    double *out;
    int sine;
    double scale;
};

struct FftArgs {
    int N, lg, Mu, Mp;
    Tables t;
    FftJob job[3];               // one after the other, `groups` workgroups each
    int groups;
    double W, H;
};

// The outputs of a thread (j of its transform's E), which are of a pair with elements that are not finite, as plain sums over the pair's
// elements (first member at p0, second at p1, stride es).
template <int PASS>
__device__ __forceinline__ void sum_directly(const FftArgs &A, const FftJob &job, int j, int E, const double *__restrict__ p0,
                                             const double *__restrict__ p1, size_t es, int n0, bool ok1, int ldo) {
    constexpr bool ROW = PASS == ROW_FWD || PASS == ROW_INV, FWD = PASS == ROW_FWD || PASS == COL_FWD;
    const int N = A.N, len = FWD ? N : ROW ? A.Mp : A.Mu, outs = PASS == ROW_FWD ? A.Mp : PASS == COL_FWD ? A.Mu : N;
    for (int i = j; i < outs; i += E) {
        double s0 = 0.0, s1 = 0.0;
        int at = FWD ? i : 0;   // i (2n + 1), or n (2i + 1), on the circle of 4N points
        for (int n = 0; n < len && !(isnan(s0) && isnan(s1)); ++n) {
            const int quad = (at >= N) + (at >= 2 * N) + (at >= 3 * N);
            const cplx z = times_i_power(A.t.T[at - quad * N], quad);
            const double f = job.sine ? z.y * ((double)n * job.scale) : z.x;
            s0 += p0[(size_t)n * es] * f;
            s1 += p1[(size_t)n * es] * f;
            at += FWD ? 2 * i : 2 * i + 1;
            at -= at >= 4 * N ? 4 * N : 0;
        }
        if constexpr (PASS == COL_FWD) {
            s0 *= disa_factor(i, n0, A.t.T[i].y, A.t.T[n0].y, A.W, A.H, N);
            if (ok1) s1 *= disa_factor(i, n0 + 1, A.t.T[i].y, A.t.T[n0 + 1].y, A.W, A.H, N);
        }
        const size_t o = ROW ? (size_t)n0 * ldo + i : (size_t)i * ldo + n0;
        job.out[o] = s0;
        if (ok1) job.out[o + (ROW ? (size_t)ldo : 1)] = s1;
    }
}

// One workgroup: G = PTS / L transforms in LDS, eight points per thread.  Row passes give each transform L / 8
// neighbouring threads, so that loads and stores run along rows; column passes deal neighbouring threads to neighbouring
// transforms (columns), and take their workgroups in XCD-major order, so that the workgroups that share the cache lines of
// neighbouring columns share an L2.
template <int PTS, int PASS, bool CHIRP>
__global__ __launch_bounds__(PTS / 8) void k_bin_fft(FftArgs A) {
    __shared__ cplx lds[lds_len(PTS)];
    constexpr bool COL = PASS == COL_FWD || PASS == COL_INV;
    const int N = A.N, lg = A.lg, L = 1 << lg, E = L >> 3, G = PTS >> lg;
    const int tid = threadIdx.x;
    const int f = COL ? (tid & (G - 1)) : tid / E, j = COL ? tid / G : (tid & (E - 1));
    const FftJob job = A.job[blockIdx.y];
    int wg = blockIdx.x;
    if (COL && A.groups % 8 == 0) wg = (wg % 8) * (A.groups / 8) + wg / 8;
    const int t = wg * G + f;                                            // transform: rows or columns 2t and 2t + 1
    constexpr bool ROW = PASS == ROW_FWD || PASS == ROW_INV;
    const int n0 = 2 * t;
    const int lim = PASS == ROW_FWD ? N : PASS == COL_FWD ? A.Mp : PASS == ROW_INV ? A.Mu : N;
    const bool ok0 = n0 < lim, ok1 = n0 + 1 < lim;
    const int ldi = PASS == ROW_FWD ? N : PASS == COL_FWD || PASS == ROW_INV ? A.Mp : N;
    const int ldo = PASS == ROW_FWD || PASS == COL_FWD ? A.Mp : N;
    cplx *x = lds + f * lds_len(L);
    const cplx *__restrict__ T = A.t.T;
    const float inv = 1.0f / (float)(2 * N);   // chirp_conj

    // ---- load: eight elements per thread at most, all in flight together ----
    cplx v[8];
    const size_t es = ROW ? 1 : (size_t)ldi, ps = ROW ? (size_t)ldi : 1;   // strides along the transform and across it
    const double *__restrict__ p0 = job.in + (ok0 ? (size_t)n0 * ps : 0);
    const double *__restrict__ p1 = job.in + (ok1 ? (size_t)(n0 + 1) * ps : 0);
    if constexpr (PASS == ROW_FWD || PASS == COL_FWD) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int n = j + r * E;
            const size_t o = n < N ? (size_t)n * es : 0;
            v[r] = cplx{p0[o], p1[o]};
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int n = j + r * E;
            if (n < N) {
                const int pos = (n & 1) ? N - 1 - (n >> 1) : n >> 1;
                cplx z = cplx{ok0 ? v[r].x : 0.0, ok1 ? v[r].y : 0.0};
                if (CHIRP) z = cmul(z, chirp_conj(T, pos, N, inv));
                x[lpos(pos)] = z;
            } else {
                x[lpos(n)] = cplx{0.0, 0.0};   // Bluestein's zero padding, N .. L - 1
            }
        }
    } else {
        // h_k of the pair from elements k and N - k
        const int K = PASS == ROW_INV ? A.Mp : A.Mu;                     // coefficients along the transform
        cplx c[8], d[8];   // (element k, element N - k) of the two
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int k = j + r * E, kn = N - k;
            const bool in0 = k < N && k < K, in1 = k < N && kn < K;
            const size_t o0 = in0 ? (size_t)k * es : 0, o1 = in1 ? (size_t)kn * es : 0;
            c[r] = cplx{p0[o0], p0[o1]};
            d[r] = cplx{p1[o0], p1[o1]};
            if (!(in0 && ok0)) c[r].x = 0.0;
            if (!(in1 && ok0)) c[r].y = 0.0;
            if (!(in0 && ok1)) d[r].x = 0.0;
            if (!(in1 && ok1)) d[r].y = 0.0;
            if (job.sine) {   // of k c_k: the cosine transform of the reversed sequence
                c[r] = cplx{(double)kn * c[r].y, (double)k * c[r].x};
                d[r] = cplx{(double)kn * d[r].y, (double)k * d[r].x};
            }
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int k = j + r * E;
            if (k < N) {
                // h = e^{i pi k / 2N} ((c_k - i c_{N-k}) + i (d_k - i d_{N-k})) / 2
                cplx z = cplx{0.5 * (c[r].x + d[r].y), 0.5 * (d[r].x - c[r].y)};
                z = cmul(z, T[k]);
                if (k == 0) z = cplx{c[r].x + c[r].y, d[r].x + d[r].y};   // (sine: 0 times element 0, element N is 0)
                z = swapped(z);
                if (CHIRP) z = cmul(z, chirp_conj(T, k, N, inv));
                v[r] = z;
            } else {
                v[r] = cplx{0.0, 0.0};
            }
            x[lpos(k)] = v[r];
        }
    }
    __syncthreads();

    // ---- transform ----
    dft<CHIRP>(x, j, lg, A.t.W);
    if constexpr (CHIRP) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int k = j + r * E;
            x[lpos(k)] = swapped(cmul(x[lpos(k)], A.t.Bh[min(k, L - k)]));
        }
        __syncthreads();
        dft<true>(x, j, lg, A.t.W);
    }
    auto get = [&](int k) {
        const cplx z = x[lpos(k)];
        return CHIRP ? cmul(swapped(z), chirp_conj(T, k, N, inv)) : z;
    };

    // ---- store ----
    double *__restrict__ out = job.out;
    bool bad = false;
    if constexpr (PASS == ROW_FWD || PASS == COL_FWD) {
        const int K = PASS == ROW_FWD ? A.Mp : A.Mu;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int k = j + r * E;
            if (k >= K || !ok0) continue;
            const cplx a = get(k), b = get(k ? N - k : 0), w = T[k];
            if (r == 0) bad = !(isfinite(a.x) && isfinite(a.y));
            // V = A + i B with A, B Hermitian; X = Re(e^{-i pi k / 2N} A), and the same of B
            double xa = 0.5 * (w.x * (a.x + b.x) + w.y * (a.y - b.y));
            double xb = 0.5 * (w.x * (a.y + b.y) - w.y * (a.x - b.x));
            if constexpr (PASS == ROW_FWD) {
                out[(size_t)n0 * ldo + k] = xa;
                if (ok1) out[(size_t)(n0 + 1) * ldo + k] = xb;
            } else {
                out[(size_t)k * ldo + n0] = xa * disa_factor(k, n0, w.y, T[n0].y, A.W, A.H, N);
                if (ok1) out[(size_t)k * ldo + n0 + 1] = xb * disa_factor(k, n0 + 1, w.y, T[n0 + 1].y, A.W, A.H, N);
            }
        }
    } else {
        const size_t eo = ROW ? 1 : (size_t)ldo, po = ROW ? (size_t)ldo : 1;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int s = j + r * E;
            if (s >= N || !ok0) continue;
            const cplx z = swapped(get((s & 1) ? N - ((s + 1) >> 1) : s >> 1));
            if (r == 0) bad = !(isfinite(z.x) && isfinite(z.y));
            const double sg = job.sine ? ((s & 1) ? -job.scale : job.scale) : 1.0;
            const size_t o = (size_t)n0 * po + (size_t)s * eo;
            out[o] = sg * z.x;
            if (ok1) out[o + po] = sg * z.y;
        }
    }
    if (bad) sum_directly<PASS>(A, job, j, E, p0, p1, es, n0, ok1, ldo);
}

int log2i(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

template <int PTS, int PASS>
hipError_t launch_pass(const BinFft &f, const FftArgs &A, int jobs, hipStream_t s) {
    const dim3 grid((unsigned)A.groups, (unsigned)jobs);
    if (f.chirp) hipLaunchKernelGGL((k_bin_fft<PTS, PASS, true>), grid, dim3(PTS / 8), 0, s, A);
    else hipLaunchKernelGGL((k_bin_fft<PTS, PASS, false>), grid, dim3(PTS / 8), 0, s, A);
    return hipGetLastError();
}

// `count`: rows or columns.
template <int PASS>
hipError_t launch_points(const BinFft &f, FftArgs A, int count, int jobs, hipStream_t s) {
    constexpr bool COL = PASS == COL_FWD || PASS == COL_INV;
    const int pts = bin_fft_points(f, COL);
    A.groups = bin_fft_workgroups(f, COL, count);
    if (pts == 2048) return launch_pass<2048, PASS>(f, A, jobs, s);
    if (pts == 4096) return launch_pass<4096, PASS>(f, A, jobs, s);
    return launch_pass<8192, PASS>(f, A, jobs, s);
}

}  // namespace

hipError_t launch_bin_fft_tables(const BinFft &f, double *tab, hipStream_t s) {
    const Tables t = tables(f, tab);
    if (f.chirp)
        hipLaunchKernelGGL(k_fft_tables_chirp, dim3(1), dim3(f.L / 8), 0, s, f.m,
                           log2i(f.L), (cplx *)t.T, (cplx *)t.W, (cplx *)t.Bh);
    else
        hipLaunchKernelGGL(k_fft_tables, dim3((unsigned)((f.m + 255) / 256)), dim3(256), 0, s, f.m, (cplx *)t.T,
                           (cplx *)t.W);
    return hipGetLastError();
}

hipError_t launch_bin_fft_coeffs(const BinFft &f, const double *tab, const double *P, double *Q, double *a, int Mu,
                                 int Mp, double W, double H, hipStream_t s) {
    FftArgs A{f.m, log2i(f.L), Mu, Mp, tables(f, tab), {}, 0, W, H};
    A.job[0] = FftJob{P, Q, 0, 1.0};
    hipError_t e = launch_points<ROW_FWD>(f, A, f.m, 1, s);
    if (e != hipSuccess) return e;
    A.job[0] = FftJob{Q, a, 0, 1.0};
    return launch_points<COL_FWD>(f, A, Mp, 1, s);
}

hipError_t launch_bin_fft_field(const BinFft &f, const double *tab, const double *a, double *R, double *Rs, double *psi,
                                double *xix, double *xiy, int Mu, int Mp, double W, double H, hipStream_t s) {
    FftArgs A{f.m, log2i(f.L), Mu, Mp, tables(f, tab), {}, 0, W, H};
    int jobs = 0;
    if (psi || xix) A.job[jobs++] = FftJob{a, R, 0, 1.0};
    if (xiy) A.job[jobs++] = FftJob{a, Rs, 1, kPi / H};
    hipError_t e = launch_points<ROW_INV>(f, A, Mu, jobs, s);
    if (e != hipSuccess) return e;
    jobs = 0;
    if (psi) A.job[jobs++] = FftJob{R, psi, 0, 1.0};
    if (xix) A.job[jobs++] = FftJob{R, xix, 1, kPi / W};
    if (xiy) A.job[jobs++] = FftJob{Rs, xiy, 0, 1.0};
    return launch_points<COL_INV>(f, A, f.m, jobs, s);
}

}  // namespace pp
