// kernels_common.hip -- precision-independent FP64 stages: split-K reduction + spectral scale +
// energy partials, the final energy sum, backward operand preparation, and the final per-block
// gradient sum.  Every reduction runs in a fixed order, so results are bitwise reproducible.
#include "common.h"

namespace pp {
namespace {

constexpr int kRedCoefs = 256;   // coefficients of a block of the split-K reduction: one wave, four a lane
constexpr int kRedBytes = 256;   // its bytes in flight per lane

// Deterministic block sum of one double per thread (butterfly inside waves, then wave order).
__device__ __forceinline__ double block_sum(double v, double *scratch) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) scratch[wave] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += scratch[k];
    return s;  // valid in thread 0
}

// Coefficients from the split-K partial contractions At = sum_s part[s]:
//   A_up = At_up / (wt_u vt_p),   a_up = s_up A_up,
//   s_up = e_u e_p / (W H (w_u^2 + v_p^2)), e_0 = 1, e_k = 2, s_00 = 0
// (the four coefficient cases of Sec. III-A written with one scale; a_00 = 0 is the
// compatibility condition).  The energy partial of this block is sum a_up A_up.
//
// Bound by reading the partials: a wave takes 256 coefficients, four per lane in vector loads, and keeps kRedBytes per lane
// (16 splits of FP32 partials) in flight, each load issued as soon as the value in its place is added.  No part of it waits
// for another wave.  The order is the one of a plain sum over the splits, so that the number in flight does not show in a
// result (the scale of the FP8 gradient's operands turns the last bit of a coefficient into 1e-8 of the gradient).
// 481 splits of 512 x 512 (504 MB): 111 us, 4.5 TB/s; 157 splits of 257 x 513: 17.5 us; 5 of 2048 x 2048: 110 us.
// (One load in a chain per coefficient took 249, 45 and 161 us; four groups of 256 threads that meet in LDS 127, 22 and 144;
// twice the bytes in flight 120 at 481 splits and the same elsewhere.)
template <typename T>
__global__ __launch_bounds__(64) void k_reduce_scale(const T *__restrict__ part, int splits, int Mu, int Mp, double W,
                                                     double H, double *__restrict__ a, double *__restrict__ epart) {
    constexpr int D = kRedBytes / (4 * sizeof(T));
    // A split's plane may begin at any element.
    typedef T Vec __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    const size_t MM = (size_t)Mu * (size_t)Mp;
    // four coefficients a lane: where fewer are left, the plane's last four; of a plane of fewer, one a lane
    const size_t idx = MM < 4 ? threadIdx.x : (size_t)blockIdx.x * kRedCoefs + 4 * threadIdx.x;
    const size_t at = MM < 4 ? idx : min(idx, MM - 4), end = MM < 4 ? min(idx + 1, MM) : MM;
    double At[4] = {};
    if (MM >= 4) {
        const T *__restrict__ p = part + at;
        Vec v[D];
#pragma unroll
        for (int k = 0; k < D; ++k) v[k] = *(const Vec *)(p + (size_t)min(k, splits - 1) * MM);
        int s = 0;
        for (; s + D < splits; s += D)
#pragma unroll
            for (int k = 0; k < D; ++k) {
#pragma unroll
                for (int c = 0; c < 4; ++c) At[c] += (double)v[k][c];
                v[k] = *(const Vec *)(p + (size_t)min(s + D + k, splits - 1) * MM);
            }
#pragma unroll
        for (int k = 0; k < D; ++k)
            if (s + k < splits)
#pragma unroll
                for (int c = 0; c < 4; ++c) At[c] += (double)v[k][c];
    } else if (at < MM) {
#pragma unroll 16
        for (int s = 0; s < splits; ++s) At[0] += (double)part[(size_t)s * MM + at];
    }
    double e = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const size_t id = at + c;
        if (id < idx || id >= end) continue;   // another lane's, or none
        const int u = (int)(id / (size_t)Mp), q = (int)(id % (size_t)Mp);
        const double wu = (double)u * kPi / W, vp = (double)q * kPi / H;
        const double wt = u ? wu : 1.0, vt = q ? vp : 1.0;
        const double A = At[c] / (wt * vt);
        const double eps = (u ? 2.0 : 1.0) * (q ? 2.0 : 1.0);
        const double sc = (u == 0 && q == 0) ? 0.0 : eps / (W * H * (wu * wu + vp * vp));
        const double av = sc * A;
        if (a) a[id] = av;
        e += av * A;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) e += __shfl_xor(e, off);
    if (threadIdx.x == 0) epart[blockIdx.x] = e;
}

// One workgroup of as many waves as there are partials for, at most kEnergyThreads (an energy of 5 blocks: 7.8 us with 64
// threads, 8.5 with 1024; the waves without partials only waited for each other).
constexpr int kEnergyThreads = 1024;

__global__ __launch_bounds__(kEnergyThreads) void k_energy_final(const double *__restrict__ epart, int nb,
                                                                 double *__restrict__ E) {
    __shared__ double scratch[kEnergyThreads / 64];
    double v = 0.0;
    const int threads = blockDim.x;
    int k = threadIdx.x;
    for (; k + 3 * threads < nb; k += 4 * threads) {
        double x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = epart[k + r * threads];
        v += (x[0] + x[1]) + (x[2] + x[3]);
    }
    for (; k < nb; k += threads) v += epart[k];
    const double s = block_sum(v, scratch);
    if (threadIdx.x == 0) *E = 0.5 * s;
}

// Operands of the row-form contractions: BxT[p][u] (K = p, epilogue over u) and By[u][p] (K = u,
// epilogue over p), a times the frequency factors of the chosen form.
template <typename T>
__global__ void k_prep_rowform(int form, const double *__restrict__ a, int Mu, int Mp, double W, double H,
                               T *__restrict__ BxT, T *__restrict__ By) {
    const size_t MM = (size_t)Mu * (size_t)Mp;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= MM) return;
    const int u = (int)(idx / (size_t)Mp), p = (int)(idx % (size_t)Mp);
    const double wt = u ? (double)u * kPi / W : 1.0, vt = p ? (double)p * kPi / H : 1.0;
    const double av = a[idx];
    double bx = av, by = av;
    if (form == ROW_FIELD) {
        bx = av / vt;
        by = av / wt;
    } else if (form == ROW_POTENTIAL) {
        bx = av / (vt * wt);
    }
    if (BxT) BxT[(size_t)p * Mu + u] = (T)bx;
    if (By) By[idx] = (T)by;
}

__global__ void k_bwd_final(const double *__restrict__ gpx, int tx, const double *__restrict__ gpy, int ty,
                            int64_t n, const double *__restrict__ dE, double *__restrict__ gx,
                            double *__restrict__ gy) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double d = dE ? *dE : 1.0;
    if (gx) {
        double sx = 0.0;
        for (int t = 0; t < tx; ++t) sx += gpx[(size_t)t * n + i];
        gx[i] = d * sx;
    }
    if (gy) {
        double sy = 0.0;
        for (int t = 0; t < ty; ++t) sy += gpy[(size_t)t * n + i];
        gy[i] = d * sy;
    }
}

}  // namespace

int reduce_scale_blocks(int Mu, int Mp) {
    const size_t MM = (size_t)Mu * (size_t)Mp;
    return (int)((MM + kRedCoefs - 1) / kRedCoefs);
}

hipError_t launch_reduce_scale(const void *part, bool part_f32, int splits, int Mu, int Mp, double W, double H,
                               double *a, double *epart, int *nblocks_out, hipStream_t s) {
    const int nb = reduce_scale_blocks(Mu, Mp);
    if (part_f32)
        hipLaunchKernelGGL(k_reduce_scale<float>, dim3(nb), dim3(64), 0, s, (const float *)part, splits, Mu, Mp, W, H, a,
                           epart);
    else
        hipLaunchKernelGGL(k_reduce_scale<double>, dim3(nb), dim3(64), 0, s, (const double *)part, splits, Mu, Mp, W, H, a,
                           epart);
    if (nblocks_out) *nblocks_out = nb;
    return hipGetLastError();
}

hipError_t launch_energy_final(const double *epart, int nblocks, double *E, hipStream_t s) {
    const int threads = nblocks < kEnergyThreads ? (nblocks + 63) / 64 * 64 : kEnergyThreads;
    hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(threads), 0, s, epart, nblocks, E);
    return hipGetLastError();
}

hipError_t launch_prep_rowform_f64(RowForm f, const double *a, int Mu, int Mp, double W, double H, double *BxT,
                                   double *By, hipStream_t s) {
    const size_t MM = (size_t)Mu * (size_t)Mp;
    hipLaunchKernelGGL(k_prep_rowform<double>, dim3((unsigned)((MM + 255) / 256)), dim3(256), 0, s, (int)f, a, Mu,
                       Mp, W, H, BxT, By);
    return hipGetLastError();
}

hipError_t launch_prep_rowform_f32(RowForm f, const double *a, int Mu, int Mp, double W, double H, float *BxT,
                                   float *By, hipStream_t s) {
    const size_t MM = (size_t)Mu * (size_t)Mp;
    hipLaunchKernelGGL(k_prep_rowform<float>, dim3((unsigned)((MM + 255) / 256)), dim3(256), 0, s, (int)f, a, Mu,
                       Mp, W, H, BxT, By);
    return hipGetLastError();
}

hipError_t launch_bwd_final(const double *gpx, int tx, const double *gpy, int ty, int64_t n, const double *dE,
                            double *gx, double *gy, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_bwd_final, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, gpx, tx, gpy, ty, n, dE, gx,
                       gy);
    return hipGetLastError();
}

}  // namespace pp
