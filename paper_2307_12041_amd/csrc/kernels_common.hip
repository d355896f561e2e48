// kernels_common.hip -- precision-independent FP64 stages: split-K reduction + spectral scale +
// energy partials, the final energy sum, backward operand preparation, and the final per-block
// gradient sum.  Every reduction runs in a fixed order, so results are bitwise reproducible.
#include "common.h"

namespace pp {
namespace {

constexpr int kRedThreads = 256;   // coefficients per block of the split-K reduction
constexpr int kRedGroups = 4;      // threads per coefficient
constexpr int kRedBatch = 32;       // splits per batch
constexpr int kRedMaxBlocks = 1 << 20;   // a grid stays below 2^32 work-items

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
// Bound by reading the partials.  A block takes 256 coefficients with kRedGroups threads each, in batches of
// kRedBatch splits: every thread has eight loads in flight, the batch meets in LDS, and the first group adds it in the order of
// the splits while the next batch is loaded.  The order is the one of a plain sum, so that neither the number of threads nor
// a change of it shows in a result (an e4m3 operand of the FP8 gradient turns the last bit of a coefficient into 2^-8 of it).
// (One thread per coefficient with its loads in a chain reached 2.0 TB/s on 481 splits of 512 x 512 (249 us, now 131:
// 3.9 TB/s) and was latency at 157 splits of 257 x 513 (45 us, now 22).)
template <typename T>
__global__ __launch_bounds__(kRedThreads * kRedGroups) void k_reduce_scale(const T *__restrict__ part, int splits, int Mu,
                                                                           int Mp, double W, double H,
                                                                           double *__restrict__ a,
                                                                           double *__restrict__ epart, int nb) {
    __shared__ T buf[kRedBatch][kRedThreads];
    __shared__ double scratch[kRedThreads * kRedGroups / 64];
    constexpr int PER = kRedBatch / kRedGroups;
    const size_t MM = (size_t)Mu * (size_t)Mp;
    const int t = threadIdx.x % kRedThreads, g = threadIdx.x / kRedThreads;
    for (int b = blockIdx.x; b < nb; b += gridDim.x) {
        const size_t idx = (size_t)b * kRedThreads + t;
        const T *__restrict__ p = part + (idx < MM ? idx : 0);
        double At = 0.0;
        T v[PER];
        auto fetch = [&](int s0) {   // splits s0 + PER g ..; past the last one the last again, which is not added
#pragma unroll
            for (int k = 0; k < PER; ++k) v[k] = p[(size_t)min(s0 + PER * g + k, splits - 1) * MM];
        };
        fetch(0);
        for (int s0 = 0; s0 < splits; s0 += kRedBatch) {
#pragma unroll
            for (int k = 0; k < PER; ++k) buf[PER * g + k][t] = v[k];
            __syncthreads();
            if (s0 + kRedBatch < splits) fetch(s0 + kRedBatch);
            if (g == 0) {
                if (s0 + kRedBatch <= splits) {
#pragma unroll
                    for (int k = 0; k < kRedBatch; ++k) At += (double)buf[k][t];
                } else {
                    for (int k = 0; k < splits - s0; ++k) At += (double)buf[k][t];
                }
            }
            __syncthreads();
        }
        double e = 0.0;
        if (g == 0 && idx < MM) {
            const int u = (int)(idx / (size_t)Mp), p = (int)(idx % (size_t)Mp);
            const double wu = (double)u * kPi / W, vp = (double)p * kPi / H;
            const double wt = u ? wu : 1.0, vt = p ? vp : 1.0;
            const double A = At / (wt * vt);
            const double eps = (u ? 2.0 : 1.0) * (p ? 2.0 : 1.0);
            const double sc = (u == 0 && p == 0) ? 0.0 : eps / (W * H * (wu * wu + vp * vp));
            const double av = sc * A;
            if (a) a[idx] = av;
            e = av * A;
        }
        const double sum = block_sum(e, scratch);
        if (threadIdx.x == 0) epart[b] = sum;
        __syncthreads();
    }
}

constexpr int kEnergyThreads = 1024;

__global__ __launch_bounds__(kEnergyThreads) void k_energy_final(const double *__restrict__ epart, int nb,
                                                                 double *__restrict__ E) {
    __shared__ double scratch[kEnergyThreads / 64];
    double v = 0.0;
    int k = threadIdx.x;
    for (; k + 3 * kEnergyThreads < nb; k += 4 * kEnergyThreads) {
        double x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = epart[k + r * kEnergyThreads];
        v += (x[0] + x[1]) + (x[2] + x[3]);
    }
    for (; k < nb; k += kEnergyThreads) v += epart[k];
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
    return (int)((MM + kRedThreads - 1) / kRedThreads);
}

hipError_t launch_reduce_scale(const void *part, bool part_f32, int splits, int Mu, int Mp, double W, double H,
                               double *a, double *epart, int *nblocks_out, hipStream_t s) {
    const int nb = reduce_scale_blocks(Mu, Mp);
    const int grid = nb < kRedMaxBlocks ? nb : kRedMaxBlocks;
    if (part_f32)
        hipLaunchKernelGGL(k_reduce_scale<float>, dim3(grid), dim3(kRedThreads * kRedGroups), 0, s, (const float *)part,
                           splits, Mu, Mp, W, H, a, epart, nb);
    else
        hipLaunchKernelGGL(k_reduce_scale<double>, dim3(grid), dim3(kRedThreads * kRedGroups), 0, s, (const double *)part,
                           splits, Mu, Mp, W, H, a, epart, nb);
    if (nblocks_out) *nblocks_out = nb;
    return hipGetLastError();
}

hipError_t launch_energy_final(const double *epart, int nblocks, double *E, hipStream_t s) {
    hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(kEnergyThreads), 0, s, epart, nblocks, E);
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
