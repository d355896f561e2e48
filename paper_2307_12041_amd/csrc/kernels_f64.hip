// kernels_f64.hip -- FP64 and FP32 paths: basis tiles generated on chip in FP64 (rounded to the
// operand type when stored), contractions on v_mfma_f64_16x16x4 (FP64) or v_mfma_f32_16x16x4 (FP32).
//
// Forward (coefficients, Sec. III-A closed forms): At[u][p] = sum_i S_iu T_ip over a K range of
// blocks, one FP64 partial per split.  Backward (field of eq. ksi integrated over each block):
// G[i][n] = sum_k A_ik B[k][n] with the sine-difference basis A generated along the K frequency
// axis, then the row dot  g_i = sum_n E_in G[i][n]  with the cosine-difference basis E.
//
// Lane layouts (16x16 output, K = 4, one value per lane for A and B): A[i][k] in lane i + 16k and
// B[k][j] in lane j + 16k for both; the output differs:
//   v_mfma_f64_16x16x4: D[i][j] in lane j + 16 (i % 4), element i / 4;
//   v_mfma_f32_16x16x4: D[i][j] in lane j + 16 (i / 4), element i % 4.
//
// What bounds these kernels (gfx950, measured with a kernel of MFMAs and VALU instructions alone): the FP64 and FP32 MFMAs run
// on the vector units, so nothing issues beside them.  A v_mfma_f64_16x16x4 takes 65-68 cycles, a v_mfma_f32_16x16x4 33, and every
// VALU instruction of any type, of the same or of another wave of the SIMD, adds 4.3 cycles, or about 8 where it
// alternates with another wave's MFMAs, plus some 12 at each change from MFMA to VALU in a wave.  Hence: as few VALU
// instructions per MFMA as possible (operand tiles copied straight into LDS, seeds by a short polynomial and shared between
// threads, long runs, wide tiles for the shorter FP32 MFMAs), and the generator in phases of its own at raised wave
// priority, so that it is not dealt between another wave's MFMAs one instruction at a time.
//
// Basis generation: every value comes from FP64 three-term recurrences f_{k+1} = 2 cos(t) f_k - f_{k-1} over runs of at most 32
// frequencies that start from exactly reduced FP64 seeds: sine differences as 2 cos(k a) sin(k b) and cosine
// differences as -2 sin(k a) sin(k b) with a = pi c / L, b = pi size / (2L) for centre c (no cancellation for narrow blocks).
#include <type_traits>

#include "basis_gen.h"
#include "common.h"

namespace pp {
namespace {

// Operand type T: the MFMA and its output row for (lane, element).
template <typename T> struct Mat;
template <> struct Mat<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mfma(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }
};
template <> struct Mat<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mfma(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// sin(pi t) and cos(pi t), |t| < 2^50: t = q / 2 + f exactly with an integer q (its low bits are read off the sum that
// rounds it) and |f| <= 1/4, then the Taylor polynomials of sin(pi f) and cos(pi f) (coefficients pi^j / j!, rounded; the first
// term left out is below 2^-58 of the result).  An infinite or NaN t gives NaN.  The callers' t is a frequency (at most 2^16) times
// a phase reduced by whole turns, so that it stays in that range however far outside the region a block lies.
__device__ __forceinline__ void sincospi_seed64(double t, double &s, double &c) {
    const double magic = 6755399441055744.0;   // 1.5 * 2^52
    const double d = fma(2.0, t, magic);
    const unsigned q = (unsigned)__builtin_bit_cast(unsigned long long, d);
    const double f = fma(-0.5, d - magic, t);
    const double x = f * f;
    double p = 7.95205400147551261e-07, r = 4.30306958703294729e-06;
    p = fma(p, x, -2.19153534478302173e-05); r = fma(r, x, -1.04638104924845705e-04);
    p = fma(p, x, 4.66302805767612554e-04);  r = fma(r, x, 1.92957430940392314e-03);
    p = fma(p, x, -7.37043094571435044e-03); r = fma(r, x, -2.58068913900140612e-02);
    p = fma(p, x, 8.21458866111282326e-02);  r = fma(r, x, 2.35330630358893206e-01);
    p = fma(p, x, -5.99264529320792105e-01); r = fma(r, x, -1.33526276885458950e+00);
    p = fma(p, x, 2.55016403987734552e+00);  r = fma(r, x, 4.05871212641676848e+00);
    p = fma(p, x, -5.16771278004997026e+00); r = fma(r, x, -4.93480220054467900e+00);
    p = fma(p, x, 3.14159265358979312e+00);  r = fma(r, x, 1.0);
    p *= f;
    const double s0 = (q & 1u) ? r : p, c0 = (q & 1u) ? p : r;
    // quarter turns: (s, c), (c, -s), (-s, -c), (-c, s)
    const unsigned long long ns = (unsigned long long)(q & 2u) << 62, nc = (unsigned long long)((q + 1u) & 2u) << 62;
    s = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, s0) ^ ns);
    c = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, c0) ^ nc);
}

struct Phasor {
    double c, s;
    __device__ __forceinline__ void set(double t) { sincospi_seed64(t, s, c); }
    __device__ __forceinline__ void rotate(const Phasor &r) {
        const double t = fma(c, r.c, -(s * r.s));
        s = fma(s, r.c, c * r.s);
        c = t;
    }
};

// One factor of a basis value over consecutive frequencies: f and the value before it.
struct Rec {
    double f, fm, t2;
    // cos (or sin) of k theta from the phasor of k theta and the one of theta
    __device__ __forceinline__ void start_cos(const Phasor &p, const Phasor &step) {
        f = p.c; fm = fma(p.c, step.c, p.s * step.s); t2 = 2.0 * step.c;
    }
    __device__ __forceinline__ void start_sin(const Phasor &p, const Phasor &step) {
        f = p.s; fm = fma(p.s, step.c, -(p.c * step.s)); t2 = 2.0 * step.c;
    }
    __device__ __forceinline__ void next() {
        const double n = fma(t2, f, -fm);
        fm = f;
        f = n;
    }
};

// Runs of one block's (or point's) basis values of one kind along one axis: the phasors of the first frequency, of one
// frequency and of the jump from a run to the thread's next one.  A thread group shares the last two: `groups` threads per
// block evaluate them in turn and exchange them through LDS.
template <int KIND>
struct BlockRuns {
    static constexpr bool kSize = KIND == RUN_SINDIFF || KIND == RUN_COSDIFF;
    Phasor pa, pb, step_a, step_b, jump_a, jump_b;
    double size;

    // Every thread of the workgroup calls this; ph: LDS for 4 phasors per block; i: the block's index of `blocks`.
    template <int GROUPS, int BLOCKS>
    __device__ __forceinline__ void init(double c, double sz, double L, int k0, int J, double2 *ph, int i, int group) {
        const double ta = gen::reduce_half_turns(c / L), tb = gen::reduce_half_turns(0.5 * sz / L);
        size = sz;
        pa.set((double)k0 * ta);
        if constexpr (kSize) pb.set((double)k0 * tb);
        constexpr int PER = (4 + GROUPS - 1) / GROUPS;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int w = group + q * GROUPS;   // 0: step of a, 1: step of b, 2: jump of a, 3: jump of b
            if (w < 4) {
                const double t = (w & 1) ? tb : ta;
                Phasor p;
                p.set((w & 2) ? (double)J * t : t);
                ph[w * BLOCKS + i] = double2{p.c, p.s};
            }
        }
        __syncthreads();
        auto get = [&](int w) { const double2 v = ph[w * BLOCKS + i]; return Phasor{v.x, v.y}; };
        step_a = get(0);
        jump_a = get(2);
        if constexpr (kSize) { step_b = get(1); jump_b = get(3); }
        __syncthreads();
    }

    // The R values at frequencies k0 .. k0 + R - 1 (the run's place), written at dst[k * stride], rounded to T; pil = pi / L.
    // (An absent block has size 0: its differences vanish by themselves.)
    template <int R, typename T>
    __device__ __forceinline__ void gen(int k0, double pil, T *dst, int stride) const {
        Rec a, b;
        if constexpr (KIND == RUN_SINDIFF || KIND == RUN_COS) a.start_cos(pa, step_a);
        else a.start_sin(pa, step_a);
        if constexpr (kSize) {
            b.start_sin(pb, step_b);
            const double m = KIND == RUN_SINDIFF ? 2.0 : -2.0;
            b.f *= m;
            b.fm *= m;
        }
        double w = (double)k0 * pil;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            double v;
            if constexpr (kSize) v = a.f * b.f;
            else if constexpr (KIND == RUN_COS) v = a.f;
            else { v = w * a.f; w = (double)(k0 + k + 1) * pil; }
            if (KIND == RUN_SINDIFF && k == 0) v = k0 == 0 ? size : v;
            dst[k * stride] = (T)v;
            a.next();
            if constexpr (kSize) b.next();
        }
    }
    __device__ __forceinline__ void jump() {
        pa.rotate(jump_a);
        if constexpr (kSize) pb.rotate(jump_b);
    }
};

// The value of the lane with the same lane % 32 in the lower (x) and in the upper half of the wave (y).
__device__ __forceinline__ void both_halves(double v, double &x, double &y) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    x = __builtin_bit_cast(double, (unsigned long long)lo[0] | (unsigned long long)hi[0] << 32);
    y = __builtin_bit_cast(double, (unsigned long long)lo[1] | (unsigned long long)hi[1] << 32);
}

constexpr int kK = 32;   // K chunk of both contractions: blocks (forward) or frequencies (row form)

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void wait_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ------------------------------------------------------------------------------------------------
// Forward: grid (tiles_u * tiles_p, splits), 256 threads as 2 x 2 waves over a TILE x TILE tile.
// LDS holds the K chunk of the two basis tiles, k-major: Xs[kb][u], Ys[kb][p].  A side's 128 threads take block j % 32 and
// runs j / 32, j / 32 + 4; the two halves of a wave hold two runs of the same blocks and share the one-frequency phasors.
// Measured at 200,050 blocks and 512 x 512: FP64 1.65 ms, FP32 (TILE 256) 0.93 ms; with a library sincospi per factor and run
// and FP32 tiles of 128: 1.73 and 1.03 ms.
// Row strides: 4 past the tile in FP64 (the 16-byte stores of 8 lanes, 8 blocks, fall on different banks; operand reads
// two-way), 16 past it in FP32 (reads free of conflicts, stores two-way).
// ------------------------------------------------------------------------------------------------
template <typename T, int TILE>
__global__ __launch_bounds__(256, TILE == 256 ? 1 : 2) void k_fwd_mat(int64_t n, int Mu, int Mp, double W, double H,
                                                                     const double *__restrict__ x,
                                                                     const double *__restrict__ y,
                                                                     const double *__restrict__ w,
                                                                     const double *__restrict__ h,
                                                                     T *__restrict__ part, int tiles_p, int64_t chunks,
                                                                     int64_t chunks_per_split) {
    typedef typename Mat<T>::v4 v4;
    constexpr int LD = TILE + (sizeof(T) == 8 ? 4 : 16);
    __shared__ __attribute__((aligned(16))) T Xs[kK * LD];
    __shared__ __attribute__((aligned(16))) T Ys[kK * LD];
    constexpr int WT = TILE / 2, S = WT / 16;
    constexpr int R = TILE >= 128 ? 32 : TILE / 4, RUNS = TILE / (4 * R);   // run length, runs per thread
    constexpr int PER = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(PER)));

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tu0 = (int)(blockIdx.x / tiles_p) * TILE, tp0 = (int)(blockIdx.x % tiles_p) * TILE;
    const int wu0 = (wave >> 1) * WT, wp0 = (wave & 1) * WT;
    const int64_t c_begin = (int64_t)blockIdx.y * chunks_per_split;
    const int64_t c_end = min(chunks, c_begin + chunks_per_split);

    const bool side_y = tid >= 128;
    const int kb = tid & 31, run = (tid >> 5) & 3;
    const double L = side_y ? H : W;
    const int f0 = (side_y ? tp0 : tu0) + run * R;
    T *dst = (side_y ? Ys : Xs) + kb * LD + run * R;

    v4 acc[S][S];
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < S; ++b) acc[a][b] = v4{(T)0, (T)0, (T)0, (T)0};

    // Block data are requested a chunk ahead, centres by the lower half of a wave and sizes by the upper one; past the last block:
    // an absent one (size 0).  Each half divides and reduces its own phase, a = pi c / L or b = pi size / (2L).
    const double *__restrict__ src = side_y ? (lane < 32 ? y : h) : (lane < 32 ? x : w);
    const double period = lane < 32 ? L : 2.0 * L;
    auto fetch = [&](int64_t c) {
        const int64_t ib = c * kK + kb;
        const bool in = ib < n;
        const double v = src[in ? ib : 0];
        return in ? v : 0.0;
    };
    double pv = c_begin < c_end ? fetch(c_begin) : 0.0;
    for (int64_t c = c_begin; c < c_end; ++c) {
        const double t = gen::reduce_half_turns(pv / period);
        double ctr, sz, ta, tb;
        both_halves(pv, ctr, sz);
        both_halves(t, ta, tb);
        if (c + 1 < c_end) pv = fetch(c + 1);
        __builtin_amdgcn_s_setprio(3);
        Phasor own, step_a, step_b;
        own.set(t);
        both_halves(own.c, step_a.c, step_b.c);
        both_halves(own.s, step_a.s, step_b.s);
        lds_barrier();   // the previous chunk has been contracted
#pragma unroll
        for (int i = 0; i < RUNS; ++i) {
            const int k0 = f0 + i * 4 * R;
            Phasor pa, pb;
            pa.set((double)k0 * ta);
            pb.set((double)k0 * tb);
            Rec a, b;
            a.start_cos(pa, step_a);
            b.start_sin(pb, step_b);
            b.f *= 2.0;
            b.fm *= 2.0;
            vec v;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                double val = a.f * b.f;
                if (k == 0) val = k0 == 0 ? sz : val;
                v[k % PER] = (T)val;
                if (k % PER == PER - 1) *(vec *)(dst + i * 4 * R + k - (PER - 1)) = v;
                a.next();
                b.next();
            }
        }
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();
#pragma unroll
        for (int ks = 0; ks < kK / 4; ++ks) {
            const int kr = ks * 4 + (lane >> 4);
            T av[S], bv[S];
#pragma unroll
            for (int a = 0; a < S; ++a) av[a] = Xs[kr * LD + wu0 + a * 16 + (lane & 15)];
#pragma unroll
            for (int b = 0; b < S; ++b) bv[b] = Ys[kr * LD + wp0 + b * 16 + (lane & 15)];
#pragma unroll
            for (int a = 0; a < S; ++a)
#pragma unroll
                for (int b = 0; b < S; ++b) acc[a][b] = Mat<T>::mfma(av[a], bv[b], acc[a][b]);
        }
    }

    T *out = part + (size_t)blockIdx.y * (size_t)Mu * (size_t)Mp;
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < S; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int u = tu0 + wu0 + a * 16 + Mat<T>::row(lane, r);
                const int p = tp0 + wp0 + b * 16 + (lane & 15);
                if (u < Mu && p < Mp) out[(size_t)u * Mp + p] = acc[a][b][r];
            }
}

// ------------------------------------------------------------------------------------------------
// Row-form contraction (the backward and the evaluation entry points): for each block (or point)
// i of a TB tile and each epilogue frequency j of a TN tile,
//     Z_ij = sum_k Bas_ik B[k][j]          (K loop over the Ka frequencies of one axis, MFMA),
//     out_i += sum_j E_ij Z_ij             (fused row-dot epilogue, FP64),
// with Bas of kind KA_KIND along the K axis and E of kind EP1 (and, if EP2 >= 0, a second
// epilogue of kind EP2 on the same Z into gpart2).  Grid (tiles_b, N tiles of the one or two contractions), 256 threads as 2 x 2
// waves; wave column wc owns the 16-column tiles 2 b + wc.  LDS: As[k][i] (generated basis of the chunk), two buffers
// Bs[k][j] of half a chunk each, filled by direct copies (global memory to LDS) while the other half is contracted; after the K
// loop the same space holds the epilogue basis of 64 columns, Es[j][i].  Two workgroups per CU.
// Measured per gradient (both axes) at 200,050 blocks and 512 x 512: FP64 3.23 ms, 65 TFLOP/s of the 71.6 that a large library product
// reaches (generator 4 %, epilogue 1 %, the rest MFMAs at 67 cycles and barriers), FP32 1.78 ms, 118 TFLOP/s (generator, copies and
// epilogue 5-6 % each); with one buffer, loads and generation between barriers: 3.83 and 2.18 ms.
// VEC: B's rows are aligned to 16 bytes and a tile row is 1024: one 16-byte copy per lane and row.  Otherwise copies of 4 bytes
// per lane.
// ------------------------------------------------------------------------------------------------
template <typename T, int TB, int TN, bool VEC, int KA_KIND, int EP1, int EP2>
__global__ __launch_bounds__(256, 2) void k_bwd_mat(int64_t n, AxisPair<BwdAxis> P) {
    typedef typename Mat<T>::v4 v4;
    const bool second = (int)blockIdx.y >= P.tiles0;
    const BwdAxis ax = P.pick(second);
    const int ntile = (int)blockIdx.y - (second ? P.tiles0 : 0);
    constexpr int LB = TB + 16, LN = TN + 16, LE = TB + 1, KH = kK / 2, EC = 64;
    constexpr int GROUPS = 256 / TB;       // threads per block
    constexpr int RA = kK / GROUPS;        // K-side run per thread per chunk
    constexpr int RE = EC / GROUPS;        // epilogue run per thread and 64 columns
    constexpr int WI = TB / 2, SI = WI / 16, SJ = TN / 32;
    constexpr int BYTES_A = kK * LB * sizeof(T), BYTES_B = 2 * KH * LN * sizeof(T), BYTES_E = EC * LE * sizeof(T),
                  BYTES_P = 4 * TB * sizeof(double2);
    constexpr int SMEM0 = BYTES_A + BYTES_B > BYTES_E ? BYTES_A + BYTES_B : BYTES_E;
    constexpr int SMEM = SMEM0 > BYTES_P ? SMEM0 : BYTES_P;
    // one LDS object: with a second one the compiler makes every LDS read wait for all copies in flight
    __shared__ __attribute__((aligned(16))) char smem[SMEM + 2 * TB * (int)sizeof(double)];
    double *red = (double *)(smem + SMEM);
    T *As = (T *)smem, *Bs = (T *)(smem + BYTES_A), *Es = (T *)smem;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t ib0 = (int64_t)blockIdx.x * TB;
    const int n0 = ntile * TN;
    const int wi0 = (wave >> 1) * WI, wc = wave & 1;
    const int gi = tid % TB, group = tid / TB;
    const int64_t ib = ib0 + gi;
    const bool valid = ib < n;

    // Copies of the KH rows from k on into buffer h: wave w copies rows w, w + 4, ..; a row past Ka is a copy of no bytes, which
    // writes zeros (its basis values are zero too, and zero times an infinite coefficient of some other row would be NaN), and
    // columns past Nb hold whatever follows in B, within the buffer's bounds (the accumulators of such columns are cleared
    // before the epilogue).  Element counts fit 32 bits (at most 2^30).
    typedef __attribute__((address_space(3))) void lds_void;
    const int elems = ax.Ka * ax.Nb;
    auto copy_half = [&](int k, int h) {
#pragma unroll
        for (int q = 0; q < KH / 4; ++q) {
            const int row = 4 * q + wave;
            // (the address stays within B: one past it cost 0.6 us of a 10 us call; max(min()) would be made on the vector unit)
            const int at = min(k + row, ax.Ka - 1) * ax.Nb + n0, over = elems - at;
            const int left = k + row < ax.Ka ? (over < TN ? over : TN) : 0;
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                (void *)((const T *)ax.B + at), (short)0, left * (int)sizeof(T), 0x00020000);
            char *dst = smem + BYTES_A + (h * KH + row) * LN * (int)sizeof(T);
            if constexpr (VEC) {
                static_assert(TN * sizeof(T) == 1024, "one copy per row");
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void *)dst, 16, lane * 16, 0, 0, 0);
            } else {
#pragma unroll
                for (int g = 0; g < TN * (int)sizeof(T) / 256; ++g)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void *)(dst + 256 * g), 4, lane * 4 + 256 * g, 0, 0,
                                                             0);
            }
        }
    };
    // The runs' init uses the LDS of As and more; the first copies follow it.
    BlockRuns<KA_KIND> runs;
    {
        const double c = valid ? ax.ca[ib] : 0.0, sz = (valid && ax.sa) ? ax.sa[ib] : 0.0;
        runs.template init<GROUPS, TB>(c, sz, ax.La, group * RA, kK, (double2 *)smem, gi, group);
    }
    copy_half(0, 0);

    v4 acc[SI][SJ];
#pragma unroll
    for (int a = 0; a < SI; ++a)
#pragma unroll
        for (int b = 0; b < SJ; ++b) acc[a][b] = v4{(T)0, (T)0, (T)0, (T)0};

    for (int k0 = 0; k0 < ax.Ka; k0 += kK) {
        __builtin_amdgcn_s_setprio(3);
        const int ka = k0 + group * RA;
        T *dst = As + (group * RA) * LB + gi;
        runs.template gen<RA>(ka, 0.0, dst, LB);
        if (k0 + kK > ax.Ka) {   // the last chunk: no basis past Ka
#pragma unroll
            for (int k = 0; k < RA; ++k)
                if (ka + k >= ax.Ka) dst[k * LB] = (T)0;
        }
        runs.jump();
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            wait_copies();
            lds_barrier();
            if (h == 0) copy_half(k0 + KH, 1);
            else if (k0 + kK < ax.Ka) copy_half(k0 + kK, 0);
#pragma unroll
            for (int ks = 0; ks < KH / 4; ++ks) {
                const int kr = ks * 4 + (lane >> 4);
                T av[SI], bw[SJ];
#pragma unroll
                for (int a = 0; a < SI; ++a) av[a] = As[(h * KH + kr) * LB + wi0 + a * 16 + (lane & 15)];
#pragma unroll
                for (int b = 0; b < SJ; ++b) bw[b] = Bs[(h * KH + kr) * LN + (2 * b + wc) * 16 + (lane & 15)];
#pragma unroll
                for (int a = 0; a < SI; ++a)
#pragma unroll
                    for (int b = 0; b < SJ; ++b) acc[a][b] = Mat<T>::mfma(av[a], bw[b], acc[a][b]);
            }
        }
        lds_barrier();
    }
    if (n0 + TN > ax.Nb) {
#pragma unroll
        for (int b = 0; b < SJ; ++b)
            if (n0 + (2 * b + wc) * 16 + (lane & 15) >= ax.Nb)
#pragma unroll
                for (int a = 0; a < SI; ++a) acc[a][b] = v4{(T)0, (T)0, (T)0, (T)0};
    }

    // Epilogue(s): row dot with the epilogue basis, 64 columns (two column tiles of each wave) at a time; the 16 lanes that
    // share a row are summed by a fixed butterfly, the two column waves in fixed order.
    auto epilogue = [&](auto kind_tag, double *__restrict__ gpart, double *__restrict__ out) {
        constexpr int EK = decltype(kind_tag)::value;
        BlockRuns<EK> er;
        {
            const double c = valid ? ax.cb[ib] : 0.0, sz = (valid && ax.sb) ? ax.sb[ib] : 0.0;
            er.template init<GROUPS, TB>(c, sz, ax.Lb, n0 + group * RE, EC, (double2 *)smem, gi, group);
        }
        const double pil = kPi / ax.Lb;
        double rs[SI][4];
#pragma unroll
        for (int a = 0; a < SI; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) rs[a][r] = 0.0;
#pragma unroll
        for (int e = 0; e < TN / EC; ++e) {
            er.template gen<RE>(n0 + e * EC + group * RE, pil, &Es[(group * RE) * LE + gi], LE);
            if (e + 1 < TN / EC) er.jump();
            __syncthreads();
#pragma unroll
            for (int a = 0; a < SI; ++a)
#pragma unroll
                for (int b = 2 * e; b < 2 * e + 2; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int il = wi0 + a * 16 + Mat<T>::row(lane, r);
                        const int jl = (2 * b + wc) * 16 - e * EC + (lane & 15);
                        rs[a][r] = fma((double)acc[a][b][r], (double)Es[jl * LE + il], rs[a][r]);
                    }
            __syncthreads();
        }
#pragma unroll
        for (int a = 0; a < SI; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double v = rs[a][r];
                v += __shfl_xor(v, 1);
                v += __shfl_xor(v, 2);
                v += __shfl_xor(v, 4);
                v += __shfl_xor(v, 8);
                rs[a][r] = v;
            }
        if ((lane & 15) == 0) {
#pragma unroll
            for (int a = 0; a < SI; ++a)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[wc * TB + wi0 + a * 16 + Mat<T>::row(lane, r)] = rs[a][r];
        }
        __syncthreads();
        if (tid < TB && ib0 + tid < n) {
            const double v = red[tid] + red[TB + tid];
            if (!ax.out.r) gpart[(size_t)ntile * (size_t)n + (size_t)(ib0 + tid)] = v;
            else if (out) out[ib0 + tid] = (ax.out.dE ? *ax.out.dE : 1.0) * v;
        }
        __syncthreads();
    };
    epilogue(std::integral_constant<int, EP1>{}, ax.gpart, ax.out.r);
    if constexpr (EP2 >= 0) epilogue(std::integral_constant<int, (EP2 >= 0 ? EP2 : 0)>{}, ax.gpart2, ax.out.r2);
}

// Row form: with fewer workgroups of 128 blocks than this the chip is better filled by tiles of 32 blocks, which take a quarter
// of the time of one tile (a gradient in FP64, tiles of 32 against 128: 512 x 512, 2,000 blocks (128 workgroups) 62 against 91
// us; 300 x 300, 4,000 blocks (192) 55 against 62; 512 x 512, 4,000 blocks (256) 114 against 94; FP32 crosses at the same place).
constexpr int64_t kFewWorkgroups = 224;

template <typename T>
hipError_t launch_fwd_mat(const FwdPlan &pl, int64_t n, int Mu, int Mp, double W, double H, const double *x,
                          const double *y, const double *w, const double *h, T *part, hipStream_t s) {
    if (pl.tu != pl.tp || pl.kb != kK) return hipErrorInvalidValue;
    dim3 grid(pl.tiles_u * pl.tiles_p, pl.splits);
    auto launch = [&](auto kernel, int tiles_p) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, n, Mu, Mp, W, H, x, y, w, h, part, tiles_p, pl.chunks,
                           pl.chunks_per_split);
        return hipGetLastError();
    };
    if (pl.tu == 64) return launch(k_fwd_mat<T, 64>, pl.tiles_p);
    if (pl.tu != 128) return hipErrorInvalidValue;
    if constexpr (sizeof(T) == 4) {
        // FP32: four tiles as one of 256 x 256 (twice the MFMAs per generated value, one workgroup per CU) where no column or row is
        // padded for it, a split is long enough for the larger prologue and stores, and the rounds of 256 workgroups are
        // nearly full; the plan's splits stay, so that the sums of a split do not change.  (128 and 256, us: 512 x 512, 13
        // chunks a split 284 and 283, 49 chunks 958 and 933; 1024 x 1024, 5 chunks 139 and 149; 3000 x 3000, 2.25 rounds, 40 chunks
        // 883 and 1095.)
        const int tu = (pl.tiles_u + 1) / 2, tp = (pl.tiles_p + 1) / 2;
        const int64_t wgs = (int64_t)tu * tp * pl.splits, rounds = (wgs + 255) / 256;
        if (pl.tiles_u % 2 == 0 && pl.tiles_p % 2 == 0 && pl.chunks_per_split >= 12 && wgs >= 480 && 100 * wgs >= 93 * 256 * rounds) {
            grid.x = tu * tp;
            return launch(k_fwd_mat<T, 256>, tp);
        }
    }
    return launch(k_fwd_mat<T, 128>, pl.tiles_p);
}

template <typename T, int TB, int TN, bool VEC, int KA_KIND, int EP1, int EP2>
hipError_t launch_rowform_tile(int64_t n, const BwdAxis &ax0, const BwdAxis *ax1, hipStream_t s) {
    AxisPair<BwdAxis> P{{ax0, ax1 ? *ax1 : ax0}, (ax0.Nb + TN - 1) / TN};
    const int tiles1 = ax1 ? (ax1->Nb + TN - 1) / TN : 0;
    dim3 grid((unsigned)((n + TB - 1) / TB), (unsigned)(P.tiles0 + tiles1));
    hipLaunchKernelGGL((k_bwd_mat<T, TB, TN, VEC, KA_KIND, EP1, EP2>), grid, dim3(256), 0, s, n, P);
    return hipGetLastError();
}

template <typename T, int KA_KIND, int EP1, int EP2>
hipError_t launch_rowform(const BwdPlan &pl, int64_t n, const BwdAxis &ax0, const BwdAxis *ax1, hipStream_t s) {
    if (ax1 && (ax1->Ka + kK - 1) / kK > 2 * ((ax0.Ka + kK - 1) / kK))
        return launch_rowform<T, KA_KIND, EP1, EP2>(pl, n, *ax1, &ax0, s);   // (see AxisPair)
    if (!(pl.tb == 128 && pl.kk == kK && (pl.tn == 128 || (pl.tn == 256 && sizeof(T) == 4)))) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    if ((ax0.out.r && ax0.Nb > pl.tn) || (ax1 && ax1->out.r && ax1->Nb > pl.tn)) return hipErrorInvalidValue;
    const auto aligned = [](const BwdAxis &ax) {
        return (size_t)ax.Nb * sizeof(T) % 16 == 0 && (uintptr_t)ax.B % 16 == 0;
    };
    const bool vec = aligned(ax0) && (!ax1 || aligned(*ax1));
    if constexpr (sizeof(T) == 4) {
        if (pl.tn == 256) return vec ? launch_rowform_tile<T, 128, 256, true, KA_KIND, EP1, EP2>(n, ax0, ax1, s)
                                     : launch_rowform_tile<T, 128, 256, false, KA_KIND, EP1, EP2>(n, ax0, ax1, s);
    }
    // at most 64 frequencies on every N axis: half a tile; few workgroups of 128 blocks: tiles of 32
    const bool half = ax0.Nb <= 64 && (!ax1 || ax1->Nb <= 64);
    const int64_t wgs = (n + 127) / 128 * ((ax0.Nb + 127) / 128 + (ax1 ? (ax1->Nb + 127) / 128 : 0));
    const bool few = wgs < kFewWorkgroups;
    if (half) return few ? launch_rowform_tile<T, 32, 64, false, KA_KIND, EP1, EP2>(n, ax0, ax1, s)
                         : launch_rowform_tile<T, 128, 64, false, KA_KIND, EP1, EP2>(n, ax0, ax1, s);
    if (few) return launch_rowform_tile<T, 32, 128, false, KA_KIND, EP1, EP2>(n, ax0, ax1, s);
    if constexpr (sizeof(T) == 8)
        if (vec) return launch_rowform_tile<T, 128, 128, true, KA_KIND, EP1, EP2>(n, ax0, ax1, s);
    return launch_rowform_tile<T, 128, 128, false, KA_KIND, EP1, EP2>(n, ax0, ax1, s);
}

template <typename T>
hipError_t launch_rowform_kind(RowForm f, const BwdPlan &pl, int64_t n, const BwdAxis &ax, const BwdAxis *ax1,
                               hipStream_t s) {
    switch (f) {
        case ROW_FIELD: return launch_rowform<T, RUN_SINDIFF, RUN_COSDIFF, -1>(pl, n, ax, ax1, s);
        case ROW_POTENTIAL: return launch_rowform<T, RUN_SINDIFF, RUN_SINDIFF, -1>(pl, n, ax, ax1, s);
        case ROW_POINT_DUAL: return launch_rowform<T, RUN_COS, RUN_COS, RUN_WSIN>(pl, n, ax, ax1, s);
        case ROW_POINT_WSIN: return launch_rowform<T, RUN_COS, RUN_WSIN, -1>(pl, n, ax, ax1, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fwd_f64(const FwdPlan &pl, int64_t n, int Mu, int Mp, double W, double H, const double *x,
                          const double *y, const double *w, const double *h, double *part, hipStream_t s) {
    return launch_fwd_mat<double>(pl, n, Mu, Mp, W, H, x, y, w, h, part, s);
}
hipError_t launch_fwd_f32(const FwdPlan &pl, int64_t n, int Mu, int Mp, double W, double H, const double *x,
                          const double *y, const double *w, const double *h, float *part, hipStream_t s) {
    return launch_fwd_mat<float>(pl, n, Mu, Mp, W, H, x, y, w, h, part, s);
}
hipError_t launch_rowform_f64(RowForm f, const BwdPlan &pl, int64_t n, const BwdAxis &ax0, const BwdAxis *ax1,
                              hipStream_t s) {
    return launch_rowform_kind<double>(f, pl, n, ax0, ax1, s);
}
hipError_t launch_rowform_f32(RowForm f, const BwdPlan &pl, int64_t n, const BwdAxis &ax0, const BwdAxis *ax1,
                              hipStream_t s) {
    return launch_rowform_kind<float>(f, pl, n, ax0, ax1, s);
}

}  // namespace pp
