// dense.hip -- the small dense FP64 parts of CP-ALS and GD (Appendix B and C)
//
//  * Gram F^T F of a factor or of an MTTKRP result, FP64 accumulation on the
//    matrix cores (FP64 MFMA), a wave's tiles in registers for R <= 64, rows
//    staged in LDS above; then a fixed-order reduction over blocks.
//  * H = G_p * G_q + reg I (Appendix A: (A kr B)^T (A kr B) = A^T A * B^T B,
//    ridge term of the regularized update).
//  * One-workgroup FP64 solve: Cholesky inverse of H, or the Moore-Penrose
//    pseudo-inverse from a parallel cyclic Jacobi eigen-decomposition when a
//    pivot shows H is numerically singular.  Working set in LDS when small.
//  * Column norms, the new Gram and the fit from R x R algebra: with
//    Fhat = M H^-1,  Fhat^T Fhat = H^-1 (M^T M) H^-1, so
//    lambda_r^2 = [H^-1 M^T M H^-1]_rr and  <X, Xhat> = <Fhat, M> =
//    trace(H^-1 M^T M) for the last mode; ||Xhat||^2 = lambda^T (G_A * G_B *
//    G_C) lambda.
//  * Row maps F = M W (W = H^-1 diag(1/lambda)) and the GD gradient -M + F H:
//    on the matrix cores up to R = 128, or over LDS-staged row tiles with the
//    R x R matrix broadcast from LDS (some small ranks) or read from memory.
//  * The row systems of the joint model's ALS, four to a wave on the matrix
//    cores.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "internal.hpp"

namespace dfacto {
namespace {

constexpr int kBlock = 256;

template <typename T>
__device__ __forceinline__ double ld(const T *p, int64_t i);
template <>
__device__ __forceinline__ double ld<float>(const float *p, int64_t i) {
    return (double)p[i];
}
template <>
__device__ __forceinline__ double ld<uint16_t>(const uint16_t *p, int64_t i) {
    return (double)__uint_as_float((uint32_t)p[i] << 16);
}

template <typename T>
__device__ __forceinline__ float ldf(const T *p, int64_t i);
template <>
__device__ __forceinline__ float ldf<float>(const float *p, int64_t i) { return p[i]; }
template <>
__device__ __forceinline__ float ldf<uint16_t>(const uint16_t *p, int64_t i) {
    return __uint_as_float((uint32_t)p[i] << 16);
}

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t b = __float_as_uint(f);
    if ((b & 0x7F800000u) == 0x7F800000u) return (uint16_t)((b >> 16) | ((b & 0xFFFFu) ? 0x40u : 0u));
    b += 0x7FFFu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

template <typename T>
__device__ __forceinline__ void st_out(T *p, int64_t i, double v);
template <>
__device__ __forceinline__ void st_out<float>(float *p, int64_t i, double v) {
    p[i] = (float)v;
}
template <>
__device__ __forceinline__ void st_out<uint16_t>(uint16_t *p, int64_t i, double v) {
    p[i] = f32_to_bf16((float)v);
}

// ---------------------------------------------------------------------------
// Gram: part[b][r][s] = sum over the rows visited by block b of F[row][r] F[row][s],
// then a fixed-order reduction over the blocks.
// ---------------------------------------------------------------------------

// Gram on the matrix cores: v_mfma_f64_16x16x4f64 multiplies a 16x4 by a
// 4x16 FP64 tile.  For F^T F, a step covers 4 rows: lane l supplies
// F[k0 + l/16][16 t + l%16] for each 16-column tile t, as the A operand
// (F^T, tile rt) and the B operand (F, tile ct); the 16x16 result D holds
// D[l/16 + 4 i][l%16] in accumulator element i of lane l (checked on the
// device against an encoded product).  Only tile pairs
// rt <= ct are computed; the lower triangle is written as their mirror.
// Each wave walks its rows 16 at a time; the waves of a block are combined
// in a fixed order through LDS.  R <= 64 (at most 4 column tiles).
typedef double double4v __attribute__((ext_vector_type(4)));
constexpr int kMfmaMaxTiles = 4;

// NT consecutive entries F[row][c0 .. c0 + NT) as FP32 bit patterns (a BF16
// value is its FP32 pattern with the low half zero), zero past the last row
// or column.  VEC: R == 16 NT and the rows are aligned for one NT-element
// vector load.
// the FP32 bits of element i (BF16: its bits in the upper half)
__device__ __forceinline__ uint32_t gram_bits(const DF_GLOBAL float *F, int64_t i) {
    return __float_as_uint(F[i]);
}
__device__ __forceinline__ uint32_t gram_bits(const DF_GLOBAL uint16_t *F, int64_t i) {
    return (uint32_t)F[i] << 16;
}

// F through a global-space pointer (the grouped kernels read it from a
// descriptor: plain loads would be flat ones, whose waits also cover the
// loads issued for the next steps)
template <typename T, int NT, bool VEC>
__device__ __forceinline__ void gram_load(const T *__restrict__ F_, int64_t row, int64_t rows,
                                          int R, int c0, uint32_t (&v)[NT]) {
    const DF_GLOBAL T *F = gptr(F_);
    if (VEC && NT == 2) {
        if (row < rows) {
            if constexpr (sizeof(T) == 4) {
                const df_u2 a = *reinterpret_cast<const DF_GLOBAL df_u2 *>(F + row * R + c0);
                v[0] = a.x;
                v[1] = a.y;
            } else {
                const uint32_t a = *reinterpret_cast<const DF_GLOBAL uint32_t *>(F + row * R + c0);
                v[0] = a << 16;
                v[1] = a & 0xFFFF0000u;
            }
        } else {
            v[0] = v[1] = 0u;
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
        v[t] = (row < rows && c0 + t < R) ? gram_bits(F, row * R + c0 + t) : 0u;
}

// Block b of nb: the launch's own block, or a grouped launch's virtual one.
template <typename T, int NT, int BS, bool VEC>
__device__ __forceinline__ void gram_mfma_body(const T *__restrict__ F, int64_t rows, int R,
                                               double *__restrict__ part, uint32_t b,
                                               uint32_t nb) {
    constexpr int NP = NT * (NT + 1) / 2;  // tile pairs rt <= ct
    constexpr int NW = BS / 64;            // waves per block
    // steps loaded per batch: the next batch's loads are in flight while the
    // current one's MFMAs run (a wave takes only a few dozen steps, so one
    // step ahead leaves the loop waiting on memory); one step for R > 32,
    // where a second would cost occupancy
    constexpr int PD = NT <= 2 ? 2 : 1;
    __shared__ double sacc[NP * 256];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int kr = lane / 16, cl = lane % 16;
    double4v acc[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) acc[q] = double4v{0.0, 0.0, 0.0, 0.0};
    const int64_t nwaves = (int64_t)nb * NW;
    const int64_t gw = (int64_t)b * NW + wave;
    // rows [16 * step, 16 * step + 16) for step = gw, gw + nwaves, ... in
    // that order; rows past the end read as zero.
    const int64_t nsteps = (rows + 15) / 16;
    // Column tile t, MFMA index c is column c * NT + t, so a lane reads the
    // NT consecutive columns cl * NT .. + NT of a row.
    auto load = [&](int64_t s0, uint32_t (&v)[PD][4][NT]) {
#pragma unroll
        for (int p = 0; p < PD; ++p)
#pragma unroll
            for (int sub = 0; sub < 4; ++sub)
                gram_load<T, NT, VEC>(F, (s0 + p * nwaves) * 16 + sub * 4 + kr, rows, R, cl * NT,
                                      v[p][sub]);
    };
    uint32_t v[PD][4][NT];
    if (gw < nsteps) load(gw, v);
    for (int64_t s0 = gw; s0 < nsteps; s0 += PD * nwaves) {
        uint32_t vn[PD][4][NT];
        load(s0 + PD * nwaves, vn);
#pragma unroll
        for (int p = 0; p < PD; ++p) {
            if (s0 + p * nwaves >= nsteps) continue;  // uniform across the wave
#pragma unroll
            for (int sub = 0; sub < 4; ++sub) {
                double x[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) x[t] = (double)__uint_as_float(v[p][sub][t]);
                int q = 0;
#pragma unroll
                for (int rt = 0; rt < NT; ++rt)
#pragma unroll
                    for (int ct = rt; ct < NT; ++ct, ++q)
                        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[rt], x[ct], acc[q], 0, 0, 0);
            }
        }
#pragma unroll
        for (int p = 0; p < PD; ++p)
#pragma unroll
            for (int sub = 0; sub < 4; ++sub)
#pragma unroll
                for (int t = 0; t < NT; ++t) v[p][sub][t] = vn[p][sub][t];
    }
    // combine the waves of the block in wave order
    for (int w = 0; w < NW; ++w) {
        if (wave == w) {
#pragma unroll
            for (int q = 0; q < NP; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = q * 256 + (kr + 4 * i) * 16 + cl;
                    sacc[e] = (w == 0) ? acc[q][i] : sacc[e] + acc[q][i];
                }
        }
        __syncthreads();
    }
    DF_GLOBAL double *pb = gptr(part) + (size_t)b * R * R;
    for (int e = threadIdx.x; e < NP * 256; e += BS) {
        int q = e / 256, rt = 0;
        while (q >= NT - rt) { q -= NT - rt; ++rt; }  // pair index -> (rt, ct)
        const int ct = rt + q;
        const int r = ((e % 256) / 16) * NT + rt, c = (e % 16) * NT + ct;
        if (r < R && c < R) {
            pb[r * R + c] = sacc[e];
            if (rt != ct) pb[c * R + r] = sacc[e];
        }
    }
}

template <typename T, int NT, int BS, bool VEC>
__global__ __launch_bounds__(BS) void k_gram_mfma(const T *__restrict__ F, int64_t rows, int R,
                                                  double *__restrict__ part) {
    gram_mfma_body<T, NT, BS, VEC>(F, rows, R, part, blockIdx.x, gridDim.x);
}

template <typename T, int NT, int BS, bool VEC>
__global__ __launch_bounds__(BS) void k_gram_mfma_group(const GramJob *__restrict__ jobs,
                                                        const uint2 *__restrict__ vb) {
    const uint2 v = vb[blockIdx.x];
    const GramJob &j = jobs[v.x];
    gram_mfma_body<T, NT, BS, VEC>((const T *)j.F, j.rows, j.R, j.part, v.y, j.nblk);
}

// Ranks above 64 (up to 16 column tiles, 136 tile pairs): a block takes
// kWidePairs of the pairs (blockIdx.y), nine per wave, whose sums fill a
// wave's registers; its rows go through LDS 16 at a time, read by all four
// waves.  What bounds it is the wait in front of each step: with one wave a SIMD
// and nothing prefetched a step's loads and its products take turns (R = 100,
// 120,000 rows: 140 to 155 us, of which the products are 23 at 68 cycles each).
// R = 100, Grams of 120,000, 61,000 and 23,000 rows on average, against 8 x 8
// register tiles on the vector units: BF16 393 -> 133 us (beside the MTTKRP; 74
// alone), FP32 330 -> 83 us (73 alone).
constexpr int kWideWavePairs = 9, kWidePairs = 4 * kWideWavePairs;

template <typename T, int NTMAX>
__global__ __launch_bounds__(kBlock) void k_gram_wide(const T *__restrict__ F, int64_t rows, int R,
                                                      double *__restrict__ part) {
    constexpr int RP = 16 * NTMAX;
    __shared__ float sx[16][RP];
    const int nt = (R + 15) / 16, npair = nt * (nt + 1) / 2;
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, kr = lane / 16, cl = lane % 16;
    // this wave's pairs (rt <= ct), in row-major order of the upper triangle
    int rt[kWideWavePairs], ct[kWideWavePairs];
    const int q0 = blockIdx.y * kWidePairs + wave * kWideWavePairs;
#pragma unroll
    for (int i = 0; i < kWideWavePairs; ++i) {
        int q = q0 + i < npair ? q0 + i : npair - 1, r = 0;
        while (q >= nt - r) q -= nt - r, ++r;
        rt[i] = r;
        ct[i] = r + q;
    }
    double4v acc[kWideWavePairs];
#pragma unroll
    for (int i = 0; i < kWideWavePairs; ++i) acc[i] = double4v{0.0, 0.0, 0.0, 0.0};
    for (int e = threadIdx.x; e < 16 * RP; e += kBlock) (&sx[0][0])[e] = 0.f;
    const int64_t nstep = (rows + 15) / 16;
    for (int64_t s = blockIdx.x; s < nstep; s += gridDim.x) {
        const int64_t r0 = s * 16;
        const int nr = (int)(rows - r0 < 16 ? rows - r0 : 16);
        __syncthreads();
        for (int e = threadIdx.x; e < 16 * R; e += kBlock) {
            const int r = e / R;
            sx[r][e - r * R] = r < nr ? ldf<T>(F, r0 * R + e) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; k += 4)
#pragma unroll
            for (int i = 0; i < kWideWavePairs; ++i)
                acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                    (double)sx[k + kr][16 * rt[i] + cl], (double)sx[k + kr][16 * ct[i] + cl],
                    acc[i], 0, 0, 0);
    }
    double *pb = part + (size_t)blockIdx.x * R * R;
#pragma unroll
    for (int i = 0; i < kWideWavePairs; ++i) {
        if (q0 + i >= npair) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * rt[i] + kr + 4 * v, c = 16 * ct[i] + cl;
            if (r < R && c < R) {
                pb[r * R + c] = acc[i][v];
                if (rt[i] != ct[i]) pb[c * R + r] = acc[i][v];
            }
        }
    }
}

// G[e] = sum_b part[b][e]: a block takes 16 entries; slice q (16 per entry)
// sums the partials b = q, q + 16, ...; the slices are combined in order.
// The first 16 partials of a slice are loaded together, then added in order.
__device__ __forceinline__ void gram_reduce_body(const double *__restrict__ part_, int nblk, int R,
                                                 double *__restrict__ G_, uint32_t b) {
    const DF_GLOBAL double *part = gptr(part_);
    DF_GLOBAL double *G = gptr(G_);
    __shared__ double sh[16][17];
    const int e = b * 16 + threadIdx.x % 16;
    const int sl = threadIdx.x / 16;
    const int RR = R * R;
    double s = 0.0;
    if (e < RR) {
        double x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int pb = sl + 16 * u;
            x[u] = pb < nblk ? part[(size_t)pb * RR + e] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (sl + 16 * u < nblk) s += x[u];
        for (int pb = sl + 256; pb < nblk; pb += 16) s += part[(size_t)pb * RR + e];
    }
    sh[sl][threadIdx.x % 16] = s;
    __syncthreads();
    if (threadIdx.x < 16 && e < RR) {
        double t = sh[0][threadIdx.x];
#pragma unroll
        for (int q = 1; q < 16; ++q) t += sh[q][threadIdx.x];
        G[e] = t;
    }
}

__global__ __launch_bounds__(kBlock) void k_gram_reduce(const double *__restrict__ part, int nblk,
                                                        int R, double *__restrict__ G) {
    gram_reduce_body(part, nblk, R, G, blockIdx.x);
}

__global__ __launch_bounds__(kBlock) void k_gram_reduce_group(const GramJob *__restrict__ jobs,
                                                              const uint2 *__restrict__ vb) {
    const uint2 v = vb[blockIdx.x];
    const GramJob &j = jobs[v.x];
    gram_reduce_body(j.part, (int)j.nblk, j.R, j.G, v.y);
}

// The three factors' Grams of a line search's trial point in one launch
// (blockIdx.y the mode), and one reduction that also forms the Hadamard
// product H = G[1] * G[2] + reg I: a block has the same 16 entries of every
// mode.  Each is bound by its launch and a round trip or two to memory (1M
// nonzeros, R = 10, per trial: three Grams, reductions and a product 30 ->
// 17 us, three trial factors 14 -> 10 us, seven launches fewer).
struct GramJobs3 {
    GramJob j[3];
};

template <typename T, int NT, int BS, bool VEC>
__global__ __launch_bounds__(BS) void k_gram_mfma3(GramJobs3 jobs) {
    const GramJob &j = jobs.j[blockIdx.y];
    if (blockIdx.x >= j.nblk) return;
    gram_mfma_body<T, NT, BS, VEC>((const T *)j.F, j.rows, j.R, j.part, blockIdx.x, j.nblk);
}

__global__ __launch_bounds__(kBlock) void k_gram_reduce3(GramJobs3 jobs, double reg,
                                                         double *__restrict__ H) {
    for (int m = 0; m < 3; ++m) {
        const GramJob &j = jobs.j[m];
        gram_reduce_body(j.part, (int)j.nblk, j.R, j.G, blockIdx.x);
        __syncthreads();
    }
    const int R = jobs.j[0].R, e = blockIdx.x * 16 + threadIdx.x;
    if (threadIdx.x < 16 && e < R * R)  // (entries this thread has just written)
        H[e] = jobs.j[1].G[e] * jobs.j[2].G[e] + (e / R == e % R ? reg : 0.0);
}

__global__ void k_hadamard(int R, const double *__restrict__ Gp, const double *__restrict__ Gq,
                           double reg, double *__restrict__ H) {
    const int e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= R * R) return;
    H[e] = Gp[e] * Gq[e] + ((e / R == e % R) ? reg : 0.0);
}

// fixed-order block reduction of one double per thread, over the first
// kBlock threads (any others only join the barriers)
__device__ double block_sum(double v, double *sh) {
    if (threadIdx.x < kBlock) sh[threadIdx.x] = v;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

__device__ double block_max(double v, double *sh) {
    if (threadIdx.x < kBlock) sh[threadIdx.x] = v;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + w]);
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// The lambda step's R x R matrices live in LDS up to this rank (4 R^2 + R
// doubles, at most 52 KB of dynamic LDS), else in global scratch.
constexpr int kLambdaSmemMaxR = 40;

// ---------------------------------------------------------------------------
// one-workgroup solve.  Working set: 3 R^2 doubles (H, A, B / V), in
// dynamic LDS when SMEM (R <= 32), else in `scratch`.  flag[0] = 1 when the
// pseudo-inverse path was taken.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double readlane_f64(double v, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// Gauss-Jordan on [H | I] in the registers of one wave (R <= 32): lane l
// holds column l of the R x 2R working matrix; the pivot and the pivot
// column's entries reach every lane by readlane.  The arithmetic (scale the
// pivot row by 1/pivot, then row_i -= a_ij * row_j) is the same, operation
// for operation, as the LDS version in k_solve.  On success columns R .. 2R-1
// (H^-1) are written to Bw (R x R, row-major); returns false at the first
// pivot that is not above tol.
template <int B, int E, typename Fn>
__device__ __forceinline__ void unroll_for(Fn &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        unroll_for<B + 1, E>(f);
    }
}

__device__ bool gauss_jordan_wave(const double *H, int R, double tol, double *Bw) {
    constexpr int RM = 32;
    const int l = threadIdx.x % 64;
    double col[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i)
        col[i] = (i < R) ? (l < R ? H[i * R + l] : (l - R == i ? 1.0 : 0.0)) : 0.0;
    bool ok = true;
    // j and i are compile-time constants, so col[] stays in registers
    unroll_for<0, RM>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if (!ok || j >= R) return;
        const double piv = readlane_f64(col[j], j);
        if (!(piv > tol)) {
            ok = false;
            return;
        }
        const double inv = 1.0 / piv;
        col[j] *= inv;
        unroll_for<0, RM>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if (i == j || i >= R) return;
            col[i] = fma(-readlane_f64(col[i], j), col[j], col[i]);
        });
        __builtin_amdgcn_sched_barrier(0);  // keep the steps apart: no hoisted readlanes
    });
    if (!ok) return false;
    if (l >= R && l < 2 * R) {
#pragma unroll
        for (int i = 0; i < RM; ++i)
            if (i < R) Bw[i * R + (l - R)] = col[i];
    }
    return true;
}

// The same Gauss-Jordan for 32 < R <= 32 NT by a block of 1024 threads, the
// matrix in their registers (thread (y, x) of 32 x 32 holds the entries (y +
// 32 a, x + 32 b)) and in place: a column of [H | I] that a step has made a
// unit column is never read again, so the column of the inverse takes its
// place.  Operation for operation the arithmetic of the other two versions.
// A step publishes its row, its column and 1 / pivot in LDS (two sets, so one
// barrier per step), then every entry takes one FMA: R steps of 0.6 us, where
// sweeping [H | I] in global memory took 28 us each (R = 100: 2782 -> 98 us
// beside the MTTKRP).  Alone the solve takes 84 us there, 60 of them the steps;
// the rest forms H in global scratch and symmetrizes the inverse from it
// (R = 128: 114 and 77; R = 64: 43).
template <int NT>
__device__ bool gauss_jordan_block(const double *__restrict__ Gp, const double *__restrict__ Gq,
                                   double reg, int R, double tol, double *__restrict__ Bw) {
    __shared__ double s_row[2][32 * NT], s_col[2][32 * NT], s_piv[2], s_inv[2];
    const int x = threadIdx.x % 32, y = threadIdx.x / 32;
    double a[NT][NT];
#pragma unroll
    for (int p = 0; p < NT; ++p)
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int i = y + 32 * p, k = x + 32 * q;
            a[p][q] = i < R && k < R ? Gp[i * R + k] * Gq[i * R + k] + (i == k ? reg : 0.0) : 0.0;
        }
    bool ok = true;
    // steps 32 t .. 32 t + 31 have their row in a[t][.] and their column in
    // a[.][t], compile-time places
    unroll_for<0, NT>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        for (int u = 0; u < 32; ++u) {
            const int j = 32 * t + u, w = u & 1;
            if (!ok || j >= R) break;  // uniform
            if (y == u) {
#pragma unroll
                for (int q = 0; q < NT; ++q) s_row[w][x + 32 * q] = a[t][q];
            }
            if (x == u) {
#pragma unroll
                for (int p = 0; p < NT; ++p) s_col[w][y + 32 * p] = a[p][t];
                if (y == u) {
                    s_piv[w] = a[t][t];
                    s_inv[w] = 1.0 / a[t][t];
                }
            }
            __syncthreads();
            ok = s_piv[w] > tol;
            const double inv = s_inv[w];
            double r[NT], c[NT];
#pragma unroll
            for (int q = 0; q < NT; ++q) r[q] = s_row[w][x + 32 * q] * inv;
#pragma unroll
            for (int p = 0; p < NT; ++p) c[p] = s_col[w][y + 32 * p];
            if (x == u) r[t] = inv;  // the new column: e_j / pivot
#pragma unroll
            for (int p = 0; p < NT; ++p)
#pragma unroll
                for (int q = 0; q < NT; ++q) {
                    const double old = q == t && x == u ? 0.0 : a[p][q];
                    a[p][q] = p == t && y == u ? r[q] : fma(-c[p], r[q], old);
                }
        }
    });
    if (!ok) return false;
#pragma unroll
    for (int p = 0; p < NT; ++p)
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int i = y + 32 * p, k = x + 32 * q;
            if (i < R && k < R) Bw[i * R + k] = a[p][q];
        }
    return true;
}

// BS threads (kBlock, or kSolveWide for launches with ranks above 32)
constexpr int kSolveWide = 1024;
constexpr int kSolveRegMaxR = 128;  // ranks that gauss_jordan_block takes

template <int BS, bool SMEM>
__device__ void solve_body(int R, const double *__restrict__ Gp, const double *__restrict__ Gq,
                           double reg, double *__restrict__ Hinv, double *__restrict__ scratch,
                           int *flag, double *dyn) {
    __shared__ double sh[kBlock];
    __shared__ int s_fail;
    __shared__ double s_c[kBlock], s_s[kBlock];
    __shared__ int s_p[kBlock], s_q[kBlock];
    const int tid = threadIdx.x;
    const int RR = R * R;
    double *base = SMEM ? dyn : scratch;
    double *H = base, *L = base + RR, *Li = base + 2 * RR;
    for (int e = tid; e < RR; e += BS) {
        H[e] = Gp[e] * Gq[e] + ((e / R == e % R) ? reg : 0.0);
        L[e] = 0.0;
        Li[e] = 0.0;
    }
    __syncthreads();
    double dm = 0.0;
    if (tid < kBlock)
        for (int r = tid; r < R; r += kBlock) dm = fmax(dm, H[r * R + r]);
    const double dmax = block_max(dm, sh);
    const double tol = (double)R * DBL_EPSILON * dmax;
    if (tid == 0) s_fail = (dmax > 0.0) ? 0 : 1;
    __syncthreads();
    // Gauss-Jordan on [H | I] without pivoting (H is symmetric): the pivot at
    // step j is the Schur-complement diagonal d_j = L_jj^2 of the Cholesky
    // factorization H = L L^T, so "every d_j > R eps max diag(H)" is the
    // Cholesky test for a numerically positive definite H.  If it fails, the
    // pseudo-inverse below is used instead.  Aw (in L) is the working copy of
    // H, Bw (in Li) starts as I and ends as H^-1.
    double *Aw = L, *Bw = Li;
    __shared__ double s_f[kBlock];
    if (R <= 32) {
        if (tid < 64 && !s_fail) {
            const bool ok = gauss_jordan_wave(H, R, tol, Bw);
            if (tid == 0 && !ok) s_fail = 1;
        }
        __syncthreads();
    } else if (BS == kSolveWide && R <= kSolveRegMaxR) {
        if (!s_fail) {
            const bool ok = R <= 64   ? gauss_jordan_block<2>(Gp, Gq, reg, R, tol, Bw)
                            : R <= 96 ? gauss_jordan_block<3>(Gp, Gq, reg, R, tol, Bw)
                                      : gauss_jordan_block<4>(Gp, Gq, reg, R, tol, Bw);
            if (tid == 0 && !ok) s_fail = 1;
        }
    } else {
        for (int e = tid; e < RR; e += BS) {
            Aw[e] = H[e];
            Bw[e] = (e / R == e % R) ? 1.0 : 0.0;
        }
        __syncthreads();
        for (int j = 0; j < R; ++j) {
            const double piv = Aw[j * R + j];
            if (!(piv > tol)) {  // uniform: every thread reads the same value
                if (tid == 0) s_fail = 1;
                break;
            }
            const double inv = 1.0 / piv;
            __syncthreads();  // all threads have read the pivot
            for (int k = tid; k < 2 * R; k += BS) {
                if (k < R) Aw[j * R + k] *= inv;
                else Bw[j * R + k - R] *= inv;
            }
            for (int i = tid; i < R; i += BS) s_f[i] = (i == j) ? 0.0 : Aw[i * R + j];
            __syncthreads();
            for (int e = tid; e < R * 2 * R; e += BS) {
                const int i = e / (2 * R), k = e % (2 * R);
                const double f = s_f[i];
                if (f == 0.0) continue;
                if (k < R) Aw[i * R + k] = fma(-f, Aw[j * R + k], Aw[i * R + k]);
                else Bw[i * R + k - R] = fma(-f, Bw[j * R + k - R], Bw[i * R + k - R]);
            }
            __syncthreads();
        }
    }
    __syncthreads();
    if (!s_fail) {
        for (int e = tid; e < RR; e += BS) {
            const int r = e / R, c = e % R;
            Hinv[e] = 0.5 * (Bw[r * R + c] + Bw[c * R + r]);
        }
        if (tid == 0) flag[0] = 0;
        return;
    }
    // pseudo-inverse: parallel cyclic Jacobi on A = H, V = I
    double *A = L, *V = Li;
    for (int e = tid; e < RR; e += BS) {
        A[e] = H[e];
        V[e] = (e / R == e % R) ? 1.0 : 0.0;
    }
    __syncthreads();
    const int n2 = (R + 1) & ~1;  // players in the round-robin schedule
    const int npair = n2 / 2;
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0, tot = 0.0;
        // the first kBlock threads sum, so that the order does not depend on BS
        for (int e = tid; tid < kBlock && e < RR; e += kBlock) {
            const double a2 = A[e] * A[e];
            tot += a2;
            if (e / R != e % R) off += a2;
        }
        off = block_sum(off, sh);
        tot = block_sum(tot, sh);
        if (off <= 1e-30 * tot || off == 0.0) break;
        for (int round = 0; round < n2 - 1; ++round) {
            for (int pi = tid; pi < npair; pi += BS) {
                auto player = [&](int pos) { return pos == 0 ? 0 : 1 + (pos - 1 + round) % (n2 - 1); };
                int p = player(pi), q = player(n2 - 1 - pi);
                if (p > q) { const int t = p; p = q; q = t; }
                double c = 1.0, s = 0.0;
                if (q < R) {
                    const double apq = A[p * R + q];
                    if (apq != 0.0) {
                        const double theta = (A[q * R + q] - A[p * R + p]) / (2.0 * apq);
                        const double t = (theta >= 0 ? 1.0 : -1.0) /
                                         (fabs(theta) + sqrt(theta * theta + 1.0));
                        c = 1.0 / sqrt(t * t + 1.0);
                        s = t * c;
                    }
                }
                s_p[pi] = p;
                s_q[pi] = q;
                s_c[pi] = c;
                s_s[pi] = s;
            }
            __syncthreads();
            // A <- A J and V <- V J (columns p, q of every disjoint pair)
            for (int e = tid; e < npair * R; e += BS) {
                const int pi = e / R, k = e % R;
                const int p = s_p[pi], q = s_q[pi];
                if (q >= R || s_s[pi] == 0.0) continue;
                const double c = s_c[pi], s = s_s[pi];
                const double akp = A[k * R + p], akq = A[k * R + q];
                A[k * R + p] = c * akp - s * akq;
                A[k * R + q] = s * akp + c * akq;
                const double vkp = V[k * R + p], vkq = V[k * R + q];
                V[k * R + p] = c * vkp - s * vkq;
                V[k * R + q] = s * vkp + c * vkq;
            }
            __syncthreads();
            // A <- J^T A (rows p, q)
            for (int e = tid; e < npair * R; e += BS) {
                const int pi = e / R, k = e % R;
                const int p = s_p[pi], q = s_q[pi];
                if (q >= R || s_s[pi] == 0.0) continue;
                const double c = s_c[pi], s = s_s[pi];
                const double apk = A[p * R + k], aqk = A[q * R + k];
                A[p * R + k] = c * apk - s * aqk;
                A[q * R + k] = s * apk + c * aqk;
            }
            __syncthreads();
        }
    }
    double wm = 0.0;
    if (tid < kBlock)
        for (int r = tid; r < R; r += kBlock) wm = fmax(wm, A[r * R + r]);
    const double wmax = block_max(wm, sh);
    const double wtol = (double)R * DBL_EPSILON * wmax;
    for (int e = tid; e < RR; e += BS) {
        const int r = e / R, s = e % R;
        double acc = 0.0;
        for (int k = 0; k < R; ++k) {
            const double w = A[k * R + k];
            if (w > wtol) acc += V[r * R + k] * V[s * R + k] / w;
        }
        Hinv[e] = acc;
    }
    if (tid == 0) flag[0] = 1;
}

template <int BS, bool SMEM>
__global__ __launch_bounds__(BS) void k_solve(int R, const double *__restrict__ Gp,
                                              const double *__restrict__ Gq, double reg,
                                              double *__restrict__ Hinv,
                                              double *__restrict__ scratch, int *flag) {
    extern __shared__ double dyn[];
    solve_body<BS, SMEM>(R, Gp, Gq, reg, Hinv, scratch, flag, dyn);
}

template <int BS, bool SMEM>
__global__ __launch_bounds__(BS) void k_solve_group(const SolveJob *__restrict__ jobs) {
    extern __shared__ double dyn[];
    const SolveJob &j = jobs[blockIdx.x];
    solve_body<BS, SMEM>(j.R, j.Gp, j.Gq, j.reg, j.Hinv, j.scratch, j.flag, dyn);
}

// ---------------------------------------------------------------------------
// lambda, new Gram, W and (last mode) fit -- one workgroup.  Working set:
// Hinv, MtM, T1 = MtM Hinv, S = Hinv T1 (4 R^2) and lambda (R), in dynamic
// LDS when SMEM, else in `scratch`.
// ---------------------------------------------------------------------------
template <bool SMEM>
__device__ void als_lambda_body(int R, int mode, const double *__restrict__ Hinv_g,
                                const double *__restrict__ MtM_g, double *__restrict__ Gn,
                                double *__restrict__ W, double *__restrict__ lambda_out,
                                const double *__restrict__ GA, const double *__restrict__ GB,
                                double normsq, double *__restrict__ fit_out,
                                double *__restrict__ scratch, double *dyn) {
    __shared__ double sh[kBlock];
    const int tid = threadIdx.x;
    const int RR = R * R;
    double *base = SMEM ? dyn : scratch;
    double *Hi = base, *MM = base + RR, *T1 = base + 2 * RR, *S = base + 3 * RR,
           *lam = base + 4 * RR;
    for (int e = tid; e < RR; e += kBlock) {
        Hi[e] = Hinv_g[e];
        MM[e] = MtM_g[e];
    }
    __syncthreads();
    for (int e = tid; e < RR; e += kBlock) {
        const int r = e / R, s = e % R;
        double acc = 0.0;
        for (int k = 0; k < R; ++k) acc += MM[r * R + k] * Hi[k * R + s];
        T1[e] = acc;
    }
    __syncthreads();
    for (int e = tid; e < RR; e += kBlock) {
        const int r = e / R, s = e % R;
        double acc = 0.0;
        for (int k = 0; k < R; ++k) acc += Hi[r * R + k] * T1[k * R + s];
        S[e] = acc;
    }
    __syncthreads();
    for (int r = tid; r < R; r += kBlock) {
        const double d = S[r * R + r];
        lam[r] = d > 0.0 ? sqrt(d) : 0.0;
        lambda_out[r] = lam[r];
    }
    __syncthreads();
    double in = 0.0, xh = 0.0;
    for (int e = tid; e < RR; e += kBlock) {
        const int r = e / R, s = e % R;
        const double lr = lam[r], ls = lam[s];
        const double g = (lr > 0.0 && ls > 0.0) ? S[e] / (lr * ls) : 0.0;
        Gn[e] = g;
        W[e] = ls > 0.0 ? Hi[e] / ls : 0.0;
        if (mode == 2) {
            in += Hi[e] * MM[e];
            xh += lr * ls * GA[e] * GB[e] * g;
        }
    }
    if (mode != 2) return;
    in = block_sum(in, sh);
    xh = block_sum(xh, sh);
    if (tid == 0) {
        double res2 = normsq + xh - 2.0 * in;
        if (res2 < 0.0) res2 = 0.0;
        *fit_out = normsq > 0.0 ? 1.0 - sqrt(res2) / sqrt(normsq) : 0.0;
    }
}

// The lambda step of ranks above kLambdaSmemMaxR, spread over the device: one
// block formed both R x R x R products from global memory (R = 100: 1103 us);
// here each of the two takes a block per 16 x 16 tile, its operands staged in
// LDS, and the rest one block (two products of 9 us and 27 us at R = 100).  Every entry's sum runs over k in order, so the
// results are bitwise those of als_lambda_body.
constexpr int kMulTile = 16, kMulK = 64;
// C = A B (R x R, row-major)
__global__ __launch_bounds__(kBlock) void k_matmul(int R, const double *__restrict__ A,
                                                   const double *__restrict__ B,
                                                   double *__restrict__ C) {
    __shared__ double sa[kMulTile][kMulK + 1], sb[kMulK][kMulTile + 1];
    const int x = threadIdx.x % kMulTile, y = threadIdx.x / kMulTile;
    const int r0 = blockIdx.y * kMulTile, c0 = blockIdx.x * kMulTile;
    double acc = 0.0;
    for (int k0 = 0; k0 < R; k0 += kMulK) {
        __syncthreads();
        for (int e = threadIdx.x; e < kMulTile * kMulK; e += kBlock) {
            const int i = e / kMulK, k = e % kMulK;
            sa[i][k] = r0 + i < R && k0 + k < R ? A[(r0 + i) * R + k0 + k] : 0.0;
            const int kb = e / kMulTile, j = e % kMulTile;
            sb[kb][j] = k0 + kb < R && c0 + j < R ? B[(k0 + kb) * R + c0 + j] : 0.0;
        }
        __syncthreads();
        const int kn = R - k0 < kMulK ? R - k0 : kMulK;
#pragma unroll 8
        for (int k = 0; k < kn; ++k) acc = fma(sa[y][k], sb[k][x], acc);
    }
    if (r0 + y < R && c0 + x < R) C[(r0 + y) * R + c0 + x] = acc;
}

// lambda, G, W and (mode 2) the fit from S = H^-1 (M^T M) H^-1
__global__ __launch_bounds__(kBlock) void k_lambda_finish(
    int R, int mode, const double *__restrict__ Hi, const double *__restrict__ MM,
    const double *__restrict__ S, double *__restrict__ Gn, double *__restrict__ W,
    double *__restrict__ lambda_out, const double *__restrict__ GA,
    const double *__restrict__ GB, double normsq, double *__restrict__ fit_out) {
    __shared__ double sh[kBlock], lam[DFACTO_MAX_R];
    const int tid = threadIdx.x, RR = R * R;
    for (int r = tid; r < R; r += kBlock) {
        const double d = S[r * R + r];
        lam[r] = d > 0.0 ? sqrt(d) : 0.0;
        lambda_out[r] = lam[r];
    }
    __syncthreads();
    double in = 0.0, xh = 0.0;
#pragma unroll 4
    for (int e = tid; e < RR; e += kBlock) {
        const double lr = lam[e / R], ls = lam[e % R], hi = Hi[e];
        const double g = (lr > 0.0 && ls > 0.0) ? S[e] / (lr * ls) : 0.0;
        Gn[e] = g;
        W[e] = ls > 0.0 ? hi / ls : 0.0;
        if (mode == 2) {
            in += hi * MM[e];
            xh += lr * ls * GA[e] * GB[e] * g;
        }
    }
    if (mode != 2) return;
    in = block_sum(in, sh);
    xh = block_sum(xh, sh);
    if (tid == 0) {
        double res2 = normsq + xh - 2.0 * in;
        if (res2 < 0.0) res2 = 0.0;
        *fit_out = normsq > 0.0 ? 1.0 - sqrt(res2) / sqrt(normsq) : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Fit from the STORED last factor (BF16 storage): the rounded factor C that
// later calls read differs from M H^-1 diag(1/lambda), so the fit is formed
// from C itself, as for the other two factors whose Grams are re-formed
// from their stored values:
//   <X, Xhat> = sum_r lambda_r sum_k C[k, r] M[k, r]   (M: mode-2 MTTKRP)
//   ||Xhat||^2 = lambda^T (G_A * G_B * G_C) lambda     (G_C from stored C)
// Partial sums of the weighted inner product per block (fit_blocks of them,
// each a fixed-order strided sum), then one block finishes.
// ---------------------------------------------------------------------------
template <typename T>
__device__ void wdot_body(const T *__restrict__ F, const float *__restrict__ X, int64_t rows,
                          int R, const double *__restrict__ lam, uint32_t b, uint32_t nb,
                          double *__restrict__ part, double *sh, double *sl) {
    for (int r = threadIdx.x; r < R; r += kBlock) sl[r] = lam[r];
    __syncthreads();
    const int64_t n = rows * (int64_t)R;
    const int64_t S = (int64_t)nb * kBlock;
    int64_t e = (int64_t)b * kBlock + threadIdx.x;
    int r = (int)(e % R);
    const int dr = (int)(S % R);
    double acc = 0.0;
    for (; e < n; e += S) {
        acc = fma(sl[r] * ld<T>(F, e), (double)X[e], acc);
        r += dr;
        if (r >= R) r -= R;
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) part[b] = acc;
}

__device__ void fit_finish_body(int R, const double *__restrict__ lam,
                                const double *__restrict__ GA, const double *__restrict__ GB,
                                const double *__restrict__ GC, const double *__restrict__ part,
                                uint32_t npart, double normsq, double *__restrict__ fit,
                                double *sh) {
    double in = 0.0, xh = 0.0;
    for (uint32_t b = threadIdx.x; b < npart; b += kBlock) in += part[b];
    for (int e = threadIdx.x; e < R * R; e += kBlock) {
        const int r = e / R, s = e % R;
        xh += lam[r] * lam[s] * GA[e] * GB[e] * GC[e];
    }
    in = block_sum(in, sh);
    xh = block_sum(xh, sh);
    if (threadIdx.x == 0) {
        double res2 = normsq + xh - 2.0 * in;
        if (res2 < 0.0) res2 = 0.0;
        *fit = normsq > 0.0 ? 1.0 - sqrt(res2) / sqrt(normsq) : 0.0;
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_wdot(const T *__restrict__ F,
                                                 const float *__restrict__ X, int64_t rows, int R,
                                                 const double *__restrict__ lam,
                                                 double *__restrict__ part) {
    __shared__ double sh[kBlock], sl[DFACTO_MAX_R];
    wdot_body<T>(F, X, rows, R, lam, blockIdx.x, gridDim.x, part, sh, sl);
}

__global__ __launch_bounds__(kBlock) void k_fit_finish(int R, const double *__restrict__ lam,
                                                       const double *__restrict__ GA,
                                                       const double *__restrict__ GB,
                                                       const double *__restrict__ GC,
                                                       const double *__restrict__ part,
                                                       uint32_t npart, double normsq,
                                                       double *__restrict__ fit) {
    __shared__ double sh[kBlock];
    fit_finish_body(R, lam, GA, GB, GC, part, npart, normsq, fit, sh);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_wdot_group(const FitJob *__restrict__ jobs,
                                                       const uint2 *__restrict__ items) {
    __shared__ double sh[kBlock], sl[DFACTO_MAX_R];
    const uint2 v = items[blockIdx.x];
    const FitJob &j = jobs[v.x];
    wdot_body<T>((const T *)j.F, j.M, j.rows, j.R, j.lambda, v.y, j.nblk, j.part, sh, sl);
}

__global__ __launch_bounds__(kBlock) void k_fit_finish_group(const FitJob *__restrict__ jobs) {
    __shared__ double sh[kBlock];
    const FitJob &j = jobs[blockIdx.x];
    fit_finish_body(j.R, j.lambda, j.GA, j.GB, j.GC, j.part, j.nblk, j.normsq, j.fit, sh);
}

__global__ __launch_bounds__(kBlock) void k_als_lambda(
    int R, int mode, const double *__restrict__ Hinv_g, const double *__restrict__ MtM_g,
    double *__restrict__ Gn, double *__restrict__ W, double *__restrict__ lambda_out,
    const double *__restrict__ GA, const double *__restrict__ GB, double normsq,
    double *__restrict__ fit_out) {
    extern __shared__ double dyn[];
    als_lambda_body<true>(R, mode, Hinv_g, MtM_g, Gn, W, lambda_out, GA, GB, normsq, fit_out,
                          nullptr, dyn);
}

template <bool SMEM>
__global__ __launch_bounds__(kBlock) void k_als_lambda_group(const LambdaJob *__restrict__ jobs) {
    extern __shared__ double dyn[];
    const LambdaJob &j = jobs[blockIdx.x];
    als_lambda_body<SMEM>(j.R, j.mode, j.Hinv, j.MtM, j.Gn, j.W, j.lambda, j.GA, j.GB, j.normsq,
                          j.fit, j.scratch, dyn);
}

// ---------------------------------------------------------------------------
// Row maps over tiles of TR = kTileElems / R consecutive rows (one contiguous
// block of memory): the tile is loaded with coalesced loads into LDS (row
// stride R + 1, conflict-free column reads), each thread computes CT = 16
// columns of one row with the R x R matrix broadcast from LDS (all lanes of a
// wave work on the same columns), and the result tile is written back with
// coalesced stores.  Instantiated for R in {4, 8, 12, 16, 32, 48}.
// ---------------------------------------------------------------------------
constexpr int kTileElems = 4096;
constexpr int kCT = 16;  // columns per thread

__host__ __device__ constexpr int tile_rows(int R) { return kTileElems / R < kBlock ? kTileElems / R : kBlock; }

// F[row, s] = sum_k M[row, k] W[k, s]   (R is a compile-time constant)
template <typename Tout, int R>
__device__ __forceinline__ void rowmap_t_body(const float *__restrict__ M, int64_t rows,
                                              const double *__restrict__ W, Tout *__restrict__ F,
                                              double *dyn, uint32_t b, uint32_t nb) {
    double *sW = dyn;                                  // R * R
    float *sM = reinterpret_cast<float *>(sW + R * R);  // TR * (R + 1)
    constexpr int TR = tile_rows(R), RS = R + 1;
    float *sO = sM + TR * RS;                          // TR * (R + 1)
    for (int e = threadIdx.x; e < R * R; e += kBlock) sW[e] = W[e];
    constexpr int tpr = kBlock / TR;                   // threads per row
    const int rr = threadIdx.x % TR, part = threadIdx.x / TR;
    const int c0 = part * kCT;
    const bool active = part < tpr && c0 < R;
    const int64_t ntile = (rows + TR - 1) / TR;
    for (int64_t tile = b; tile < ntile; tile += nb) {
        const int64_t r0 = tile * TR;
        const int nr = (int)((rows - r0) < TR ? (rows - r0) : TR);
        __syncthreads();
        for (int e = threadIdx.x; e < nr * R; e += kBlock) sM[(e / R) * RS + e % R] = M[r0 * R + e];
        __syncthreads();
        if (active && rr < nr) {
            double acc[kCT];
#pragma unroll
            for (int s = 0; s < kCT; ++s) acc[s] = 0.0;
            const float *m = sM + rr * RS;
#pragma unroll 4
            for (int k = 0; k < R; ++k) {
                const double mk = m[k];
                const double *w = sW + k * R + c0;
#pragma unroll
                for (int s = 0; s < kCT; ++s)
                    if (c0 + s < R) acc[s] = fma(mk, w[s], acc[s]);
            }
#pragma unroll
            for (int s = 0; s < kCT; ++s)
                if (c0 + s < R) sO[rr * RS + c0 + s] = (float)acc[s];
        }
        __syncthreads();
        for (int e = threadIdx.x; e < nr * R; e += kBlock)
            st_out<Tout>(F, r0 * R + e, (double)sO[(e / R) * RS + e % R]);
    }
}

template <typename Tout, int R>
__global__ __launch_bounds__(kBlock) void k_rowmap_t(const float *__restrict__ M, int64_t rows,
                                                     const double *__restrict__ W,
                                                     Tout *__restrict__ F) {
    extern __shared__ double dyn[];
    rowmap_t_body<Tout, R>(M, rows, W, F, dyn, blockIdx.x, gridDim.x);
}

template <typename Tout, int R>
__global__ __launch_bounds__(kBlock) void k_rowmap_t_group(const RowmapJob *__restrict__ jobs,
                                                           const uint2 *__restrict__ vb) {
    extern __shared__ double dyn[];
    const uint2 v = vb[blockIdx.x];
    const RowmapJob &j = jobs[v.x];
    rowmap_t_body<Tout, R>(j.M, j.rows, j.W, (Tout *)j.F, dyn, v.y, j.nblk);
}

// G[row, s] = -G[row, s] + sum_k F[row, k] H[k, s]  (G holds the MTTKRP);
// partial[block] = sum over the block's rows of <F[row,:], M[row,:]>.
template <typename T, int R>
__global__ __launch_bounds__(kBlock) void k_gd_rows_t(float *__restrict__ G,
                                                      const T *__restrict__ F, int64_t rows,
                                                      const double *__restrict__ H,
                                                      double *__restrict__ partial) {
    extern __shared__ double dyn[];
    __shared__ double sh[kBlock];
    double *sH = dyn;
    float *sF = reinterpret_cast<float *>(sH + R * R);
    constexpr int TR = tile_rows(R), RS = R + 1;
    float *sM = sF + TR * RS;
    for (int e = threadIdx.x; e < R * R; e += kBlock) sH[e] = H[e];
    constexpr int tpr = kBlock / TR;
    const int rr = threadIdx.x % TR, part = threadIdx.x / TR;
    const int c0 = part * kCT;
    const bool active = part < tpr && c0 < R;
    const int64_t ntile = (rows + TR - 1) / TR;
    double inner = 0.0;
    for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const int64_t r0 = tile * TR;
        const int nr = (int)((rows - r0) < TR ? (rows - r0) : TR);
        __syncthreads();
        for (int e = threadIdx.x; e < nr * R; e += kBlock) {
            const int o = (e / R) * RS + e % R;
            sF[o] = ldf<T>(F, r0 * R + e);
            sM[o] = G[r0 * R + e];
        }
        __syncthreads();
        double acc[kCT];
        if (active && rr < nr) {
#pragma unroll
            for (int s = 0; s < kCT; ++s) acc[s] = 0.0;
            const float *f = sF + rr * RS;
#pragma unroll 4
            for (int k = 0; k < R; ++k) {
                const double fk = f[k];
                const double *h = sH + k * R + c0;
#pragma unroll
                for (int s = 0; s < kCT; ++s)
                    if (c0 + s < R) acc[s] = fma(fk, h[s], acc[s]);
            }
        }
        __syncthreads();  // every thread has read its F row: sF can take the output
        if (active && rr < nr) {
            const float *mrow = sM + rr * RS;
#pragma unroll
            for (int s = 0; s < kCT; ++s) {
                if (c0 + s < R) {
                    const double m = mrow[c0 + s];
                    inner = fma((double)sF[rr * RS + c0 + s], m, inner);
                }
            }
        }
        __syncthreads();
        if (active && rr < nr) {
            const float *mrow = sM + rr * RS;
#pragma unroll
            for (int s = 0; s < kCT; ++s)
                if (c0 + s < R) sF[rr * RS + c0 + s] = (float)(acc[s] - (double)mrow[c0 + s]);
        }
        __syncthreads();
        for (int e = threadIdx.x; e < nr * R; e += kBlock) G[r0 * R + e] = sF[(e / R) * RS + e % R];
    }
    const double tot = block_sum(inner, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

size_t tile_lds_bytes(int R) {
    return sizeof(double) * (size_t)R * R + 2 * sizeof(float) * (size_t)tile_rows(R) * (R + 1);
}

// Generic versions for ranks above kRowAnyMaxR: rows staged in LDS, the matrix
// read from memory (its FMAs' bound; the matrix-core kernels below would hold
// 256 registers of it a wave at R = 256).
template <typename Tout>
__global__ __launch_bounds__(kBlock) void k_rowmap_g(const float *__restrict__ M, int64_t rows,
                                                     int R, const double *__restrict__ W,
                                                     Tout *__restrict__ F) {
    __shared__ float sM[kBlock * 4];
    const int rpp = (kBlock * 4) / R > 0 ? (kBlock * 4) / R : 1;  // rows per pass staged
    const int64_t npass = (rows + rpp - 1) / rpp;
    for (int64_t pass = blockIdx.x; pass < npass; pass += gridDim.x) {
        const int64_t r0 = pass * rpp;
        const int nr = (int)((rows - r0) < rpp ? (rows - r0) : rpp);
        __syncthreads();
        for (int e = threadIdx.x; e < nr * R; e += kBlock) sM[e] = M[r0 * R + e];
        __syncthreads();
        for (int e = threadIdx.x; e < nr * R; e += kBlock) {
            const int rr = e / R, s = e % R;
            double acc = 0.0;
            const float *m = sM + rr * R;
            for (int k = 0; k < R; ++k) acc = fma((double)m[k], W[k * R + s], acc);
            st_out<Tout>(F, r0 * R + e, acc);
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_gd_rows_g(float *__restrict__ G, const T *__restrict__ F,
                                                      int64_t rows, int R,
                                                      const double *__restrict__ H,
                                                      double *__restrict__ partial) {
    __shared__ double sF[kBlock * 2];
    __shared__ double sh[kBlock];
    const int rpp = (kBlock * 2) / R > 0 ? (kBlock * 2) / R : 1;
    const int64_t npass = (rows + rpp - 1) / rpp;
    double inner = 0.0;
    for (int64_t pass = blockIdx.x; pass < npass; pass += gridDim.x) {
        const int64_t r0 = pass * rpp;
        const int nr = (int)((rows - r0) < rpp ? (rows - r0) : rpp);
        __syncthreads();
        for (int e = threadIdx.x; e < nr * R; e += kBlock) sF[e] = ld<T>(F, r0 * R + e);
        __syncthreads();
        for (int e = threadIdx.x; e < nr * R; e += kBlock) {
            const int rr = e / R, s = e % R;
            const double *f = sF + rr * R;
            double acc = 0.0;
            for (int k = 0; k < R; ++k) acc = fma(f[k], H[k * R + s], acc);
            const double m = (double)G[r0 * R + e];
            inner = fma(f[s], m, inner);
            G[r0 * R + e] = (float)(acc - m);
        }
    }
    const double tot = block_sum(inner, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kBlock) void k_gd_f(int R, const double *__restrict__ GA,
                                                 const double *__restrict__ GB,
                                                 const double *__restrict__ GC,
                                                 const double *__restrict__ partial, int npartial,
                                                 double normsq, double reg, double *__restrict__ f) {
    __shared__ double sh[kBlock];
    double in = 0.0;
    for (int b = threadIdx.x; b < npartial; b += kBlock) in += partial[b];
    double xh = 0.0, tr = 0.0;
    for (int e = threadIdx.x; e < R * R; e += kBlock) {
        xh += GA[e] * GB[e] * GC[e];
        if (e / R == e % R) tr += GA[e] + GB[e] + GC[e];
    }
    in = block_sum(in, sh);
    xh = block_sum(xh, sh);
    tr = block_sum(tr, sh);
    if (threadIdx.x == 0) *f = 0.5 * (normsq - 2.0 * in + xh) + 0.5 * reg * tr;
}

// ---- GD step: trial factors and the squared gradient norm ----------------
// out = F - alpha * G, formed in FP64 from the stored factor and the FP32
// gradient, stored in the factor dtype (BF16: FP32 then nearest-even BF16)
template <typename T>
struct TrialJobs3 {
    const T *F[3];
    const float *G[3];
    T *out[3];
    int64_t n[3];
};

template <typename T>  // (blockIdx.y the mode)
__global__ __launch_bounds__(kBlock) void k_trial_factors(TrialJobs3<T> jobs, double alpha) {
    const int m = blockIdx.y;
    const T *__restrict__ F = jobs.F[m];
    const float *__restrict__ G = jobs.G[m];
    T *__restrict__ out = jobs.out[m];
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < jobs.n[m];
         e += (int64_t)gridDim.x * kBlock)
        st_out<T>(out, e, ld<T>(F, e) - alpha * (double)G[e]);
}

// per-block partial sums of x^2 in FP64 (grid-stride, fixed order)
__global__ __launch_bounds__(kBlock) void k_sumsq_f32(const float *__restrict__ x, int64_t n,
                                                      double *__restrict__ part) {
    __shared__ double sh[kBlock];
    double acc = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kBlock) {
        const double v = (double)x[e];
        acc += v * v;
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

__global__ __launch_bounds__(kBlock) void k_sum_parts(const double *__restrict__ part, int n,
                                                      double *__restrict__ out) {
    __shared__ double sh[kBlock];
    double acc = 0.0;
    for (int b = threadIdx.x; b < n; b += kBlock) acc += part[b];
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) *out = acc;
}

// Raw 4-element runs (kept undecoded while in flight: half the registers of
// doubles for FP32, a quarter for BF16).
template <typename T>
struct Run4;
template <>
struct Run4<float> {
    float4 v;
    __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
    __device__ __forceinline__ void zero() { v = make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ __forceinline__ double operator[](int i) const {
        return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
    }
};
template <>
struct Run4<uint16_t> {
    uint2 v;
    __device__ __forceinline__ void load(const uint16_t *p) { v = *reinterpret_cast<const uint2 *>(p); }
    __device__ __forceinline__ void zero() { v = make_uint2(0u, 0u); }
    __device__ __forceinline__ double operator[](int i) const {
        const uint32_t w = i < 2 ? v.x : v.y;
        return __uint_as_float((i % 2 == 0) ? (w << 16) : (w & 0xFFFF0000u));
    }
};
__device__ __forceinline__ void store4d(float *p, const double4v &a) {
    *reinterpret_cast<float4 *>(p) = make_float4((float)a[0], (float)a[1], (float)a[2], (float)a[3]);
}
__device__ __forceinline__ void store4d(uint16_t *p, const double4v &a) {
    uint2 w;
    w.x = (uint32_t)f32_to_bf16((float)a[0]) | ((uint32_t)f32_to_bf16((float)a[1]) << 16);
    w.y = (uint32_t)f32_to_bf16((float)a[2]) | ((uint32_t)f32_to_bf16((float)a[3]) << 16);
    *reinterpret_cast<uint2 *>(p) = w;
}

// ---- joint matrix completion + tensor factorization ----------------------
// The row systems of the joint ALS (R <= 32).  An entry of a row in a ratings
// stream carries v = the other factor's row, named by the fiber's header
// (by_mid) or by the nonzero itself (the third factor is a row of ones), and
// the rating y; the row is x with
//   (sum v^T v + mu H + lam I) x = sum y v + mu M[row],  all in FP64.
//
// Four rows a wave, every product on the matrix cores: v_mfma_f64_4x4x4 takes
// four independent 4 x 4 x 4 products, one per row ("system").  Lane
// (i, b, j) = (lane / 16, lane / 4 % 4, lane % 4) belongs to system b and
// holds element (i, j) of each 4 x 4 block of its S; the same register is the
// instruction's right operand, and as the left one stands for the block's
// transpose.  Kept are the blocks on and above the diagonal (NB = 4 blocks a
// side for R <= 16, 8 for R <= 32) and the right-hand side as one more block
// column, used in its column j = 0.  Unknown i of block c is column
// joint_col(c, i): lane j's 16-byte loads of a factor row are then whole
// operands.  Columns beyond R are decoupled unit equations.
//
// What bounds it: FP64 issue -- 44 products of 16 cycles per four entries of
// four rows, and 250 products with about as much scalar-pivot arithmetic per
// solve of four -- at three waves a SIMD (168 registers; at R > 16 k_joint_rows
// keeps 17 to 19 more, and 32 to 34 scalars, in scratch).  One row a wave with
// the columns broadcast through LDS was bound by LDS bandwidth, one 512-byte
// broadcast read per multiply-add.  10M + 4M nonzeros, 400K users, 200K items,
// R = 32, users and items together: rows 4594 -> 1206 us, split rows (segments
// and their solves) 1476 -> 305 us.
constexpr int kJointRM = 32;            // largest rank
constexpr int kJointRP = kJointRM + 1;  // k_joint_small: padded LDS row
constexpr int kJointK = kJointRM / 2;   // its columns of P^-1 per lane
constexpr int kJointB = 32;             // its entries per batch
constexpr int kJointWood = 7;           // its most nonzeros a row

template <int NB>
struct JointSys {
    static constexpr int kS = NB * (NB + 1) / 2;
    static constexpr int kAll = kS + NB;  // blocks of S, then of the right-hand side
    double s[kS], b[NB];
};

template <int NB>
__device__ __host__ constexpr int joint_at(int r, int c) {  // block (r, c), r <= c
    return r * NB - r * (r - 1) / 2 + c - r;
}

__device__ __forceinline__ int joint_col(int c, int i) { return (c & 4) * 4 + 4 * i + (c & 3); }

// the lane, opaque: what a lane's place decides is formed again for each
// group of rows (kept across the loop it would spill)
__device__ __forceinline__ int joint_lane() {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    return l;
}

__device__ __forceinline__ double mfma4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

template <int ctrl>
__device__ __forceinline__ double dpp(double v) {
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(x & 0xffffffffll), ctrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), ctrl, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
// lane t of each quad's v in all four of its lanes
template <int t>
__device__ __forceinline__ double quad_bcast(double v) {
    return dpp<t * 0x55>(v);
}
// the four systems' sum, in all of them (rotations within 16 lanes)
__device__ __forceinline__ double systems_sum(double v) {
    v += dpp<0x128>(v);
    return v + dpp<0x124>(v);
}

// P = mu H + lam I in a workgroup's LDS (16 elements a block), unit equations beyond R
template <int NB>
__device__ __forceinline__ void joint_base(double *P, const double *__restrict__ H, int R, double mu,
                                           double lam) {
    int r = 0, c = 0;
    for (int q = threadIdx.x >> 4, at = 0; q < JointSys<NB>::kS; q += 4) {
        for (; at < q; ++at)
            if (++c == NB) c = ++r;
        const int row = joint_col(r, (threadIdx.x >> 2) & 3), col = joint_col(c, threadIdx.x & 3);
        double v = row == col ? 1.0 : 0.0;
        if (row < R && col < R) v = mu * H[row * R + col] + (row == col ? lam : 0.0);
        P[q * 16 + (threadIdx.x & 15)] = v;
    }
    __syncthreads();
}

// S = P
template <int NB>
__device__ __forceinline__ void joint_start(JointSys<NB> &S, const double *P, int l) {
    const int at = (l >> 4) * 4 + (l & 3);
    asm volatile("" ::: "memory");  // read here, not kept in registers
#pragma unroll
    for (int q = 0; q < JointSys<NB>::kS; ++q) S.s[q] = P[q * 16 + at];
}

// b = mu M[row] (zero without M, or for a system without a row)
template <int NB>
__device__ __forceinline__ void joint_rhs(JointSys<NB> &S, const float *__restrict__ M, int64_t row,
                                          int R, double mu, bool mine, int l) {
    const int i = l >> 4, j = l & 3;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        const int col = joint_col(c, i);
        const double m = M ? mu * (double)M[row * R + min(col, R - 1)] : 0.0;
        S.b[c] = mine && j == 0 && col < R ? m : 0.0;
    }
}

// the 16 bits of my system's lanes in a ballot, in the order 4 i + j
__device__ __forceinline__ uint32_t joint_mask(uint64_t m, int b) {
    const uint64_t y = m >> (4 * b);
    return (uint32_t)((y & 0xFull) | ((y >> 12) & 0xF0ull) | ((y >> 24) & 0xF00ull) |
                      ((y >> 36) & 0xF000ull));
}

// Adds the entries [e, e1) of each system's range (per system; empty ranges
// allowed): S += v^T v, rhs += y v.  `mid` is the index named by the header
// open at e.  Returns the system's number of nonzeros.  A step takes 16 entries per
// system, one a lane, closes up the nonzeros (a permutation within the
// system's 16 lanes) and adds them four at a time.
template <typename T, int NB, bool VEC>
__device__ __forceinline__ uint32_t joint_gather(const uint2 *__restrict__ st, uint32_t e,
                                                 uint32_t e1, uint32_t mid,
                                                 const T *__restrict__ F, bool by_mid, int R,
                                                 JointSys<NB> &S, int l) {
    const int i = l >> 4, b = (l >> 2) & 3, j = l & 3, pos = 4 * i + j;
    uint32_t total = 0, n = 0, most = 0;  // `most`: n's maximum over the four systems
    int qi = 0, qy = 0;
    e += (uint32_t)pos;
    // loads are clamped, not branched around (the stream has an entry, F a row)
    uint2 w = st[e < e1 ? e : 0];
    // one loop around the products with its one exit at the end (a nest, or an
    // exit at the refill, would keep S twice)
    uint32_t t = 0;
    bool more = false;
    do {
        if (4 * t >= most) {
            const bool in = e < e1;
            const uint64_t hb = __ballot(in && (w.x & kHdrBit));
            const uint64_t nb = __ballot(in && !(w.x & kHdrBit));
            const uint32_t hm = joint_mask(hb, b), nm = joint_mask(nb, b);
            uint32_t idx = w.x & kIdxMask;
            if (by_mid) {
                const uint32_t upto = hm & ((2u << pos) - 1u);
                const int at = 31 - __clz((int)(upto | 1u)), last = 31 - __clz((int)(hm | 1u));
                const uint32_t own =
                    (uint32_t)__shfl((int)idx, (at >> 2) * 16 + 4 * b + (at & 3));
                const uint32_t end =
                    (uint32_t)__shfl((int)idx, (last >> 2) * 16 + 4 * b + (last & 3));
                idx = upto ? own : mid;
                if (hm) mid = end;
            }
            // nonzeros first, in stream order, the rest behind them
            n = (uint32_t)__popc(nm);
            const uint32_t below = (1u << pos) - 1u;
            const uint32_t slot = ((nm >> pos) & 1u) ? (uint32_t)__popc(nm & below)
                                                     : n + (uint32_t)__popc(~nm & below);
            const int to = (int)(((slot >> 2) * 16 + 4 * (uint32_t)b + (slot & 3)) * 4);
            qi = __builtin_amdgcn_ds_permute(to, (int)idx);
            qy = __builtin_amdgcn_ds_permute(to, (int)w.y);
            total += n;
            most = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                most = max(most, (uint32_t)__popcll(nb & (0x000F000F000F000Full << (4 * q))));
            t = 0;
            e += 16;
            more = __ballot(e < e1) != 0;
            w = st[e < e1 ? e : 0];  // the next step's, in flight meanwhile
        }
        {
            const int src = 16 * (int)t + 4 * b + i;  // slot 4 t + i
            const uint32_t at = (uint32_t)__shfl(qi, src), yb = (uint32_t)__shfl(qy, src);
            const bool ok = 4 * t + (uint32_t)i < n;
            const T *f = F + (int64_t)(ok ? at : 0u) * R;
            double v[NB];
            if (VEC) {
                Run4<T> run[NB / 4];
#pragma unroll
                for (int q = 0; q < NB / 4; ++q) run[q].load(f + min(16 * q + 4 * j, R - 4));
#pragma unroll
                for (int c = 0; c < NB; ++c)
                    v[c] = ok && joint_col(c, j) < R ? run[c / 4][c % 4] : 0.0;
            } else {
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    const double x = ld<T>(f, min(joint_col(c, j), R - 1));
                    v[c] = ok && joint_col(c, j) < R ? x : 0.0;
                }
            }
            const double y = ok && j == 0 ? (double)__uint_as_float(yb) : 0.0;
#pragma unroll
            for (int r = 0; r < NB; ++r) {
#pragma unroll
                for (int c = r; c < NB; ++c)
                    S.s[joint_at<NB>(r, c)] = mfma4(v[r], v[c], S.s[joint_at<NB>(r, c)]);
                S.b[r] = mfma4(v[r], y, S.b[r]);
            }
        }
        ++t;
    } while (4 * t < most || more);
    return total;
}

// 1 / sqrt(d), d > 0 and normal: the estimate and one third-order step
// (r + r e (1/2 + 3/8 e), e = 1 - d r^2: past 2^-26 this leaves the rounding)
__device__ __forceinline__ double joint_rsqrt(double d) {
    const double r = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * r, r, 1.0);
    return fma(r * e, fma(e, 0.375, 0.5), r);
}

// one pivot of a diagonal block: a's rows below are eliminated, u keeps
// the inverse unit factor's transpose and ds the pivots' inverse roots
template <int t>
__device__ __forceinline__ void joint_pivot(double &a, double &u, double &ds, bool &ok, bool pad,
                                            double tol, int i, int j) {
    const double row = mfma4(i == t ? 1.0 : 0.0, a, 0.0);  // a[t][j] in every i
    const double d = quad_bcast<t>(row);                    // the Schur-complement pivot
    ok = ok & (pad | (d > tol));  // (no branches)
    const double inv = joint_rsqrt(d);
    ds = j == t ? inv : ds;
    if (t < 3) {
        const double m = j > t ? row * (inv * inv) : 0.0;
        const double ca = quad_bcast<t>(a), cu = quad_bcast<t>(u);
        a = fma(-ca, m, a);
        u = fma(-cu, m, u);
    }
}

// S x = b for the wave's four systems; x comes back in S.b.  Blocked Cholesky
// S = U^T U with the pivot test d > R eps max diag(S); the inverse of each
// diagonal block of U takes the block's place.  Returns whether the system
// passed (its x is meaningless otherwise; the other systems don't see it).
template <int NB>
__device__ __forceinline__ bool joint_solve(JointSys<NB> &S, int R, int l) {
    const int i = l >> 4, j = l & 3;
    double dm = 0.0;
#pragma unroll
    for (int c = 0; c < NB; ++c)
        if (i == j && joint_col(c, j) < R) dm = fmax(dm, S.s[joint_at<NB>(c, c)]);
#pragma unroll
    for (int o = 1; o < 64; o = o == 2 ? 16 : 2 * o) dm = fmax(dm, __shfl_xor(dm, o, 64));
    const double tol = (double)R * DBL_EPSILON * dm;
    bool ok = dm > 0.0;
    const double eye = i == j ? 1.0 : 0.0;
#pragma unroll
    for (int p = 0; p < NB; ++p) {
        double a = S.s[joint_at<NB>(p, p)], u = eye, ds = 0.0;
        joint_pivot<0>(a, u, ds, ok, joint_col(p, 0) >= R, tol, i, j);
        joint_pivot<1>(a, u, ds, ok, joint_col(p, 1) >= R, tol, i, j);
        joint_pivot<2>(a, u, ds, ok, joint_col(p, 2) >= R, tol, i, j);
        joint_pivot<3>(a, u, ds, ok, joint_col(p, 3) >= R, tol, i, j);
        u *= ds;
        S.s[joint_at<NB>(p, p)] = u;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = p + 1; c < NB; ++c)
            S.s[joint_at<NB>(p, c)] = mfma4(u, S.s[joint_at<NB>(p, c)], 0.0);
        S.b[p] = mfma4(u, S.b[p], 0.0);
#pragma unroll
        for (int r = p + 1; r < NB; ++r) {
            const double nu = -S.s[joint_at<NB>(p, r)];
#pragma unroll
            for (int c = r; c < NB; ++c)
                S.s[joint_at<NB>(r, c)] =
                    mfma4(nu, S.s[joint_at<NB>(p, c)], S.s[joint_at<NB>(r, c)]);
            S.b[r] = mfma4(nu, S.b[p], S.b[r]);
        }
    }
    // U x = y, a product with the unit block transposing each left operand
#pragma unroll
    for (int p = NB - 1; p >= 0; --p) {
        S.b[p] = mfma4(mfma4(S.s[joint_at<NB>(p, p)], eye, 0.0), S.b[p], 0.0);
#pragma unroll
        for (int r = 0; r < p; ++r)
            S.b[r] = mfma4(-mfma4(S.s[joint_at<NB>(r, p)], eye, 0.0), S.b[p], S.b[r]);
        __builtin_amdgcn_sched_barrier(0);  // few transposes in flight
    }
    return ok;
}

// out[row] = x (zeros when the system failed), by the lanes j = 0
template <typename T, int NB>
__device__ __forceinline__ void joint_store(const JointSys<NB> &S, bool ok, int64_t row, int R,
                                            bool vec, T *__restrict__ out, int l) {
    const int i = l >> 4;
    T *o = out + row * R;
#pragma unroll
    for (int q = 0; q < NB / 4; ++q) {
        const int col = 16 * q + 4 * i;
        double4v x;
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = ok ? S.b[4 * q + c] : 0.0;
        if (vec) {
            if (col < R) store4d(o + col, x);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (col + c < R) st_out<T>(o, col + c, x[c]);
        }
    }
}

// every row of at most kJointLight entries, four a wave (persistent grid: a
// workgroup forms P once).  A row of at most kJointWood nonzeros in one batch
// that fails the test raises *need instead of *flag: k_joint_small decides.
template <typename T, int NB, bool VEC>
__global__ __launch_bounds__(64, 3) void k_joint_rows(
    const uint2 *__restrict__ st, const uint2 *__restrict__ range, int64_t nrows,
    const T *__restrict__ F, bool by_mid, int R, const float *__restrict__ M,
    const double *__restrict__ H, double mu, double lam, T *__restrict__ out,
    int *__restrict__ flag, int *__restrict__ need) {
    using Sys = JointSys<NB>;
    __shared__ double P[Sys::kS * 16];
    joint_base<NB>(P, H, R, mu, lam);
    for (int64_t g = blockIdx.x; 4 * g < nrows; g += gridDim.x) {
        const int l = joint_lane(), i = l >> 4, b = (l >> 2) & 3, j = l & 3;
        const int64_t row = 4 * g + b;
        uint2 rg = row < nrows ? range[row] : make_uint2(0u, 0u);
        const bool mine = row < nrows && rg.y - rg.x <= (uint32_t)kJointLight;
        if (!mine) rg = make_uint2(0u, 0u);
        Sys S;
        joint_start<NB>(S, P, l);
        joint_rhs<NB>(S, M, mine ? row : 0, R, mu, mine, l);
        const uint32_t n = joint_gather<T, NB, VEC>(st, rg.x, rg.y, 0u, F, by_mid, R, S, l);
        const bool ok = joint_solve<NB>(S, R, l);
        if (mine && j == 0) {
            joint_store<T, NB>(S, ok, row, R, VEC, out, l);
            if (!ok && i == 0)
                atomicOr(rg.y - rg.x <= (uint32_t)kJointB && n <= (uint32_t)kJointWood ? need : flag,
                         1);
        }
    }
}

// One segment of a heavy row: its entries over the 16 systems of four waves,
// added up in a fixed order to one partial system (kAll blocks of 16).
template <typename T, int NB, bool VEC>
__global__ __launch_bounds__(256, 3) void k_joint_segments(
    const uint2 *__restrict__ st, const uint2 *__restrict__ seg, int64_t nseg,
    const T *__restrict__ F, bool by_mid, int R, double *__restrict__ part) {
    using Sys = JointSys<NB>;
    __shared__ double red[4][Sys::kAll * 16];
    const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int i = l >> 4, b = (l >> 2) & 3, j = l & 3, pos = 4 * i + j;
    for (int64_t q = blockIdx.x; q < nseg; q += gridDim.x) {
        const uint2 sg = seg[q];
        const uint32_t len = (((sg.y - sg.x + 15) / 16 + 15) / 16) * 16;  // per system
        const uint32_t e0 = min(sg.y, sg.x + (uint32_t)(4 * wv + b) * len);
        const uint32_t e1 = min(sg.y, e0 + len);
        // the header open at e0 is at most one fiber before it, and the row's
        // first entry is a header
        uint32_t mid = 0;
        if (by_mid) {
            bool open = e0 < e1 && !(st[e0].x & kHdrBit);
            for (uint32_t back = 1; __ballot(open) != 0; back += 16) {
                const uint32_t d = back + (uint32_t)pos;
                const uint2 w = open && d <= e0 ? st[e0 - d] : make_uint2(0u, 0u);
                const uint32_t hm = joint_mask(__ballot((w.x & kHdrBit) != 0), b);
                const int at = __ffs((int)(hm | 0x10000u)) - 1;  // the nearest
                const uint32_t m =
                    (uint32_t)__shfl((int)(w.x & kIdxMask), ((at >> 2) & 3) * 16 + 4 * b + (at & 3));
                if (open && hm) {
                    mid = m;
                    open = false;
                }
                if (back + 16 > e0) open = false;
            }
        }
        Sys S;
#pragma unroll
        for (int x = 0; x < Sys::kS; ++x) S.s[x] = 0.0;
#pragma unroll
        for (int x = 0; x < NB; ++x) S.b[x] = 0.0;
        joint_gather<T, NB, VEC>(st, e0, e1, mid, F, by_mid, R, S, l);
#pragma unroll
        for (int x = 0; x < Sys::kAll; ++x) {
            double v = x < Sys::kS ? S.s[x < Sys::kS ? x : 0] : S.b[x < Sys::kS ? 0 : x - Sys::kS];
            v = systems_sum(v);
            if (b == 0) red[wv][x * 16 + pos] = v;
        }
        __syncthreads();
        for (int x = threadIdx.x; x < Sys::kAll * 16; x += 256)
            part[q * (Sys::kAll * 16) + x] = ((red[0][x] + red[1][x]) + red[2][x]) + red[3][x];
        __syncthreads();
    }
}

// heavy rows, four a wave: the sum of a row's partial systems in segment
// order (part begins with segment seg0's), solved
template <typename T, int NB>
__global__ __launch_bounds__(64, 2) void k_joint_heavy(const uint4 *__restrict__ heavy,
                                                    int64_t nheavy, int64_t seg0, int R, bool vec,
                                                    const double *__restrict__ part,
                                                    const float *__restrict__ M,
                                                    const double *__restrict__ H, double mu,
                                                    double lam, T *__restrict__ out,
                                                    int *__restrict__ flag) {
    using Sys = JointSys<NB>;
    __shared__ double P[Sys::kS * 16];
    joint_base<NB>(P, H, R, mu, lam);
    for (int64_t g = blockIdx.x; 4 * g < nheavy; g += gridDim.x) {
        const int l = joint_lane(), i = l >> 4, b = (l >> 2) & 3, j = l & 3;
        const bool mine = 4 * g + b < nheavy;
        // (row, first segment, segments, 0)
        const uint4 hv = mine ? heavy[4 * g + b] : make_uint4(0u, 0u, 0u, 0u);
        const int64_t row = (int64_t)hv.x;
        Sys S;
        joint_start<NB>(S, P, l);
        joint_rhs<NB>(S, M, row, R, mu, mine, l);
        for (uint32_t q = hv.y; q < hv.y + hv.z; ++q) {
            const double *pt = part + ((int64_t)q - seg0) * (Sys::kAll * 16) + 4 * i + j;
            double v[Sys::kAll];  // all loads in flight
#pragma unroll
            for (int x = 0; x < Sys::kAll; ++x) v[x] = pt[x * 16];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < Sys::kS; ++x) S.s[x] += v[x];
#pragma unroll
            for (int x = 0; x < NB; ++x) S.b[x] += v[Sys::kS + x];
        }
        const bool ok = joint_solve<NB>(S, R, l);
        if (mine && j == 0) {
            joint_store<T, NB>(S, ok, row, R, vec, out, l);
            if (!ok && i == 0) atomicOr(flag, 1);
        }
    }
}

// lane `src`'s v (src uniform) in every lane
__device__ __forceinline__ double lane_bcast(double v, int src) {
    const long long x = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(x & 0xffffffffll), src);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(x >> 32), src);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// One batch [b, min(b + 32, e1)) of a ratings stream: the nonzeros'
// vectors go, compacted in stream order, to rows 0 .. n-1 of V (columns
// beyond R zero) and their ratings to Yb; returns n.  A header opens the batch.
template <typename T>
__device__ int joint_load_batch(const uint2 *__restrict__ st, uint32_t b, uint32_t e1,
                                const T *__restrict__ F, bool by_mid, int R, double *V,
                                double *Yb) {
    const int h = threadIdx.x >> 5, t = threadIdx.x & 31;
    // entry t of the batch in lanes t and t + 32
    const uint32_t e = b + (uint32_t)t;
    const bool in = e < e1;
    const uint2 w = in ? st[e] : make_uint2(0u, 0u);
    const bool hdr = in && (w.x & kHdrBit);
    const bool nz = in && !(w.x & kHdrBit);
    const uint64_t hm = __ballot(hdr) & 0xffffffffull;
    const uint64_t nm = __ballot(nz) & 0xffffffffull;
    const uint64_t upto = hm & ((2ull << t) - 1ull);
    const uint32_t midx = w.x & kIdxMask;
    const uint32_t mid = (uint32_t)__shfl((int)midx, upto ? 63 - __clzll((long long)upto) : 0);
    if (nz) {
        const int slot = __popcll(nm & ((1ull << t) - 1ull));
        const T *f = F + (int64_t)(by_mid ? mid : w.x) * R;
#pragma unroll
        for (int k = 0; k < kJointK; ++k) {
            const int q = 2 * k + h;
            V[slot * kJointRP + q] = q < R ? ld<T>(f, q) : 0.0;
        }
        if (h == 0) Yb[slot] = (double)__uint_as_float(w.y);
    }
    __syncthreads();
    return __popcll(nm);
}

// A row of at most kJointWood entries (vectors v_e in rows of V, ratings in
// Yb) solved without factorizing its own S = P + V^T V, from P^-1 (the same
// for every row of the mode).  With b = sum_e y_e v_e + mu m the
// Sherman-Morrison-Woodbury identity and S^-1 V^T = P^-1 V^T K^-1 give
//   z = P^-1 mu m,  u_e = P^-1 v_e,  K = I + [v_e . u_f],
//   t = [y_e - v_e . z],  K w = t,  x = z + sum_e w_e u_e.
// The ratings enter behind K^-1: with them in z, x would be the difference of
// two terms of size P^-1 V^T y, far above x where P is small beside V^T V,
// which is when a row comes here.
// P^-1 = ws * Pinv (R x R, row-major), or ws * I when Pinv is null.  K is
// symmetric positive definite with eigenvalues >= 1 and is solved by
// Gauss-Jordan without pivoting, lane (e, f) = e * 8 + f holding K[e][f]
// and lane (e, n) holding t[e].  U (kJointRM rows of kJointRP doubles, apart
// from V's first n rows) holds u_e and z; Bb (32 doubles) carries mu m.
template <typename T>
__device__ void joint_woodbury(int n, const double *V, const double *Yb, double mu, double m,
                               const double *__restrict__ Pinv, double ws, int R, int64_t row,
                               T *__restrict__ out, double *U, double *Bb) {
    const int l = threadIdx.x, h = l >> 5, r = l & 31;
    double wr[kJointK];  // P^-1[r][2k + h]
#pragma unroll
    for (int k = 0; k < kJointK; ++k) {
        const int q = 2 * k + h;
        wr[k] = (r < R && q < R) ? (Pinv ? ws * Pinv[r * R + q] : (q == r ? ws : 0.0)) : 0.0;
    }
    if (h == 0) Bb[r] = mu * m;
    __syncthreads();
    double zp = 0.0;
#pragma unroll
    for (int k = 0; k < kJointK; ++k) zp = fma(wr[k], Bb[2 * k + h], zp);
    const double z = zp + __shfl_xor(zp, 32, 64);  // the halves' sums, equal in both
    for (int e = 0; e < n; ++e) {
        double up = 0.0;
#pragma unroll
        for (int k = 0; k < kJointK; ++k) up = fma(wr[k], V[e * kJointRP + 2 * k + h], up);
        const double u = up + __shfl_xor(up, 32, 64);
        if (h == 0) U[e * kJointRP + r] = u;
    }
    if (h == 0) U[n * kJointRP + r] = z;
    __syncthreads();
    // G[e][f] = a_e . v_f for e <= n (a_e = u_e, a_n = z) and f < n
    const int ge = l >> 3, gf = l & 7;
    double g = 0.0;
    if (ge <= n && gf < n) {
#pragma unroll 4
        for (int q = 0; q < kJointRM; ++q) g = fma(U[ge * kJointRP + q], V[gf * kJointRP + q], g);
    }
    const double tv = __shfl(g, n * 8 + ge, 64);  // v_ge . z
    double a = 0.0;
    if (ge < n && gf < n) a = g + (ge == gf ? 1.0 : 0.0);
    if (ge < n && gf == n) a = Yb[ge] - tv;
    for (int j = 0; j < n; ++j) {
        const double inv = 1.0 / lane_bcast(a, j * 9);  // K's pivot at step j
        const double rowj = __shfl(a, j * 8 + gf, 64);
        const double colj = __shfl(a, ge * 8 + j, 64);
        a = ge == j ? rowj * inv : fma(-colj * inv, rowj, a);
    }
    double x = z;
    for (int e = 0; e < n; ++e) x = fma(lane_bcast(a, e * 8 + n), U[e * kJointRP + r], x);
    if (h == 0 && r < R) st_out<T>(out, row * R + r, x);
    __syncthreads();  // U, V and Bb are free again
}

// Short rows whose own system is too close to singular for the pivot test
// although P is not (a tiny lam and few ratings): all short rows once more by
// the Woodbury identity, from P^-1.  Does nothing unless a short row raised
// *need; without a valid P^-1 (*pflag != 0) such a row is a failure.
template <typename T>
__global__ __launch_bounds__(64) void k_joint_small(const uint2 *__restrict__ st,
                                                    const uint2 *__restrict__ range, int64_t nrows,
                                                    const T *__restrict__ F, bool by_mid, int R,
                                                    const float *__restrict__ M, double mu,
                                                    const double *__restrict__ Pinv, double ws,
                                                    const int *__restrict__ pflag,
                                                    T *__restrict__ out, int *__restrict__ flag,
                                                    const int *__restrict__ need) {
    __shared__ double V[kJointB * kJointRP], Yb[kJointB], Bb[32];
    if (*need == 0) return;
    if (Pinv && *pflag != 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(flag, 1);
        return;
    }
    const int r = threadIdx.x & 31;
    for (int64_t row = blockIdx.x; row < nrows; row += gridDim.x) {
        const uint2 rg = range[row];
        if (rg.y - rg.x > (uint32_t)kJointB) continue;
        const int n = rg.y > rg.x ? joint_load_batch<T>(st, rg.x, rg.y, F, by_mid, R, V, Yb) : 0;
        if (n > kJointWood) {
            __syncthreads();
            continue;
        }
        const double m = (M && r < R) ? (double)M[row * R + r] : 0.0;
        joint_woodbury<T>(n, V, Yb, mu, m, Pinv, ws, R, row, out, V + 16 * kJointRP, Bb);
    }
}

// G = mu G + lam F - RY (RY may be null): the joint gradient from the
// tensor part -M + F H, the ridge term and the ratings part
template <typename T>
__global__ __launch_bounds__(kBlock) void k_joint_combine(float *__restrict__ G,
                                                          const T *__restrict__ F,
                                                          const float *__restrict__ RY, double mu,
                                                          double lam, int64_t n) {
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kBlock) {
        double g = mu * (double)G[e] + lam * ld<T>(F, e);
        if (RY) g -= (double)RY[e];
        G[e] = (float)g;
    }
}

// per-block partial sums of F[e] * X[e] in FP64 (grid-stride, fixed order)
template <typename T>
__global__ __launch_bounds__(kBlock) void k_dot_parts(const T *__restrict__ F,
                                                      const float *__restrict__ X, int64_t n,
                                                      double *__restrict__ part) {
    __shared__ double sh[kBlock];
    double acc = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)kBlock + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * kBlock)
        acc = fma(ld<T>(F, e), (double)X[e], acc);
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// f = mu f_tensor + lam/2 (tr G_A + tr G_B + tr G_C)
//     + 1/2 (||Y||^2 - <A, Y B> - <A, residual(Y) B>)
// (the ratings term: sum r^2 = sum r y - sum r (a.b) = ||Y||^2 - <A,YB> - <A,RB>)
__global__ __launch_bounds__(kBlock) void k_joint_f(const double *__restrict__ ft,
                                                    const double *__restrict__ GA,
                                                    const double *__restrict__ GB,
                                                    const double *__restrict__ GC, int R,
                                                    const double *__restrict__ part, int npart,
                                                    double normsq_y, double mu, double lam,
                                                    double *__restrict__ f) {
    __shared__ double sh[kBlock];
    double in = 0.0, tr = 0.0;
    for (int b = threadIdx.x; b < npart; b += kBlock) in += part[b];
    for (int r = threadIdx.x; r < R; r += kBlock) tr += GA[r * R + r] + GB[r * R + r] + GC[r * R + r];
    in = block_sum(in, sh);
    tr = block_sum(tr, sh);
    if (threadIdx.x == 0) *f = mu * ft[0] + 0.5 * lam * tr + 0.5 * (normsq_y - in);
}

// ---------------------------------------------------------------------------
// Row maps on the matrix cores, R = 16 * NCT (16, 32, 48, 64).
//
// A wave takes 16 rows X[r0 .. r0+16) at a time and forms out^T = W^T X^T with
// FP64 MFMA 16x16x4 steps: the R x R matrix is the A operand and stays in
// registers for the whole kernel (4 * NCT^2 doubles per lane), the rows are
// the B operand.  Two index permutations make every lane's memory accesses
// 4 consecutive elements wide:
//  * contraction index: at step t, lane group g = lane / 16 contributes
//    k = 16 * (t / 4) + 4 * g + t % 4, so a lane reads columns
//    16 * c + 4 * g .. + 4 of its row for c = 0 .. NCT-1;
//  * output index: MFMA output row m of column tile c is column
//    16 * c + 4 * (m % 4) + m / 4, so the 4 accumulator entries of a lane are
//    columns 16 * c + 4 * g .. + 4 of row r0 + lane % 16 -- the same columns
//    it read.
// Accumulation is FP64; the next tile's rows are loaded before the current
// tile's MFMAs.
// ---------------------------------------------------------------------------
// wa[c][t] = W[k(t)][16 c + column of MFMA row lane % 16]
template <int NCT>
__device__ __forceinline__ void load_rmat(const double *__restrict__ W, int lane,
                                          double (&wa)[NCT][4 * NCT]) {
    constexpr int R = 16 * NCT;
    const int g = lane / 16, m = lane % 16;
    const int col = 4 * (m % 4) + m / 4;
#pragma unroll
    for (int c = 0; c < NCT; ++c)
#pragma unroll
        for (int t = 0; t < 4 * NCT; ++t) {
            const int k = 16 * (t / 4) + 4 * g + t % 4;
            wa[c][t] = W[k * R + 16 * c + col];
        }
}

// the 4 * NCT entries of row `row` that this lane reads (zero past the last row)
template <int NCT, typename T>
__device__ __forceinline__ void load_rowrun(const T *__restrict__ X, int64_t row, int64_t rows,
                                            int g, Run4<T> (&v)[NCT]) {
    constexpr int R = 16 * NCT;
    if (row < rows) {
#pragma unroll
        for (int c = 0; c < NCT; ++c) v[c].load(X + row * R + 16 * c + 4 * g);
    } else {
#pragma unroll
        for (int c = 0; c < NCT; ++c) v[c].zero();
    }
}

// F[row, s] = sum_k M[row, k] W[k, s]
template <typename Tout, int NCT>
__device__ __forceinline__ void rowmap_mfma_body(const float *__restrict__ M, int64_t rows,
                                                 const double *__restrict__ W,
                                                 Tout *__restrict__ F, uint32_t b, uint32_t nb) {
    constexpr int R = 16 * NCT, S = 4 * NCT;
    const int lane = threadIdx.x % 64, g = lane / 16;
    double wa[NCT][S];
    load_rmat<NCT>(W, lane, wa);
    const int64_t ntile = (rows + 15) / 16;
    const int64_t nw = (int64_t)nb * (kBlock / 64);
    int64_t tile = (int64_t)b * (kBlock / 64) + threadIdx.x / 64;
    Run4<float> x[NCT];
    load_rowrun<NCT>(M, tile * 16 + lane % 16, rows, g, x);
    for (; tile < ntile; tile += nw) {
        const int64_t row = tile * 16 + lane % 16;
        Run4<float> xn[NCT];
        load_rowrun<NCT>(M, row + 16 * nw, rows, g, xn);
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
            double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int t = 0; t < S; ++t)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(wa[c][t], x[t / 4][t % 4], acc, 0, 0, 0);
            if (row < rows) store4d(F + row * R + 16 * c + 4 * g, acc);
        }
#pragma unroll
        for (int c = 0; c < NCT; ++c) x[c] = xn[c];
    }
}

template <typename Tout, int NCT>
__global__ __launch_bounds__(kBlock) void k_rowmap_mfma(const float *__restrict__ M, int64_t rows,
                                                        const double *__restrict__ W,
                                                        Tout *__restrict__ F) {
    rowmap_mfma_body<Tout, NCT>(M, rows, W, F, blockIdx.x, gridDim.x);
}

template <typename Tout, int NCT>
__global__ __launch_bounds__(kBlock) void k_rowmap_mfma_group(const RowmapJob *__restrict__ jobs,
                                                              const uint2 *__restrict__ vb) {
    const uint2 v = vb[blockIdx.x];
    const RowmapJob &j = jobs[v.x];
    rowmap_mfma_body<Tout, NCT>(j.M, j.rows, j.W, (Tout *)j.F, v.y, j.nblk);
}

// G[row, s] = -G[row, s] + sum_k F[row, k] H[k, s]  (G holds the MTTKRP on
// entry); partial[block] = sum over the block's rows of <F[row,:], G[row,:]>
// (the entry values).
template <typename T, int NCT>
__global__ __launch_bounds__(kBlock) void k_gd_rows_mfma(float *__restrict__ G,
                                                         const T *__restrict__ F, int64_t rows,
                                                         const double *__restrict__ H,
                                                         double *__restrict__ partial) {
    constexpr int R = 16 * NCT, S = 4 * NCT;
    __shared__ double sh[kBlock];
    const int lane = threadIdx.x % 64, g = lane / 16;
    double wa[NCT][S];
    load_rmat<NCT>(H, lane, wa);
    const int64_t ntile = (rows + 15) / 16;
    const int64_t nw = (int64_t)gridDim.x * (kBlock / 64);
    int64_t tile = (int64_t)blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
    double inner = 0.0;
    Run4<T> f[NCT];
    Run4<float> m[NCT];
    load_rowrun<NCT>(F, tile * 16 + lane % 16, rows, g, f);
    load_rowrun<NCT>((const float *)G, tile * 16 + lane % 16, rows, g, m);
    for (; tile < ntile; tile += nw) {
        const int64_t row = tile * 16 + lane % 16;
        Run4<T> fn[NCT];
        Run4<float> mn[NCT];
        load_rowrun<NCT>(F, row + 16 * nw, rows, g, fn);
        load_rowrun<NCT>((const float *)G, row + 16 * nw, rows, g, mn);
#pragma unroll
        for (int t = 0; t < S; ++t) inner = fma(f[t / 4][t % 4], m[t / 4][t % 4], inner);
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
            double4v acc = {-m[c][0], -m[c][1], -m[c][2], -m[c][3]};
#pragma unroll
            for (int t = 0; t < S; ++t)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(wa[c][t], f[t / 4][t % 4], acc, 0, 0, 0);
            if (row < rows) store4d(G + row * R + 16 * c + 4 * g, acc);
        }
#pragma unroll
        for (int c = 0; c < NCT; ++c) {
            f[c] = fn[c];
            m[c] = mn[c];
        }
    }
    const double tot = block_sum(inner, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// Row maps of any rank up to 128 (and of any alignment).  A block takes 16 RS
// rows at a time through LDS, coalesced both ways.  Its four waves are RS row
// tiles times 4 / RS pairs of output column tiles; a wave keeps its pair's
// R x 32 part of the matrix in registers as the A operand, the rows are the B
// operand.  The per-element loops read both factors of every FMA from LDS:
// R = 100, the same three factors 381 -> 124 us on average; gradient rows at
// R = 10, 350,000 rows 190 -> 73 us (beside the MTTKRP).
template <int NCT>
struct RowAny {
    static constexpr int RS = NCT <= 2 ? 4 : (NCT <= 4 ? 2 : 1);  // row tiles per block
    static constexpr int TR = 16 * RS;                           // rows per block and step
    static constexpr int RP = 16 * NCT + 1;                      // LDS row
    static constexpr int S = 4 * NCT;                            // contraction steps
};

// wa[c][t] = W[4 t + lane / 16][16 (2 cg + c) + lane % 16], zero beyond R
template <int NCT>
__device__ __forceinline__ void load_any(const double *__restrict__ W, int R, int cg,
                                         double (&wa)[2][RowAny<NCT>::S]) {
    const int lane = threadIdx.x % 64;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int t = 0; t < RowAny<NCT>::S; ++t) {
            const int k = 4 * t + lane / 16, col = 16 * (2 * cg + c) + lane % 16;
            wa[c][t] = k < R && col < R ? W[k * R + col] : 0.0;
        }
}

// F[row, s] = sum_k M[row, k] W[k, s]
template <typename Tout, int NCT>
__global__ __launch_bounds__(kBlock) void k_rowmap_any(const float *__restrict__ M, int64_t rows,
                                                       int R, const double *__restrict__ W,
                                                       Tout *__restrict__ F) {
    using A = RowAny<NCT>;
    __shared__ float sx[A::TR * A::RP], so[A::TR * A::RP];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int rs = wave % A::RS, cg = wave / A::RS;
    double wa[2][A::S];
    load_any<NCT>(W, R, cg, wa);
    for (int e = threadIdx.x; e < A::TR * A::RP; e += kBlock) sx[e] = 0.f;
    const int64_t ntile = (rows + A::TR - 1) / A::TR;
    for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const int64_t r0 = tile * A::TR;
        const int n = (int)(rows - r0 < A::TR ? rows - r0 : A::TR) * R;
        __syncthreads();
        for (int e = threadIdx.x; e < n; e += kBlock) {
            const int r = e / R;
            sx[r * A::RP + e - r * R] = M[r0 * R + e];
        }
        __syncthreads();
        const float *x = sx + (16 * rs + lane % 16) * A::RP + lane / 16;
        double4v acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int t = 0; t < A::S; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                if (2 * cg + c < NCT)
                    acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(wa[c][t], (double)x[4 * t],
                                                                  acc[c], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < 2; ++c)
            if (2 * cg + c < NCT) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    so[(16 * rs + lane % 16) * A::RP + 16 * (2 * cg + c) + lane / 16 + 4 * v] =
                        (float)acc[c][v];
            }
        __syncthreads();
        for (int e = threadIdx.x; e < n; e += kBlock) {
            const int r = e / R;
            st_out<Tout>(F, r0 * R + e, (double)so[r * A::RP + e - r * R]);
        }
    }
}

// G[row, s] = -G[row, s] + sum_k F[row, k] H[k, s]  (G holds the MTTKRP);
// partial[block] = sum over the block's rows of <F[row,:], M[row,:]>.
template <typename T, int NCT>
__global__ __launch_bounds__(kBlock) void k_gd_rows_any(float *__restrict__ G,
                                                        const T *__restrict__ F, int64_t rows,
                                                        int R, const double *__restrict__ H,
                                                        double *__restrict__ partial) {
    using A = RowAny<NCT>;
    __shared__ float sx[A::TR * A::RP], so[A::TR * A::RP];
    __shared__ double sh[kBlock];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int rs = wave % A::RS, cg = wave / A::RS;
    double wa[2][A::S];
    load_any<NCT>(H, R, cg, wa);
    for (int e = threadIdx.x; e < A::TR * A::RP; e += kBlock) sx[e] = so[e] = 0.f;
    double inner = 0.0;
    const int64_t ntile = (rows + A::TR - 1) / A::TR;
    for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const int64_t r0 = tile * A::TR;
        const int n = (int)(rows - r0 < A::TR ? rows - r0 : A::TR) * R;
        __syncthreads();
        for (int e = threadIdx.x; e < n; e += kBlock) {
            const int r = e / R, o = r * A::RP + e - r * R;
            const float f = ldf<T>(F, r0 * R + e), m = G[r0 * R + e];
            sx[o] = f;
            so[o] = m;
            inner = fma((double)f, (double)m, inner);
        }
        __syncthreads();
        const float *x = sx + (16 * rs + lane % 16) * A::RP + lane / 16;
        float *m = so + (16 * rs + lane % 16) * A::RP + 32 * cg + lane / 16;
        double4v acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int t = 0; t < A::S; ++t)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                if (2 * cg + c < NCT)
                    acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(wa[c][t], (double)x[4 * t],
                                                                  acc[c], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < 2; ++c)
            if (2 * cg + c < NCT) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float *o = m + 16 * c + 4 * v;
                    *o = (float)(acc[c][v] - (double)*o);
                }
            }
        __syncthreads();
        for (int e = threadIdx.x; e < n; e += kBlock) {
            const int r = e / R;
            G[r0 * R + e] = so[r * A::RP + e - r * R];
        }
    }
    const double tot = block_sum(inner, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

constexpr int kRowAnyMaxR = 128;

// f(integral_constant<int, NCT>) for the column tiles of rank R <= kRowAnyMaxR
template <typename Fn>
void with_tiles(int R, Fn &&f) {
    switch ((R + 15) / 16) {
        case 1: return f(std::integral_constant<int, 1>{});
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 7: return f(std::integral_constant<int, 7>{});
        default: return f(std::integral_constant<int, 8>{});
    }
}

unsigned rows_grid_any(int64_t rows, int R) {
    const int nct = (R + 15) / 16, tr = 16 * (nct <= 2 ? 4 : (nct <= 4 ? 2 : 1));
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((rows + tr - 1) / tr, 2048));
}

// ranks with a matrix-core row kernel; the rows must start 16-byte aligned
// (FP32) or 8-byte aligned (BF16)
bool mfma_rows_ok(int R, const void *a, size_t ea, const void *b, size_t eb) {
    if (!(R == 16 || R == 32 || R == 48 || R == 64)) return false;
    return (uintptr_t)a % (4 * ea) == 0 && (uintptr_t)b % (4 * eb) == 0;
}

unsigned rows_grid_mfma(int64_t rows) {
    const int64_t ntile = (rows + 15) / 16;
    const int64_t want = (ntile + 4 * 4 - 1) / (4 * 4);  // about 4 tiles per wave
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(want, 2048));
}

template <typename Tout>
void rowmap_mfma(hipStream_t s, const float *M, int64_t rows, int R, const double *W, void *F) {
    const dim3 grid(rows_grid_mfma(rows)), block(kBlock);
    switch (R) {
        case 16: hipLaunchKernelGGL((k_rowmap_mfma<Tout, 1>), grid, block, 0, s, M, rows, W, (Tout *)F); break;
        case 32: hipLaunchKernelGGL((k_rowmap_mfma<Tout, 2>), grid, block, 0, s, M, rows, W, (Tout *)F); break;
        case 48: hipLaunchKernelGGL((k_rowmap_mfma<Tout, 3>), grid, block, 0, s, M, rows, W, (Tout *)F); break;
        default: hipLaunchKernelGGL((k_rowmap_mfma<Tout, 4>), grid, block, 0, s, M, rows, W, (Tout *)F); break;
    }
}

template <typename T>
void gd_rows_mfma(hipStream_t s, float *G, const void *F, int64_t rows, int R, const double *H,
                  double *partial) {
    const dim3 grid(rows_grid_mfma(rows)), block(kBlock);
    const T *Ft = (const T *)F;
    switch (R) {
        case 16: hipLaunchKernelGGL((k_gd_rows_mfma<T, 1>), grid, block, 0, s, G, Ft, rows, H, partial); break;
        case 32: hipLaunchKernelGGL((k_gd_rows_mfma<T, 2>), grid, block, 0, s, G, Ft, rows, H, partial); break;
        case 48: hipLaunchKernelGGL((k_gd_rows_mfma<T, 3>), grid, block, 0, s, G, Ft, rows, H, partial); break;
        default: hipLaunchKernelGGL((k_gd_rows_mfma<T, 4>), grid, block, 0, s, G, Ft, rows, H, partial); break;
    }
}

bool tiled_rows_ok(int R) {  // ranks with a compile-time LDS-tiled row kernel (<= ~51 KB LDS)
    return R == 4 || R == 8 || R == 12 || R == 16 || R == 32 || R == 48;
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

GramPlan gram_plan(int64_t rows, int R, const void *F, dfacto_dtype dtype) {
    GramPlan g;
    g.nt = (R + 15) / 16;
    const int bs = g.nt <= 2 ? 1024 : 256;  // 16 waves per block when the registers allow
    // Short factors (batched members): eight 16-row steps per wave, so that a
    // block's fixed costs (combining its waves' sums in LDS, writing its
    // partial R x R block) stay small beside its work.  Longer ones: two, so
    // that a single Gram spreads over enough blocks to fill the device.
    const int64_t per_blk = 16 * (rows < 65536 ? 8 : 2) * (bs / 64);
    const int64_t want = (rows + per_blk - 1) / per_blk;
    g.nblk = (int)std::max<int64_t>(1, std::min<int64_t>(want, 256));
    const size_t es = dtype == DFACTO_F32 ? 4 : 2;
    g.vec = R == 32 && (uintptr_t)F % (2 * es) == 0;
    return g;
}

// the partial-sum buffer of the stream the Gram is launched on
static dfacto_ctx::Slot gram_slot(const dfacto_ctx *ctx) {
    return (ctx->side && ctx->stream == ctx->side) ? dfacto_ctx::kPartialSide
                                                   : dfacto_ctx::kPartial;
}

void launch_gram(dfacto_ctx *ctx, const void *F, dfacto_dtype dtype, int64_t rows, int R,
                 double *G) {
    hipStream_t s = ctx->stream;
    if (R <= 16 * kMfmaMaxTiles) {
        const GramPlan gp = gram_plan(rows, R, F, dtype);
        const int nt = gp.nt, nblk = gp.nblk;
        const bool vec2 = gp.vec;
        double *part = (double *)ws_get(ctx, gram_slot(ctx),
                                        sizeof(double) * 256 * (size_t)R * R);
#define GM(T, NTV, V)                                                                              \
    hipLaunchKernelGGL((k_gram_mfma<T, NTV, (NTV <= 2 ? 1024 : 256), V>), dim3(nblk),              \
                       dim3(NTV <= 2 ? 1024 : 256), 0, s, (const T *)F, rows, R, part)
        if (dtype == DFACTO_F32) {
            if (nt == 1) GM(float, 1, false);
            else if (nt == 2 && vec2) GM(float, 2, true);
            else if (nt == 2) GM(float, 2, false);
            else if (nt == 3) GM(float, 3, false);
            else GM(float, 4, false);
        } else {
            if (nt == 1) GM(uint16_t, 1, false);
            else if (nt == 2 && vec2) GM(uint16_t, 2, true);
            else if (nt == 2) GM(uint16_t, 2, false);
            else if (nt == 3) GM(uint16_t, 3, false);
            else GM(uint16_t, 4, false);
        }
#undef GM
        hipLaunchKernelGGL(k_gram_reduce, dim3((R * R + 15) / 16), dim3(kBlock), 0, s, part, nblk, R,
                           G);
        DF_LAUNCHED();
        return;
    }
    const int nt = (R + 15) / 16, npair = nt * (nt + 1) / 2;
    // at least four 16-row steps per block
    const int nblk = (int)std::max<int64_t>(1, std::min<int64_t>((rows + 63) / 64, 256));
    // sized for the largest block count so that the buffer never moves between calls
    double *part = (double *)ws_get(ctx, gram_slot(ctx), sizeof(double) * 256 * (size_t)R * R);
    const dim3 grid(nblk, (npair + kWidePairs - 1) / kWidePairs);
#define GRAM_LAUNCH(T)                                                                          \
    if (nt <= 8)                                                                                \
        hipLaunchKernelGGL((k_gram_wide<T, 8>), grid, dim3(kBlock), 0, s, (const T *)F, rows, R, \
                           part);                                                               \
    else                                                                                        \
        hipLaunchKernelGGL((k_gram_wide<T, 16>), grid, dim3(kBlock), 0, s, (const T *)F, rows, R, \
                           part)
    if (dtype == DFACTO_F32) {
        GRAM_LAUNCH(float);
    } else {
        GRAM_LAUNCH(uint16_t);
    }
#undef GRAM_LAUNCH
    hipLaunchKernelGGL(k_gram_reduce, dim3((R * R + 15) / 16), dim3(kBlock), 0, s, part, nblk, R, G);
    DF_LAUNCHED();
}

void launch_hadamard(dfacto_ctx *ctx, int R, const double *Gp, const double *Gq, double reg,
                     double *H) {
    hipLaunchKernelGGL(k_hadamard, dim3((R * R + kBlock - 1) / kBlock), dim3(kBlock), 0, ctx->stream,
                       R, Gp, Gq, reg, H);
    DF_LAUNCHED();
}

void launch_solve(dfacto_ctx *ctx, int R, const double *Gp, const double *Gq, double reg,
                  double *Hinv, double *scratch, int *flag) {
    if (R <= 32)
        hipLaunchKernelGGL((k_solve<kBlock, true>), dim3(1), dim3(kBlock),
                           sizeof(double) * 3 * R * R, ctx->stream, R, Gp, Gq, reg, Hinv, scratch,
                           flag);
    else
        hipLaunchKernelGGL((k_solve<kSolveWide, false>), dim3(1), dim3(kSolveWide), 0, ctx->stream,
                           R, Gp, Gq, reg, Hinv, scratch, flag);
    DF_LAUNCHED();
}

void launch_als_lambda(dfacto_ctx *ctx, int R, int mode, const double *Hinv, const double *MtM,
                       double *Gn, double *W, double *lambda_out, const double *GA,
                       const double *GB, double normsq, double *fit_out, double *scratch) {
    if (R <= kLambdaSmemMaxR)
        hipLaunchKernelGGL(k_als_lambda, dim3(1), dim3(kBlock), sizeof(double) * (4 * R * R + R),
                           ctx->stream, R, mode, Hinv, MtM, Gn, W, lambda_out, GA, GB, normsq,
                           fit_out);
    else {
        double *T1 = scratch, *S = scratch + (size_t)R * R;
        const unsigned nt = (unsigned)(R + kMulTile - 1) / kMulTile;
        hipLaunchKernelGGL(k_matmul, dim3(nt, nt), dim3(kBlock), 0, ctx->stream, R, MtM, Hinv, T1);
        hipLaunchKernelGGL(k_matmul, dim3(nt, nt), dim3(kBlock), 0, ctx->stream, R, Hinv, T1, S);
        hipLaunchKernelGGL(k_lambda_finish, dim3(1), dim3(kBlock), 0, ctx->stream, R, mode, Hinv,
                           MtM, S, Gn, W, lambda_out, GA, GB, normsq, fit_out);
    }
    DF_LAUNCHED();
}

static unsigned rows_grid_generic(int64_t rows, int R, int per_pass_elems) {
    const int rpp = std::max(1, per_pass_elems / R);
    const int64_t npass = (rows + rpp - 1) / rpp;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(npass, 8192));
}

static unsigned rows_grid_tiles(int64_t rows, int R) {
    const int64_t nt = (rows + tile_rows(R) - 1) / tile_rows(R);
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(nt, 2048));
}

template <typename Tout, int RC>
void rowmap_tiled(hipStream_t s, const float *M, int64_t rows, const double *W, void *F) {
    hipLaunchKernelGGL((k_rowmap_t<Tout, RC>), dim3(rows_grid_tiles(rows, RC)), dim3(kBlock),
                       tile_lds_bytes(RC), s, M, rows, W, (Tout *)F);
}

template <typename T, int RC>
void gd_rows_tiled(hipStream_t s, float *G, const void *F, int64_t rows, const double *H,
                   double *partial) {
    hipLaunchKernelGGL((k_gd_rows_t<T, RC>), dim3(rows_grid_tiles(rows, RC)), dim3(kBlock),
                       tile_lds_bytes(RC), s, G, (const T *)F, rows, H, partial);
}

// Dispatch a tiled row kernel on the compile-time rank; false if R has none.
template <template <typename, int> class K, typename T, typename... A>
bool dispatch_tiled(int R, A... args) {
    switch (R) {
        case 4: K<T, 4>::run(args...); return true;
        case 8: K<T, 8>::run(args...); return true;
        case 12: K<T, 12>::run(args...); return true;
        case 16: K<T, 16>::run(args...); return true;
        case 32: K<T, 32>::run(args...); return true;
        case 48: K<T, 48>::run(args...); return true;
        default: return false;
    }
}
template <typename T, int RC>
struct RowmapK {
    static void run(hipStream_t s, const float *M, int64_t rows, const double *W, void *F) {
        rowmap_tiled<T, RC>(s, M, rows, W, F);
    }
};
template <typename T, int RC>
struct GdRowsK {
    static void run(hipStream_t s, float *G, const void *F, int64_t rows, const double *H,
                    double *partial) {
        gd_rows_tiled<T, RC>(s, G, F, rows, H, partial);
    }
};

void launch_rowmap(dfacto_ctx *ctx, const float *M, int64_t rows, int R, const double *W, void *F,
                   dfacto_dtype dtype) {
    if (rows <= 0) return;
    hipStream_t s = ctx->stream;
    const size_t ef = dtype == DFACTO_F32 ? 4 : 2;
    if (mfma_rows_ok(R, M, 4, F, ef)) {
        if (dtype == DFACTO_F32) rowmap_mfma<float>(s, M, rows, R, W, F);
        else rowmap_mfma<uint16_t>(s, M, rows, R, W, F);
        DF_LAUNCHED();
        return;
    }
    const bool done = dtype == DFACTO_F32
                          ? dispatch_tiled<RowmapK, float>(R, s, M, rows, W, F)
                          : dispatch_tiled<RowmapK, uint16_t>(R, s, M, rows, W, F);
    if (!done && R <= kRowAnyMaxR) {
        with_tiles(R, [&](auto nc) {
            constexpr int NCT = decltype(nc)::value;
            const dim3 g(rows_grid_any(rows, R)), b(kBlock);
            if (dtype == DFACTO_F32)
                hipLaunchKernelGGL((k_rowmap_any<float, NCT>), g, b, 0, s, M, rows, R, W,
                                   (float *)F);
            else
                hipLaunchKernelGGL((k_rowmap_any<uint16_t, NCT>), g, b, 0, s, M, rows, R, W,
                                   (uint16_t *)F);
        });
    } else if (!done) {
        const unsigned g = rows_grid_generic(rows, R, kBlock * 4);
        if (dtype == DFACTO_F32)
            hipLaunchKernelGGL(k_rowmap_g<float>, dim3(g), dim3(kBlock), 0, s, M, rows, R, W,
                               (float *)F);
        else
            hipLaunchKernelGGL(k_rowmap_g<uint16_t>, dim3(g), dim3(kBlock), 0, s, M, rows, R, W,
                               (uint16_t *)F);
    }
    DF_LAUNCHED();
}

int gd_rows_partials(int64_t rows, int R, const float *G, const void *F, dfacto_dtype dtype) {
    if (mfma_rows_ok(R, G, 4, F, dtype == DFACTO_F32 ? 4 : 2)) return (int)rows_grid_mfma(rows);
    return (int)(tiled_rows_ok(R)     ? rows_grid_tiles(rows, R)
                 : R <= kRowAnyMaxR ? rows_grid_any(rows, R)
                                      : rows_grid_generic(rows, R, kBlock * 2));
}

void launch_gd_rows(dfacto_ctx *ctx, float *G, const void *F, dfacto_dtype dtype, int64_t rows,
                    int R, const double *H, double *inner_partial) {
    if (rows <= 0) return;
    hipStream_t s = ctx->stream;
    if (mfma_rows_ok(R, G, 4, F, dtype == DFACTO_F32 ? 4 : 2)) {
        if (dtype == DFACTO_F32) gd_rows_mfma<float>(s, G, F, rows, R, H, inner_partial);
        else gd_rows_mfma<uint16_t>(s, G, F, rows, R, H, inner_partial);
        DF_LAUNCHED();
        return;
    }
    const bool done = dtype == DFACTO_F32
                          ? dispatch_tiled<GdRowsK, float>(R, s, G, F, rows, H, inner_partial)
                          : dispatch_tiled<GdRowsK, uint16_t>(R, s, G, F, rows, H, inner_partial);
    if (!done && R <= kRowAnyMaxR) {
        with_tiles(R, [&](auto nc) {
            constexpr int NCT = decltype(nc)::value;
            const dim3 g(rows_grid_any(rows, R)), b(kBlock);
            if (dtype == DFACTO_F32)
                hipLaunchKernelGGL((k_gd_rows_any<float, NCT>), g, b, 0, s, G, (const float *)F,
                                   rows, R, H, inner_partial);
            else
                hipLaunchKernelGGL((k_gd_rows_any<uint16_t, NCT>), g, b, 0, s, G,
                                   (const uint16_t *)F, rows, R, H, inner_partial);
        });
    } else if (!done) {
        const unsigned g = (unsigned)gd_rows_partials(rows, R, G, F, dtype);
        if (dtype == DFACTO_F32)
            hipLaunchKernelGGL(k_gd_rows_g<float>, dim3(g), dim3(kBlock), 0, s, G,
                               (const float *)F, rows, R, H, inner_partial);
        else
            hipLaunchKernelGGL(k_gd_rows_g<uint16_t>, dim3(g), dim3(kBlock), 0, s, G,
                               (const uint16_t *)F, rows, R, H, inner_partial);
    }
    DF_LAUNCHED();
}

void launch_gd_f(dfacto_ctx *ctx, int R, const double *GA, const double *GB, const double *GC,
                 const double *inner_partial, int npartial, double normsq, double reg,
                 double *f_out) {
    hipLaunchKernelGGL(k_gd_f, dim3(1), dim3(kBlock), 0, ctx->stream, R, GA, GB, GC, inner_partial,
                       npartial, normsq, reg, f_out);
    DF_LAUNCHED();
}

unsigned stream_grid(int64_t n) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + kBlock - 1) / kBlock, 4096));
}

void launch_trial_factors(dfacto_ctx *ctx, void *const F[3], float *const G[3], double alpha,
                          void *const out[3], dfacto_dtype dtype, const int64_t n[3]) {
    const dim3 grid(stream_grid(std::max({n[0], n[1], n[2]})), 3);
    auto go = [&](auto *tag, auto kernel) {
        using T = std::remove_pointer_t<decltype(tag)>;
        TrialJobs3<T> j;
        for (int m = 0; m < 3; ++m) {
            j.F[m] = (const T *)F[m];
            j.G[m] = G[m];
            j.out[m] = (T *)out[m];
            j.n[m] = n[m];
        }
        hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, ctx->stream, j, alpha);
    };
    if (dtype == DFACTO_F32) go((float *)nullptr, k_trial_factors<float>);
    else go((uint16_t *)nullptr, k_trial_factors<uint16_t>);
    DF_LAUNCHED();
}

size_t trial_gram_doubles(int64_t rows, int R) {
    if (R > 16 * kMfmaMaxTiles) return 0;  // one Gram at a time, in launch_gram's own buffer
    return (size_t)gram_plan(rows, R, nullptr, DFACTO_F32).nblk * R * R;
}

void launch_trial_grams(dfacto_ctx *ctx, void *const F[3], dfacto_dtype dtype,
                        const int64_t rows[3], int R, double *const G[3], double reg, double *H,
                        double *const part[3]) {
    if (R > 16 * kMfmaMaxTiles) {
        for (int m = 0; m < 3; ++m) launch_gram(ctx, F[m], dtype, rows[m], R, G[m]);
        launch_hadamard(ctx, R, G[1], G[2], reg, H);
        return;
    }
    GramJobs3 jobs;
    unsigned nblk = 1;
    bool vec = true;
    int nt = 1;
    for (int m = 0; m < 3; ++m) {
        const GramPlan gp = gram_plan(rows[m], R, F[m], dtype);
        jobs.j[m] = GramJob{F[m], rows[m], R, (uint32_t)gp.nblk, part[m], G[m]};
        nblk = std::max(nblk, (unsigned)gp.nblk);
        vec = vec && gp.vec;
        nt = gp.nt;
    }
#define GM3(T, NTV, V)                                                                      \
    hipLaunchKernelGGL((k_gram_mfma3<T, NTV, (NTV <= 2 ? 1024 : 256), V>), dim3(nblk, 3),   \
                       dim3(NTV <= 2 ? 1024 : 256), 0, ctx->stream, jobs)
    if (dtype == DFACTO_F32) {
        if (nt == 1) GM3(float, 1, false);
        else if (nt == 2 && vec) GM3(float, 2, true);
        else if (nt == 2) GM3(float, 2, false);
        else if (nt == 3) GM3(float, 3, false);
        else GM3(float, 4, false);
    } else {
        if (nt == 1) GM3(uint16_t, 1, false);
        else if (nt == 2 && vec) GM3(uint16_t, 2, true);
        else if (nt == 2) GM3(uint16_t, 2, false);
        else if (nt == 3) GM3(uint16_t, 3, false);
        else GM3(uint16_t, 4, false);
    }
#undef GM3
    hipLaunchKernelGGL(k_gram_reduce3, dim3((R * R + 15) / 16), dim3(kBlock), 0, ctx->stream, jobs,
                       reg, H);
    DF_LAUNCHED();
}

void launch_sumsq3(dfacto_ctx *ctx, const float *const x[3], const int64_t n[3], double *part,
                   double *out) {
    for (int m = 0; m < 3; ++m)
        hipLaunchKernelGGL(k_sumsq_f32, dim3(kSumsqBlocks), dim3(kBlock), 0, ctx->stream, x[m],
                           n[m], part + m * kSumsqBlocks);
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(kBlock), 0, ctx->stream, part,
                       3 * kSumsqBlocks, out);
    DF_LAUNCHED();
}

// workgroups of `block` threads of `kernel` that one CU holds at once (>= 1)
template <typename K>
int resident_blocks(K kernel, int block) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, block, 0) != hipSuccess || n < 1)
        n = 1;
    return n;
}

size_t joint_part_doubles(int R, int64_t nseg) {
    return (size_t)nseg * 16 * (R <= 16 ? JointSys<4>::kAll : JointSys<8>::kAll);
}

namespace {
template <typename T, int NB, bool VEC>
void joint_rows_t(dfacto_ctx *ctx, const dfacto_tensor *Y, int m, int64_t nrows, const T *F, int R,
                  const float *M, const double *H, double mu, double lam, const double *Pinv,
                  double ws, const int *pflag, T *out, int *flag, int *need, double *part) {
    hipStream_t s = ctx->stream;
    // (an empty stream is never used, only read)
    const uint2 *st = Y->mode[m].nentry > 0 ? Y->mode[m].stream : (const uint2 *)flag;
    const bool by_mid = m == 1;
    // persistent: the grid is what the device holds at once, so no
    // workgroup waits for a second round
    static const int occ = resident_blocks(k_joint_rows<T, NB, VEC>, 64);
    const unsigned grid = (unsigned)std::min<int64_t>((nrows + 3) / 4,
                                                      (int64_t)std::max(1, ctx->num_cu) * occ);
    hipLaunchKernelGGL((k_joint_rows<T, NB, VEC>), dim3(grid), dim3(64), 0, s, st, Y->row_range[m], nrows,
                       F, by_mid, R, M, H, mu, lam, out, flag, need);
    hipLaunchKernelGGL(k_joint_small<T>, dim3(grid), dim3(64), 0, s, st, Y->row_range[m], nrows, F,
                       by_mid, R, M, mu, Pinv, ws, pflag, out, flag, need);
    const auto &cut = Y->batch[m];
    for (size_t q = 0; q + 1 < cut.size(); ++q) {
        const auto [row0, seg0] = cut[q];
        const int64_t rows = cut[q + 1].first - row0, segs = cut[q + 1].second - seg0;
        hipLaunchKernelGGL((k_joint_segments<T, NB, VEC>), dim3((unsigned)segs), dim3(256), 0, s,
                           st, Y->seg_range[m] + seg0, segs, F, by_mid, R, part);
        hipLaunchKernelGGL((k_joint_heavy<T, NB>), dim3((unsigned)((rows + 3) / 4)), dim3(64), 0,
                           s, Y->heavy[m] + row0, rows, seg0, R, VEC, part, M, H, mu, lam, out,
                           flag);
    }
    DF_LAUNCHED();
}
}  // namespace

void launch_joint_rows(dfacto_ctx *ctx, const dfacto_tensor *Y, int m, int64_t nrows,
                       const void *F, int R, const float *M, const double *H, double mu, double lam,
                       const double *Pinv, double ws, const int *pflag, void *out,
                       dfacto_dtype dtype, int *flag, int *need, double *part) {
    if (nrows <= 0) return;
    // rows of whole 4-element runs (R % 4 == 0) on their alignment are loaded
    // and stored a run at a time, others by element
    const size_t al = 4 * elem_size(dtype) - 1;
    const bool vec = R % 4 == 0 && (((uintptr_t)F | (uintptr_t)out) & al) == 0;
#define DF_JOINT_V(T, NB, V)                                                                   \
    joint_rows_t<T, NB, V>(ctx, Y, m, nrows, (const T *)F, R, M, H, mu, lam, Pinv, ws, pflag,  \
                           (T *)out, flag, need, part)
#define DF_JOINT(T, NB)                        \
    {                                          \
        if (vec) DF_JOINT_V(T, NB, true);      \
        else DF_JOINT_V(T, NB, false);         \
    }
    if (dtype == DFACTO_F32) {
        if (R <= 16) DF_JOINT(float, 4)
        else DF_JOINT(float, 8)
    } else {
        if (R <= 16) DF_JOINT(uint16_t, 4)
        else DF_JOINT(uint16_t, 8)
    }
#undef DF_JOINT_V
#undef DF_JOINT
}

void launch_joint_combine(dfacto_ctx *ctx, float *G, const void *F, const float *RY, double mu,
                          double lam, int64_t n, dfacto_dtype dtype) {
    if (n <= 0) return;
    if (dtype == DFACTO_F32)
        hipLaunchKernelGGL(k_joint_combine<float>, dim3(stream_grid(n)), dim3(kBlock), 0,
                           ctx->stream, G, (const float *)F, RY, mu, lam, n);
    else
        hipLaunchKernelGGL(k_joint_combine<uint16_t>, dim3(stream_grid(n)), dim3(kBlock), 0,
                           ctx->stream, G, (const uint16_t *)F, RY, mu, lam, n);
    DF_LAUNCHED();
}

uint32_t fit_blocks(int64_t rows, int R) {
    const int64_t n = rows * (int64_t)R;
    return (uint32_t)std::min<int64_t>(64, std::max<int64_t>(1, (n + 16383) / 16384));
}

void launch_fit_stored(dfacto_ctx *ctx, const void *F, dfacto_dtype dtype, const float *M,
                       int64_t rows, int R, const double *lambda, const double *GA,
                       const double *GB, const double *GC, double normsq, double *part,
                       double *fit) {
    const uint32_t nb = fit_blocks(rows, R);
    if (dtype == DFACTO_F32)
        hipLaunchKernelGGL(k_wdot<float>, dim3(nb), dim3(kBlock), 0, ctx->stream,
                           (const float *)F, M, rows, R, lambda, part);
    else
        hipLaunchKernelGGL(k_wdot<uint16_t>, dim3(nb), dim3(kBlock), 0, ctx->stream,
                           (const uint16_t *)F, M, rows, R, lambda, part);
    hipLaunchKernelGGL(k_fit_finish, dim3(1), dim3(kBlock), 0, ctx->stream, R, lambda, GA, GB, GC,
                       part, nb, normsq, fit);
    DF_LAUNCHED();
}

void launch_fit_group(dfacto_ctx *ctx, dfacto_dtype dtype, const FitJob *d_jobs, uint32_t n,
                      const uint2 *d_items, uint32_t nitems) {
    if (nitems > 0) {
        if (dtype == DFACTO_F32)
            hipLaunchKernelGGL(k_wdot_group<float>, dim3(nitems), dim3(kBlock), 0, ctx->stream,
                               d_jobs, d_items);
        else
            hipLaunchKernelGGL(k_wdot_group<uint16_t>, dim3(nitems), dim3(kBlock), 0,
                               ctx->stream, d_jobs, d_items);
    }
    hipLaunchKernelGGL(k_fit_finish_group, dim3(n), dim3(kBlock), 0, ctx->stream, d_jobs);
    DF_LAUNCHED();
}

void launch_dot_parts(dfacto_ctx *ctx, const void *F, const float *X, int64_t n, double *part,
                      dfacto_dtype dtype) {
    if (dtype == DFACTO_F32)
        hipLaunchKernelGGL(k_dot_parts<float>, dim3(kSumsqBlocks), dim3(kBlock), 0, ctx->stream,
                           (const float *)F, X, n, part);
    else
        hipLaunchKernelGGL(k_dot_parts<uint16_t>, dim3(kSumsqBlocks), dim3(kBlock), 0,
                           ctx->stream, (const uint16_t *)F, X, n, part);
    DF_LAUNCHED();
}

void launch_joint_f(dfacto_ctx *ctx, const double *ft, const double *GA, const double *GB,
                    const double *GC, int R, const double *part, int npart, double normsq_y,
                    double mu, double lam, double *f) {
    hipLaunchKernelGGL(k_joint_f, dim3(1), dim3(kBlock), 0, ctx->stream, ft, GA, GB, GC, R, part,
                       npart, normsq_y, mu, lam, f);
    DF_LAUNCHED();
}

// ---- grouped launches (many tensors, one launch per kernel class) ---------
void launch_gram_group(dfacto_ctx *ctx, dfacto_dtype dtype, int nt, bool vec,
                       const GramJob *d_jobs, const uint2 *d_vb, uint32_t nvb) {
    if (nvb == 0) return;
    hipStream_t s = ctx->stream;
#define GMG(T, NTV, V)                                                                         \
    hipLaunchKernelGGL((k_gram_mfma_group<T, NTV, (NTV <= 2 ? 1024 : 256), V>), dim3(nvb),     \
                       dim3(NTV <= 2 ? 1024 : 256), 0, s, d_jobs, d_vb)
    if (dtype == DFACTO_F32) {
        if (nt == 1) GMG(float, 1, false);
        else if (nt == 2 && vec) GMG(float, 2, true);
        else if (nt == 2) GMG(float, 2, false);
        else if (nt == 3) GMG(float, 3, false);
        else GMG(float, 4, false);
    } else {
        if (nt == 1) GMG(uint16_t, 1, false);
        else if (nt == 2 && vec) GMG(uint16_t, 2, true);
        else if (nt == 2) GMG(uint16_t, 2, false);
        else if (nt == 3) GMG(uint16_t, 3, false);
        else GMG(uint16_t, 4, false);
    }
#undef GMG
    DF_LAUNCHED();
}

uint32_t gram_reduce_blocks(int R) { return (uint32_t)((R * R + 15) / 16); }

void launch_gram_reduce_group(dfacto_ctx *ctx, const GramJob *d_jobs, const uint2 *d_vb,
                              uint32_t nvb) {
    if (nvb == 0) return;
    hipLaunchKernelGGL(k_gram_reduce_group, dim3(nvb), dim3(kBlock), 0, ctx->stream, d_jobs, d_vb);
    DF_LAUNCHED();
}

void launch_solve_group(dfacto_ctx *ctx, int maxR, const SolveJob *d_jobs, uint32_t n) {
    if (n == 0) return;
    if (maxR <= 32)
        hipLaunchKernelGGL((k_solve_group<kBlock, true>), dim3(n), dim3(kBlock),
                           sizeof(double) * 3 * maxR * maxR, ctx->stream, d_jobs);
    else
        hipLaunchKernelGGL((k_solve_group<kSolveWide, false>), dim3(n), dim3(kSolveWide), 0,
                           ctx->stream, d_jobs);
    DF_LAUNCHED();
}

void launch_lambda_group(dfacto_ctx *ctx, int maxR, const LambdaJob *d_jobs, uint32_t n) {
    if (n == 0) return;
    if (maxR <= kLambdaSmemMaxR)
        hipLaunchKernelGGL(k_als_lambda_group<true>, dim3(n), dim3(kBlock),
                           sizeof(double) * (4 * maxR * maxR + maxR), ctx->stream, d_jobs);
    else
        hipLaunchKernelGGL(k_als_lambda_group<false>, dim3(n), dim3(kBlock), 0, ctx->stream,
                           d_jobs);
    DF_LAUNCHED();
}

RowmapPlan rowmap_plan(int R, const float *M, const void *F, dfacto_dtype dtype, int64_t rows) {
    RowmapPlan p;
    if (mfma_rows_ok(R, M, 4, F, dtype == DFACTO_F32 ? 4 : 2)) {
        p.kind = RowmapPlan::kMfma;
        p.nblk = rows_grid_mfma(rows);
    } else if (tiled_rows_ok(R)) {
        p.kind = RowmapPlan::kTiled;
        p.nblk = rows_grid_tiles(rows, R);
    } else {
        p.kind = RowmapPlan::kGeneric;
        p.nblk = 0;
    }
    return p;
}

void launch_rowmap_group(dfacto_ctx *ctx, dfacto_dtype dtype, int kind, int R,
                         const RowmapJob *d_jobs, const uint2 *d_vb, uint32_t nvb) {
    if (nvb == 0) return;
    hipStream_t s = ctx->stream;
    const dim3 grid(nvb), block(kBlock);
    auto mfma = [&](auto tag) {
        using Tout = decltype(tag);
        switch (R) {
            case 16: hipLaunchKernelGGL((k_rowmap_mfma_group<Tout, 1>), grid, block, 0, s, d_jobs, d_vb); break;
            case 32: hipLaunchKernelGGL((k_rowmap_mfma_group<Tout, 2>), grid, block, 0, s, d_jobs, d_vb); break;
            case 48: hipLaunchKernelGGL((k_rowmap_mfma_group<Tout, 3>), grid, block, 0, s, d_jobs, d_vb); break;
            case 64: hipLaunchKernelGGL((k_rowmap_mfma_group<Tout, 4>), grid, block, 0, s, d_jobs, d_vb); break;
            default: throw Error{DFACTO_E_UNSUPPORTED, "no grouped row map for this rank"};
        }
    };
    auto tiled = [&](auto tag) {
        using Tout = decltype(tag);
        const size_t lds = tile_lds_bytes(R);
        switch (R) {
            case 4: hipLaunchKernelGGL((k_rowmap_t_group<Tout, 4>), grid, block, lds, s, d_jobs, d_vb); break;
            case 8: hipLaunchKernelGGL((k_rowmap_t_group<Tout, 8>), grid, block, lds, s, d_jobs, d_vb); break;
            case 12: hipLaunchKernelGGL((k_rowmap_t_group<Tout, 12>), grid, block, lds, s, d_jobs, d_vb); break;
            case 16: hipLaunchKernelGGL((k_rowmap_t_group<Tout, 16>), grid, block, lds, s, d_jobs, d_vb); break;
            case 32: hipLaunchKernelGGL((k_rowmap_t_group<Tout, 32>), grid, block, lds, s, d_jobs, d_vb); break;
            case 48: hipLaunchKernelGGL((k_rowmap_t_group<Tout, 48>), grid, block, lds, s, d_jobs, d_vb); break;
            default: throw Error{DFACTO_E_UNSUPPORTED, "no grouped row map for this rank"};
        }
    };
    if (kind == RowmapPlan::kMfma) {
        if (dtype == DFACTO_F32) mfma(float{});
        else mfma(uint16_t{});
    } else if (kind == RowmapPlan::kTiled) {
        if (dtype == DFACTO_F32) tiled(float{});
        else tiled(uint16_t{});
    } else {
        throw Error{DFACTO_E_UNSUPPORTED, "no grouped row map for this rank"};
    }
    DF_LAUNCHED();
}

}  // namespace dfacto
