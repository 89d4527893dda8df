// mttkrp.hip -- fused DFacTo MTTKRP for gfx950 (Section 3, Algorithm 1,
// all R rank columns at once).
//
// For output mode n with coordinate roles (root, mid, leaf), DFacTo computes
//   stage 1: value(M^r) <- (Xhat)^T f_leaf_r        (one value per fiber)
//   stage 2: n_r        <- M^r f_mid_r              (one value per root)
// (Lemma 2: column r of X1 (C kr B) is [unvec((X2)^T b_r)]^T c_r; Lemmas 3
// and 4: only nonempty fibers matter and their pattern is fixed).  Here both
// products run in one pass over the mode's stream for all R columns: a group
// of G lanes owns the rank columns (CPL consecutive columns per lane, so a
// factor-row gather is one coalesced 4*CPL-byte load per lane) and walks one
// work chunk of the stream.  The fiber partial P (the paper's value(M^r),
// materialized only in registers) accumulates val * F_leaf[leaf, :]; at the
// next header it is folded into the root accumulator as P * F_mid[mid, :];
// at a new root the accumulator is written out.
//
// Work chunks always start at a header and are balanced in entries, so a
// heavy root is spread over many groups.  A root that begins before the
// chunk (no ROOT bit on the chunk's first header) is written to a per-chunk
// carry slot; the fix-up kernels add the carries of each such root to the
// owner's row in a fixed order.  No floating-point atomics: results are
// deterministic.  The fix-up launches also zero-fill the empty output rows.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "internal.hpp"

namespace dfacto {
namespace {

// Tuning knobs (compile-time; the defaults are the measured best).
#ifndef DFACTO_UNROLL
#define DFACTO_UNROLL 8
#endif
#ifndef DFACTO_MAX_CPL
#define DFACTO_MAX_CPL 8
#endif
#ifndef DFACTO_NT_STREAM
#define DFACTO_NT_STREAM 0
#endif
// At least 5 waves per SIMD: the gathers are latency-bound, and the FP32
// CPL = 4 kernel sits right at the 96-register limit for 5 waves.  Whole-wave
// groups (G = 64) keep the compiler's choice (they would spill).
#ifndef DFACTO_WAVES_PER_EU
#define DFACTO_WAVES_PER_EU 5
#endif
// Eight columns per lane hold twice the gathered data per batch: 4 waves
// per SIMD (128 registers) keep them out of scratch.
#define MTTKRP_OCCUPANCY                                                               \
    __attribute__((amdgpu_waves_per_eu(G <= 32 ? (CPL >= 8 ? 4 : DFACTO_WAVES_PER_EU) : 1)))

constexpr int kBlock = 256;
constexpr int kUnroll = DFACTO_UNROLL;  // the residual kernel's entries in flight per group
static_assert(kStreamPad >= kUnroll && kStreamPad >= 32, "stream padding must cover a batch");

// f(integral_constant<int, I>) for I = B .. E-1, so I is usable as a constant
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

__device__ __forceinline__ uint2 load_entry(const uint2 *p) {
#if DFACTO_NT_STREAM
    const unsigned long long x =
        __builtin_nontemporal_load(reinterpret_cast<const unsigned long long *>(p));
    return make_uint2((uint32_t)x, (uint32_t)(x >> 32));
#else
    return *p;
#endif
}

__device__ __forceinline__ uint2 load_entry(const DF_GLOBAL uint2 *p) {
#if DFACTO_NT_STREAM
    const unsigned long long x =
        __builtin_nontemporal_load(reinterpret_cast<const DF_GLOBAL unsigned long long *>(p));
    return make_uint2((uint32_t)x, (uint32_t)(x >> 32));
#else
    const df_u2 x = *reinterpret_cast<const DF_GLOBAL df_u2 *>(p);
    return make_uint2(x.x, x.y);
#endif
}

// ---- factor-row loads: CPL consecutive columns, widened to FP32 ----------
template <typename T, int CPL>
struct RowLoad;

template <>
struct RowLoad<float, 4> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[4]) {
        const float4 x = *reinterpret_cast<const float4 *>(p);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    }
    static __device__ __forceinline__ void load(const DF_GLOBAL float *p, float (&v)[4]) {
        const df_f4 x = *reinterpret_cast<const DF_GLOBAL df_f4 *>(p);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    }
};
template <>
struct RowLoad<float, 2> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[2]) {
        const float2 x = *reinterpret_cast<const float2 *>(p);
        v[0] = x.x; v[1] = x.y;
    }
    static __device__ __forceinline__ void load(const DF_GLOBAL float *p, float (&v)[2]) {
        const df_f2 x = *reinterpret_cast<const DF_GLOBAL df_f2 *>(p);
        v[0] = x.x; v[1] = x.y;
    }
};
template <>
struct RowLoad<float, 1> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[1]) { v[0] = *p; }
    static __device__ __forceinline__ void load(const DF_GLOBAL float *p, float (&v)[1]) { v[0] = *p; }
};

template <>
struct RowLoad<float, 8> {
    static __device__ __forceinline__ void load(const float *p, float (&v)[8]) {
        const float4 x = *reinterpret_cast<const float4 *>(p);
        const float4 y = *reinterpret_cast<const float4 *>(p + 4);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
    }
    static __device__ __forceinline__ void load(const DF_GLOBAL float *p, float (&v)[8]) {
        const df_f4 x = *reinterpret_cast<const DF_GLOBAL df_f4 *>(p);
        const df_f4 y = *reinterpret_cast<const DF_GLOBAL df_f4 *>(p + 4);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
    }
};

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

template <>
struct RowLoad<uint16_t, 8> {
    static __device__ __forceinline__ void load(const uint16_t *p, float (&v)[8]) {
        const uint4 x = *reinterpret_cast<const uint4 *>(p);
        v[0] = bf16_lo(x.x); v[1] = bf16_hi(x.x); v[2] = bf16_lo(x.y); v[3] = bf16_hi(x.y);
        v[4] = bf16_lo(x.z); v[5] = bf16_hi(x.z); v[6] = bf16_lo(x.w); v[7] = bf16_hi(x.w);
    }
    static __device__ __forceinline__ void load(const DF_GLOBAL uint16_t *p, float (&v)[8]) {
        const df_u4 x = *reinterpret_cast<const DF_GLOBAL df_u4 *>(p);
        v[0] = bf16_lo(x.x); v[1] = bf16_hi(x.x); v[2] = bf16_lo(x.y); v[3] = bf16_hi(x.y);
        v[4] = bf16_lo(x.z); v[5] = bf16_hi(x.z); v[6] = bf16_lo(x.w); v[7] = bf16_hi(x.w);
    }
};
template <>
struct RowLoad<uint16_t, 4> {
    static __device__ __forceinline__ void load(const uint16_t *p, float (&v)[4]) {
        const uint2 x = *reinterpret_cast<const uint2 *>(p);
        v[0] = bf16_lo(x.x); v[1] = bf16_hi(x.x); v[2] = bf16_lo(x.y); v[3] = bf16_hi(x.y);
    }
    static __device__ __forceinline__ void load(const DF_GLOBAL uint16_t *p, float (&v)[4]) {
        const df_u2 x = *reinterpret_cast<const DF_GLOBAL df_u2 *>(p);
        v[0] = bf16_lo(x.x); v[1] = bf16_hi(x.x); v[2] = bf16_lo(x.y); v[3] = bf16_hi(x.y);
    }
};
template <>
struct RowLoad<uint16_t, 2> {
    static __device__ __forceinline__ void load(const uint16_t *p, float (&v)[2]) {
        const uint32_t x = *reinterpret_cast<const uint32_t *>(p);
        v[0] = bf16_lo(x); v[1] = bf16_hi(x);
    }
    static __device__ __forceinline__ void load(const DF_GLOBAL uint16_t *p, float (&v)[2]) {
        const uint32_t x = *reinterpret_cast<const DF_GLOBAL uint32_t *>(p);
        v[0] = bf16_lo(x); v[1] = bf16_hi(x);
    }
};
template <>
struct RowLoad<uint16_t, 1> {
    static __device__ __forceinline__ void load(const uint16_t *p, float (&v)[1]) {
        v[0] = __uint_as_float((uint32_t)(*p) << 16);
    }
    static __device__ __forceinline__ void load(const DF_GLOBAL uint16_t *p, float (&v)[1]) {
        v[0] = __uint_as_float((uint32_t)(*p) << 16);
    }
};

template <int CPL>
__device__ __forceinline__ void store_vec(float *p, const float (&v)[CPL]) {
    if constexpr (CPL == 8) {
        *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4 *>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
    } else if constexpr (CPL == 4) {
        *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
    } else if constexpr (CPL == 2) {
        *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
    } else {
        p[0] = v[0];
    }
}

template <int CPL>
__device__ __forceinline__ void store_vec(DF_GLOBAL float *p, const float (&v)[CPL]) {
    if constexpr (CPL == 8) {
        *reinterpret_cast<DF_GLOBAL df_f4 *>(p) = df_f4{v[0], v[1], v[2], v[3]};
        *reinterpret_cast<DF_GLOBAL df_f4 *>(p + 4) = df_f4{v[4], v[5], v[6], v[7]};
    } else if constexpr (CPL == 4) {
        *reinterpret_cast<DF_GLOBAL df_f4 *>(p) = df_f4{v[0], v[1], v[2], v[3]};
    } else if constexpr (CPL == 2) {
        *reinterpret_cast<DF_GLOBAL df_f2 *>(p) = df_f2{v[0], v[1]};
    } else {
        p[0] = v[0];
    }
}

// CPL consecutive floats of LDS
template <int CPL>
__device__ __forceinline__ void store_lds(float *p, const float (&v)[CPL]) {
    if constexpr (CPL == 2) *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
    else p[0] = v[0];
}
template <int CPL>
__device__ __forceinline__ void load_lds(const float *p, float (&v)[CPL]) {
    if constexpr (CPL == 2) {
        const float2 x = *reinterpret_cast<const float2 *>(p);
        v[0] = x.x; v[1] = x.y;
    } else {
        v[0] = p[0];
    }
}

template <int CPL>
__device__ __forceinline__ void load_f32(const DF_GLOBAL float *p, float (&v)[CPL]) {
    RowLoad<float, CPL>::load(p, v);
}

template <int CPL>
__device__ __forceinline__ void load_f32(const float *p, float (&v)[CPL]) {
    RowLoad<float, CPL>::load(p, v);
}

// ---- factor-row sources ------------------------------------------------------
// load(w, c, v): the row that stream entry w gathers -- the leaf row for a
// nonzero, the mid row for a header -- columns of block c (CPL per lane),
// widened to FP32.  Lanes whose columns lie beyond R read column 0 instead
// (in bounds, never stored), so every gather is issued without a branch and
// the loads of a batch stay in flight together.
// SMALL: every row index is below 2^24, so row offsets are one 24-bit
// multiply (idx * R < 2^32) instead of 64-bit arithmetic.

// Rows straight from the two factor tables in device memory.
template <typename T, int CPL, int NCH, bool SMALL>
struct GlobalRows {
    const DF_GLOBAL T *leafb[NCH], *midb[NCH];
    int R;
    __device__ __forceinline__ GlobalRows(const T *Fleaf, const T *Fmid, int R_, int G, int lane)
        : R(R_) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int col = (c * G + lane) * CPL;
            leafb[c] = gptr(Fleaf) + (col < R ? col : 0);
            midb[c] = gptr(Fmid) + (col < R ? col : 0);
        }
    }
    __device__ __forceinline__ size_t off(uint32_t idx) const {
        if constexpr (SMALL) return (size_t)(uint32_t)__umul24(idx, (uint32_t)R);
        else return (size_t)idx * (size_t)R;
    }
    __device__ __forceinline__ void load(const uint2 &w, int c, float (&v)[CPL]) const {
        const bool hdr = (int32_t)w.x < 0;  // kHdrBit is the sign bit
        RowLoad<T, CPL>::load((hdr ? midb[c] : leafb[c]) + off(w.x & kIdxMask), v);
    }
};

// CPL elements of T at byte offset `off` of a buffer resource; an offset
// past the buffer's end loads zeros and makes no memory request.
template <typename T, int CPL>
struct BufLoad;
template <>
struct BufLoad<float, 4> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                float (&v)[4]) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        v[0] = __uint_as_float(x[0]); v[1] = __uint_as_float(x[1]);
        v[2] = __uint_as_float(x[2]); v[3] = __uint_as_float(x[3]);
    }
};
template <>
struct BufLoad<float, 2> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                float (&v)[2]) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        v[0] = __uint_as_float(x[0]); v[1] = __uint_as_float(x[1]);
    }
};
template <>
struct BufLoad<float, 1> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                float (&v)[1]) {
        v[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    }
};
template <>
struct BufLoad<float, 8> {  // two 16-byte loads
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                float (&v)[8]) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        const auto y = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16u, 0, 0);
        v[0] = __uint_as_float(x[0]); v[1] = __uint_as_float(x[1]);
        v[2] = __uint_as_float(x[2]); v[3] = __uint_as_float(x[3]);
        v[4] = __uint_as_float(y[0]); v[5] = __uint_as_float(y[1]);
        v[6] = __uint_as_float(y[2]); v[7] = __uint_as_float(y[3]);
    }
};
template <>
struct BufLoad<uint16_t, 8> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                float (&v)[8]) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        v[0] = bf16_lo(x[0]); v[1] = bf16_hi(x[0]); v[2] = bf16_lo(x[1]); v[3] = bf16_hi(x[1]);
        v[4] = bf16_lo(x[2]); v[5] = bf16_hi(x[2]); v[6] = bf16_lo(x[3]); v[7] = bf16_hi(x[3]);
    }
};
template <>
struct BufLoad<uint16_t, 4> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                float (&v)[4]) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        v[0] = bf16_lo(x[0]); v[1] = bf16_hi(x[0]); v[2] = bf16_lo(x[1]); v[3] = bf16_hi(x[1]);
    }
};
template <>
struct BufLoad<uint16_t, 2> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                float (&v)[2]) {
        const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
        v[0] = bf16_lo(x); v[1] = bf16_hi(x);
    }
};
template <>
struct BufLoad<uint16_t, 1> {
    static __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                                float (&v)[1]) {
        v[0] = __uint_as_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0) << 16);
    }
};

// ---- residual kernel -------------------------------------------------------
// The joint model's ratings term: the MTTKRP with each nonzero's value x
// replaced by x - xhat, xhat = sum_r F_root[root, r] F_mid[mid, r]
// F_leaf[leaf, r] (the CP model at that entry), so the output is the MTTKRP
// of the residual restricted to the stored entries.  One work chunk (gid) per
// lane group of G lanes (lane = 0 .. G-1), its factor rows from `src`; the dot
// product is reduced across the group's lanes by xor shuffles (every lane
// ends with the same sum: each step adds two commuted operands).
template <typename T, int CPL, int G, int NCH, bool SMALL, class Src>
__device__ __forceinline__ void mttkrp_res_chunk(const uint2 *__restrict__ st_,
                                                 const uint32_t *__restrict__ cstart,
                                                 uint32_t nchunk, const Src &src, int R,
                                                 float *__restrict__ out_,
                                                 float *__restrict__ carry_, uint32_t gid,
                                                 int lane, const T *__restrict__ Froot) {
    if (gid >= nchunk) return;
    const uint32_t cs = gptr(cstart)[gid], ce = gptr(cstart)[gid + 1];
    if (cs >= ce) return;
    const DF_GLOBAL uint2 *__restrict__ st = gptr(st_);
    DF_GLOBAL float *__restrict__ out = gptr(out_);
    DF_GLOBAL float *__restrict__ carry = gptr(carry_);

    int col[NCH];
    bool act[NCH];
    const DF_GLOBAL T *rootb[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        col[c] = (c * G + lane) * CPL;
        act[c] = col[c] < R;
        rootb[c] = gptr(Froot) + (act[c] ? col[c] : 0);
    }
    auto row_off = [&](uint32_t idx) -> size_t {
        if constexpr (SMALL) return (size_t)(uint32_t)__umul24(idx, (uint32_t)R);
        else return (size_t)idx * (size_t)R;
    };
    float acc[NCH][CPL], p[NCH][CPL], mrow[NCH][CPL];
    float rrow[NCH][CPL];  // the root's factor row
    const uint2 h0 = load_entry(st + cs);
    uint32_t row = h0.y;
    bool cont = !(h0.x & kRootBit);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[c][q] = p[c][q] = 0.f;
        src.load(h0, c, mrow[c]);  // h0 is a header: its mid row
        RowLoad<T, CPL>::load(rootb[c] + row_off(row), rrow[c]);
    }

    auto flush = [&](uint32_t r_out, bool is_cont) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (!act[c]) continue;
            DF_GLOBAL float *dst =
                is_cont ? carry + (size_t)gid * R + col[c] : out + row_off(r_out) + col[c];
            store_vec<CPL>(dst, acc[c]);
        }
    };

    // Gathers of one batch: every entry's factor row, without branches.
    // Entries at or past the chunk end are still valid stream entries (the
    // next chunk's, or the padding sentinels with index 0), so these loads
    // are in bounds; their values are ignored.
    auto gather = [&](const uint2 (&w)[kUnroll], float (&g)[kUnroll][NCH][CPL]) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
#pragma unroll
            for (int c = 0; c < NCH; ++c) src.load(w[u], c, g[u][c]);
    };
    // One stream entry, without data-dependent branches except the (rarer)
    // write of a finished output row.  A header closes the fiber segment --
    // stage 2 of Algorithm 1, acc += P * F_mid[mid] -- and opens the next
    // one (P = 0, new mid row); a nonzero accumulates stage 1, P += x *
    // F_leaf[leaf].
    auto step = [&](const uint2 &w, const float (&g)[NCH][CPL]) {
        const bool hdr = (int32_t)w.x < 0;
        float part = 0.f;
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int q = 0; q < CPL; ++q)
                part = fmaf(act[c] ? rrow[c][q] * mrow[c][q] : 0.f, g[c][q], part);
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) part += __shfl_xor(part, o, G);
        const float v = hdr ? 0.f : __uint_as_float(w.y) - part;
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
                const float a2 = fmaf(p[c][q], mrow[c][q], acc[c][q]);
                acc[c][q] = hdr ? a2 : acc[c][q];
                p[c][q] = fmaf(v, g[c][q], hdr ? 0.f : p[c][q]);
                mrow[c][q] = hdr ? g[c][q] : mrow[c][q];
            }
        if (hdr && (w.x & kRootBit)) {
            flush(row, cont);
#pragma unroll
            for (int c = 0; c < NCH; ++c)
#pragma unroll
                for (int q = 0; q < CPL; ++q) acc[c][q] = 0.f;
            cont = false;
            row = w.y;
#pragma unroll
            for (int c = 0; c < NCH; ++c) RowLoad<T, CPL>::load(rootb[c] + row_off(row), rrow[c]);
        }
    };

    // Stream entries of a batch.  With groups of at most 32 lanes, lane l
    // loads only entries l, l + G, ... of the batch (8 bytes each) and the
    // group shares them through ds_swizzle (the LDS crossbar), so the vector
    // memory path carries each entry once instead of once per lane.  A
    // 64-lane group is the whole wave and loads the batch directly.
    constexpr bool kShare = G <= 32;
    constexpr int KL = kShare ? (kUnroll + G - 1) / G : kUnroll;  // entries held per lane
    auto load_batch = [&](uint32_t at, uint2 (&wl)[KL]) {
#pragma unroll
        for (int k = 0; k < KL; ++k)
            wl[k] = kShare ? load_entry(st + at + lane + G * k) : load_entry(st + at + k);
    };
    auto expand = [&](const uint2 (&wl)[KL], uint2 (&w)[kUnroll]) {
        static_for<0, kUnroll>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            if constexpr (kShare) {
                // bit-mask swizzle: source lane = (lane & ~(G-1)) | (u % G), within 32 lanes
                constexpr int pat = (0x1F & ~(G - 1)) | ((u % G) << 5);
                w[u].x = (uint32_t)__builtin_amdgcn_ds_swizzle((int)wl[u / G].x, pat);
                w[u].y = (uint32_t)__builtin_amdgcn_ds_swizzle((int)wl[u / G].y, pat);
            } else {
                w[u] = wl[u];
            }
        });
    };

    // Full batches.  The next batch's entries are requested right after the
    // current batch's gathers, so their latency overlaps the gathers.  The
    // stream padding (>= 64 entries) keeps the look-ahead in bounds.
    uint32_t e = cs + 1;
    uint2 wn[KL];
    load_batch(e, wn);
    for (; e + kUnroll <= ce; e += kUnroll) {
        uint2 w[kUnroll];
        expand(wn, w);
        float g[kUnroll][NCH][CPL];
        gather(w, g);
        load_batch(e + kUnroll, wn);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) step(w[u], g[u]);
    }
    // Last, partial batch (fewer than kUnroll entries left).
    if (e < ce) {
        uint2 w[kUnroll];
        expand(wn, w);
        float g[kUnroll][NCH][CPL];
        gather(w, g);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            if (e + u < ce) step(w[u], g[u]);
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[c][q] = fmaf(p[c][q], mrow[c][q], acc[c][q]);
    flush(row, cont);
}

// ---- main kernel: lane groups with execution masks -------------------------
// One work chunk per group of G lanes, CPL columns per lane (NCH blocks of
// them for a whole wave, G = 64).  A wave's groups meet headers and nonzeros at
// different entries, so selecting per lane what each entry does cost 22 of the
// 45 vector instructions per entry.  Here what an entry does is kept as
// execution masks: one ballot per batch tells which lanes' entries are
// headers, and for each entry the scalar unit spreads its bit over every
// group's lanes; a masked FMA then costs one vector instruction per column
// and nothing where it does not apply (about 20 per entry in all).  The lane
// that loads an entry also forms its row's address, once for its group.
// What bounds it at scale: the misses of its gathers.  Its loads alone (the
// gather probe's pattern 0) take 91 to 100% of its time, and two rates limit
// them: lines from beyond L2 (uniformly drawn rows of the same tables get 53 to
// 56 G/s, 6.8 to 7.2 TB/s of 128-byte lines) and L1 misses (rows that all lie
// in L2: 142 to 150 G/s).  By the counters, R = 32: 50M nonzeros 47.8 G/s (FP32)
// and 50.5 (BF16) from beyond L2, 91 and 93% of that limit, and 104 and 105 G/s
// L1 misses, 70 and 74%; 100M relabeled 43.3 and 40.8 (80 and 72%), 111 and 108
// (74 and 75%).  R = 8 to 32 take nearly the same time: a row is one line.
// Three modes, before and after: 50M, R = 32 FP32 2140 -> 2060 us, BF16 2046 ->
// 1905, R = 8 2181 -> 1799; 100M relabeled, R = 32 BF16 3244 -> 2948, R = 10
// FP32 3108 -> 3043, R = 100 BF16 11018 -> 8250.
//
// p += v * g in the lanes of `m` (V: the constraint of v, "v" or "s")
#define DF_MASKED_ADD(V)                                                                       \
    if constexpr (CPL == 1) {                                                                  \
        asm("s_mov_b64 exec, %[m]\n\t"                                                         \
            "v_fmac_f32 %[p0], %[v], %[g0]\n\t"                                                \
            "s_mov_b64 exec, -1"                                                               \
            : [p0] "+v"(p[0])                                                                  \
            : [m] "s"(m), [v] V(v), [g0] "v"(g[0]));                                           \
    } else if constexpr (CPL == 2) {                                                           \
        asm("s_mov_b64 exec, %[m]\n\t"                                                         \
            "v_fmac_f32 %[p0], %[v], %[g0]\n\t"                                                \
            "v_fmac_f32 %[p1], %[v], %[g1]\n\t"                                                \
            "s_mov_b64 exec, -1"                                                               \
            : [p0] "+v"(p[0]), [p1] "+v"(p[1])                                                 \
            : [m] "s"(m), [v] V(v), [g0] "v"(g[0]), [g1] "v"(g[1]));                           \
    } else {                                                                                   \
        for (int q = 0; q < CPL; q += 4)                                                       \
            asm("s_mov_b64 exec, %[m]\n\t"                                                     \
                "v_fmac_f32 %[p0], %[v], %[g0]\n\t"                                            \
                "v_fmac_f32 %[p1], %[v], %[g1]\n\t"                                            \
                "v_fmac_f32 %[p2], %[v], %[g2]\n\t"                                            \
                "v_fmac_f32 %[p3], %[v], %[g3]\n\t"                                            \
                "s_mov_b64 exec, -1"                                                           \
                : [p0] "+v"(p[q]), [p1] "+v"(p[q + 1]), [p2] "+v"(p[q + 2]),                   \
                  [p3] "+v"(p[q + 3])                                                          \
                : [m] "s"(m), [v] V(v), [g0] "v"(g[q]), [g1] "v"(g[q + 1]),                    \
                  [g2] "v"(g[q + 2]), [g3] "v"(g[q + 3]));                                     \
    }
template <int CPL>
__device__ __forceinline__ void masked_add(uint64_t m, float v, const float (&g)[CPL],
                                           float (&p)[CPL]) {
    DF_MASKED_ADD("v")
}
template <int CPL>  // v uniform
__device__ __forceinline__ void masked_add_s(uint64_t m, uint32_t v, const float (&g)[CPL],
                                             float (&p)[CPL]) {
    DF_MASKED_ADD("s")
}
#undef DF_MASKED_ADD

// acc += p * mrow, p = 0 * g + 0, mrow = g in the lanes of `m`
template <int CPL>
__device__ __forceinline__ void masked_close(uint64_t m, const float (&g)[CPL], float (&p)[CPL],
                                             float (&acc)[CPL], float (&mrow)[CPL]) {
    if constexpr (CPL == 1) {
        asm("s_mov_b64 exec, %[m]\n\t"
            "v_fmac_f32 %[a0], %[p0], %[r0]\n\t"
            "v_fma_f32 %[p0], 0, %[g0], 0\n\t"
            "v_mov_b32 %[r0], %[g0]\n\t"
            "s_mov_b64 exec, -1"
            : [a0] "+v"(acc[0]), [p0] "+v"(p[0]), [r0] "+v"(mrow[0])
            : [m] "s"(m), [g0] "v"(g[0]));
    } else {
        for (int q = 0; q < CPL; q += 2)
            asm("s_mov_b64 exec, %[m]\n\t"
                "v_fmac_f32 %[a0], %[p0], %[r0]\n\t"
                "v_fmac_f32 %[a1], %[p1], %[r1]\n\t"
                "v_fma_f32 %[p0], 0, %[g0], 0\n\t"
                "v_fma_f32 %[p1], 0, %[g1], 0\n\t"
                "v_mov_b32 %[r0], %[g0]\n\t"
                "v_mov_b32 %[r1], %[g1]\n\t"
                "s_mov_b64 exec, -1"
                : [a0] "+v"(acc[q]), [a1] "+v"(acc[q + 1]), [p0] "+v"(p[q]), [p1] "+v"(p[q + 1]),
                  [r0] "+v"(mrow[q]), [r1] "+v"(mrow[q + 1])
                : [m] "s"(m), [g0] "v"(g[q]), [g1] "v"(g[q + 1]));
    }
}

// the bits of `b` (one per G-lane group, at the group's first lane) spread
// over the lanes of their groups
template <int G>
__device__ __forceinline__ uint64_t spread_groups(uint64_t b) {
    if constexpr (G == 64) {
        return (b & 1) ? ~0ull : 0ull;
    } else {
        constexpr uint32_t k = G == 32 ? 0xFFFFFFFFu : (1u << (G & 31)) - 1u;
        return ((uint64_t)((uint32_t)(b >> 32) * k) << 32) | (uint32_t)((uint32_t)b * k);
    }
}

// Entries per batch: as many rows in flight as the registers allow.  FP32 rows
// at four columns per lane keep two batches of eight (one batch is gathered
// while the other is added up: R = 32, 50M nonzeros 2112 -> 2058 us; 16 in one
// batch spill, 3170); narrower ones one batch of 16 (R = 16: 1885 us against
// 1965 at 8, 2008 at 24, and 3028 with two batches).  BF16 rows at four columns
// over two or four lanes, which only a tuned group tries, hold more entries a
// lane and take eight.
template <typename T, int CPL, int G, int NCH>
constexpr int batch_entries() {
    if (G == 64) return CPL * NCH == 1 ? 32 : (CPL * NCH == 2 ? 16 : 8);
    return CPL <= 2 || (CPL == 4 && sizeof(T) == 2 && G >= 8) ? 16 : 8;
}

// No probe: the product itself.  A probe (below) walks the same chunk with the
// same requests for stream entries and rows, only adds up what it loads, and
// may replace the address that an entry gathers from.
struct NoProbe {
    static constexpr int kPat = -1;
};

// TWO: FP32 rows at four columns per lane in two batches (else in one)
template <typename T, int CPL, int G, int NCH, bool TWO, class Probe = NoProbe>
__device__ __forceinline__ void mttkrp_group_chunk(const uint2 *__restrict__ st_,
                                                   const uint32_t *__restrict__ cstart,
                                                   uint32_t nchunk, const T *__restrict__ Fleaf,
                                                   const T *__restrict__ Fmid, int R,
                                                   float *__restrict__ out_,
                                                   float *__restrict__ carry_, uint32_t gid,
                                                   int lane, const Probe &probe = Probe{}) {
    constexpr int PAT = Probe::kPat;
    constexpr bool WAVE = G == 64;
    constexpr int U = batch_entries<T, CPL, G, NCH>();
    constexpr int KL = (U + G - 1) / G;  // entries held per lane
    constexpr uint64_t kFirst = G == 2    ? 0x5555555555555555ull
                                : G == 4  ? 0x1111111111111111ull
                                : G == 8  ? 0x0101010101010101ull
                                : G == 16 ? 0x0001000100010001ull
                                : G == 32 ? 0x0000000100000001ull
                                          : 1ull;
    const DF_GLOBAL uint2 *__restrict__ st = gptr(st_);
    DF_GLOBAL float *__restrict__ out = gptr(out_);
    DF_GLOBAL float *__restrict__ carry = gptr(carry_);
    // every lane of the wave stays active: a group without a chunk walks an
    // empty one
    if constexpr (WAVE) gid = __builtin_amdgcn_readfirstlane(gid);
    const uint32_t gc = gid < nchunk ? gid : nchunk - 1;
    uint32_t cs = gptr(cstart)[gc], ce = gptr(cstart)[gc + 1];
    if constexpr (WAVE) {
        cs = __builtin_amdgcn_readfirstlane(cs);
        ce = __builtin_amdgcn_readfirstlane(ce);
    }
    const bool live = gid < nchunk && cs < ce;
    const uint32_t last = live ? ce : cs;  // == cs: nothing to do
    // lanes past the last column repeat the group's first lane's
    int col[NCH];
    uint32_t colb[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        col[c] = (c * G + lane) * CPL;
        if (col[c] >= R) col[c] = 0;
        colb[c] = (uint32_t)col[c] * (uint32_t)sizeof(T);
    }
    const uint32_t rowb = (uint32_t)R * (uint32_t)sizeof(T);
    uint32_t nmax = live ? ce - cs - 1 : 0u, nmin = nmax;
    if constexpr (!WAVE) {
#pragma unroll
        for (int o = G; o < 64; o <<= 1) {
            nmax = max(nmax, (uint32_t)__shfl_xor((int)nmax, o));
            nmin = min(nmin, (uint32_t)__shfl_xor((int)nmin, o));
        }
        nmax = __builtin_amdgcn_readfirstlane(nmax);
        nmin = __builtin_amdgcn_readfirstlane(nmin);
    }

    auto fetch = [&](uint32_t at, uint2 (&wl)[KL]) {
#pragma unroll
        for (int k = 0; k < KL; ++k) {
            const uint32_t e = at + (uint32_t)lane + G * k;
            wl[k] = load_entry(st + (e < last ? e : last));
        }
    };
    float acc[NCH][CPL], p[NCH][CPL], mrow[NCH][CPL];
    const uint2 h0 = load_entry(st + cs);
    DF_GLOBAL float *dst[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[c][q] = p[c][q] = 0.f;
        if constexpr (PAT > 0) continue;
        RowLoad<T, CPL>::load(
            (const DF_GLOBAL T *)((const DF_GLOBAL char *)gptr(Fmid) + colb[c] +
                                  (uint64_t)(live ? h0.x & kIdxMask : 0u) * rowb),
            mrow[c]);
        if constexpr (PAT < 0)
            dst[c] = ((h0.x & kRootBit) ? out + (size_t)h0.y * R : carry + (size_t)gc * R) + col[c];
    }

    struct Batch {
        uint64_t hdr[KL], nz[KL], root[KL];
        uint32_t y[KL];
        float g[U][NCH][CPL];
    };
    auto bcast = [&](uint32_t x, auto uc) -> uint32_t {
        constexpr int u = decltype(uc)::value;
        if constexpr (WAVE) {
            return (uint32_t)__builtin_amdgcn_readlane((int)x, u);
        } else {
            // bit-mask swizzle: source lane = (lane & ~(G-1)) | (u % G), within 32 lanes
            constexpr int pat = (0x1F & ~(G - 1)) | ((u % G) << 5);
            return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, pat);
        }
    };
    auto issue = [&](Batch &b, uint32_t at, const uint2 (&wl)[KL]) {
        uint32_t lo[KL], hi[KL];
#pragma unroll
        for (int k = 0; k < KL; ++k) {
            const bool v = at + (uint32_t)lane + G * k < last;
            const bool h = (int32_t)wl[k].x < 0;
            uint64_t a;
            if constexpr (PAT <= 0)
                a = (uint64_t)(uintptr_t)(h ? Fmid : Fleaf) + (uint64_t)(wl[k].x & kIdxMask) * rowb;
            else
                a = probe.place(wl[k].x, at + (uint32_t)lane + G * k, (uint64_t)(uintptr_t)Fleaf,
                                (uint64_t)(uintptr_t)Fmid, rowb);
            lo[k] = (uint32_t)a;
            hi[k] = (uint32_t)(a >> 32);
            b.hdr[k] = __ballot(v && h);
            b.nz[k] = __ballot(v && !h);
            b.root[k] = __ballot(v && h && (wl[k].x & kRootBit));
            b.y[k] = wl[k].y;
        }
        static_for<0, U>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            if constexpr (PAT == 3) {  // nothing gathered: the entries alone
                const float y = __uint_as_float(bcast(b.y[u / G], uc) & 0x3F7FFFFFu);
#pragma unroll
                for (int q = 0; q < CPL; ++q) b.g[u][0][q] = y;
            } else {
                const uint32_t l = bcast(lo[u / G], uc), h = bcast(hi[u / G], uc);
                if constexpr (PAT >= 5) {
                    probe.load(l, h, colb[0], b.g[u][0]);
                } else {
                    const DF_GLOBAL char *a =
                        (const DF_GLOBAL char *)(uintptr_t)(((uint64_t)h << 32) | l);
#pragma unroll
                    for (int c = 0; c < NCH; ++c)
                        RowLoad<T, CPL>::load((const DF_GLOBAL T *)(a + colb[c]), b.g[u][c]);
                }
            }
        });
    };
    auto add = [&](const Batch &b, auto fullc) {
        static_for<0, U>([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            constexpr int k = u / G, sh = u % G;
            constexpr bool full = decltype(fullc)::value;
            if constexpr (PAT >= 0) {
                const bool have = full || __builtin_amdgcn_inverse_ballot_w64(spread_groups<G>(
                                              ((b.nz[k] | b.hdr[k]) >> sh) & kFirst));
#pragma unroll
                for (int q = 0; q < CPL; ++q) acc[0][q] += have ? b.g[u][0][q] : 0.f;
                return;
            }
            const uint32_t y = bcast(b.y[k], uc);
            const uint64_t hm = spread_groups<G>((b.hdr[k] >> sh) & kFirst);
            const uint64_t nm = full ? ~hm : spread_groups<G>((b.nz[k] >> sh) & kFirst);
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                if constexpr (WAVE) masked_add_s<CPL>(nm, y, b.g[u][c], p[c]);
                else masked_add<CPL>(nm, __uint_as_float(y), b.g[u][c], p[c]);
                masked_close<CPL>(hm, b.g[u][c], p[c], acc[c], mrow[c]);
            }
            const uint64_t rb = (b.root[k] >> sh) & kFirst;
            if (rb) {
                if (WAVE || __builtin_amdgcn_inverse_ballot_w64(spread_groups<G>(rb))) {
#pragma unroll
                    for (int c = 0; c < NCH; ++c) {
                        store_vec<CPL>(dst[c], acc[c]);
#pragma unroll
                        for (int q = 0; q < CPL; ++q) acc[c][q] = 0.f;
                        dst[c] = out + (size_t)y * R + col[c];
                    }
                }
            }
        });
    };
    uint2 wn[KL];
    fetch(cs + 1, wn);
    if constexpr (WAVE || (TWO && CPL == 4 && sizeof(T) == 4)) {
        // Each batch's entries are requested before the rows of the batch
        // ahead of it, so that waiting for them leaves those rows in flight.
        if (nmax > 0) {
            uint2 wm[KL];
            Batch a, b;
            fetch(cs + 1 + U, wm);
            issue(a, cs + 1, wn);
            for (uint32_t i = 0; i < nmax; i += 2 * U) {
                fetch(cs + 1 + i + 2 * U, wn);
                issue(b, cs + 1 + i + U, wm);
                add(a, std::false_type{});
                fetch(cs + 1 + i + 3 * U, wm);
                issue(a, cs + 1 + i + 2 * U, wn);
                add(b, std::false_type{});
            }
        }
    } else {
        uint32_t i = 0;
        for (; i + U <= nmin; i += U) {
            Batch b;
            issue(b, cs + 1 + i, wn);
            fetch(cs + 1 + i + U, wn);
            add(b, std::true_type{});
        }
        for (; i < nmax; i += U) {
            Batch b;
            issue(b, cs + 1 + i, wn);
            fetch(cs + 1 + i + U, wn);
            add(b, std::false_type{});
        }
    }
    if constexpr (PAT >= 0) {  // a sum per lane (of the first mid row too), so nothing is elided
        float sum = 0.f;
#pragma unroll
        for (int q = 0; q < CPL; ++q) sum += PAT == 0 ? acc[0][q] + mrow[0][q] : acc[0][q];
        if (gid < nchunk) out[(size_t)gid * G + lane] = sum;
        return;
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[c][q] = fmaf(p[c][q], mrow[c][q], acc[c][q]);
        if (live) store_vec<CPL>(dst[c], acc[c]);
    }
}

template <typename T, int CPL, int G, int NCH>
__global__ __launch_bounds__(kBlock) MTTKRP_OCCUPANCY void k_mttkrp(
    const uint2 *__restrict__ st, const uint32_t *__restrict__ cstart, uint32_t nchunk,
    const T *__restrict__ Fleaf, const T *__restrict__ Fmid, int R, float *__restrict__ out,
    float *__restrict__ carry) {
    mttkrp_group_chunk<T, CPL, G, NCH, true>(st, cstart, nchunk, Fleaf, Fmid, R, out, carry,
                                             (blockIdx.x * (uint32_t)kBlock + threadIdx.x) / G,
                                             threadIdx.x % G);
}

// ---- one block per chunk ---------------------------------------------------
// For tensors with too few chunks to fill the device with lane groups: a
// lane group walks its chunk's 512 entries one batch after another, so a call
// on a small tensor lasts as long as that walk's memory round trips (65 us),
// however little there is to do.  Here a block takes one chunk and W = CPL * G
// columns; Algorithm 1's two stages run one after the other, each spread over
// the block's lane groups:
//   stage 1: a group forms the P of the fibers whose headers lie in its share
//     of the entries, all their leaf rows in flight at once, and leaves P and
//     the mid row in LDS;
//   stage 2: a group adds P * mid row over the fibers of whole output rows.
// Every fiber's and every row's sum runs in stream order, so the result is
// bitwise that of mttkrp_group_chunk.  What bounds it is the chain of round
// trips of a block (about a third each of the time in front of the stages, in
// stage 1 and in stage 2) times the rounds of blocks, so blocks are kept small:
// LDS for the R columns there are (R = 10: 32 KB, five blocks a CU, not 47 KB
// and three), and stage 1 takes ten entries at once by selects (59 registers;
// sixteen with branches 100).  1M nonzeros, R = 10, a mode: 53 -> 43 us; either
// change alone 51.
constexpr int kBlkEntries = 640;  // a chunk of chunk_len <= 512: one more segment at most
constexpr int kBlkFibers = kBlkEntries / 2;
static_assert(kBlkEntries >= DFACTO_CHUNK_DEFAULT + kFiberCap, "a chunk fits the block's LDS");

template <typename T, int CPL, int G>
__global__ __launch_bounds__(kBlock, 5) void k_mttkrp_block(
    const uint2 *__restrict__ st_, const uint32_t *__restrict__ cstart,
    const T *__restrict__ Fleaf, const T *__restrict__ Fmid, int R, float *__restrict__ out_,
    float *__restrict__ carry_, int ld) {
    constexpr int W = CPL * G, NG = kBlock / G, U = 10;
    constexpr int kWords = kBlkEntries / 64, kFWords = kBlkFibers / 64;
    __shared__ uint2 ent[kBlkEntries];
    extern __shared__ float Ps[];  // P, then the mid rows: ld floats a segment
    float *Ms = Ps + kBlkFibers * ld;
    __shared__ uint32_t frow[kBlkFibers];               // the row of each segment's header
    __shared__ uint64_t hmask[kWords], rmask[kFWords];  // headers; segments that open a row
    __shared__ int before[kWords + 1];                  // headers before each word of hmask
    const DF_GLOBAL uint2 *__restrict__ st = gptr(st_);
    const uint32_t gid = blockIdx.x, cs = gptr(cstart)[gid];
    const int L = (int)min(gptr(cstart)[gid + 1] - cs, (uint32_t)kBlkEntries);
    if (L <= 0) return;
    const int tid = threadIdx.x, g = tid / G, lane = tid % G;

    if (tid < kFWords) rmask[tid] = 0;
    for (int i = tid; i < kBlkEntries; i += kBlock) {
        const uint2 w = i < L ? load_entry(st + cs + i) : make_uint2(0u, 0u);
        ent[i] = w;
        const uint64_t m = __ballot((int32_t)w.x < 0);
        if (tid % 64 == 0) hmask[i / 64] = m;
    }
    __syncthreads();
    if (tid <= kWords) {
        int n = 0;
#pragma unroll
        for (int w = 0; w < kWords; ++w) n += w < tid ? __popcll(hmask[w]) : 0;
        before[tid] = n;
    }
    // the first header from entry b on (L: none), and the headers before b
    auto next_head = [&](int b) {
        int w = b >> 6;
        if (b >= L) return L;
        uint64_t m = hmask[w] & (~0ull << (b & 63));
        while (!m && ++w < kWords) m = hmask[w];
        return m ? 64 * w + __ffsll((unsigned long long)m) - 1 : L;
    };
    auto heads_before = [&](int b) {
        return b >= L ? before[kWords]
                      : before[b >> 6] + __popcll(hmask[b >> 6] & ~(~0ull << (b & 63)));
    };
    const int share = (L + NG - 1) / NG;
    const int beg = next_head(g * share), end = next_head((g + 1) * share);
    __syncthreads();
    const int nf = before[kWords], f0 = heads_before(g * share);
    for (int i = tid; i < L; i += kBlock) {
        const uint2 w = ent[i];
        if ((int32_t)w.x >= 0) continue;
        const int f = heads_before(i);
        frow[f] = w.y;
        if (w.x & kRootBit) atomicOr((uint32_t *)rmask + (f >> 5), 1u << (f & 31));
    }

    // stage 1
    const int c0 = blockIdx.y * W + lane * CPL;
    const uint32_t colb = (uint32_t)(c0 < R ? c0 : blockIdx.y * W) * (uint32_t)sizeof(T);
    const uint32_t rowb = (uint32_t)R * (uint32_t)sizeof(T);
    const uint64_t leaf0 = (uint64_t)(uintptr_t)Fleaf + colb, mid0 = (uint64_t)(uintptr_t)Fmid + colb;
    {
        const bool mine = lane * CPL < ld;
        int pos = (f0 - 1) * ld + lane * CPL;
        float p[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) p[q] = 0.f;
        for (int at = beg; at < end; at += U) {
            uint2 w[U];
            float r[U][CPL];
#pragma unroll
            for (int u = 0; u < U; ++u) w[u] = ent[min(at + u, end - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u)
                RowLoad<T, CPL>::load(
                    (const DF_GLOBAL T *)(uintptr_t)(((int32_t)w[u].x < 0 ? mid0 : leaf0) +
                                                     (uint64_t)(w[u].x & kIdxMask) * rowb),
                    r[u]);
            // Headers and nonzeros by selects: a wave's groups stand at both.
            // A header stores its mid row, a nonzero the P up to it (its
            // fiber's last one stays).  A header leaves P = 0, or NaN for an
            // Inf or NaN in the mid row, as the lane groups have it for all
            // but a chunk's first segment.
            static_for<0, U>([&](auto uc) {
                constexpr int u = decltype(uc)::value;
                const bool h = (int32_t)w[u].x < 0;
                const float y = h ? 0.f : __uint_as_float(w[u].y);
                float v[CPL];
#pragma unroll
                for (int q = 0; q < CPL; ++q) {
                    p[q] = fmaf(y, r[u][q], h ? 0.f : p[q]);
                    if (u == 0 && at == 0) p[q] = 0.f;
                    v[q] = h ? r[u][q] : p[q];
                }
                pos += h ? ld : 0;
                if (at + u < end && mine) store_lds<CPL>(Ps + pos + (h ? kBlkFibers * ld : 0), v);
            });
        }
    }
    __syncthreads();

    // stage 2: the rows that open in the group's share of the segments (and,
    // group 0, the row that the chunk begins in)
    auto next_row = [&](int f) {  // the first segment from f on that opens a row
        if (f >= nf) return nf;
        int w = f >> 6;
        uint64_t m = rmask[w] & (~0ull << (f & 63));
        while (!m && ++w < kFWords) m = rmask[w];
        return m ? 64 * w + __ffsll((unsigned long long)m) - 1 : nf;
    };
    const int fshare = (nf + NG - 1) / NG;
    const int stop = next_row((g + 1) * fshare);
    DF_GLOBAL float *out = gptr(out_), *carry = gptr(carry_);
    for (int f = g == 0 ? 0 : next_row(g * fshare); f < stop;) {
        const bool opens = (rmask[f >> 6] >> (f & 63)) & 1;
        const uint32_t row = frow[f];
        const int e = next_row(f + 1);
        float acc[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[q] = 0.f;
        const int at = f * ld + min(lane * CPL, ld - CPL);
        const float *ps = Ps + at, *ms = Ms + at;
#pragma unroll 4
        for (; f < e; ++f, ps += ld, ms += ld) {
            float p[CPL], m[CPL];
            load_lds<CPL>(ps, p);
            load_lds<CPL>(ms, m);
#pragma unroll
            for (int q = 0; q < CPL; ++q) acc[q] = fmaf(p[q], m[q], acc[q]);
        }
        if (c0 < R)
            store_vec<CPL>((opens ? out + (size_t)row * R : carry + (size_t)gid * R) + c0, acc);
    }
}

template <typename T, int CPL, int G, int NCH, bool SMALL>
__global__ __launch_bounds__(kBlock) void k_mttkrp_res(
    const uint2 *__restrict__ st, const uint32_t *__restrict__ cstart, uint32_t nchunk,
    const T *__restrict__ Fleaf, const T *__restrict__ Fmid, const T *__restrict__ Froot, int R,
    float *__restrict__ out, float *__restrict__ carry) {
    const int lane = threadIdx.x % G;
    const GlobalRows<T, CPL, NCH, SMALL> src(Fleaf, Fmid, R, G, lane);
    mttkrp_res_chunk<T, CPL, G, NCH, SMALL>(st, cstart, nchunk, src, R, out, carry,
                                            (blockIdx.x * (uint32_t)kBlock + threadIdx.x) / G,
                                            lane, Froot);
}

// Grouped MTTKRP over many tensors of one kernel shape: a persistent grid
// walks the work items (tensor, first chunk of kBlock / G * kper
// consecutive chunks) in a fixed order, item blockIdx.x, blockIdx.x +
// gridDim.x, ...; each lane group takes kper consecutive chunks of its item
// in turn.  Every chunk writes its own rows and carry, so the grid, the
// shape and kper change no result.  One batch in flight for every form: a
// second one does not fit beside the member's fields and the loops (FP32 at
// four columns then spilled 9 to 64 registers; an iteration of eight tensors of
// 2M nonzeros, R = 48 2206 us with it, 2186 without, R = 64 3098 and 3086,
// R = 32 1188 and 1187).
template <typename T, int CPL, int G, int NCH>
__global__ __launch_bounds__(kBlock) MTTKRP_OCCUPANCY void k_mttkrp_group(
    const GroupMttkrp *__restrict__ desc, const uint2 *__restrict__ items, uint32_t nitems,
    uint32_t kper) {
    const int lane = threadIdx.x % G;
    const uint32_t first = (threadIdx.x / G) * kper;
    for (uint32_t it = blockIdx.x; it < nitems; it += gridDim.x) {
        const uint2 w = items[it];
        const GroupMttkrp &d = desc[w.x];
        for (uint32_t q = 0; q < kper; ++q)
            mttkrp_group_chunk<T, CPL, G, NCH, false>(d.stream, d.chunk_start, d.nchunk,
                                                      (const T *)d.Fleaf, (const T *)d.Fmid, d.R,
                                                      d.out, d.carry, w.y + first + q, lane);
    }
}

// ---- gather ceiling --------------------------------------------------------
// The main kernel's memory requests without its arithmetic and its stores of
// rows: mttkrp_group_chunk itself, with the same work chunks, lane groups,
// batches, address sharing and row loads, but every gathered row is only
// summed.  PAT selects the row that an entry gathers:
//   0  the entry's own row (leaf for a nonzero, mid for a header): the
//      MTTKRP's exact sequence of loads;
//   1  a row drawn uniformly from the same table (hash of the position);
//   2  a row among the table's first 4096 (a working set that stays in L2);
//   3  none: the stream is read, nothing is gathered;
//   4  a row among the table's first 32;
//   5  a row of a 128-row table in LDS;
//   6-9 leaf rows (a header's mid index modulo the leaf rows) by buffer loads:
//      6 every offset out of range, 7 the entry's own row, 8 half of the
//      entries (a hash bit) from the LDS table and half own rows, split by a
//      branch, 9 the same half split without a branch (an out-of-range buffer
//      load beside an LDS load).
// Each lane writes its sum to sink[chunk * G + lane].
__device__ __forceinline__ uint32_t probe_hash(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7feb352dU;
    x ^= x >> 15;
    x *= 0x846ca68bU;
    x ^= x >> 16;
    return x;
}

constexpr int kProbeLdsRows = 128, kProbeLdsRowElems = 64;
constexpr uint32_t kProbeOut = 0xFFFFFF00u;  // past the end of every probed table

template <typename T, int CPL, int PAT>
struct GatherProbe {
    static constexpr int kPat = PAT;
    uint32_t nleaf, nmid;
    const T *lds;  // kProbeLdsRows rows of kProbeLdsRowElems (5, 8, 9)
    __amdgpu_buffer_rsrc_t rsrc;  // the leaf table (6 to 9)
    // what the lane that holds entry `x` at stream position `e` shares: an
    // address (1, 2, 4), an LDS offset (5), the leaf row's offset and, above it,
    // the LDS offset with the top bit for the LDS half (8, 9)
    __device__ __forceinline__ uint64_t place(uint32_t x, uint32_t e, uint64_t leaf, uint64_t mid,
                                              uint32_t rowb) const {
        const bool hdr = (int32_t)x < 0;
        const uint32_t h = probe_hash(e);
        constexpr uint32_t ldsb = kProbeLdsRowElems * (uint32_t)sizeof(T);
        if constexpr (PAT == 1 || PAT == 2 || PAT == 4) {
            const uint32_t n = hdr ? nmid : nleaf, lim = PAT == 2 ? 4096u : 32u;
            const uint32_t idx = PAT == 1 ? (uint32_t)(((uint64_t)h * n) >> 32)
                                          : (h & (lim - 1)) % (n < lim ? n : lim);
            return (hdr ? mid : leaf) + (uint64_t)idx * rowb;
        } else if constexpr (PAT == 5) {
            return (h & (kProbeLdsRows - 1)) * ldsb;
        } else if constexpr (PAT >= 7) {
            const uint32_t own = ((x & kIdxMask) % nleaf) * rowb;
            if constexpr (PAT == 7) return own;
            return ((uint64_t)((h >> 25) * ldsb | (h << 31)) << 32) | own;
        } else {
            return 0;
        }
    }
    __device__ __forceinline__ void load(uint32_t lo, uint32_t hi, uint32_t colb,
                                         float (&v)[CPL]) const {
        auto from_lds = [&](uint32_t off, float (&o)[CPL]) {
            RowLoad<T, CPL>::load((const T *)((const char *)lds + off + colb), o);
        };
        if constexpr (PAT == 5) {
            from_lds(lo, v);
        } else if constexpr (PAT == 6) {
            BufLoad<T, CPL>::load(rsrc, kProbeOut, v);
        } else if constexpr (PAT == 7) {
            BufLoad<T, CPL>::load(rsrc, lo + colb, v);
        } else if constexpr (PAT == 8) {
            if (hi >> 31) from_lds(hi & 0x7FFFFFFFu, v);
            else BufLoad<T, CPL>::load(rsrc, lo + colb, v);
        } else {
            float gv[CPL], lv[CPL];
            BufLoad<T, CPL>::load(rsrc, hi >> 31 ? kProbeOut : lo + colb, gv);
            from_lds(hi >> 31 ? hi & 0x7FFFFFFFu : 0u, lv);
#pragma unroll
            for (int q = 0; q < CPL; ++q) v[q] = hi >> 31 ? lv[q] : gv[q];
        }
    }
};

template <typename T, int CPL, int G, int PAT>
__global__ __launch_bounds__(kBlock) MTTKRP_OCCUPANCY void k_gather_probe(
    const uint2 *__restrict__ st, const uint32_t *__restrict__ cstart, uint32_t nchunk,
    const T *__restrict__ Fleaf, const T *__restrict__ Fmid, int R, uint32_t nleaf,
    uint32_t nmid, float *__restrict__ sink) {
    constexpr bool kLds = PAT == 5 || PAT == 8 || PAT == 9;
    __shared__ alignas(16) T lds_rows[kLds ? kProbeLdsRows * kProbeLdsRowElems : 1];
    if constexpr (kLds) {
        const uint64_t have = (uint64_t)nleaf * (uint64_t)R;
        const uint32_t nfill = have < (uint64_t)kProbeLdsRowElems ? (uint32_t)have
                                                                   : (uint32_t)kProbeLdsRowElems;
        for (int x = threadIdx.x; x < kProbeLdsRows * kProbeLdsRowElems; x += kBlock)
            lds_rows[x] = Fleaf[(uint32_t)x % nfill];
        __syncthreads();
    }
    GatherProbe<T, CPL, PAT> probe;
    probe.nleaf = nleaf;
    probe.nmid = nmid;
    probe.lds = lds_rows;
    const uint64_t bytes = (uint64_t)nleaf * R * sizeof(T);
    probe.rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)Fleaf, (short)0, (int)(bytes < kProbeOut ? bytes : kProbeOut), 0x00020000);
    // (8 and 9, two loads an entry, have no registers for a second batch)
    mttkrp_group_chunk<T, CPL, G, 1, (PAT < 8)>(st, cstart, nchunk, Fleaf, Fmid, R, sink, sink,
                                                (blockIdx.x * (uint32_t)kBlock + threadIdx.x) / G,
                                                threadIdx.x % G, probe);
}

// ---- fix-up: carries of split rows, and empty rows ------------------------
// out[row] += carry[c0] + ... + carry[c0 + n - 1], in chunk order (one lane
// group; col/act are the lane's column blocks)
template <int CPL, int NCH>
__device__ __forceinline__ void add_run(const float *__restrict__ carry_, int R,
                                        float *__restrict__ out_, uint32_t row, uint32_t c0,
                                        uint32_t n, const int (&col)[NCH], const bool (&act)[NCH]) {
    const DF_GLOBAL float *__restrict__ carry = gptr(carry_);
    DF_GLOBAL float *__restrict__ out = gptr(out_);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if (!act[c]) continue;
        float acc[CPL];
        load_f32<CPL>(out + (size_t)row * R + col[c], acc);
        for (uint32_t k = 0; k < n; ++k) {
            float v[CPL];
            load_f32<CPL>(carry + (size_t)(c0 + k) * R + col[c], v);
#pragma unroll
            for (int q = 0; q < CPL; ++q) acc[q] += v[q];
        }
        store_vec<CPL>(out + (size_t)row * R + col[c], acc);
    }
}

template <int CPL, int NCH>
__device__ __forceinline__ void zero_row(float *__restrict__ out_, int R, uint32_t row,
                                         const int (&col)[NCH], const bool (&act)[NCH]) {
    DF_GLOBAL float *__restrict__ out = gptr(out_);
    float z[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) z[q] = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
        if (act[c]) store_vec<CPL>(out + (size_t)row * R + col[c], z);
}

// Short runs: one lane group per run adds its <= kShortRun carries in chunk
// order; the groups after the runs zero-fill the empty output rows.
template <int CPL, int G, int NCH>
__device__ __forceinline__ void short_runs(uint32_t gid, const uint32_t *__restrict__ runs,
                                           uint32_t nruns, const float *__restrict__ carry, int R,
                                           float *__restrict__ out,
                                           const uint32_t *__restrict__ empty_rows,
                                           uint32_t nempty, uint32_t nempty_groups) {
    const int lane = threadIdx.x % G;
    int col[NCH];
    bool act[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        col[c] = (c * G + lane) * CPL;
        act[c] = col[c] < R;
    }
    if (gid < nruns) {
        add_run<CPL, NCH>(carry, R, out, runs[3 * gid], runs[3 * gid + 1], runs[3 * gid + 2], col,
                          act);
        return;
    }
    const uint32_t eg = gid - nruns;
    if (eg >= nempty_groups) return;
    for (uint32_t r = eg; r < nempty; r += nempty_groups)
        zero_row<CPL, NCH>(out, R, empty_rows[r], col, act);
}

// Long runs: one workgroup per run; kBlock / G slices each sum a strided
// subset of the carries, then a fixed-order tree over the slices (so the
// result is deterministic) is added to the row.
constexpr int kLongBlock = 1024;

template <int CPL, int G, int NCH>
__device__ __forceinline__ void long_run(const float *__restrict__ carry_, int R,
                                         float *__restrict__ out_, uint32_t row, uint32_t c0,
                                         uint32_t n) {
    const DF_GLOBAL float *__restrict__ carry = gptr(carry_);
    DF_GLOBAL float *__restrict__ out = gptr(out_);
    constexpr int S = kLongBlock / G;
    constexpr int W = CPL * NCH;  // floats per thread
    __shared__ float sh[kLongBlock * W];
    const int slice = threadIdx.x / G, lane = threadIdx.x % G;
    float acc[NCH][CPL];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
        for (int q = 0; q < CPL; ++q) acc[c][q] = 0.f;
        const int col = (c * G + lane) * CPL;
        if (col >= R) continue;
        // eight loads in flight, then the adds in the same order as one at
        // a time (k, k + S, k + 2S, ...): the sum is bitwise the same
        uint32_t k = slice;
        for (; k + 7u * S < n; k += 8u * S) {
            float v[8][CPL];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                load_f32<CPL>(carry + (size_t)(c0 + k + u * S) * R + col, v[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int q = 0; q < CPL; ++q) acc[c][q] += v[u][q];
        }
        for (; k < n; k += S) {
            float v[CPL];
            load_f32<CPL>(carry + (size_t)(c0 + k) * R + col, v);
#pragma unroll
            for (int q = 0; q < CPL; ++q) acc[c][q] += v[q];
        }
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int q = 0; q < CPL; ++q) sh[threadIdx.x * W + c * CPL + q] = acc[c][q];
    __syncthreads();
    for (int half = S / 2; half > 0; half >>= 1) {
        if (slice < half) {
#pragma unroll
            for (int w = 0; w < W; ++w)
                sh[threadIdx.x * W + w] += sh[(threadIdx.x + half * G) * W + w];
        }
        __syncthreads();
    }
    if (slice == 0) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int col = (c * G + lane) * CPL;
            if (col >= R) continue;
            float o[CPL];
            load_f32<CPL>(out + (size_t)row * R + col, o);
#pragma unroll
            for (int q = 0; q < CPL; ++q) o[q] += sh[threadIdx.x * W + c * CPL + q];
            store_vec<CPL>(out + (size_t)row * R + col, o);
        }
    }
}

// Every fix-up of one MTTKRP in one launch (short runs, long runs and empty
// rows own disjoint output rows): blocks [0, nlong) take a long run each, the
// blocks after them the short runs and then the empty rows, one lane group
// each.
template <int CPL, int G, int NCH>
__global__ __launch_bounds__(kLongBlock) void k_fix(
    const uint32_t *__restrict__ runs_long, uint32_t nlong, const uint32_t *__restrict__ runs,
    uint32_t nruns, const float *__restrict__ carry, int R, float *__restrict__ out,
    const uint32_t *__restrict__ empty_rows, uint32_t nempty, uint32_t nempty_groups) {
    if (blockIdx.x < nlong) {
        long_run<CPL, G, NCH>(carry, R, out, runs_long[3 * blockIdx.x],
                              runs_long[3 * blockIdx.x + 1], runs_long[3 * blockIdx.x + 2]);
        return;
    }
    short_runs<CPL, G, NCH>(((blockIdx.x - nlong) * (uint32_t)kLongBlock + threadIdx.x) / G, runs,
                            nruns, carry, R, out, empty_rows, nempty, nempty_groups);
}

// Grouped fix-ups: runs as (tensor, row, c0, n), empty rows as (tensor, row).
template <int CPL, int G, int NCH>
__global__ __launch_bounds__(kBlock) void k_fix_short_group(const GroupMttkrp *__restrict__ desc,
                                                            const uint4 *__restrict__ runs,
                                                            uint32_t nruns,
                                                            const uint2 *__restrict__ empty,
                                                            uint32_t nempty) {
    const uint32_t gid = (blockIdx.x * (uint32_t)kBlock + threadIdx.x) / G;
    const int lane = threadIdx.x % G;
    uint32_t t;
    if (gid < nruns) t = runs[gid].x;
    else if (gid - nruns < nempty) t = empty[gid - nruns].x;
    else return;
    const GroupMttkrp &d = desc[t];
    int col[NCH];
    bool act[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        col[c] = (c * G + lane) * CPL;
        act[c] = col[c] < d.R;
    }
    if (gid < nruns) {
        const uint4 r = runs[gid];
        add_run<CPL, NCH>(d.carry, d.R, d.out, r.y, r.z, r.w, col, act);
    } else {
        zero_row<CPL, NCH>(d.out, d.R, empty[gid - nruns].y, col, act);
    }
}

template <int CPL, int G, int NCH>
__global__ __launch_bounds__(kLongBlock) void k_fix_long_group(const GroupMttkrp *__restrict__ desc,
                                                               const uint4 *__restrict__ runs) {
    const uint4 r = runs[blockIdx.x];
    const GroupMttkrp &d = desc[r.x];
    long_run<CPL, G, NCH>(d.carry, d.R, d.out, r.y, r.z, r.w);
}

// ---- relabeled tables ------------------------------------------------------
// out[r] = in[perm[r]], rows of vr elements of V (a row of R factor entries
// in 16-, 8-, 4- or 2-byte pieces)
template <typename V, bool WIDE>
__global__ __launch_bounds__(256) void k_permute_rows(const V *__restrict__ in,
                                                      const uint32_t *__restrict__ perm,
                                                      int64_t rows, int vr, V *__restrict__ out) {
    const int64_t n = rows * vr;
    for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        int64_t r, c;
        if constexpr (WIDE) {
            r = e / vr;
            c = e - r * vr;
        } else {
            r = (uint32_t)e / (uint32_t)vr;
            c = (uint32_t)e - (uint32_t)r * (uint32_t)vr;
        }
        out[e] = in[(int64_t)perm[r] * vr + c];
    }
}

// out[r * S + c] = in[perm[r] * R + c] for c < R, 0 for R <= c < S (S a
// power of two: the row and column of an element are a shift and a mask)
template <typename T>
__global__ __launch_bounds__(256) void k_permute_pad(const T *__restrict__ in,
                                                     const uint32_t *__restrict__ perm,
                                                     int64_t rows, int R, int log2S,
                                                     T *__restrict__ out) {
    const int64_t n = rows << log2S;
    const int64_t mask = ((int64_t)1 << log2S) - 1;
    for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const int64_t r = e >> log2S;
        const int c = (int)(e & mask);
        out[e] = c < R ? in[(int64_t)perm[r] * R + c] : T(0);
    }
}

// out[r * R + c] = in[r * S + c]: a padded MTTKRP result back to R columns
__global__ __launch_bounds__(256) void k_unpad_rows(const float *__restrict__ in, int64_t rows,
                                                    int R, int log2S, float *__restrict__ out) {
    const int64_t n = rows * R;
    for (int64_t e = blockIdx.x * 256ll + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        const int64_t r = e / R;
        out[e] = in[(r << log2S) + (e - r * R)];
    }
}

// ---- dispatch --------------------------------------------------------------
template <int V>
using IntC = std::integral_constant<int, V>;
template <typename T>
struct TypeC {
    using type = T;
};

// f(TypeC<T>, IntC<CPL>, IntC<G>, IntC<NCH>) for the kernel shape
template <typename F>
void with_shape(dfacto_dtype dtype, const MttkrpShape &sh, F &&f) {
    auto by_g = [&](auto tc, auto cplc) {
        constexpr int CPL = decltype(cplc)::value;
        if (sh.nch == 1) {
            switch (sh.g) {
                case 2: return f(tc, cplc, IntC<2>{}, IntC<1>{});
                case 4: return f(tc, cplc, IntC<4>{}, IntC<1>{});
                case 8: return f(tc, cplc, IntC<8>{}, IntC<1>{});
                case 16: return f(tc, cplc, IntC<16>{}, IntC<1>{});
                case 32: return f(tc, cplc, IntC<32>{}, IntC<1>{});
                default: return f(tc, cplc, IntC<64>{}, IntC<1>{});
            }
        }
        if constexpr (CPL < 4) {
            if (sh.nch == 2) return f(tc, cplc, IntC<64>{}, IntC<2>{});
        }
        if constexpr (CPL == 1) {
            return f(tc, cplc, IntC<64>{}, IntC<4>{});
        }
        throw Error{DFACTO_E_UNSUPPORTED, "no MTTKRP kernel for this rank"};
    };
    auto by_cpl = [&](auto tc) {
        switch (sh.cpl) {
#if DFACTO_MAX_CPL >= 8
            case 8: return by_g(tc, IntC<8>{});
#endif
            case 4: return by_g(tc, IntC<4>{});
            case 2: return by_g(tc, IntC<2>{});
            default: return by_g(tc, IntC<1>{});
        }
    };
    if (dtype == DFACTO_F32) by_cpl(TypeC<float>{});
    else by_cpl(TypeC<uint16_t>{});
}

// The forms that rows of a type are walked in: eight columns per lane only for
// BF16 (mttkrp_shape); the main kernel's rows take at least five lanes, or
// single columns (main_shape).
template <typename T, int CPL>
constexpr bool form_ok() {
    return CPL < 8 || sizeof(T) == 2;
}
template <typename T, int CPL, int G>
constexpr bool main_form_ok() {
    return form_ok<T, CPL>() && (CPL == 1 || G >= 8);
}

// The tables the main kernel gathers from, their row stride (the kernel's
// column count), and for padded tables the padded output rows the kernel
// writes (rows_out of them), copied back to R columns after the fix-ups.
struct Tables {
    const void *leaf = nullptr, *mid = nullptr;
    int stride = 0;
    float *pad_out = nullptr;
    int64_t rows_out = 0;
};

// The block-per-chunk kernel where it is the faster one (false: not launched).
// A mode takes about 10 us and 8 ns per block (8 columns; 11 ns for 16), the
// lane groups 50 to 65 us however few chunks there are, until about 6000 chunks
// fill the device.  Three modes, FP32, by blocks and by lane groups: 78 chunks,
// R = 8 41 and 156 us (a pass limited by its launches); 1950, R = 8 82 and 187,
// R = 16 97 and 187, R = 32 (two slices) 159 and 174; 3902, R = 8 125 and 193,
// R = 16 161 and 191, but R = 32 283 and 180; 5464, R = 8 158 and 197, R = 16
// 206 and 192; 7806, R = 8 209 and 206, R = 16 281 and 204.
bool launch_block(dfacto_ctx *ctx, const ModeData &md, int R, dfacto_dtype dtype,
                  const MttkrpShape &sh, const Tables &tb, float *out, float *carry) {
    if (md.chunk_len > DFACTO_CHUNK_DEFAULT) return false;
    const bool even = sh.cpl >= 2, narrow = R <= 8;
    const unsigned slices = narrow ? 1u : (unsigned)(R + 15) / 16;
    if ((uint64_t)md.nchunk * slices > (uint64_t)(narrow ? 20 : 16) * ctx->num_cu) return false;
    auto go = [&](auto tc, auto cplc, auto gc) {
        using T = typename decltype(tc)::type;
        constexpr int CPL = decltype(cplc)::value, W = CPL * decltype(gc)::value;
        const int ld = (std::min(R, W) + CPL - 1) / CPL * CPL;
        hipLaunchKernelGGL((k_mttkrp_block<T, CPL, decltype(gc)::value>),
                           dim3((unsigned)md.nchunk, slices), dim3(kBlock),
                           sizeof(float) * 2 * kBlkFibers * (size_t)ld, ctx->stream, md.stream,
                           md.chunk_start, (const T *)tb.leaf, (const T *)tb.mid, R, out, carry, ld);
    };
    auto by_type = [&](auto tc) {
        if (narrow) go(tc, IntC<1>{}, IntC<8>{});
        else if (even) go(tc, IntC<2>{}, IntC<8>{});
        else go(tc, IntC<1>{}, IntC<16>{});
    };
    if (dtype == DFACTO_F32) by_type(TypeC<float>{});
    else by_type(TypeC<uint16_t>{});
    return true;
}

// The lane groups of the main kernel, from the fix-ups' shape `sh` (which sets
// the order of the carries' sums and so stays as it is).  Microseconds for
// three modes; "a x b": b lanes of a columns:
//  * at least five lanes per row: with fewer a wave holds more groups, and
//    nearly every entry finds one of them storing a row.  50M nonzeros, FP32:
//    R = 8 1x8 1799 against 4x2 2310; R = 16 2x8 1885 against 4x4 2112.
//  * BF16 rows of at most eight lanes: two columns per lane (a 4-byte load),
//    half the registers per row and so more rows in flight.  R = 32, 50M:
//    2x16 1905 against 4x8 1976; 100M relabeled 2950 against 3071 (8x4: 3085).
//  * the same for FP32 while the chunks are too few to fill the device with
//    eight-lane groups: R = 32, 1M nonzeros 185 against 273, 3M (8500 chunks)
//    240 against 296, but 10M (28,000 chunks) 557 against 510.
MttkrpShape main_shape(MttkrpShape sh, int R, dfacto_dtype dtype, int64_t nchunk, int num_cu) {
    if (sh.nch != 1) return sh;
    while (sh.cpl > 1 && (R + sh.cpl - 1) / sh.cpl <= 4) sh.cpl /= 2;
    if (sh.cpl == 4 && (R + 3) / 4 <= 8 && (dtype == DFACTO_BF16 || nchunk < 48 * (int64_t)num_cu))
        sh.cpl = 2;
    const int lanes = (R + sh.cpl - 1) / sh.cpl;
    sh.g = 2;
    while (sh.g < lanes) sh.g <<= 1;
    return sh;
}

// fix/ev: when set, the carry fix-ups go to stream `fix`, ordered after the
// main kernel by `ev` recorded on ctx's stream; carry_in: the carries' buffer
// (else the context's carry workspace); sh: the fix-ups' shape
void run(dfacto_ctx *ctx, const ModeData &md, int R, dfacto_dtype dtype, const MttkrpShape &sh,
         const Tables &tb, float *out, bool small, const void *Froot = nullptr,
         float *carry_in = nullptr, hipStream_t fix = nullptr, hipEvent_t ev = nullptr) {
    hipStream_t s = ctx->stream;
    const uint32_t nchunk = (uint32_t)md.nchunk;
    float *const out_user = out;
    const int R_user = R;
    if (tb.pad_out) {  // the kernels see padded rows of tb.stride columns
        R = tb.stride;
        out = tb.pad_out;
    }
    float *carry = carry_in ? carry_in
                            : (float *)ws_get(ctx, dfacto_ctx::kCarry,
                                              sizeof(float) *
                                                  (size_t)std::max<int64_t>(md.nchunk, 1) * R);
    if (nchunk > 0 && Froot) {
        with_shape(dtype, sh, [&](auto tc, auto cplc, auto gc, auto nchc) {
            using T = typename decltype(tc)::type;
            constexpr int CPL = decltype(cplc)::value, G = decltype(gc)::value,
                          NCH = decltype(nchc)::value;
            const unsigned blocks = (nchunk + kBlock / G - 1) / (kBlock / G);
            auto go = [&](auto kern) {
                hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBlock), 0, s, md.stream,
                                   md.chunk_start, nchunk, (const T *)tb.leaf,
                                   (const T *)tb.mid, (const T *)Froot, R, out, carry);
            };
            if (small) go(k_mttkrp_res<T, CPL, G, NCH, true>);
            else go(k_mttkrp_res<T, CPL, G, NCH, false>);
        });
    } else if (nchunk > 0) {
        prof_mark(ctx);
        const MttkrpShape ms = main_shape(sh, R, dtype, md.nchunk, ctx->num_cu);
        if (!launch_block(ctx, md, R, dtype, sh, tb, out, carry))
            with_shape(dtype, ms, [&](auto tc, auto cplc, auto gc, auto nchc) {
                using T = typename decltype(tc)::type;
                constexpr int CPL = decltype(cplc)::value, G = decltype(gc)::value,
                              NCH = decltype(nchc)::value;
                if constexpr (main_form_ok<T, CPL, G>()) {
                    const unsigned blocks = (nchunk + kBlock / G - 1) / (kBlock / G);
                    hipLaunchKernelGGL((k_mttkrp<T, CPL, G, NCH>), dim3(blocks), dim3(kBlock), 0,
                                       s, md.stream, md.chunk_start, nchunk, (const T *)tb.leaf,
                                       (const T *)tb.mid, R, out, carry);
                } else {
                    throw Error{DFACTO_E_UNSUPPORTED, "no MTTKRP kernel for this form"};
                }
            });
        prof_mark(ctx);
    }
    if (fix) {
        DF_HIP(hipEventRecord(ev, s));
        DF_HIP(hipStreamWaitEvent(fix, ev, 0));
        s = fix;
    }
    const uint32_t nempty = (uint32_t)md.nempty;
    const uint32_t egroups = nempty == 0 ? 0u : std::min<uint32_t>(nempty, 65536u);
    const uint64_t groups = (uint64_t)md.nruns_short + egroups;
    with_shape(DFACTO_F32, sh, [&](auto, auto cplc, auto gc, auto nchc) {
        constexpr int CPL = decltype(cplc)::value, G = decltype(gc)::value,
                      NCH = decltype(nchc)::value;
        constexpr int gpl = kLongBlock / G;  // lane groups per fix-up block
        const uint64_t fblocks = (uint64_t)md.nruns_long + (groups + gpl - 1) / gpl;
        if (fblocks > 0)
            hipLaunchKernelGGL((k_fix<CPL, G, NCH>), dim3((unsigned)fblocks), dim3(kLongBlock), 0,
                               s, md.runs_long, (uint32_t)md.nruns_long, md.runs_short,
                               (uint32_t)md.nruns_short, carry, R, out, md.empty_rows, nempty,
                               egroups);
    });
    if (tb.pad_out && tb.rows_out > 0) {
        int log2S = 0;
        while ((1 << log2S) < tb.stride) ++log2S;
        const int64_t n = tb.rows_out * R_user;
        hipLaunchKernelGGL(k_unpad_rows, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 65536)),
                           dim3(256), 0, s, tb.pad_out, tb.rows_out, R_user, log2S, out_user);
    }
    DF_LAUNCHED();
}

}  // namespace

// Row stride of a relabeled mode's gathered copies: rows shorter than a cache
// line (128 bytes) are padded to a power-of-two number of columns, so that no
// row straddles two lines (R = 10 FP32: 40 -> 64 bytes, 13.7 -> 12.3 ms per
// paper-shape launch as measured at R = 16); longer rows keep R.
int table_stride(int R, dfacto_dtype dtype) {
    if ((size_t)R * elem_size(dtype) >= 128) return R;
    int S = 1;
    while (S < R) S <<= 1;
    return S;
}

// Floats per padded output set of a tensor's relabeled modes (0 without
// padding), and the bytes of `sets` of them.
size_t pad_out_stride(const dfacto_tensor *t, int R, dfacto_dtype dtype) {
    const int S = table_stride(R, dtype);
    if (S == R) return 0;
    int64_t rows = 0;
    for (int m = 0; m < 3; ++m)
        if (t->mode[m].perm_leaf) rows = std::max<int64_t>(rows, t->dims[t->mode[m].root]);
    return ((size_t)rows * S + 63) & ~(size_t)63;
}

size_t pad_out_bytes(const dfacto_tensor *t, int R, dfacto_dtype dtype, int sets) {
    return sizeof(float) * pad_out_stride(t, R, dtype) * (size_t)sets;
}

// The column count the main kernel works with for tensor t (the padded
// stride when its relabeled modes pad their rows).
int kernel_cols(const dfacto_tensor *t, int R, dfacto_dtype dtype) {
    return pad_out_stride(t, R, dtype) ? table_stride(R, dtype) : R;
}

namespace {

// Byte offset of the mid table after `rows` leaf rows of `rowb` bytes: a
// whole number of rows that is a multiple of 256 bytes.
size_t mid_offset(int64_t rows, size_t rowb) {
    size_t g = 256, b = rowb;  // gcd(rowb, 256)
    while (b) {
        const size_t r = g % b;
        g = b;
        b = r;
    }
    const size_t m = 256 / g;  // rows per 256-byte multiple
    return ((size_t)rows + m - 1) / m * m * rowb;
}

// rows x R entries of dtype from F into `out` in the order of perm
void launch_permute(dfacto_ctx *ctx, const void *F, const uint32_t *perm, int64_t rows, int R,
                    dfacto_dtype dtype, void *out) {
    if (rows <= 0) return;
    const size_t rowb = (size_t)R * elem_size(dtype);
    auto al = [&](size_t a) {
        return rowb % a == 0 && (uintptr_t)F % a == 0 && (uintptr_t)out % a == 0;
    };
    auto go = [&](auto vt, size_t vb) {
        using V = typename decltype(vt)::type;
        const int vr = (int)(rowb / vb);
        const int64_t n = rows * vr;
        const unsigned grid = (unsigned)std::min<int64_t>((n + 255) / 256, 65536);
        if (n < ((int64_t)1 << 32))
            hipLaunchKernelGGL((k_permute_rows<V, false>), dim3(grid), dim3(256), 0, ctx->stream,
                               (const V *)F, perm, rows, vr, (V *)out);
        else
            hipLaunchKernelGGL((k_permute_rows<V, true>), dim3(grid), dim3(256), 0, ctx->stream,
                               (const V *)F, perm, rows, vr, (V *)out);
    };
    if (al(16)) go(TypeC<uint4>{}, 16);
    else if (al(8)) go(TypeC<uint2>{}, 8);
    else if (al(4)) go(TypeC<uint32_t>{}, 4);
    else go(TypeC<uint16_t>{}, 2);
    DF_LAUNCHED();
}

// The tables a mode's main kernel gathers from: the factors themselves, or
// for a relabeled mode copies permuted into rank order -- the leaf table,
// then the mid table (mid_offset), in the context's permutation workspace
// or in `buf`.
Tables gather_tables(dfacto_ctx *ctx, const dfacto_tensor *t, int mode, int R, dfacto_dtype dtype,
                     const void *Fleaf, const void *Fmid, void *buf = nullptr, int pad_set = -1) {
    const ModeData &md = t->mode[mode];
    Tables tb;
    tb.stride = R;
    if (!md.perm_leaf) {
        tb.leaf = Fleaf;
        tb.mid = Fmid;
        return tb;
    }
    const int S = pad_set >= 0 ? table_stride(R, dtype) : R;
    if (S != R) {  // rows padded to S (a power of two) columns; see table_stride
        const int64_t dl = t->dims[md.leaf], dm = t->dims[md.mid];
        const size_t es = elem_size(dtype);
        const size_t off_mid = mid_offset(dl, (size_t)S * es);
        char *w = (char *)ws_get(ctx, dfacto_ctx::kPerm, off_mid + (size_t)dm * S * es);
        int log2S = 0;
        while ((1 << log2S) < S) ++log2S;
        auto pad = [&](const void *F, const uint32_t *perm, int64_t rows, void *o) {
            if (rows <= 0) return;
            const unsigned grid =
                (unsigned)std::min<int64_t>((((int64_t)rows << log2S) + 255) / 256, 65536);
            if (dtype == DFACTO_F32)
                hipLaunchKernelGGL(k_permute_pad<float>, dim3(grid), dim3(256), 0, ctx->stream,
                                   (const float *)F, perm, rows, R, log2S, (float *)o);
            else
                hipLaunchKernelGGL(k_permute_pad<uint16_t>, dim3(grid), dim3(256), 0,
                                   ctx->stream, (const uint16_t *)F, perm, rows, R, log2S,
                                   (uint16_t *)o);
            DF_LAUNCHED();
        };
        pad(Fleaf, md.perm_leaf, dl, w);
        pad(Fmid, md.perm_mid, dm, w + off_mid);
        tb.leaf = w;
        tb.mid = w + off_mid;
        tb.stride = S;
        tb.rows_out = t->dims[md.root];
        float *po = (float *)ws_get(ctx, dfacto_ctx::kPadOut, pad_out_bytes(t, R, dtype, pad_set + 1));
        tb.pad_out = po + (size_t)pad_set * pad_out_stride(t, R, dtype);
        return tb;
    }
    const int64_t dl = t->dims[md.leaf], dm = t->dims[md.mid];
    const size_t es = elem_size(dtype);
    const size_t off_mid = mid_offset(dl, (size_t)R * es);
    const size_t total = off_mid + (size_t)dm * R * es;
    char *w = buf ? (char *)buf : (char *)ws_get(ctx, dfacto_ctx::kPerm, total);
    launch_permute(ctx, Fleaf, md.perm_leaf, dl, R, dtype, w);
    launch_permute(ctx, Fmid, md.perm_mid, dm, R, dtype, w + off_mid);
    tb.leaf = w;
    tb.mid = w + off_mid;
    return tb;
}

}  // namespace

void relabeled_tables(const dfacto_tensor *t, int mode, int R, dfacto_dtype dtype, void *buf,
                      const void **leaf, const void **mid) {
    const ModeData &md = t->mode[mode];
    *leaf = buf;
    *mid = (char *)buf + mid_offset(t->dims[md.leaf], (size_t)R * elem_size(dtype));
}

void launch_relabeled_tables(dfacto_ctx *ctx, const dfacto_tensor *t, int mode, int R,
                             dfacto_dtype dtype, const void *Fleaf, const void *Fmid, void *buf) {
    const ModeData &md = t->mode[mode];
    const void *l, *m;
    relabeled_tables(t, mode, R, dtype, buf, &l, &m);
    launch_permute(ctx, Fleaf, md.perm_leaf, t->dims[md.leaf], R, dtype, (void *)l);
    launch_permute(ctx, Fmid, md.perm_mid, t->dims[md.mid], R, dtype, (void *)m);
}

size_t perm_bytes(const dfacto_tensor *t, int R, dfacto_dtype dtype) {
    size_t b = 0;
    // the padded copies of dfacto_mttkrp & co. (the grouped and fixed-array
    // paths keep R columns, fewer bytes)
    const size_t rowb = (size_t)table_stride(R, dtype) * elem_size(dtype);
    for (int m = 0; m < 3; ++m) {
        const ModeData &md = t->mode[m];
        if (!md.perm_leaf) continue;
        b = std::max(b, mid_offset(t->dims[md.leaf], rowb) + (size_t)t->dims[md.mid] * rowb);
    }
    return b;
}

MttkrpShape mttkrp_shape(int R, dfacto_dtype dtype, const void *Fleaf, const void *Fmid,
                         const float *out, bool relabeled) {
    const size_t es = dtype == DFACTO_BF16 ? 2 : 4;
    auto al = [&](size_t a) {
        return ((uintptr_t)Fleaf % a == 0) && ((uintptr_t)Fmid % a == 0) &&
               ((uintptr_t)out % (a * 4 / es) == 0);
    };
    const bool aligned8 = al(8 * es), aligned4 = al(4 * es), aligned2 = al(2 * es);
    int cpl = 1;
    // Eight columns per lane only for BF16 (one 16-byte load per lane): a
    // gather instruction then fetches 16 rows of 64 bytes instead of 8.  For
    // FP32 eight columns are two loads per lane, no fewer instructions.  Only
    // for relabeled gathers (where the most-gathered rows share lines and the
    // wider loads pay: 13.1 -> 12.7 ms per paper-shape launch; with plain
    // gathers they cost 7%: 0.66 -> 0.70 ms at 50M nonzeros), and not below
    // R = 32, where groups of one or two lanes would share each batch of
    // stream entries over too few lanes.
    if (dtype == DFACTO_BF16 && relabeled && R % 8 == 0 && R >= 32 && aligned8 &&
        DFACTO_MAX_CPL >= 8)
        cpl = 8;
    else if (R % 4 == 0 && aligned4 && DFACTO_MAX_CPL >= 4) cpl = 4;
    else if (R % 2 == 0 && aligned2 && DFACTO_MAX_CPL >= 2) cpl = 2;
    const int lanes = (R + cpl - 1) / cpl;
    if (lanes <= 64) {
        int g = 2;
        while (g < lanes) g <<= 1;
        return {cpl, g, 1};
    }
    int nch = (lanes + 63) / 64;
    nch = nch <= 2 ? 2 : 4;
    return {cpl, 64, nch};
}

bool mttkrp_small(const dfacto_tensor *t, int mode) {
    // 24-bit row offsets when every index of the leaf, mid and output factor
    // is below 2^24 (then idx * R < 2^32 for R <= 256)
    const ModeData &md = t->mode[mode];
    return t->dims[md.root] < (1 << 24) && t->dims[md.leaf] < (1 << 24) &&
           t->dims[md.mid] < (1 << 24);
}

void launch_mttkrp(dfacto_ctx *ctx, const dfacto_tensor *t, int mode, int R, dfacto_dtype dtype,
                   const void *Fleaf, const void *Fmid, float *out) {
    const ModeData &md = t->mode[mode];
    if (ctx->profiling && md.nchunk > 0) {
        const double sf = dtype == DFACTO_BF16 ? 2.0 : 4.0;
        ctx->prof_bytes += 8.0 * (double)t->nnz + 8.0 * (double)md.nfib + 8.0 * (double)md.nroot +
                           4.0 * (double)t->dims[md.root] * R +
                           sf * (double)(t->dims[md.leaf] + t->dims[md.mid]) * R;
        ctx->prof_flops += 2.0 * R * (double)(t->nnz + md.nfib);
    }
    const bool sm = mttkrp_small(t, mode);
    const Tables tb = gather_tables(ctx, t, mode, R, dtype, Fleaf, Fmid, nullptr, 0);
    const MttkrpShape sh =
        tb.pad_out ? mttkrp_shape(tb.stride, dtype, tb.leaf, tb.mid, tb.pad_out, true)
                   : mttkrp_shape(R, dtype, Fleaf, Fmid, out, md.perm_leaf != nullptr);
    run(ctx, md, R, dtype, sh, tb, out, sm);
}

size_t mttkrp_buffers(const dfacto_tensor *t, int mode, int R, dfacto_dtype dtype,
                      size_t *carry_bytes) {
    const ModeData &md = t->mode[mode];
    *carry_bytes = (sizeof(float) * (size_t)std::max<int64_t>(md.nchunk, 1) * R + 255) &
                   ~(size_t)255;
    if (!md.perm_leaf) return 0;
    const size_t rowb = (size_t)R * elem_size(dtype);
    return mid_offset(t->dims[md.leaf], rowb) + (size_t)t->dims[md.mid] * rowb;
}

void launch_mttkrp_in(dfacto_ctx *ctx, const dfacto_tensor *t, int mode, int R,
                      dfacto_dtype dtype, const void *Fleaf, const void *Fmid, float *out,
                      float *carry, void *perm) {
    const ModeData &md = t->mode[mode];
    const MttkrpShape sh = mttkrp_shape(R, dtype, Fleaf, Fmid, out, md.perm_leaf != nullptr);
    const bool sm = mttkrp_small(t, mode);
    const Tables tb = gather_tables(ctx, t, mode, R, dtype, Fleaf, Fmid, perm);
    run(ctx, md, R, dtype, sh, tb, out, sm, nullptr, carry);
}

void launch_mttkrp_split(dfacto_ctx *ctx, const dfacto_tensor *t, int mode, int R,
                         dfacto_dtype dtype, const void *Fleaf, const void *Fmid, float *out,
                         float *carry, hipStream_t fix, hipEvent_t ev) {
    const ModeData &md = t->mode[mode];
    if (ctx->profiling && md.nchunk > 0) {
        const double sf = dtype == DFACTO_BF16 ? 2.0 : 4.0;
        ctx->prof_bytes += 8.0 * (double)t->nnz + 8.0 * (double)md.nfib + 8.0 * (double)md.nroot +
                           4.0 * (double)t->dims[md.root] * R +
                           sf * (double)(t->dims[md.leaf] + t->dims[md.mid]) * R;
        ctx->prof_flops += 2.0 * R * (double)(t->nnz + md.nfib);
    }
    const bool sm = mttkrp_small(t, mode);
    const Tables tb = gather_tables(ctx, t, mode, R, dtype, Fleaf, Fmid, nullptr, mode);
    const MttkrpShape sh =
        tb.pad_out ? mttkrp_shape(tb.stride, dtype, tb.leaf, tb.mid, tb.pad_out, true)
                   : mttkrp_shape(R, dtype, Fleaf, Fmid, out, md.perm_leaf != nullptr);
    run(ctx, md, R, dtype, sh, tb, out, sm, nullptr, carry, fix, ev);
}

void launch_mttkrp_resid(dfacto_ctx *ctx, const dfacto_tensor *t, int mode, int R,
                         dfacto_dtype dtype, const void *Fleaf, const void *Fmid,
                         const void *Froot, float *out) {
    const ModeData &md = t->mode[mode];
    // the root rows share the alignment rule of the gathered rows
    MttkrpShape sh = mttkrp_shape(R, dtype, Fleaf, Fmid, out, false);
    const MttkrpShape sr = mttkrp_shape(R, dtype, Froot, Froot, out, false);
    if (sr.cpl < sh.cpl) sh = sr;
    const bool sm = mttkrp_small(t, mode);
    const Tables tb = gather_tables(ctx, t, mode, R, dtype, Fleaf, Fmid);
    run(ctx, md, R, dtype, sh, tb, out, sm, Froot);
}

void launch_gather_probe(dfacto_ctx *ctx, const dfacto_tensor *t, int mode, int R,
                         dfacto_dtype dtype, const void *Fleaf, const void *Fmid, int pattern,
                         float *sink) {
    const ModeData &md = t->mode[mode];
    // the tables, row stride and lane groups that launch_mttkrp's call would
    // have with an output aligned as the sink
    auto shape = [&](int cols, const void *leaf, const void *mid) {
        const MttkrpShape sh = mttkrp_shape(cols, dtype, leaf, mid, sink, md.perm_leaf != nullptr);
        return main_shape(sh, cols, dtype, md.nchunk, ctx->num_cu);
    };
    const int S = kernel_cols(t, R, dtype);
    if (shape(S, Fleaf, Fmid).nch != 1)
        throw Error{DFACTO_E_UNSUPPORTED, "the gather probe takes R <= 64 * CPL"};
    if ((pattern == 5 || pattern >= 8) && S > kProbeLdsRowElems)
        throw Error{DFACTO_E_UNSUPPORTED, "the LDS patterns take R <= 64"};
    if (pattern >= 6 && (uint64_t)t->dims[md.leaf] * S * elem_size(dtype) >= kProbeOut)
        throw Error{DFACTO_E_UNSUPPORTED, "the buffer patterns take a leaf table below 4 GB"};
    const uint32_t nchunk = (uint32_t)md.nchunk;
    if (nchunk == 0) return;
    const uint32_t nleaf = (uint32_t)t->dims[md.leaf], nmid = (uint32_t)t->dims[md.mid];
    const Tables tb = gather_tables(ctx, t, mode, R, dtype, Fleaf, Fmid, nullptr, 0);
    const MttkrpShape sh =
        tb.pad_out ? shape(tb.stride, tb.leaf, tb.mid) : shape(R, Fleaf, Fmid);
    with_shape(dtype, sh, [&](auto tc, auto cplc, auto gc, auto) {
        using T = typename decltype(tc)::type;
        constexpr int CPL = decltype(cplc)::value, G = decltype(gc)::value;
        if constexpr (main_form_ok<T, CPL, G>()) {
            const unsigned blocks = (nchunk + kBlock / G - 1) / (kBlock / G);
            auto go = [&](auto kern) {
                prof_mark(ctx);
                hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBlock), 0, ctx->stream, md.stream,
                                   md.chunk_start, nchunk, (const T *)tb.leaf, (const T *)tb.mid,
                                   tb.stride, nleaf, nmid, sink);
                prof_mark(ctx);
            };
            switch (pattern) {
                case 0: return go(k_gather_probe<T, CPL, G, 0>);
                case 1: return go(k_gather_probe<T, CPL, G, 1>);
                case 2: return go(k_gather_probe<T, CPL, G, 2>);
                case 3: return go(k_gather_probe<T, CPL, G, 3>);
                case 4: return go(k_gather_probe<T, CPL, G, 4>);
                case 5: return go(k_gather_probe<T, CPL, G, 5>);
                case 6: return go(k_gather_probe<T, CPL, G, 6>);
                case 7: return go(k_gather_probe<T, CPL, G, 7>);
                case 8: return go(k_gather_probe<T, CPL, G, 8>);
                default: return go(k_gather_probe<T, CPL, G, 9>);
            }
        } else {
            throw Error{DFACTO_E_UNSUPPORTED, "no gather probe for this form"};
        }
    });
    DF_LAUNCHED();
}

MttkrpShape mttkrp_main_shape(const dfacto_ctx *ctx, const MttkrpShape &sh, int R,
                              dfacto_dtype dtype, int64_t nchunk) {
    return main_shape(sh, R, dtype, nchunk, ctx->num_cu);
}

unsigned mttkrp_group_chunks_per_item(const MttkrpShape &sh, unsigned kper) {
    return (unsigned)(kBlock / sh.g) * kper;
}

void launch_mttkrp_group(dfacto_ctx *ctx, dfacto_dtype dtype, const MttkrpShape &sh,
                         const GroupMttkrp *d_desc, const uint2 *d_items, uint32_t nitems,
                         unsigned grid, unsigned kper) {
    if (nitems == 0) return;
    if (kper < 1 || grid < 1) throw Error{DFACTO_E_INVALID, "grouped MTTKRP launch shape"};
    with_shape(dtype, sh, [&](auto tc, auto cplc, auto gc, auto nchc) {
        using T = typename decltype(tc)::type;
        constexpr int CPL = decltype(cplc)::value;
        if constexpr (form_ok<T, CPL>())
            hipLaunchKernelGGL((k_mttkrp_group<T, CPL, decltype(gc)::value,
                                               decltype(nchc)::value>),
                               dim3(grid), dim3(kBlock), 0, ctx->stream, d_desc, d_items, nitems,
                               kper);
        else
            throw Error{DFACTO_E_UNSUPPORTED, "no grouped MTTKRP kernel for this form"};
    });
    DF_LAUNCHED();
}

void launch_fix_group(dfacto_ctx *ctx, const MttkrpShape &sh, const GroupMttkrp *d_desc,
                      const uint4 *d_short, uint32_t nshort, const uint2 *d_empty,
                      uint32_t nempty, const uint4 *d_long, uint32_t nlong) {
    hipStream_t s = ctx->stream;
    // the fix-up kernels do not depend on the factor type
    with_shape(DFACTO_F32, sh, [&](auto, auto cplc, auto gc, auto nchc) {
        constexpr int CPL = decltype(cplc)::value, G = decltype(gc)::value,
                      NCH = decltype(nchc)::value;
        const uint64_t groups = (uint64_t)nshort + nempty;
        if (groups > 0) {
            const unsigned blocks = (unsigned)((groups + kBlock / G - 1) / (kBlock / G));
            hipLaunchKernelGGL((k_fix_short_group<CPL, G, NCH>), dim3(blocks), dim3(kBlock), 0, s,
                               d_desc, d_short, nshort, d_empty, nempty);
        }
        if (nlong > 0)
            hipLaunchKernelGGL((k_fix_long_group<CPL, G, NCH>), dim3(nlong), dim3(kLongBlock), 0,
                               s, d_desc, d_long);
    });
    DF_LAUNCHED();
}

}  // namespace dfacto
