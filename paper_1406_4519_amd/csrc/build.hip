// build.hip -- on-device construction of the three fiber-compressed
// flattenings (DFacTo, Section 2.1 eq. (1); Section 3, the CSR storage of
// (X2)^T without zero rows and the precomputed pattern of M^r, Lemmas 3-4).
//
// Pipeline (all on the device, one host readback per size that must be
// known to allocate):
//   validate and pack each coordinate into one 64-bit key (i, k, j), sort the
//   values with it (stable LSD radix) -> merge duplicates (sum in input
//   order) -> ||X||^2 -> from the (i, k, j) order a stable sort by j alone is
//   mode 1's order (j, i, k), and from that a sort by k alone mode 2's (k, j,
//   i), so each takes only that field's digits -> per mode: fiber starts,
//   fiber segments of at most kFiberCap nonzeros, the interleaved
//   header/nonzero stream, empty output rows, work chunks.
// The key carries all three indices through every sort, so nothing is gathered
// by a permutation.  Sizes whose indices need more than 64 bits together take
// the coordinates as three arrays and sort permutations instead.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "internal.hpp"

namespace dfacto {
namespace {

constexpr int kThreads = 256;

inline unsigned grid_for(int64_t n, int per_block = kThreads) {
    int64_t g = (n + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > (1 << 20)) g = 1 << 20;  // grid-stride beyond this
    return (unsigned)g;
}

#define GRID_STRIDE(e, n)                                                           \
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (n);       \
         e += (int64_t)gridDim.x * blockDim.x)

int bits_for(int64_t d) {  // bits needed to store indices 0 .. d-1
    int b = 0;
    while (((int64_t)1 << b) < d) ++b;
    return b;
}

// ---------------------------------------------------------------------------
// simple elementwise kernels
// ---------------------------------------------------------------------------

__global__ void k_validate(const uint32_t *__restrict__ i, const uint32_t *__restrict__ j,
                           const uint32_t *__restrict__ k, const float *__restrict__ v,
                           int64_t n, uint32_t I, uint32_t J, uint32_t K,
                           uint32_t *__restrict__ flag) {
    uint32_t bad = 0;
    GRID_STRIDE(e, n) {
        if (i[e] >= I || j[e] >= J || k[e] >= K) bad |= 1u;
        if (!isfinite(v[e])) bad |= 2u;
    }
    if (bad) atomicOr(flag, bad);
}

// the same check, packing (i, k, j) into a key of bK + bJ lower bits
__global__ void k_pack(const uint32_t *__restrict__ i, const uint32_t *__restrict__ j,
                       const uint32_t *__restrict__ k, const float *__restrict__ v, int64_t n,
                       uint32_t I, uint32_t J, uint32_t K, int bK, int bJ,
                       uint64_t *__restrict__ key, uint32_t *__restrict__ val,
                       uint32_t *__restrict__ flag) {
    uint32_t bad = 0;
    GRID_STRIDE(e, n) {
        const uint32_t a = i[e], b = j[e], c = k[e];
        const float x = v[e];
        if (a >= I || b >= J || c >= K) bad |= 1u;
        if (!isfinite(x)) bad |= 2u;
        // an index out of range may spill into its neighbours' bits: the
        // build stops before anything but the sort has read the key
        key[e] = ((uint64_t)a << (bK + bJ)) | ((uint64_t)c << bJ) | b;
        val[e] = __float_as_uint(x);
    }
    if (bad) atomicOr(flag, bad);
}

__global__ void k_iota(uint32_t *__restrict__ p, int64_t n) {
    GRID_STRIDE(e, n) p[e] = (uint32_t)e;
}

// key = (a << sa) | (b << sb) | c   from coordinate arrays, optionally
// gathered through a permutation.
__global__ void k_make_key(uint64_t *__restrict__ key, const uint32_t *__restrict__ a, int sa,
                           const uint32_t *__restrict__ b, int sb,
                           const uint32_t *__restrict__ c, const uint32_t *__restrict__ perm,
                           int64_t n) {
    GRID_STRIDE(e, n) {
        const int64_t s = perm ? perm[e] : e;
        uint64_t x = 0;
        if (a) x |= (uint64_t)a[s] << sa;
        if (b) x |= (uint64_t)b[s] << sb;
        if (c) x |= (uint64_t)c[s];
        key[e] = x;
    }
}

__global__ void k_gather4(const uint32_t *__restrict__ perm, int64_t n,
                          const uint32_t *__restrict__ a, const uint32_t *__restrict__ b,
                          const uint32_t *__restrict__ c, const float *__restrict__ v,
                          uint32_t *__restrict__ oa, uint32_t *__restrict__ ob,
                          uint32_t *__restrict__ oc, float *__restrict__ ov) {
    GRID_STRIDE(e, n) {
        const uint32_t s = perm[e];
        oa[e] = a[s];
        ob[e] = b[s];
        oc[e] = c[s];
        ov[e] = v[s];
    }
}

// ---------------------------------------------------------------------------
// coordinates in a mode's order: packed keys, or three arrays
// ---------------------------------------------------------------------------
struct PackedCoords {
    const uint64_t *key;
    int sr, sm, sl;           // each field's lowest bit
    uint32_t mr, mm, ml;      // and mask
    __device__ uint32_t root(int64_t e) const { return (uint32_t)(key[e] >> sr) & mr; }
    __device__ uint32_t mid(int64_t e) const { return (uint32_t)(key[e] >> sm) & mm; }
    __device__ uint32_t leaf(int64_t e) const { return (uint32_t)(key[e] >> sl) & ml; }
    // bit 0: entry e opens a fiber, bit 1: and a root
    __device__ uint32_t opens(int64_t e) const {
        if (e == 0) return 3u;
        const uint64_t d = key[e] ^ key[e - 1];
        return ((uint32_t)(d >> sr) & mr) ? 3u : (((uint32_t)(d >> sm) & mm) ? 1u : 0u);
    }
    __device__ bool same(int64_t e, int64_t f) const { return key[e] == key[f]; }
};
struct ArrayCoords {
    const uint32_t *r, *m, *l;
    __device__ uint32_t root(int64_t e) const { return r[e]; }
    __device__ uint32_t mid(int64_t e) const { return m[e]; }
    __device__ uint32_t leaf(int64_t e) const { return l[e]; }
    __device__ uint32_t opens(int64_t e) const {
        if (e == 0 || r[e] != r[e - 1]) return 3u;
        return m[e] != m[e - 1] ? 1u : 0u;
    }
    __device__ bool same(int64_t e, int64_t f) const {
        return r[e] == r[f] && m[e] == m[f] && l[e] == l[f];
    }
};

// Tiles of the passes below: each wave takes kTileSlots * 64 consecutive
// entries, 64 at a time.
constexpr int kTileSlots = 8, kTileWave = kTileSlots * 64, kTile = (kThreads / 64) * kTileWave;

__device__ __forceinline__ int64_t tile_entry(int q) {
    return (int64_t)blockIdx.x * kTile + (threadIdx.x >> 6) * kTileWave + q * 64 +
           (threadIdx.x & 63);
}

// the block's sum of one count per wave (the same in every lane of a wave);
// *before: of the waves before this one
__device__ __forceinline__ uint32_t waves_sum(uint32_t c, uint32_t *before) {
    __shared__ uint32_t sh[kThreads / 64];
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = c;
    __syncthreads();
    uint32_t t = 0, b = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
        if (w == (int)(threadIdx.x >> 6)) b = t;
        t += sh[w];
    }
    *before = b;
    return t;
}

// distinct coordinates per tile of the sorted entries
template <class C>
__global__ __launch_bounds__(kThreads) void k_tile_distinct(C c, int64_t n,
                                                            uint32_t *__restrict__ cnt) {
    uint32_t k = 0;
#pragma unroll
    for (int q = 0; q < kTileSlots; ++q) {
        const int64_t e = tile_entry(q);
        k += (uint32_t)__popcll(__ballot(e < n && (e == 0 || !c.same(e, e - 1))));
    }
    uint32_t b;
    const uint32_t t = waves_sum(k, &b);
    if (threadIdx.x == 0) cnt[blockIdx.x] = t;
}

// Sum each run of equal coordinates in order; store(o, e, sum) writes the o-th
// distinct one, entry e.  Runs of more than kRunShort entries are listed as
// (o, e) and left to k_merge_long: adding up the 100,000 draws of a skewed
// tensor's most frequent coordinate in one thread took 16 ms, a memory round
// trip per entry (50M draws now: 0.73 + 0.54 ms; one global atomic per listed
// run instead of per tile: 2.25 + 0.6).
constexpr int kRunShort = 16;
template <class C, class Store>
__global__ __launch_bounds__(kThreads) void k_merge(C c, const float *__restrict__ v, int64_t n,
                                                    const uint32_t *__restrict__ off, Store store,
                                                    uint2 *__restrict__ longs,
                                                    uint32_t *__restrict__ nlong) {
    __shared__ uint2 sl[kTile / (kRunShort + 1) + 2];  // the long runs that begin here
    __shared__ uint32_t nsl;
    if (threadIdx.x == 0) nsl = 0;
    uint64_t mask[kTileSlots];
    uint32_t k = 0;
#pragma unroll
    for (int q = 0; q < kTileSlots; ++q) {
        const int64_t e = tile_entry(q);
        mask[q] = __ballot(e < n && (e == 0 || !c.same(e, e - 1)));
        k += (uint32_t)__popcll(mask[q]);
    }
    uint32_t o;
    (void)waves_sum(k, &o);
    o += off[blockIdx.x];
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < kTileSlots; ++q) {
        const int64_t e = tile_entry(q);
        const uint32_t at = o + (uint32_t)__popcll(mask[q] & ~(~0ull << lane));
        bool lng = false;
        if ((mask[q] >> lane) & 1) {
            float sum = v[e];
            int64_t t = e + 1;
            if (lane == 63 || !((mask[q] >> (lane + 1)) & 1))
                for (; t < n && t <= e + kRunShort && c.same(t, e); ++t) sum += v[t];
            lng = t == e + kRunShort + 1;
            if (!lng) store(at, e, sum);
        }
        if (lng) sl[atomicAdd(&nsl, 1u)] = make_uint2(at, (uint32_t)e);
        o += (uint32_t)__popcll(mask[q]);
    }
    // the tile's runs take consecutive places in the list: one global atomic
    __syncthreads();
    __shared__ uint32_t place;
    if (threadIdx.x == 0 && nsl) place = atomicAdd(nlong, nsl);
    __syncthreads();
    for (uint32_t r = threadIdx.x; r < nsl; r += kThreads) longs[place + r] = sl[r];
}

// One wave per listed run: its end by a search with 64 probes at a time, then
// 1024 values at a time through LDS, added in order while the next ones are in
// flight.  Bound by the chain of adds.
constexpr int kLongSlots = 16, kLongBatch = 64 * kLongSlots;
template <class C, class Store>
__global__ __launch_bounds__(64) void k_merge_long(C c, const float *__restrict__ v, int64_t n,
                                                   Store store, const uint2 *__restrict__ longs,
                                                   const uint32_t *__restrict__ nlong) {
    __shared__ alignas(16) float x[kLongBatch];
    const int lane = threadIdx.x;
    for (uint32_t r = blockIdx.x; r < *nlong; r += gridDim.x) {
        const uint2 w = longs[r];
        const int64_t e = w.y;
        // the run is [e, end): lo is in it, hi is not
        int64_t lo = e, hi = n, step = 1;
        while (hi - lo > 1) {
            const int64_t t = lo + (lane + 1) * step;
            const uint64_t in = __ballot(t < hi && c.same(t, e));
            const int k = __popcll(in);  // sorted: the first k probes
            if (k < 64) hi = lo + (k + 1) * step < hi ? lo + (k + 1) * step : hi;
            lo += k * step;
            step = k == 64 ? step * 64 : (hi - lo + 62) / 64;
            if (step < 1) step = 1;
        }
        const int64_t end = hi;
        float next[kLongSlots];
        auto load = [&](int64_t at) {
#pragma unroll
            for (int q = 0; q < kLongSlots; ++q) {
                const int64_t t = at + q * 64 + lane;
                next[q] = v[t < end ? t : end - 1];
            }
        };
        load(e);
        float sum = 0.f;
        for (int64_t at = e; at < end; at += kLongBatch) {
            const int have = (int)(end - at < kLongBatch ? end - at : kLongBatch);
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kLongSlots; ++q) x[q * 64 + lane] = next[q];
            __syncthreads();
            load(at + kLongBatch);
            int k = 0;
            if (at == e) sum = x[k++];  // the first value itself
            for (; k < have && (k & 63); ++k) sum += x[k];
            for (; k + 64 <= have; k += 64) {
                float4 a[16];  // all reads ahead of the chain of adds
#pragma unroll
                for (int q = 0; q < 16; ++q) a[q] = *(const float4 *)(x + k + 4 * q);
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    sum += a[q].x; sum += a[q].y; sum += a[q].z; sum += a[q].w;
                }
            }
            for (; k < have; ++k) sum += x[k];
        }
        if (lane == 0) store(w.x, e, sum);
    }
}

struct StorePacked {
    const uint64_t *key;
    uint64_t *ok;
    uint32_t *ov;
    __device__ void operator()(uint32_t o, int64_t e, float sum) const {
        ok[o] = key[e];
        ov[o] = __float_as_uint(sum);
    }
};
struct StoreArrays {
    ArrayCoords c;
    uint32_t *a, *b, *l;
    float *ov;
    __device__ void operator()(uint32_t o, int64_t e, float sum) const {
        a[o] = c.r[e];
        b[o] = c.m[e];
        l[o] = c.l[e];
        ov[o] = sum;
    }
};

// per-block partial sums of squares, fixed order
__global__ void k_sumsq_partial(const float *__restrict__ v, int64_t n, double *__restrict__ part) {
    __shared__ double sh[kThreads];
    double s = 0.0;
    GRID_STRIDE(e, n) {
        const double x = v[e];
        s += x * x;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void k_sum_f64_final(const double *__restrict__ part, int n, double *__restrict__ out) {
    __shared__ double sh[kThreads];
    double s = 0.0;
    for (int e = threadIdx.x; e < n; e += kThreads) s += part[e];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0];
}

// ---------------------------------------------------------------------------
// exclusive scan of u32 by sum or maximum (three phases, recursive on blocks)
// ---------------------------------------------------------------------------
constexpr int kScanIpt = 8;
constexpr int kScanTile = kThreads * kScanIpt;

struct ScanSum {
    __device__ static uint32_t op(uint32_t a, uint32_t b) { return a + b; }
};
struct ScanMax {
    __device__ static uint32_t op(uint32_t a, uint32_t b) { return a > b ? a : b; }
};

template <class Op>
__global__ void k_scan_reduce(const uint32_t *__restrict__ in, int64_t n,
                              uint32_t *__restrict__ bsum) {
    __shared__ uint32_t sh[kThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
    for (int q = 0; q < kScanIpt; ++q) {
        const int64_t e = base + (int64_t)q * kThreads + threadIdx.x;
        if (e < n) s = Op::op(s, in[e]);
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] = Op::op(sh[threadIdx.x], sh[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = sh[0];
}

template <class Op>
__global__ void k_scan_apply(const uint32_t *__restrict__ in, uint32_t *__restrict__ out,
                             int64_t n, const uint32_t *__restrict__ boff) {
    __shared__ uint32_t sh[kThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanIpt;
    uint32_t v[kScanIpt];
    uint32_t s = 0;
    for (int q = 0; q < kScanIpt; ++q) {
        const int64_t e = base + q;
        v[q] = (e < n) ? in[e] : 0u;
        s = Op::op(s, v[q]);
    }
    // Hillis-Steele over kThreads values in LDS
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < kThreads; off <<= 1) {
        const uint32_t y = ((int)threadIdx.x >= off) ? sh[threadIdx.x - off] : 0u;
        __syncthreads();
        sh[threadIdx.x] = Op::op(sh[threadIdx.x], y);
        __syncthreads();
    }
    uint32_t run = Op::op(threadIdx.x ? sh[threadIdx.x - 1] : 0u, boff ? boff[blockIdx.x] : 0u);
    for (int q = 0; q < kScanIpt; ++q) {
        const int64_t e = base + q;
        if (e < n) out[e] = run;
        run = Op::op(run, v[q]);
    }
}

// ---------------------------------------------------------------------------
// stable LSD radix sort of (u64 key, u32 value) pairs, digits of at most 8 bits
//
// Bound by HBM: a pass reads the keys for the histograms, then reads and
// writes keys and values (32 bytes per pair).  A tile's pairs are put in digit
// order in LDS first, so that each digit's run leaves as one piece of
// consecutive stores: 50M pairs 478 + 120 us per pass -> 311 + 100 (3.9 TB/s).
// ---------------------------------------------------------------------------
constexpr int kRadixSlots = 16;  // pairs per thread
constexpr int kRadixTile = kThreads * kRadixSlots;
constexpr int kRadixWaves = kThreads / 64;

__global__ __launch_bounds__(kThreads) void k_radix_hist(const uint64_t *__restrict__ keys,
                                                         int64_t n, int shift, uint32_t dmask,
                                                         uint32_t *__restrict__ hist,
                                                         int64_t nblk, bool own) {
    __shared__ uint32_t h[kRadixWaves][256];
    const int tid = threadIdx.x;
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) h[w][tid] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRadixTile;
#pragma unroll
    for (int q = 0; q < kRadixSlots; ++q) {
        const int64_t e = base + (int64_t)q * kThreads + tid;
        if (e < n) atomicAdd(&h[tid / 64][(uint32_t)(keys[e] >> shift) & dmask], 1u);
    }
    __syncthreads();
    if ((uint32_t)tid <= dmask) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kRadixWaves; ++w) c += h[w][tid];
        hist[own ? (int64_t)blockIdx.x * 256 + tid : (int64_t)tid * nblk + blockIdx.x] = c;
    }
}

// A wave takes kRadixSlots * 64 consecutive pairs, 64 at a time; a pair's rank
// among its digit's is the digits of earlier waves, of the wave's earlier
// slots, and of earlier lanes, the last from one ballot per digit bit.  The
// tile's first position for digit d is offs[d * nblk + tile] (the exclusive
// scan of the histograms in (digit, tile) order); with kOwn the block forms it
// itself from the histograms, kept in (tile, digit) order (few tiles: nblk reads
// per thread and a scan over the digits, two launches per pass instead of five).
constexpr int64_t kRadixOwnMax = 256;  // most tiles for kOwn
template <bool kOwn>
__global__ __launch_bounds__(kThreads) void k_radix_scatter(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
    uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n, int shift, int bits,
    const uint32_t *__restrict__ offs, int64_t nblk) {
    __shared__ uint64_t sk[kRadixTile];
    __shared__ uint32_t sv[kRadixTile];
    __shared__ uint32_t s_cnt[kRadixWaves][256];  // digits of a wave; then of the waves before it
    __shared__ uint32_t s_base[256], s_gbase[256];  // a digit's first place in LDS and in kout
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t dmask = (1u << bits) - 1u;
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) s_cnt[w][tid] = 0;
    if constexpr (kOwn) {  // offs holds the histograms here
        uint32_t tot = 0, pre = 0;
        if ((uint32_t)tid <= dmask) {
#pragma unroll 32
            for (int b = 0; b < (int)nblk; ++b) {
                const uint32_t c = offs[b * 256 + tid];
                tot += c;
                pre += (b < (int)blockIdx.x) ? c : 0u;
            }
        }
        s_base[tid] = tot;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {
            const uint32_t v = tid >= o ? s_base[tid - o] : 0u;
            __syncthreads();
            s_base[tid] += v;
            __syncthreads();
        }
        s_gbase[tid] = s_base[tid] - tot + pre;
    } else if ((uint32_t)tid <= dmask) {
        s_gbase[tid] = offs[(int64_t)tid * nblk + blockIdx.x];
    }
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRadixTile;
    const int cnt = (int)(n - base < kRadixTile ? n - base : kRadixTile);
    const int first = wave * (kRadixSlots * 64) + lane;
    uint64_t key[kRadixSlots];
    uint32_t val[kRadixSlots], rank[kRadixSlots];
#pragma unroll
    for (int q = 0; q < kRadixSlots; ++q) {
        const int x = first + 64 * q;
        key[q] = x < cnt ? kin[base + x] : 0ull;
        val[q] = x < cnt ? vin[base + x] : 0u;
    }
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int q = 0; q < kRadixSlots; ++q) {
        const bool valid = first + 64 * q < cnt;
        const uint32_t d = (uint32_t)(key[q] >> shift) & dmask;
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            if (b >= bits) break;  // uniform
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(bit);
            m &= bit ? bal : ~bal;
        }
        const uint32_t before = (uint32_t)__popcll(m & lt);
        // only this wave touches its row of s_cnt, and a wave's LDS operations
        // are in order
        rank[q] = valid ? ((volatile uint32_t *)s_cnt[wave])[d] + before : 0u;
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) ((volatile uint32_t *)s_cnt[wave])[d] += (uint32_t)__popcll(m);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kRadixWaves; ++w) {
            const uint32_t x = s_cnt[w][tid];
            s_cnt[w][tid] = c;
            c += x;
        }
        s_base[tid] = c;
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {
            const uint32_t v = tid >= o ? s_base[tid - o] : 0u;
            __syncthreads();
            s_base[tid] += v;
            __syncthreads();
        }
        s_base[tid] -= c;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kRadixSlots; ++q) {
        if (first + 64 * q >= cnt) continue;
        const uint32_t d = (uint32_t)(key[q] >> shift) & dmask;
        const uint32_t x = s_base[d] + s_cnt[wave][d] + rank[q];
        if (x < (uint32_t)kRadixTile) {  // always true
            sk[x] = key[q];
            sv[x] = val[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kRadixSlots; ++q) {
        const int x = q * kThreads + tid;
        if (x >= cnt) continue;
        const uint64_t k = sk[x];
        const uint32_t d = (uint32_t)(k >> shift) & dmask;
        const uint32_t pos = s_gbase[d] + (uint32_t)x - s_base[d];
        if ((int64_t)pos < n) {  // always true for consistent histograms
            kout[pos] = k;
            vout[pos] = sv[x];
        }
    }
}

// ---------------------------------------------------------------------------
// per-mode stream construction
// ---------------------------------------------------------------------------

// Pass 1: fibers per tile, and 1 + the tile's last fiber start (0: none).
template <class C>
__global__ __launch_bounds__(kThreads) void k_tile_fibers(C c, int64_t n,
                                                          uint32_t *__restrict__ nfib,
                                                          uint32_t *__restrict__ last) {
    __shared__ uint32_t sl[kThreads / 64];
    uint32_t k = 0, l = 0;
#pragma unroll
    for (int q = 0; q < kTileSlots; ++q) {
        const int64_t e = tile_entry(q);
        const uint64_t m = __ballot(e < n && c.opens(e));
        if (m) l = (uint32_t)(e - (threadIdx.x & 63)) + 64u - (uint32_t)__clzll((long long)m);
        k += (uint32_t)__popcll(m);
    }
    if ((threadIdx.x & 63) == 0) sl[threadIdx.x >> 6] = l;
    uint32_t b;
    const uint32_t t = waves_sum(k, &b);
    if (threadIdx.x == 0) {
        nfib[blockIdx.x] = t;
        uint32_t x = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) x = sl[w] ? sl[w] : x;
        last[blockIdx.x] = x;
    }
}

// The header bits of this thread's entries: a header precedes a nonzero at
// every fiber start and every kFiberCap nonzeros inside a fiber.  open: 1 + the
// last fiber start before the tile (an exclusive maximum scan of pass 1's).
// Returns the wave's headers; root[q]: which entries open an output row.
template <class C>
__device__ __forceinline__ uint32_t tile_headers(const C &c, int64_t n, uint32_t open,
                                                 uint64_t (&head)[kTileSlots],
                                                 uint64_t (&root)[kTileSlots]) {
    __shared__ uint32_t sl[kThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t l = 0;
#pragma unroll
    for (int q = 0; q < kTileSlots; ++q) {
        const int64_t e = tile_entry(q);
        const uint32_t o = e < n ? c.opens(e) : 0u;
        head[q] = __ballot(o & 1u);
        root[q] = __ballot(o & 2u);
        if (head[q]) l = (uint32_t)(e - lane) + 64u - (uint32_t)__clzll((long long)head[q]);
    }
    if (lane == 0) sl[wave] = l;
    __syncthreads();
    for (int w = 0; w < wave; ++w) open = sl[w] ? sl[w] : open;
    uint32_t k = 0;
#pragma unroll
    for (int q = 0; q < kTileSlots; ++q) {
        const int64_t e = tile_entry(q);
        const uint64_t f = head[q], upto = f & ~((~0ull << 1) << lane);
        const uint32_t start = upto ? (uint32_t)(e - lane) + 63u - (uint32_t)__clzll((long long)upto)
                                    : open - 1u;
        head[q] = __ballot(e < n && (((uint32_t)e - start) % (uint32_t)kFiberCap) == 0u);
        if (f) open = (uint32_t)(e - lane) + 64u - (uint32_t)__clzll((long long)f);
        k += (uint32_t)__popcll(head[q]);
    }
    return k;
}

// Pass 2: headers per tile; mark[row] = 0 for every row with a nonzero
template <class C>
__global__ __launch_bounds__(kThreads) void k_tile_headers(C c, int64_t n, int64_t nrows,
                                                           const uint32_t *__restrict__ open,
                                                           uint32_t *__restrict__ nhdr,
                                                           uint32_t *__restrict__ mark) {
    uint64_t head[kTileSlots], root[kTileSlots];
    const uint32_t k = tile_headers(c, n, open[blockIdx.x], head, root);
#pragma unroll
    for (int q = 0; q < kTileSlots; ++q)
        if ((root[q] >> (threadIdx.x & 63)) & 1) {
            const uint32_t r = c.root(tile_entry(q));
            if (r < nrows) mark[r] = 0u;
        }
    uint32_t b;
    const uint32_t t = waves_sum(k, &b);
    if (threadIdx.x == 0) nhdr[blockIdx.x] = t;
}

// Pass 3: f(q, e, header, opens a row, headers before e) for every entry
template <class C, class Fn>
__device__ __forceinline__ void tile_walk(const C &c, int64_t n, uint32_t open, uint32_t hoff,
                                          Fn &&f) {
    uint64_t head[kTileSlots], root[kTileSlots];
    const uint32_t k = tile_headers(c, n, open, head, root);
    uint32_t h;
    (void)waves_sum(k, &h);
    h += hoff;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < kTileSlots; ++q) {
        const int64_t e = tile_entry(q);
        if (e < n)
            f(e, (bool)((head[q] >> lane) & 1), (bool)((root[q] >> lane) & 1),
              h + (uint32_t)__popcll(head[q] & ~(~0ull << lane)));
        h += (uint32_t)__popcll(head[q]);
    }
}

// the stream; inv_leaf / inv_mid (or null): the relabeled index of each row
template <class C>
__global__ __launch_bounds__(kThreads) void k_emit_stream(
    C c, const uint32_t *__restrict__ val, int64_t n, int64_t L, const uint32_t *__restrict__ open,
    const uint32_t *__restrict__ hoff, const uint32_t *__restrict__ inv_leaf,
    const uint32_t *__restrict__ inv_mid, uint2 *__restrict__ st) {
    tile_walk(c, n, open[blockIdx.x], hoff[blockIdx.x],
              [&](int64_t e, bool h, bool r, uint32_t before) {
                  const uint32_t pos = (uint32_t)e + before + (h ? 1u : 0u);
                  if ((int64_t)pos >= L) return;  // never when the scan is consistent
                  if (h) {
                      const uint32_t m = c.mid(e);
                      st[pos - 1] = make_uint2(kHdrBit | (r ? kRootBit : 0u) |
                                                   (inv_mid ? inv_mid[m] : m),
                                               c.root(e));
                  }
                  const uint32_t l = c.leaf(e);
                  st[pos] = make_uint2(inv_leaf ? inv_leaf[l] : l, val[e]);
              });
}

// the keys that count_rows sorts: every leaf index / every header's mid index
template <class C>
__global__ void k_leaf_keys(C c, int64_t n, uint64_t *__restrict__ key,
                            uint32_t *__restrict__ val) {
    GRID_STRIDE(e, n) {
        key[e] = c.leaf(e);
        val[e] = 0u;
    }
}
template <class C>
__global__ __launch_bounds__(kThreads) void k_mid_keys(C c, int64_t n, int64_t nhdr,
                                                       const uint32_t *__restrict__ open,
                                                       const uint32_t *__restrict__ hoff,
                                                       uint64_t *__restrict__ key,
                                                       uint32_t *__restrict__ val) {
    tile_walk(c, n, open[blockIdx.x], hoff[blockIdx.x],
              [&](int64_t e, bool h, bool, uint32_t before) {
                  if (!h || (int64_t)before >= nhdr) return;
                  key[before] = c.mid(e);
                  val[before] = 0u;
              });
}

// Gathers per row: every nonzero gathers its leaf row, every header (fiber
// start or segment start) its mid row.  Skewed indices put millions of
// counts on a few rows, so the counts are not accumulated with atomics (they
// serialize on those rows' addresses): the gathered indices are radix-sorted
// and each row's count is the length of its run.
// [beg[r], end[r]) = the run of row r in the sorted keys (rows absent from
// the keys keep the zeros they were filled with)
__global__ void k_run_bounds(const uint64_t *__restrict__ key, int64_t n,
                             uint32_t *__restrict__ beg, uint32_t *__restrict__ end) {
    GRID_STRIDE(e, n) {
        const uint64_t k = key[e];
        if (e == 0 || key[e - 1] != k) beg[k] = (uint32_t)e;
        if (e == n - 1 || key[e + 1] != k) end[k] = (uint32_t)(e + 1);
    }
}

__global__ void k_run_lengths(const uint32_t *__restrict__ beg, const uint32_t *__restrict__ end,
                              int64_t rows, uint32_t *__restrict__ cnt) {
    GRID_STRIDE(r, rows) cnt[r] = end[r] - beg[r];
}

// sort key: count descending (a stable sort keeps equal counts in index order)
__global__ void k_count_keys(const uint32_t *__restrict__ cnt, int64_t n,
                             uint64_t *__restrict__ key, uint32_t *__restrict__ idx) {
    GRID_STRIDE(e, n) {
        key[e] = (uint64_t)(0xFFFFFFFFu - cnt[e]);
        idx[e] = (uint32_t)e;
    }
}

__global__ void k_invert(const uint32_t *__restrict__ perm, int64_t n, uint32_t *__restrict__ inv) {
    GRID_STRIDE(e, n) inv[perm[e]] = (uint32_t)e;
}

__global__ void k_fill_pad(uint2 *__restrict__ st, int64_t from, int64_t count) {
    GRID_STRIDE(e, count) st[from + e] = make_uint2(kHdrBit | kRootBit, 0u);
}

__global__ void k_fill_u32(uint32_t *__restrict__ p, int64_t n, uint32_t v) {
    GRID_STRIDE(e, n) p[e] = v;
}

__global__ void k_compact_rows(const uint32_t *__restrict__ mark, const uint32_t *__restrict__ pos,
                               int64_t n, uint32_t *__restrict__ out) {
    GRID_STRIDE(e, n) {
        if (mark[e]) out[pos[e]] = (uint32_t)e;
    }
}

// chunk c starts at the first header at or after c * len (or at the end): a
// wave looks at 64 entries at a time (a header comes every kFiberCap + 1 at
// least).  heads[c]: that entry (a chunk at the end counts as opening a row).
__global__ void k_chunk_starts(const uint2 *__restrict__ st, int64_t nentry, int64_t nchunk,
                               int len, uint32_t *__restrict__ cs, uint2 *__restrict__ heads) {
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t c = blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6); c <= nchunk;
         c += waves) {
        int64_t p = c == nchunk ? nentry : c * (int64_t)len;
        uint2 h = make_uint2(kHdrBit | kRootBit, 0u);
        while (p < nentry) {
            const uint2 w = p + lane < nentry ? st[p + lane] : make_uint2(0u, 0u);
            const uint64_t m = __ballot((w.x & kHdrBit) != 0u);
            if (m) {
                const int l = __ffsll((unsigned long long)m) - 1;
                p += l;
                h = make_uint2((uint32_t)__shfl((int)w.x, l), (uint32_t)__shfl((int)w.y, l));
                break;
            }
            p += 64;
        }
        if (p > nentry) p = nentry;
        if (lane == 0) {
            cs[c] = (uint32_t)p;
            heads[c] = h;
        }
    }
}

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------

// Transient build buffers, stream-ordered (from the context's memory
// source, freed on the build stream), so building one tensor never waits for
// unrelated work on the device.
struct Scratch {
    hipStream_t s;
    DevMem mem;
    std::vector<void *> ptrs;
    Scratch(hipStream_t st, const DevMem &m) : s(st), mem(m) {}
    ~Scratch() {
        for (void *p : ptrs) mem.free(p, s);
    }
    template <typename T>
    T *alloc(int64_t n) {
        void *p = nullptr;
        const size_t bytes = sizeof(T) * (size_t)std::max<int64_t>(n, 1);
        if (mem.arena && (p = mem.arena->take(bytes))) return (T *)p;  // freed with the arena
        if (mem.alloc(&p, bytes, s) != hipSuccess) {
            (void)hipGetLastError();
            throw Error{DFACTO_E_NOMEM, "device allocation of " + std::to_string(bytes) +
                                            " bytes failed while building the flattenings"};
        }
        ptrs.push_back(p);
        return (T *)p;
    }
    void release(void *p) {
        for (auto &q : ptrs)
            if (q == p) {
                mem.free(q, s);
                q = nullptr;
            }
    }
};

// Tensor memory.  Once the counts are known a build reserves all that the
// flattenings take as one allocation (tensor_reserve) and carves the arrays
// from it; other arrays up to kSlabTake bytes share slabs of kSlabBytes.
constexpr size_t kSlabTake = (size_t)256 << 10, kSlabBytes = (size_t)1 << 20;

size_t tensor_round(size_t bytes) {
    return (std::max<size_t>(bytes, 1) + 255) & ~(size_t)255;
}

void *tensor_raw(dfacto_tensor *t, size_t bytes) {
    void *p = nullptr;
    const hipError_t e =
        t->alloc_stream ? t->mem.alloc(&p, bytes, t->alloc_stream) : hipMalloc(&p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        throw Error{DFACTO_E_NOMEM, "device allocation of " + std::to_string(bytes) +
                                        " bytes failed for the flattenings"};
    }
    t->allocations.push_back(p);
    t->bytes += bytes;
    return p;
}

void tensor_reserve(dfacto_tensor *t, size_t bytes) {
    t->slab = (char *)tensor_raw(t, bytes);
    t->slab_left = bytes;
}

void *tensor_alloc_bytes(dfacto_tensor *t, size_t bytes) {
    bytes = tensor_round(bytes);
    if (bytes > t->slab_left) {
        if (bytes > kSlabTake) return tensor_raw(t, bytes);
        tensor_reserve(t, kSlabBytes);
    }
    void *p = t->slab;
    t->slab += bytes;
    t->slab_left -= bytes;
    return p;
}

template <typename T>
T *tensor_alloc(dfacto_tensor *t, int64_t n) {
    return (T *)tensor_alloc_bytes(t, sizeof(T) * (size_t)std::max<int64_t>(n, 1));
}

template <class Op>
void scan_exclusive(const uint32_t *in, uint32_t *out, int64_t n, hipStream_t s,
                    const DevMem *mem) {
    if (n <= 0) return;
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb == 1) {
        hipLaunchKernelGGL(k_scan_apply<Op>, dim3(1), dim3(kThreads), 0, s, in, out, n,
                           (const uint32_t *)nullptr);
        return;
    }
    Scratch sc(s, mem ? *mem : DevMem{});
    uint32_t *bsum = sc.alloc<uint32_t>(nb), *boff = sc.alloc<uint32_t>(nb);
    hipLaunchKernelGGL(k_scan_reduce<Op>, dim3((unsigned)nb), dim3(kThreads), 0, s, in, n, bsum);
    scan_exclusive<Op>(bsum, boff, nb, s, &sc.mem);
    hipLaunchKernelGGL(k_scan_apply<Op>, dim3((unsigned)nb), dim3(kThreads), 0, s, in, out, n,
                       (const uint32_t *)boff);
}

// Pairs by the key bits [lo, hi): `from` (kept) if given, else (keys, vals),
// into (keys, vals) by way of (kalt, valt).
struct PairBuf {
    uint64_t *key = nullptr;
    uint32_t *val = nullptr;
};
void radix_sort(PairBuf &ab, PairBuf &alt, int64_t n, int lo, int hi, Scratch &sc, hipStream_t s,
                const PairBuf *from = nullptr) {
    const int bits = n <= 1 ? 0 : hi - lo, passes = (bits + 7) / 8;
    if (passes == 0) {
        if (from) {
            DF_HIP(hipMemcpyAsync(ab.key, from->key, sizeof(uint64_t) * (size_t)n,
                                  hipMemcpyDeviceToDevice, s));
            DF_HIP(hipMemcpyAsync(ab.val, from->val, sizeof(uint32_t) * (size_t)n,
                                  hipMemcpyDeviceToDevice, s));
        }
        return;
    }
    const int64_t nblk = (n + kRadixTile - 1) / kRadixTile;
    uint32_t *hist = sc.alloc<uint32_t>(256 * nblk);
    uint32_t *offs = sc.alloc<uint32_t>(256 * nblk);
    int shift = lo;
    for (int p = 0; p < passes; ++p) {
        const int b = (hi - shift + passes - p - 1) / (passes - p);  // digits of even width
        const PairBuf src = p == 0 && from ? *from : ab;
        const PairBuf dst = p == 0 && from ? ab : alt;
        const uint32_t dmask = (1u << b) - 1u;
        hipLaunchKernelGGL(k_radix_hist, dim3((unsigned)nblk), dim3(kThreads), 0, s, src.key, n,
                           shift, dmask, hist, nblk, nblk <= kRadixOwnMax);
        if (nblk <= kRadixOwnMax) {
            hipLaunchKernelGGL(k_radix_scatter<true>, dim3((unsigned)nblk), dim3(kThreads), 0, s,
                               src.key, src.val, dst.key, dst.val, n, shift, b, hist, nblk);
        } else {
            scan_exclusive<ScanSum>(hist, offs, ((int64_t)dmask + 1) * nblk, s, &sc.mem);
            hipLaunchKernelGGL(k_radix_scatter<false>, dim3((unsigned)nblk), dim3(kThreads), 0, s,
                               src.key, src.val, dst.key, dst.val, n, shift, b, offs, nblk);
        }
        if (!(p == 0 && from)) std::swap(ab, alt);
        shift += b;
    }
    DF_LAUNCHED();
    sc.release(hist);
    sc.release(offs);
}

void radix_sort(uint64_t *&keys, uint32_t *&vals, uint64_t *&kalt, uint32_t *&valt, int64_t n,
                int bits, Scratch &sc, hipStream_t s) {
    PairBuf a{keys, vals}, b{kalt, valt};
    radix_sort(a, b, n, 0, bits, sc, s);
    keys = a.key, vals = a.val, kalt = b.key, valt = b.val;
}

// Rows split across chunks: a maximal sequence of chunks whose first header
// continues the same row (no ROOT bit) forms one run of carries, (row, first
// chunk, chunks).  One block per mode walks the chunks 1024 at a time; the
// chunk that ends a sequence (its head opens a row, or continues another one)
// writes the run before it, at its place in chunk order.  The next 1024 heads
// are loaded a step ahead.
struct RunJob {
    const uint2 *heads;
    uint32_t nchunk;
    uint32_t *shortr, *longr, *count;  // count: short runs, long runs
};
constexpr int kRunBlock = 1024;

__global__ __launch_bounds__(kRunBlock) void k_runs(const RunJob j0, const RunJob j1,
                                                    const RunJob j2) {
    const RunJob &j = blockIdx.x == 0 ? j0 : blockIdx.x == 1 ? j1 : j2;
    __shared__ uint32_t s_pos[kRunBlock / 64], s_ns[kRunBlock / 64], s_nl[kRunBlock / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint2 none = make_uint2(kHdrBit | kRootBit, 0u);
    auto head = [&](uint32_t c) { return c < j.nchunk ? j.heads[c] : none; };
    uint32_t open = 0, ns = 0, nl = 0;  // 1 + the last sequence start so far; runs written
    uint2 hn = head(tid), gn = tid ? head(tid - 1) : none;  // this chunk's head, the one before
    for (uint32_t base = 0; base <= j.nchunk; base += kRunBlock) {
        const uint32_t c = base + tid;
        bool ends = false;
        const uint2 hc = hn, gc = gn;
        hn = head(c + kRunBlock);
        gn = head(c + kRunBlock - 1);
        if (c < j.nchunk)
            ends = c == 0 || (hc.x & kRootBit) || (gc.x & kRootBit) || gc.y != hc.y;
        else
            ends = c == j.nchunk;
        const uint64_t m = __ballot(ends), below = m & ~(~0ull << lane);
        if (lane == 0) s_pos[wave] = m ? c + 64u - (uint32_t)__clzll((long long)m) : 0u;
        __syncthreads();
        uint32_t prev = open;
        for (int w = 0; w < wave; ++w) prev = s_pos[w] ? s_pos[w] : prev;
        if (below) prev = c - (uint32_t)lane + 64u - (uint32_t)__clzll((long long)below);
        for (int w = 0; w < kRunBlock / 64; ++w) open = s_pos[w] ? s_pos[w] : open;
        // the sequence [prev - 1, c) ends here: a run if its head continues a row
        uint32_t row = 0, n = 0;
        if (ends && prev) {
            const uint2 h = head(prev - 1);
            if (!(h.x & kRootBit)) row = h.y, n = c - (prev - 1);
        }
        const uint64_t bs = __ballot(n > 0 && n <= (uint32_t)kShortRun),
                       bl = __ballot(n > (uint32_t)kShortRun);
        if (lane == 0) {
            s_ns[wave] = (uint32_t)__popcll(bs);
            s_nl[wave] = (uint32_t)__popcll(bl);
        }
        __syncthreads();
        uint32_t at_s = ns, at_l = nl;
        for (int w = 0; w < kRunBlock / 64; ++w) {
            if (w < wave) at_s += s_ns[w], at_l += s_nl[w];
            ns += s_ns[w], nl += s_nl[w];
        }
        if (n > 0) {
            const bool sh = n <= (uint32_t)kShortRun;
            const uint32_t q = (sh ? at_s : at_l) +
                               (uint32_t)__popcll((sh ? bs : bl) & ~(~0ull << lane));
            uint32_t *o = (sh ? j.shortr : j.longr) + 3 * (size_t)q;
            o[0] = row;
            o[1] = prev - 1;
            o[2] = n;
        }
        __syncthreads();  // s_pos, s_ns, s_nl are free again
    }
    if (tid == 0) {
        j.count[0] = ns;
        j.count[1] = nl;
    }
}

// most runs of each kind among n chunks
int64_t most_short(int64_t n) { return n; }
int64_t most_long(int64_t n) { return n / (kShortRun + 1) + 1; }

// cnt[r] = occurrences of row r < rows among the m indices that fill(key,
// val) writes as sort keys
template <class Fill>
void count_rows(int64_t m, int64_t rows, uint32_t *cnt, Scratch &sc, hipStream_t s, Fill &&fill) {
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(rows)), dim3(kThreads), 0, s, cnt, rows, 0u);
    DF_LAUNCHED();
    if (m == 0) return;
    uint64_t *key = sc.alloc<uint64_t>(m), *kalt = sc.alloc<uint64_t>(m);
    uint32_t *val = sc.alloc<uint32_t>(m), *valt = sc.alloc<uint32_t>(m);
    fill(key, val);
    DF_LAUNCHED();
    radix_sort(key, val, kalt, valt, m, bits_for(rows), sc, s);
    uint32_t *beg = sc.alloc<uint32_t>(rows), *end = sc.alloc<uint32_t>(rows);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(rows)), dim3(kThreads), 0, s, beg, rows, 0u);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(rows)), dim3(kThreads), 0, s, end, rows, 0u);
    hipLaunchKernelGGL(k_run_bounds, dim3(grid_for(m)), dim3(kThreads), 0, s, key, m, beg, end);
    hipLaunchKernelGGL(k_run_lengths, dim3(grid_for(rows)), dim3(kThreads), 0, s, beg, end, rows,
                       cnt);
    DF_LAUNCHED();
    sc.release(end);
    sc.release(beg);
    sc.release(valt);
    sc.release(val);
    sc.release(kalt);
    sc.release(key);
}

// The order of a gathered table's rows by decreasing gather count (ties by
// index): perm[r] = the row ranked r (tensor memory).
uint32_t *relabel_order(dfacto_tensor *t, const uint32_t *cnt, int64_t rows, Scratch &sc,
                        hipStream_t s) {
    uint64_t *key = sc.alloc<uint64_t>(rows), *kalt = sc.alloc<uint64_t>(rows);
    uint32_t *idx = sc.alloc<uint32_t>(rows), *ialt = sc.alloc<uint32_t>(rows);
    hipLaunchKernelGGL(k_count_keys, dim3(grid_for(rows)), dim3(kThreads), 0, s, cnt, rows, key,
                       idx);
    DF_LAUNCHED();
    radix_sort(key, idx, kalt, ialt, rows, 32, sc, s);
    uint32_t *perm = tensor_alloc<uint32_t>(t, rows);
    DF_HIP(hipMemcpyAsync(perm, idx, sizeof(uint32_t) * (size_t)rows, hipMemcpyDeviceToDevice, s));
    return perm;
}

// What the counting passes leave for a mode's stream: per tile the open fiber
// and the headers before it, per row the empty-row mark and its scan.
struct ModeCount {
    uint32_t *open = nullptr, *hoff = nullptr, *nfib = nullptr, *fib_off = nullptr,
             *nhdr = nullptr, *mark = nullptr, *rpos = nullptr;
    int64_t fibers = 0, headers = 0, empty = 0;
};

// Enqueue a mode's counting passes over its n > 0 nonzeros c (in root, mid,
// leaf order).
template <class C>
ModeCount count_mode(int64_t nrows, const C &c, int64_t n, Scratch &sc, hipStream_t s) {
    const int64_t nt = (n + kTile - 1) / kTile;
    const dim3 grid((unsigned)nt), block(kThreads);
    ModeCount k;
    uint32_t *last = sc.alloc<uint32_t>(nt);
    k.nfib = sc.alloc<uint32_t>(nt);
    k.fib_off = sc.alloc<uint32_t>(nt);
    k.open = sc.alloc<uint32_t>(nt);
    k.nhdr = sc.alloc<uint32_t>(nt);
    k.hoff = sc.alloc<uint32_t>(nt);
    k.mark = sc.alloc<uint32_t>(nrows);
    k.rpos = sc.alloc<uint32_t>(nrows);
    hipLaunchKernelGGL(k_tile_fibers<C>, grid, block, 0, s, c, n, k.nfib, last);
    scan_exclusive<ScanMax>(last, k.open, nt, s, &sc.mem);
    scan_exclusive<ScanSum>(k.nfib, k.fib_off, nt, s, &sc.mem);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nrows)), block, 0, s, k.mark, nrows, 1u);
    hipLaunchKernelGGL(k_tile_headers<C>, grid, block, 0, s, c, n, nrows, k.open, k.nhdr, k.mark);
    scan_exclusive<ScanSum>(k.nhdr, k.hoff, nt, s, &sc.mem);
    scan_exclusive<ScanSum>(k.mark, k.rpos, nrows, s, &sc.mem);
    DF_LAUNCHED();
    return k;
}

// out[q] = *a[q] + *b[q] (b null: *a[q]): totals of scans and flags gathered
// for one copy to the host (each copy costs the host 20 us)
constexpr int kMostTotals = 9;
struct Totals {
    const uint32_t *a[kMostTotals], *b[kMostTotals];
};
__global__ void k_totals(const Totals t, int n, uint32_t *__restrict__ out) {
    const int q = threadIdx.x;
    if (q < n) out[q] = *t.a[q] + (t.b[q] ? *t.b[q] : 0u);
}
void read_totals(const Totals &t, int n, uint32_t *h, Scratch &sc, hipStream_t s) {
    uint32_t *out = sc.alloc<uint32_t>(kMostTotals);
    hipLaunchKernelGGL(k_totals, dim3(1), dim3(64), 0, s, t, n, out);
    DF_LAUNCHED();
    DF_HIP(hipMemcpyAsync(h, out, sizeof(uint32_t) * n, hipMemcpyDeviceToHost, s));
    DF_HIP(hipStreamSynchronize(s));
}

// A mode of an empty tensor.
void empty_mode(dfacto_ctx *ctx, dfacto_tensor *t, int m) {
    hipStream_t s = ctx->stream;
    ModeData &md = t->mode[m];
    const int64_t nrows = t->dims[md.root];
    Scratch sc(s, ctx->mem);
    md.chunk_len = t->chunk_len;
    md.nentry = 0;
    md.nfib = md.nroot = 0;
    md.stream = tensor_alloc<uint2>(t, kStreamPad);
    hipLaunchKernelGGL(k_fill_pad, dim3(1), dim3(kThreads), 0, s, md.stream, (int64_t)0,
                       (int64_t)kStreamPad);
    md.nchunk = 0;
    md.chunk_start = tensor_alloc<uint32_t>(t, 1);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(kThreads), 0, s, md.chunk_start, (int64_t)1, 0u);
    md.nempty = nrows;
    md.empty_rows = tensor_alloc<uint32_t>(t, nrows);
    uint32_t *mark = sc.alloc<uint32_t>(nrows);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nrows)), dim3(kThreads), 0, s, mark, nrows, 1u);
    uint32_t *pos = sc.alloc<uint32_t>(nrows);
    scan_exclusive_u32(mark, pos, nrows, s, &sc.mem);
    hipLaunchKernelGGL(k_compact_rows, dim3(grid_for(nrows)), dim3(kThreads), 0, s, mark, pos,
                       nrows, md.empty_rows);
    DF_LAUNCHED();
    DF_HIP(hipStreamSynchronize(s));
}

// The sizes of mode m's flattening from its counts; returns the bytes of its
// arrays (those that emit_mode allocates).
size_t size_mode(dfacto_tensor *t, int m, int64_t n, const ModeCount &k) {
    ModeData &md = t->mode[m];
    md.chunk_len = t->chunk_len;
    md.nfib = k.fibers;
    md.nempty = k.empty;
    md.nroot = t->dims[md.root] - md.nempty;
    md.nentry = n + k.headers;
    if (md.nentry > (int64_t)0xFFFFFFFFu - (1 << 20))
        throw Error{DFACTO_E_UNSUPPORTED, "nonzeros plus fiber headers exceed 2^32 - 2^20"};
    md.nchunk = (md.nentry + md.chunk_len - 1) / md.chunk_len;
    size_t b = tensor_round(sizeof(uint2) * (size_t)(md.nentry + kStreamPad)) +
               tensor_round(sizeof(uint32_t) * (size_t)md.nempty) +
               tensor_round(sizeof(uint32_t) * (size_t)(md.nchunk + 1)) +
               tensor_round(sizeof(uint32_t) * 3 * (size_t)most_short(md.nchunk)) +
               tensor_round(sizeof(uint32_t) * 3 * (size_t)most_long(md.nchunk));
    if (t->relabel)
        b += tensor_round(sizeof(uint32_t) * (size_t)t->dims[md.leaf]) +
             tensor_round(sizeof(uint32_t) * (size_t)t->dims[md.mid]);
    return b;
}

// Mode m's flattening from its nonzeros (c, val), their counts and size_mode's
// sizes; heads: its chunks' first headers (nchunk + 1), from which finish_runs
// forms the run lists.
template <class C>
void emit_mode(dfacto_ctx *ctx, dfacto_tensor *t, int m, const C &c, const uint32_t *val,
               int64_t n, const ModeCount &k, uint2 *heads, Scratch &sc) {
    hipStream_t s = ctx->stream;
    ModeData &md = t->mode[m];
    const int64_t nrows = t->dims[md.root], nhdr = k.headers, L = md.nentry;
    const dim3 tiles((unsigned)((n + kTile - 1) / kTile));
    // relabeled gathers: ranks by decreasing gather count per gathered table
    const uint32_t *inv_leaf = nullptr, *inv_mid = nullptr;
    if (t->relabel) {
        const int64_t dl = t->dims[md.leaf], dm = t->dims[md.mid];
        uint32_t *cl = sc.alloc<uint32_t>(dl), *cm = sc.alloc<uint32_t>(dm);
        count_rows(n, dl, cl, sc, s, [&](uint64_t *key, uint32_t *kv) {
            hipLaunchKernelGGL(k_leaf_keys<C>, dim3(grid_for(n)), dim3(kThreads), 0, s, c, n, key,
                               kv);
        });
        count_rows(nhdr, dm, cm, sc, s, [&](uint64_t *key, uint32_t *kv) {
            hipLaunchKernelGGL(k_mid_keys<C>, tiles, dim3(kThreads), 0, s, c, n, nhdr, k.open,
                               k.hoff, key, kv);
        });
        md.perm_leaf = relabel_order(t, cl, dl, sc, s);
        md.perm_mid = relabel_order(t, cm, dm, sc, s);
        uint32_t *il = sc.alloc<uint32_t>(dl), *im = sc.alloc<uint32_t>(dm);
        hipLaunchKernelGGL(k_invert, dim3(grid_for(dl)), dim3(kThreads), 0, s, md.perm_leaf, dl, il);
        hipLaunchKernelGGL(k_invert, dim3(grid_for(dm)), dim3(kThreads), 0, s, md.perm_mid, dm, im);
        DF_LAUNCHED();
        inv_leaf = il;
        inv_mid = im;
    }
    md.stream = tensor_alloc<uint2>(t, L + kStreamPad);
    hipLaunchKernelGGL(k_emit_stream<C>, tiles, dim3(kThreads), 0, s, c, val, n, L, k.open, k.hoff,
                       inv_leaf, inv_mid, md.stream);
    hipLaunchKernelGGL(k_fill_pad, dim3(1), dim3(kThreads), 0, s, md.stream, L,
                       (int64_t)kStreamPad);
    md.empty_rows = tensor_alloc<uint32_t>(t, md.nempty);
    hipLaunchKernelGGL(k_compact_rows, dim3(grid_for(nrows)), dim3(kThreads), 0, s, k.mark, k.rpos,
                       nrows, md.empty_rows);
    // work chunks
    md.chunk_start = tensor_alloc<uint32_t>(t, md.nchunk + 1);
    hipLaunchKernelGGL(k_chunk_starts, dim3(grid_for(md.nchunk + 1, kThreads / 64)),
                       dim3(kThreads), 0, s, md.stream, L, md.nchunk, md.chunk_len,
                       md.chunk_start, heads);
    DF_LAUNCHED();
}

// The run lists of all three modes (n > 0); waits.
void finish_runs(dfacto_tensor *t, uint2 *const (&heads)[3], Scratch &sc, hipStream_t s) {
    uint32_t *count = sc.alloc<uint32_t>(6);
    RunJob j[3];
    for (int m = 0; m < 3; ++m) {
        ModeData &md = t->mode[m];
        md.runs_short = tensor_alloc<uint32_t>(t, 3 * most_short(md.nchunk));
        md.runs_long = tensor_alloc<uint32_t>(t, 3 * most_long(md.nchunk));
        j[m] = {heads[m], (uint32_t)md.nchunk, md.runs_short, md.runs_long, count + 2 * m};
    }
    hipLaunchKernelGGL(k_runs, dim3(3), dim3(kRunBlock), 0, s, j[0], j[1], j[2]);
    DF_LAUNCHED();
    uint32_t h[6];
    DF_HIP(hipMemcpyAsync(h, count, sizeof(h), hipMemcpyDeviceToHost, s));
    DF_HIP(hipStreamSynchronize(s));  // and ||X||^2
    for (int m = 0; m < 3; ++m) {
        t->mode[m].nruns_short = h[2 * m];
        t->mode[m].nruns_long = h[2 * m + 1];
    }
}

// 1 where a stream entry opens an output row (a ROOT header)
__global__ void k_root_flags(const uint2 *__restrict__ st, int64_t n, uint32_t *__restrict__ f) {
    GRID_STRIDE(e, n) f[e] = ((st[e].x & (kHdrBit | kRootBit)) == (kHdrBit | kRootBit)) ? 1u : 0u;
}

// the q-th row opening of the stream at pos[q] covers [pos[q], pos[q+1])
__global__ void k_row_ranges(const uint2 *__restrict__ st, const uint32_t *__restrict__ flag,
                             const uint32_t *__restrict__ off, int64_t n, uint32_t *__restrict__ pos) {
    GRID_STRIDE(e, n) if (flag[e]) pos[off[e]] = (uint32_t)e;
}

__global__ void k_store_ranges(const uint2 *__restrict__ st, const uint32_t *__restrict__ pos,
                               int64_t nroot, int64_t n, uint2 *__restrict__ range) {
    GRID_STRIDE(q, nroot) {
        const uint32_t b = pos[q];
        const uint32_t e = (q + 1 < nroot) ? pos[q + 1] : (uint32_t)n;
        range[st[b].y] = make_uint2(b, e);
    }
}

}  // namespace

void scan_exclusive_u32(const uint32_t *in, uint32_t *out, int64_t n, hipStream_t s,
                        const DevMem *mem) {
    scan_exclusive<ScanSum>(in, out, n, s, mem);
}

void build_row_ranges(dfacto_ctx *ctx, dfacto_tensor *t) {
    hipStream_t s = ctx->stream;
    Scratch sc(s, ctx->mem);
    for (int m = 0; m < 2; ++m) {
        const ModeData &md = t->mode[m];
        const int64_t rows = t->dims[md.root], n = md.nentry;
        uint2 *range = tensor_alloc<uint2>(t, rows);
        DF_HIP(hipMemsetAsync(range, 0, sizeof(uint2) * (size_t)rows, s));
        if (n > 0 && md.nroot > 0) {
            uint32_t *flag = sc.alloc<uint32_t>(n), *off = sc.alloc<uint32_t>(n);
            uint32_t *pos = sc.alloc<uint32_t>(md.nroot);
            hipLaunchKernelGGL(k_root_flags, dim3(grid_for(n)), dim3(kThreads), 0, s, md.stream, n,
                               flag);
            scan_exclusive_u32(flag, off, n, s, &sc.mem);
            hipLaunchKernelGGL(k_row_ranges, dim3(grid_for(n)), dim3(kThreads), 0, s, md.stream,
                               flag, off, n, pos);
            hipLaunchKernelGGL(k_store_ranges, dim3(grid_for(md.nroot)), dim3(kThreads), 0, s,
                               md.stream, pos, md.nroot, n, range);
            DF_LAUNCHED();
        }
        t->row_range[m] = range;
    }
    // rows longer than kJointLight entries become at most kJointMaxSegs
    // segments of kJointSeg entries or more
    std::vector<uint2> hr, seg[2];
    std::vector<uint4> heavy[2];
    for (int m = 0; m < 2; ++m) {
        const int64_t rows = t->dims[t->mode[m].root];
        hr.resize((size_t)rows);
        DF_HIP(hipMemcpyAsync(hr.data(), t->row_range[m], sizeof(uint2) * (size_t)rows,
                              hipMemcpyDeviceToHost, s));
        DF_HIP(hipStreamSynchronize(s));
        for (int64_t r = 0; r < rows; ++r) {
            const uint32_t b = hr[r].x, e = hr[r].y;
            if (e - b <= (uint32_t)kJointLight) continue;
            const uint32_t len = std::max<uint32_t>(
                kJointSeg, (e - b + kJointMaxSegs - 1) / kJointMaxSegs);
            const uint32_t first = (uint32_t)seg[m].size(), n = (e - b + len - 1) / len;
            if (t->batch[m].empty() || first + n - t->batch[m].back().second > kJointBatch)
                t->batch[m].push_back({(int64_t)heavy[m].size(), (int64_t)first});
            t->batch_segs = std::max<int64_t>(t->batch_segs, first + n - t->batch[m].back().second);
            heavy[m].push_back(make_uint4((uint32_t)r, first, n, 0u));
            for (uint32_t x = 0; x < n; ++x)
                seg[m].push_back(make_uint2(b + x * len, x + 1 < n ? b + (x + 1) * len : e));
        }
        t->nseg[m] = (int64_t)seg[m].size();
        t->nheavy[m] = (int64_t)heavy[m].size();
        t->batch[m].push_back({t->nheavy[m], t->nseg[m]});
        t->seg_range[m] = tensor_alloc<uint2>(t, t->nseg[m]);
        t->heavy[m] = tensor_alloc<uint4>(t, t->nheavy[m]);
        if (t->nseg[m] > 0) {
            DF_HIP(hipMemcpyAsync(t->seg_range[m], seg[m].data(), sizeof(uint2) * seg[m].size(),
                                  hipMemcpyHostToDevice, s));
            DF_HIP(hipMemcpyAsync(t->heavy[m], heavy[m].data(), sizeof(uint4) * heavy[m].size(),
                                  hipMemcpyHostToDevice, s));
        }
    }
    DF_HIP(hipStreamSynchronize(s));
}

namespace {

// ||X||^2 in FP64, fixed reduction order (lands when the build next waits)
void start_normsq(dfacto_tensor *t, const float *v, int64_t n, Scratch &sc, hipStream_t s) {
    const unsigned nb = std::min<unsigned>(grid_for(n), 1024u);
    double *part = sc.alloc<double>(nb), *tot = sc.alloc<double>(1);
    hipLaunchKernelGGL(k_sumsq_partial, dim3(nb), dim3(kThreads), 0, s, v, n, part);
    hipLaunchKernelGGL(k_sum_f64_final, dim3(1), dim3(kThreads), 0, s, part, (int)nb, tot);
    DF_LAUNCHED();
    DF_HIP(hipMemcpyAsync(&t->normsq, tot, sizeof(double), hipMemcpyDeviceToHost, s));
}

// The distinct coordinates among n sorted ones, and their first places per
// tile (*off); throws for bad input (*flag, from the check), waits.
template <class C>
int64_t count_distinct(const C &c, int64_t n, const uint32_t *flag, uint32_t **off, Scratch &sc,
                       hipStream_t s) {
    const int64_t nt = (n + kTile - 1) / kTile;
    uint32_t *cnt = sc.alloc<uint32_t>(nt);
    *off = sc.alloc<uint32_t>(nt);
    hipLaunchKernelGGL(k_tile_distinct<C>, dim3((unsigned)nt), dim3(kThreads), 0, s, c, n, cnt);
    scan_exclusive<ScanSum>(cnt, *off, nt, s, &sc.mem);
    DF_LAUNCHED();
    uint32_t h[2];
    read_totals(Totals{{flag, *off + nt - 1}, {nullptr, cnt + nt - 1}}, 2, h, sc, s);
    if (h[0] & 1u) throw Error{DFACTO_E_RANGE, "a coordinate is not below its dimension"};
    if (h[0] & 2u) throw Error{DFACTO_E_NUMERIC, "a tensor value is NaN or Inf"};
    return (int64_t)h[1];
}

// merge the duplicates of n sorted coordinates into nd distinct ones
template <class C, class Store>
void merge(const C &c, const float *v, int64_t n, const uint32_t *off, const Store &store,
           Scratch &sc, hipStream_t s) {
    const int64_t most = n / (kRunShort + 1) + 1;  // runs longer than kRunShort
    uint2 *longs = sc.alloc<uint2>(most);
    uint32_t *nlong = sc.alloc<uint32_t>(1);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(kThreads), 0, s, nlong, (int64_t)1, 0u);
    hipLaunchKernelGGL((k_merge<C, Store>), dim3((unsigned)((n + kTile - 1) / kTile)),
                       dim3(kThreads), 0, s, c, v, n, off, store, longs, nlong);
    hipLaunchKernelGGL((k_merge_long<C, Store>),
                       dim3((unsigned)std::min<int64_t>(most, 4096)), dim3(64), 0, s, c, v, n,
                       store, longs, nlong);
    DF_LAUNCHED();
    sc.release(longs);
}

// one wait for the counts of several modes
void read_counts(dfacto_tensor *t, ModeCount *k, const int *modes, int count, int64_t n,
                 Scratch &sc, hipStream_t s) {
    const int64_t nt = (n + kTile - 1) / kTile;
    Totals w{};
    for (int q = 0; q < count; ++q) {
        const int64_t nrows = t->dims[t->mode[modes[q]].root];
        const uint32_t **a = w.a + 3 * q, **b = w.b + 3 * q;
        a[0] = k[q].fib_off + nt - 1, b[0] = k[q].nfib + nt - 1;
        a[1] = k[q].hoff + nt - 1, b[1] = k[q].nhdr + nt - 1;
        a[2] = k[q].rpos + nrows - 1, b[2] = k[q].mark + nrows - 1;
    }
    uint32_t h[kMostTotals];
    read_totals(w, 3 * count, h, sc, s);
    for (int q = 0; q < count; ++q) {
        k[q].fibers = h[3 * q];
        k[q].headers = h[3 * q + 1];
        k[q].empty = h[3 * q + 2];
    }
}

// indices of at most 64 bits together
void build_packed(dfacto_ctx *ctx, dfacto_tensor *t, const uint32_t *d_i, const uint32_t *d_j,
                  const uint32_t *d_k, const float *d_val, int bI, int bJ, int bK,
                  Scratch &sc, uint2 *(&heads)[3]) {
    hipStream_t s = ctx->stream;
    const int64_t n = t->nnz;
    auto pairs = [&](int64_t m) { return PairBuf{sc.alloc<uint64_t>(m), sc.alloc<uint32_t>(m)}; };
    auto drop = [&](PairBuf &b) {
        sc.release(b.key);
        sc.release(b.val);
        b = PairBuf{};
    };
    uint32_t *flag = sc.alloc<uint32_t>(1);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(kThreads), 0, s, flag, (int64_t)1, 0u);
    PairBuf x[3] = {pairs(n), pairs(n), PairBuf{}};
    hipLaunchKernelGGL(k_pack, dim3(grid_for(n)), dim3(kThreads), 0, s, d_i, d_j, d_k, d_val, n,
                       (uint32_t)t->dims[0], (uint32_t)t->dims[1], (uint32_t)t->dims[2], bK, bJ,
                       x[0].key, x[0].val, flag);
    DF_LAUNCHED();
    radix_sort(x[0], x[1], n, 0, bI + bK + bJ, sc, s);
    auto mask = [](int b) { return (uint32_t)(((uint64_t)1 << b) - 1); };
    const int sh[3] = {bK + bJ, 0, bJ};  // of i, j, k
    const uint32_t mk[3] = {mask(bI), mask(bJ), mask(bK)};
    auto coords = [&](int m, const PairBuf &b) {
        const ModeData &md = t->mode[m];
        return PackedCoords{b.key,       sh[md.root], sh[md.mid], sh[md.leaf],
                            mk[md.root], mk[md.mid],  mk[md.leaf]};
    };
    uint32_t *off;
    const int64_t nd = count_distinct(coords(0, x[0]), n, flag, &off, sc, s);
    if (nd < n) {
        merge(coords(0, x[0]), (const float *)x[0].val, n, off,
              StorePacked{x[0].key, x[1].key, x[1].val}, sc, s);
        std::swap(x[0], x[1]);
    }
    t->nnz = nd;
    start_normsq(t, (const float *)x[0].val, nd, sc, s);
    // x[0]: mode 0's order; mode 1's by j from it, mode 2's by k from mode 1's
    PairBuf alt = pairs(nd);
    ModeCount k[3];
    static const int modes[3] = {0, 1, 2};
    k[0] = count_mode(t->dims[0], coords(0, x[0]), nd, sc, s);
    radix_sort(x[1], alt, nd, 0, bJ, sc, s, &x[0]);
    k[1] = count_mode(t->dims[1], coords(1, x[1]), nd, sc, s);
    x[2] = pairs(nd);
    radix_sort(x[2], alt, nd, bJ, bJ + bK, sc, s, &x[1]);
    drop(alt);
    k[2] = count_mode(t->dims[2], coords(2, x[2]), nd, sc, s);
    read_counts(t, k, modes, 3, nd, sc, s);
    size_t bytes = 0;
    for (int m = 0; m < 3; ++m) bytes += size_mode(t, m, nd, k[m]);
    tensor_reserve(t, bytes);
    for (int m = 0; m < 3; ++m) {
        heads[m] = sc.alloc<uint2>(t->mode[m].nchunk + 1);
        emit_mode(ctx, t, m, coords(m, x[m]), x[m].val, nd, k[m], heads[m], sc);
        drop(x[m]);
    }
}

// indices of more than 64 bits together
void build_arrays(dfacto_ctx *ctx, dfacto_tensor *t, const uint32_t *d_i, const uint32_t *d_j,
                  const uint32_t *d_k, const float *d_val, int bI, int bJ, int bK,
                  Scratch &sc, uint2 *(&heads)[3]) {
    hipStream_t s = ctx->stream;
    const int64_t n = t->nnz;
    // coordinates and values are checked here and the outcome read with the
    // distinct count below: until then only sort keys (any bits) and
    // permutation-indexed copies depend on them
    uint32_t *flag = sc.alloc<uint32_t>(1);
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(kThreads), 0, s, flag, (int64_t)1, 0u);
    hipLaunchKernelGGL(k_validate, dim3(grid_for(n)), dim3(kThreads), 0, s, d_i, d_j, d_k, d_val,
                       n, (uint32_t)t->dims[0], (uint32_t)t->dims[1], (uint32_t)t->dims[2], flag);
    DF_LAUNCHED();
    uint64_t *key = sc.alloc<uint64_t>(n), *kalt = sc.alloc<uint64_t>(n);
    uint32_t *perm = sc.alloc<uint32_t>(n), *palt = sc.alloc<uint32_t>(n);
    hipLaunchKernelGGL(k_iota, dim3(grid_for(n)), dim3(kThreads), 0, s, perm, n);
    // mode-0 order (i, k, j)
    hipLaunchKernelGGL(k_make_key, dim3(grid_for(n)), dim3(kThreads), 0, s, key,
                       (const uint32_t *)nullptr, 0, (const uint32_t *)nullptr, 0, d_j,
                       (const uint32_t *)nullptr, n);
    radix_sort(key, perm, kalt, palt, n, bJ, sc, s);
    hipLaunchKernelGGL(k_make_key, dim3(grid_for(n)), dim3(kThreads), 0, s, key, d_i, bK, d_k, 0,
                       (const uint32_t *)nullptr, (const uint32_t *)perm, n);
    radix_sort(key, perm, kalt, palt, n, bI + bK, sc, s);
    sc.release(key);
    sc.release(kalt);
    // gather into sorted coordinates and merge duplicates
    uint32_t *si = sc.alloc<uint32_t>(n), *sj = sc.alloc<uint32_t>(n), *sk = sc.alloc<uint32_t>(n);
    float *sv = sc.alloc<float>(n);
    hipLaunchKernelGGL(k_gather4, dim3(grid_for(n)), dim3(kThreads), 0, s, perm, n, d_i, d_j, d_k,
                       d_val, si, sj, sk, sv);
    const ArrayCoords sorted{si, sk, sj};
    uint32_t *off;
    const int64_t nd = count_distinct(sorted, n, flag, &off, sc, s);
    uint32_t *di = sc.alloc<uint32_t>(nd), *dj = sc.alloc<uint32_t>(nd), *dk = sc.alloc<uint32_t>(nd);
    float *dv = sc.alloc<float>(nd);
    merge(sorted, sv, n, off, StoreArrays{sorted, di, dk, dj, dv}, sc, s);
    sc.release(si);
    sc.release(sj);
    sc.release(sk);
    sc.release(sv);
    t->nnz = nd;
    start_normsq(t, dv, nd, sc, s);
    // modes 1 and 2: stable sort by (root, mid) from the mode-0 order
    uint64_t *key2 = sc.alloc<uint64_t>(nd), *kalt2 = sc.alloc<uint64_t>(nd);
    uint32_t *p2 = perm, *palt2 = palt;  // n >= nd
    uint32_t *gr = sc.alloc<uint32_t>(nd), *gm = sc.alloc<uint32_t>(nd), *gl = sc.alloc<uint32_t>(nd);
    float *gv = sc.alloc<float>(nd);
    const uint32_t *coord[3] = {di, dj, dk};
    const int bits[3] = {bI, bJ, bK};
    for (int m = 0; m < 3; ++m) {
        const ModeData &md = t->mode[m];
        ArrayCoords c{di, dk, dj};
        const float *v = dv;
        if (m > 0) {
            hipLaunchKernelGGL(k_iota, dim3(grid_for(nd)), dim3(kThreads), 0, s, p2, nd);
            hipLaunchKernelGGL(k_make_key, dim3(grid_for(nd)), dim3(kThreads), 0, s, key2,
                               coord[md.root], bits[md.mid], coord[md.mid], 0,
                               (const uint32_t *)nullptr, (const uint32_t *)nullptr, nd);
            radix_sort(key2, p2, kalt2, palt2, nd, bits[md.root] + bits[md.mid], sc, s);
            hipLaunchKernelGGL(k_gather4, dim3(grid_for(nd)), dim3(kThreads), 0, s, p2, nd,
                               coord[md.root], coord[md.mid], coord[md.leaf], dv, gr, gm, gl, gv);
            DF_LAUNCHED();
            c = ArrayCoords{gr, gm, gl};
            v = gv;
        }
        Scratch scm(s, ctx->mem);
        ModeCount k = count_mode(t->dims[md.root], c, nd, scm, s);
        read_counts(t, &k, &m, 1, nd, scm, s);
        (void)size_mode(t, m, nd, k);
        heads[m] = sc.alloc<uint2>(md.nchunk + 1);
        emit_mode(ctx, t, m, c, (const uint32_t *)v, nd, k, heads[m], scm);
    }
}

}  // namespace

void build_tensor(dfacto_ctx *ctx, dfacto_tensor *t, const uint32_t *d_i, const uint32_t *d_j,
                  const uint32_t *d_k, const float *d_val) {
    hipStream_t s = ctx->stream;
    const int64_t n = t->nnz;
    Scratch sc(s, ctx->mem);
    static const int ROOT[3] = {0, 1, 2}, MID[3] = {2, 0, 1}, LEAF[3] = {1, 2, 0};
    for (int m = 0; m < 3; ++m) {
        t->mode[m].root = ROOT[m];
        t->mode[m].mid = MID[m];
        t->mode[m].leaf = LEAF[m];
    }
    if (n == 0) {
        t->normsq = 0.0;
        for (int m = 0; m < 3; ++m) empty_mode(ctx, t, m);
        return;
    }
    const int bI = bits_for(t->dims[0]), bJ = bits_for(t->dims[1]), bK = bits_for(t->dims[2]);
    uint2 *heads[3];
    if (bI + bJ + bK <= 64) build_packed(ctx, t, d_i, d_j, d_k, d_val, bI, bJ, bK, sc, heads);
    else build_arrays(ctx, t, d_i, d_j, d_k, d_val, bI, bJ, bK, sc, heads);
    finish_runs(t, heads, sc, s);
}

}  // namespace dfacto
