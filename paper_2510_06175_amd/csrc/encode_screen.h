// Nearest-centroid search (Eq. 2) of the tiled cache-fill and K-Means kernels: a matrix-core screen
// followed by the exact comparison.
//
// What is written is, bit for bit, what the plain search writes: the centroid with the smallest
// squared distance, summed directly in fp32 in channel order, lowest index among equals.  The
// matrix cores only tell which centroids can possibly be that one:
//   score(c) = sigma (x . c - |c|^2 / 2)      (largest score <=> smallest distance)
// for the 64 tokens of a tile against 32 centroids at a time, as v_mfma_f32_32x32x16_f16 products:
// rows = 32 centroids, columns = 32 tokens, and along k
//   [ c          | c          | -sigma |c|^2 / 2 as two fp16 parts ]   (A)
//   [ hi(sigma x)| lo(sigma x)| 1 1                               ]   (B)
// (hi + lo: sigma x to 22 bits; the centroids are fp16 already; sigma, a power of two per
// sub-space, keeps the low parts out of the fp16 denormal range).  At d = 8 that is 18 of 16 places:
// the low parts of the last two channels are left out, which costs a wider margin instead of a
// second MFMA.  The screen's error is bounded (below), so every centroid that can win or tie has a
// score within `margin` of the best one.
// A lane keeps, of the 128 scores it sees per token, only the maximum of each accumulator register
// over the 8 blocks of 32 centroids (16 "groups" of 8 centroids): one v_max3_f32 per two scores,
// which is the least that looks at every score.  A score within the margin marks its group, and the
// centroids of the marked groups (normally one group) get the exact distance.  (Keeping the
// maximum of every block as well, so that a mark names one centroid, costs as many v_max3_f32 again;
// going over the 8 centroids of a group costs half of that.)
//
// What bounds it: vector-ALU instructions.  Per wavefront, sub-space and tile 128 + 16 for the maxima,
// 64 for the marks, about 110 per round of exact distances, 50 for operands and the rest.
// 65536 tokens x 8 heads, d = 4, keys / values: 459 / 398 us with block maxima, 338 / 276 us without;
// both in turn 604 us, 540 us with four wavefronts per SIMD instead of two;
// 10007 tokens x 8 heads, d = 8, 12-bit codes: 511 / 498 us, 236 / 203 us (one MFMA per block, marks
// once per search instead of once per 256 centroids).
//
// Error bound, in score units (T = sum_j |x_j| max|c_j| + max|c|^2 / 2 bounds the sum of the
// magnitudes of a score's terms), per score:
//   split of sigma x                                                        <= 2^-22 sigma T
//   fp32 |c|^2 (d roundings) and its two parts                  <= (d 2^-24 + 2^-22) sigma T
//   fp32 accumulation of n products (n = 2 d + 2, 16 at d = 8), every addition
//   taken as truncating                                                 <= n 2^-23 sigma T
//   fp16 parts below 2^-14 taken as flushed to zero: <= 2^-14 (d max|c_j| + 3), whatever sigma
//   d = 8: the low parts left out,                     <= (|lo_6| + |lo_7|) max|c_j|
// Two scores are compared, so twice that.  The exact distances themselves carry (d + 2) 2^-24
// relative rounding each: a centroid is safely worse when its true distance exceeds the best's, D, by
// 2 (d + 2) 2^-24 D, i.e. its score lies (d + 2) 2^-24 sigma D below; sigma D = sigma |x|^2 - 2 best.
// (5 % are added to cover the margin's own rounding and what the screen's error does to D.)
// A token whose scaled sub-vector leaves the fp16 range (or holds an infinity or a NaN) has no
// finite best score; a codebook whose |c|^2 does not fit, or that holds an infinity or a NaN, gets
// a NaN sigma: either way the wavefront falls back to the plain search for that tile.
#pragma once
#include "common.h"

namespace vecinfer {

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// LDS table of one codebook of C centroids: one entry per centroid with everything the MFMA's A operand
// needs of it, so that a lane fetches its operand with one 16-byte read and no register moves:
//   d = 2:  8 bytes  [ c0 c1 | n n' ]                 d = 4: 12 bytes  [ c0 .. c3 | n n' ]
//   d = 8: 20 bytes  [ n n' | c0 .. c7 ]
// (c: the fp16 centroid, n n': -sigma |c|^2 / 2 in two fp16 parts).  A 16-byte read of the last entries
// runs into the 16 spare bytes at the end.
// C = 256: the codebook of one sub-space (8-bit codes); C = 2^b: the one codebook a KV head's
// sub-spaces share (10- / 12-bit codes).
template <int d, int C = kCentroids>
struct ScreenTab {
    static constexpr int kEntry = d == 8 ? 20 : (d == 4 ? 12 : 8);
    static constexpr int kCen = d == 8 ? 4 : 0;             // offset of the centroid in its entry
    static constexpr int kNorm = d == 8 ? 0 : 2 * d;        // offset of its norm
    static constexpr int kBytes = C * kEntry + 16;
};

struct ScreenConsts {
    float sigma, cmax, nmax;
};

// A value that every lane holds, in a scalar register.
__device__ __forceinline__ float uniform(float v)
{
    return __uint_as_float((unsigned)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v)));
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// sigma: the power of two that brings max |c|^2 / 2 to about 2^10 (within 2^-14 .. 2^14).
// Centroids too large for the fp16 parts of -sigma |c|^2 / 2 (or not finite: nm is then infinite): no
// screen for this codebook; a NaN sigma makes every margin NaN, which sends every tile to the plain
// search.
__device__ __forceinline__ float screen_sigma(float nm)
{
    int e = 9 - ilogbf(fmaxf(0.5f * nm, 1e-30f));
    e = e < -14 ? -14 : (e > 14 ? 14 : e);
    const float sigma = ldexpf(1.0f, e);
    return 0.5f * sigma * nm < 60000.0f ? sigma : __builtin_nanf("");
}

template <int d>
__device__ __forceinline__ void screen_store_norm(unsigned char *tab, int c, float sigma, float n)
{
    const float v = -0.5f * sigma * n;
    const _Float16 hi = (_Float16)v;
    const f16x2 h = {hi, (_Float16)(v - (float)hi)};
    *reinterpret_cast<f16x2 *>(tab + c * ScreenTab<d>::kEntry + ScreenTab<d>::kNorm) = h;
}

// The fp16 values of centroid c -> its entry; returns |c|^2 (fp32) and folds max |c_j| into cm.
template <int d>
__device__ __forceinline__ float screen_store_centroid(const __half *src, unsigned char *tab, int c, float &cm)
{
    typedef _Float16 f16xd __attribute__((ext_vector_type(d)));
    const f16xd raw = *reinterpret_cast<const f16xd *>(src + (size_t)c * d);
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < d; ++j) {
        const float v = (float)raw[j];
        s = fmaf(v, v, s);
        cm = fmaxf(cm, fabsf(v));
    }
    unsigned w[d / 2];
    __builtin_memcpy(w, &raw, 2 * d);
#pragma unroll
    for (int j = 0; j < d / 2; ++j)
        *reinterpret_cast<unsigned *>(tab + c * ScreenTab<d>::kEntry + ScreenTab<d>::kCen + 4 * j) = w[j];
    return s;
}

// Tables of one sub-space's codebook `src` [256][d] fp16 (in memory), built by one wavefront: the
// one that searches the sub-space.
template <int d>
__device__ __forceinline__ ScreenConsts screen_prepare(const __half *src, unsigned char *tab, int lane)
{
    float n[4], cm = 0.f, nm = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        n[i] = screen_store_centroid<d>(src, tab, lane + 64 * i, cm);
        nm = fmaxf(nm, n[i] < INFINITY ? n[i] : INFINITY);
    }
    cm = wave_max(cm);
    nm = wave_max(nm);
    const float sigma = screen_sigma(nm);
#pragma unroll
    for (int i = 0; i < 4; ++i) screen_store_norm<d>(tab, lane + 64 * i, sigma, n[i]);
    if (lane < 4) *reinterpret_cast<unsigned *>(tab + ScreenTab<d>::kBytes - 16 + 4 * lane) = 0u;   // the spare bytes
    return ScreenConsts{uniform(sigma), uniform(cm), uniform(nm)};
}

// Tables of a shared codebook `src` [C][d] fp16, built by the whole workgroup of BLOCK threads
// (`red_s`: 2 BLOCK / 64 floats of LDS scratch).  Ends with a barrier: the tables are complete.
template <int d, int C, int BLOCK>
__device__ __forceinline__ ScreenConsts screen_prepare_shared(const __half *src, unsigned char *tab, float *red_s)
{
    constexpr int PER = C / BLOCK, NW = BLOCK / 64;
    static_assert(C % BLOCK == 0, "whole rounds");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float n[PER], cm = 0.f, nm = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        n[i] = screen_store_centroid<d>(src, tab, tid + BLOCK * i, cm);
        nm = fmaxf(nm, n[i] < INFINITY ? n[i] : INFINITY);
    }
    cm = wave_max(cm);
    nm = wave_max(nm);
    if (lane == 0) {
        red_s[wave] = cm;
        red_s[NW + wave] = nm;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        cm = fmaxf(cm, red_s[w]);
        nm = fmaxf(nm, red_s[NW + w]);
    }
    const float sigma = screen_sigma(nm);
#pragma unroll
    for (int i = 0; i < PER; ++i) screen_store_norm<d>(tab, tid + BLOCK * i, sigma, n[i]);
    if (tid < 4) *reinterpret_cast<unsigned *>(tab + ScreenTab<d, C>::kBytes - 16 + 4 * tid) = 0u;        // the spare bytes
    __syncthreads();
    return ScreenConsts{uniform(sigma), uniform(cm), uniform(nm)};
}

// The fp16 centroid at p (4-byte aligned).
template <int d>
__device__ __forceinline__ void screen_load_centroid(const unsigned char *p, _Float16 (&cen)[d])
{
    unsigned w[d / 2];
#pragma unroll
    for (int j = 0; j < d / 2; ++j) w[j] = *reinterpret_cast<const unsigned *>(p + 4 * j);
    __builtin_memcpy(cen, w, 2 * d);
}

// A constant in a scalar register that the compiler does not see through.
__device__ __forceinline__ float opaque(float v)
{
    asm("" : "+s"(v));
    return v;
}

// Bits of the squared distance of x to a centroid: the fp16 centroid widened (exact), differences
// squared and summed in channel order in fp32.  The difference is a fused multiply-add by -1, which
// rounds the same value once and takes the fp16 operand as it is (v_fma_mix_f32 in place of a
// conversion and a subtraction).
template <int d>
__device__ __forceinline__ unsigned dist_bits(const float (&x)[d], const _Float16 (&cen)[d])
{
    const float minus1 = opaque(-1.0f);
    float dist = 0.f;
#pragma unroll
    for (int j = 0; j < d; ++j) {
        const float t = fmaf((float)cen[j], minus1, x[j]);
        dist = fmaf(t, t, dist);
    }
    return __float_as_uint(dist);
}

template <int d>
__device__ __forceinline__ unsigned screen_dist_bits(const float (&x)[d], const unsigned char *tab, int c)
{
    _Float16 cen[d];
    screen_load_centroid<d>(tab + c * ScreenTab<d>::kEntry + ScreenTab<d>::kCen, cen);
    return dist_bits<d>(x, cen);
}

// The plain search of one token's sub-vector x over the C centroids (the same address in every
// lane: broadcast reads): groups of 8, the group minimum against the running best (strict "<":
// the earliest group wins), the winning group re-evaluated for the lowest index at the minimum.
template <int d, int C = kCentroids>
__device__ __forceinline__ void plain_search(const float (&x)[d], const unsigned char *tab, int &arg_out,
                                             unsigned &best_out)
{
    unsigned best = 0x7f800000u;            // +inf
    int best_group = 0;
#pragma unroll 2
    for (int c0 = 0; c0 < C; c0 += 8) {
        unsigned gmin = screen_dist_bits<d>(x, tab, c0);
#pragma unroll
        for (int k = 1; k < 8; ++k) {
            const unsigned v = screen_dist_bits<d>(x, tab, c0 + k);
            gmin = v < gmin ? v : gmin;
        }
        if (gmin < best) {
            best = gmin;
            best_group = c0;
        }
    }
    int arg = best_group;
#pragma unroll
    for (int k = 7; k >= 0; --k)
        if (screen_dist_bits<d>(x, tab, best_group + k) == best) arg = best_group + k;
    arg_out = arg;
    best_out = best;
}

// What a search needs of the tile's tokens: lane l holds token l's sub-vector and margin, and both
// B operands (cb = 0: tokens 0 .. 31, cb = 1: tokens 32 .. 63; column = lane % 32) are made of the
// lanes' own halves by exchanging 32-lane halves between two registers.
template <int d>
struct ScreenTokens {
    float x[d];
    float mg;          // margin but for the part that depends on the best score
    float sx2;         // sigma |x|^2
    f16x8 b[2];
};

__device__ __forceinline__ unsigned pack2(_Float16 a, _Float16 b)
{
    const f16x2 v = {a, b};
    return __builtin_bit_cast(unsigned, v);
}

__device__ __forceinline__ f16x8 as_f16x8(unsigned a, unsigned b, unsigned c, unsigned e)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = {a, b, c, e};
    return __builtin_bit_cast(f16x8, v);
}

// k-slots 0 .. 7 belong to lanes 0 .. 31, 8 .. 15 to lanes 32 .. 63:
//   d = 2   [ hi0 hi1 1 1 0 0 0 0           | lo0 lo1 0 .. 0            ]
//   d = 4   [ hi0 .. hi3 1 1 0 0            | lo0 .. lo3 0 .. 0         ]
//   d = 8   [ hi0 .. hi7                    | 1 1 lo0 .. lo5            ]   (A: [ c0 .. c7 | n n' c0 .. c5 ])
// v_permlane32_swap(a, b) exchanges the upper half of a with the lower half of b: with a = the lane's
// word for k-slots 0 .. 7 and b = its word for 8 .. 15, a becomes the word of cb = 0 and b that of cb = 1.
template <int d>
__device__ __forceinline__ ScreenTokens<d> screen_tokens(const float *x_s, int XS, int ch0, const ScreenConsts &k, int lane)
{
    ScreenTokens<d> o;
    float l1 = 0.f, l2 = 0.f, dropped = 0.f;
    _Float16 hi[d], lo[d];
#pragma unroll
    for (int j = 0; j < d; ++j) {
        o.x[j] = x_s[lane * XS + ch0 + j];
        l1 += fabsf(o.x[j]);
        l2 = fmaf(o.x[j], o.x[j], l2);
        const float xs = o.x[j] * k.sigma;
        hi[j] = (_Float16)xs;
        const float rest = xs - (float)hi[j];
        lo[j] = (_Float16)rest;
        if (d == 8 && j >= 6) dropped += fabsf(rest);
    }
    constexpr float kT = 2.1f * (0x1p-22f + d * 0x1p-24f + 0x1p-22f + (d == 8 ? 16 : 2 * d + 2) * 0x1p-23f);
    o.mg = k.sigma * kT * (l1 * k.cmax + 0.5f * k.nmax) + 0x1p-13f * ((float)d * k.cmax + 3.0f);
    if (d == 8) o.mg += 2.1f * dropped * k.cmax;
    o.sx2 = k.sigma * l2;
    const unsigned ones = 0x3c003c00u;                      // 1.0, 1.0
    unsigned a[4], b[4];
    if constexpr (d == 8) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            a[j] = pack2(hi[2 * j], hi[2 * j + 1]);
            b[j] = j == 0 ? ones : pack2(lo[2 * j - 2], lo[2 * j - 1]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < d / 2; ++j) {
            a[j] = pack2(hi[2 * j], hi[2 * j + 1]);
            b[j] = pack2(lo[2 * j], lo[2 * j + 1]);
        }
    }
    constexpr int kWords = d == 8 ? 4 : d / 2;              // words that are exchanged
#pragma unroll
    for (int j = 0; j < kWords; ++j) {
        auto sw = __builtin_amdgcn_permlane32_swap(a[j], b[j], false, false);
        a[j] = sw[0];
        b[j] = sw[1];
    }
    if constexpr (d != 8) {
        a[d / 2] = b[d / 2] = lane < 32 ? ones : 0u;        // the same in both operands
#pragma unroll
        for (int j = d / 2 + 1; j < 4; ++j) a[j] = b[j] = 0u;
    }
    o.b[0] = as_f16x8(a[0], a[1], a[2], a[3]);
    o.b[1] = as_f16x8(b[0], b[1], b[2], b[3]);
    return o;
}

// A operand of the 32 centroids from `row0`: 16 bytes of the lane's entry.  What lies behind the
// entry (the next one, or the zeroed spare bytes) meets zeros in the B operand and is finite.
template <int d>
__device__ __forceinline__ f16x8 screen_a(const unsigned char *lane_tab, int row0)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4), aligned(4)));
    const u32x4 w = *reinterpret_cast<const u32x4 *>(lane_tab + row0 * ScreenTab<d>::kEntry);
    return __builtin_bit_cast(f16x8, (unsigned __attribute__((ext_vector_type(4))))w);
}

// This lane's base for screen_a.
template <int d>
__device__ __forceinline__ const unsigned char *screen_lane_tab(const unsigned char *tab, int lane)
{
    return tab + (lane & 31) * ScreenTab<d>::kEntry + (d == 8 && lane < 32 ? 4 : 0);
}

// Scores of the tile's 64 tokens against NB x 32 centroids from row0; gm: per accumulator register
// ("group" of NB centroids) the maximum over the blocks of 32.  A step is two blocks for one of
// the two operands: two MFMAs and 16 v_max3_f32, which take about as long.
// DEPTH = 2 (workgroups that leave a SIMD two wavefronts): the MFMAs of a step are issued ahead of the
// maxima of the step before, so that the matrix cores and the vector ALU work side by side within
// the wavefront.  DEPTH = 1 (four wavefronts per SIMD, which do that among themselves): one set of
// results, 32 registers less, which is what brings the kernel to 128.  (Not quite with 32 sub-spaces, two searches
// per wavefront: the keys' fills spill 7, 5 and 3 registers at D = 128, d = 4 and 2, and D = 64, d = 2, the values' fill
// at D = 128, d = 4 spills one.)
// (The fences keep it at that: left alone the compiler issues many more MFMAs first, whose
// results then spill.)
template <int d, int NB, int DEPTH>
__device__ __forceinline__ void screen_groups(const unsigned char *lane_tab, int row0, const ScreenTokens<d> &o,
                                              float (&gm)[2][16])
{
    const f32x16 z16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // (as a third operand of the first maxima: a plain fmaxf of two MFMA results would quiet both first)
    const float lowest = opaque(-INFINITY);
    if constexpr (DEPTH == 1) {
        f16x8 a[2] = {screen_a<d>(lane_tab, row0), screen_a<d>(lane_tab, row0 + 32)};
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            f32x16 v[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) v[u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[u], o.b[t & 1], z16, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (t % 2 == 1 && t + 1 < NB) {                  // the next pair of blocks' operands
                a[0] = screen_a<d>(lane_tab, row0 + 32 * (t + 1));
                a[1] = screen_a<d>(lane_tab, row0 + 32 * (t + 2));
            }
#pragma unroll
            for (int r = 0; r < 16; ++r)
                gm[t & 1][r] = fmaxf(fmaxf(t < 2 ? lowest : gm[t & 1][r], v[0][r]), v[1][r]);
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }
    f32x16 v[2][2];
    f16x8 a[2], next[2] = {screen_a<d>(lane_tab, row0), screen_a<d>(lane_tab, row0 + 32)};
#pragma unroll
    for (int t = 0; t <= NB; ++t) {
        if (t % 2 == 0) {
            a[0] = next[0];
            a[1] = next[1];
        } else if (t + 1 < NB) {                             // the next pair of blocks' operands, a step ahead
            next[0] = screen_a<d>(lane_tab, row0 + 32 * (t + 1));
            next[1] = screen_a<d>(lane_tab, row0 + 32 * (t + 2));
        }
        if (t < NB) {
#pragma unroll
            for (int u = 0; u < 2; ++u) v[t & 1][u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[u], o.b[t & 1], z16, 0, 0, 0);
        }
        if (t > 0) {
            const int p = (t - 1) & 1;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                gm[p][r] = fmaxf(fmaxf(t <= 2 ? lowest : gm[p][r], v[p][0][r]), v[p][1][r]);
        }
        if (t > 0 && t < NB) {
            if (t % 2 == 1 && t + 1 < NB) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int n>
__device__ __forceinline__ float max_of(const float (&v)[n])
{
    float m = n > 1 ? fmaxf(v[0], v[1]) : v[0];
#pragma unroll
    for (int r = 2; r + 1 < n; r += 2) m = fmaxf(fmaxf(m, v[r]), v[r + 1]);
    if (n > 2 && n % 2) m = fmaxf(m, v[n - 1]);
    return m;
}

// Bit r set where v[r] > thr: the sign bit of thr - v[r], shifted into the mask (one subtraction and
// one v_alignbit each).
template <int n>
__device__ __forceinline__ unsigned marks_above(const float (&v)[n], float thr, unsigned m = 0u)
{
#pragma unroll
    for (int r = n - 1; r >= 0; --r) m = __builtin_amdgcn_alignbit(m, __float_as_uint(thr - v[r]), 31);
    return m;
}

// Thresholds (best score - margin) of the two operands' tokens from the lanes' maxima `bm` of both;
// returns the own token's.
template <int d>
__device__ __forceinline__ float screen_thresholds(const float (&bm)[2], const ScreenTokens<d> &o, float (&thr)[2])
{
    // own token: its best over the rows of lanes 0 .. 31 and over those of lanes 32 .. 63
    auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(bm[0]), __float_as_uint(bm[1]), false, false);
    const float best = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    constexpr float kD = 1.05f * (d + 2) * 0x1p-24f;
    const float own = best - fmaf(kD, fmaxf(fmaf(-2.0f, best, o.sx2), 0.0f), o.mg);
    auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(own), __float_as_uint(own), false, false);
    thr[0] = __uint_as_float(both[0]);
    thr[1] = __uint_as_float(both[1]);
    return own;
}

// Exact distances of the N centroids row, row + 32, .. (row: this lane's): (best, arg) keeps the
// smallest (distance bits, index).
template <int d, int N>
__device__ __forceinline__ void screen_eval(const float (&x)[d], const unsigned char *tab, int row, unsigned &best, int &arg)
{
    const unsigned char *const p = tab + row * ScreenTab<d>::kEntry + ScreenTab<d>::kCen;
    // (channel by channel over all N: independent chains side by side)
    const float minus1 = opaque(-1.0f);
    _Float16 cen[N][d];
    float dist[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        screen_load_centroid<d>(p + i * 32 * ScreenTab<d>::kEntry, cen[i]);
        dist[i] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < d; ++j)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float t = fmaf((float)cen[i][j], minus1, x[j]);
            dist[i] = fmaf(t, t, dist[i]);
        }
    unsigned v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __float_as_uint(dist[i]);
    unsigned m = v[0];
#pragma unroll
    for (int i = 1; i < N; ++i) m = v[i] < m ? v[i] : m;
    int at = N - 1;
#pragma unroll
    for (int i = N - 2; i >= 0; --i) at = v[i] == m ? i : at;
    const int c = row + 32 * at;
    if (m < best || (m == best && c < arg)) {
        best = m;
        arg = c;
    }
}

// Row (within a block of 32 centroids) of accumulator register r & 15 in lanes 32 (r >> 4) ..
__device__ __forceinline__ int screen_row(unsigned r)
{
    return (int)(8u * ((r >> 2) & 3u) + 4u * ((r >> 4) & 1u) + (r & 3u));
}

// The wavefront's 64 tokens (rows of x_s, channels ch0 .. ch0 + d) against the sub-space whose
// table is `tab`.  Returns the code of token `lane` and the bits of its squared distance; false
// if some token of the wavefront has no usable scores (the caller then runs the plain search; same for
// every lane).
template <int d, int DEPTH>
__device__ __forceinline__ bool screen_search(const float *x_s, int XS, int ch0, const unsigned char *tab,
                                              const ScreenConsts &k, int lane, int &arg_out, unsigned &best_out)
{
    const ScreenTokens<d> o = screen_tokens<d>(x_s, XS, ch0, k, lane);
    float gm[2][16];
    screen_groups<d, kCentroids / 32, DEPTH>(screen_lane_tab<d>(tab, lane), 0, o, gm);
    // ---- groups within the margin of the token's best score
    const float bm[2] = {max_of(gm[0]), max_of(gm[1])};
    float thr[2];
    const float own_thr = screen_thresholds<d>(bm, o, thr);
    auto sw = __builtin_amdgcn_permlane32_swap(marks_above(gm[0], thr[0]), marks_above(gm[1], thr[1]), false, false);
    unsigned marks = sw[0] | sw[1] << 16;                   // own token: groups of lanes 0 .. 31, of lanes 32 .. 63
    // ---- exact distances of the marked groups' centroids.  A lane that has run out of marks while
    // another has not goes over group 31 (its real distances can only repeat what is known).
    unsigned best = 0x7f800000u;
    int arg = 0;
    do {
        const unsigned r = (unsigned)__builtin_ctz(marks | 0x80000000u);
        marks &= marks - 1u;
        screen_eval<d, kCentroids / 32>(o.x, tab, screen_row(r), best, arg);
    } while (__any(marks != 0u));
    arg_out = arg;
    best_out = best;
    // no screen result for a token whose scaled operands left the fp16 range (infinite or NaN
    // scores), and none where nothing finite was found
    return !__any(best >= 0x7f800000u || !(fabsf(own_thr) < INFINITY));
}

// The same for a codebook of C = 2^b centroids shared by the sub-spaces: the centroids are gone through
// in chunks, and a token keeps, in each half of the wavefront, the maxima of its 16 groups over the
// whole codebook and the maximum of every chunk.  A score within the margin marks its group and
// its chunk, so the marked (chunk, group) pairs - normally one - hold every centroid that can win or
// tie.  (Per chunk of 512 centroids that is 48 vector-ALU instructions on top of the 256 of the maxima
// themselves; marking groups chunk by chunk took 140 per 256 centroids.)
template <int d, int C>
__device__ __forceinline__ bool screen_search_shared(const float *x_s, int XS, int ch0, const unsigned char *tab,
                                                     const ScreenConsts &k, int lane, int &arg_out,
                                                     unsigned &best_out)
{
    constexpr int NCH = C >= 4096 ? 8 : 4, NB = C / 32 / NCH;     // chunks; blocks of 32 centroids per chunk
    static_assert(NCH <= 8 && NB % 2 == 0 && NB * NCH * 32 == C, "whole chunks, chunk marks in 8 bits");
    const ScreenTokens<d> o = screen_tokens<d>(x_s, XS, ch0, k, lane);
    const unsigned char *const lane_tab = screen_lane_tab<d>(tab, lane);
    float run[2][16], cm[2][NCH];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) run[cb][r] = -INFINITY;
#pragma unroll
        for (int i = 0; i < NCH; ++i) cm[cb][i] = -INFINITY;
    }
#pragma unroll 1
    for (int ch = 0; ch < NCH; ++ch) {
        float gm[2][16];
        screen_groups<d, NB, 2>(lane_tab, ch * NB * 32, o, gm);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            // (the chunk maxima move up a place per iteration, so that no register is indexed by ch)
#pragma unroll
            for (int i = 0; i + 1 < NCH; ++i) cm[cb][i] = cm[cb][i + 1];
            cm[cb][NCH - 1] = max_of(gm[cb]);
#pragma unroll
            for (int r = 0; r < 16; ++r) run[cb][r] = fmaxf(run[cb][r], gm[cb][r]);
        }
    }
    const float bm[2] = {max_of(cm[0]), max_of(cm[1])};
    float thr[2];
    const float own_thr = screen_thresholds<d>(bm, o, thr);
    unsigned m[2];                                          // groups in bits 0 .. 15, chunks from bit 16
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) m[cb] = marks_above(run[cb], thr[cb], marks_above(cm[cb], thr[cb]));
    auto sw = __builtin_amdgcn_permlane32_swap(m[0], m[1], false, false);
    // own token: the marks of lanes 0 .. 31's rows, then those of lanes 32 .. 63's
    unsigned cur = sw[0], next = sw[1];
    unsigned half = 0u;
    if (cur == 0u) {
        cur = next;
        next = 0u;
        half = 16u;
    }
    unsigned groups = cur & 0xffffu, chunks = cur >> 16;
    unsigned best = 0x7f800000u;
    int arg = 0;
    do {
        // (a lane without marks left goes over some pair again: it can only repeat what is known)
        const unsigned r = (unsigned)__builtin_ctz(groups | 0x8000u), ch = (unsigned)__builtin_ctz(chunks | 1u << (NCH - 1));
        screen_eval<d, NB>(o.x, tab, (int)ch * NB * 32 + screen_row(r + half), best, arg);
        groups &= groups - 1u;
        if (groups == 0u) {
            chunks &= chunks - 1u;
            if (chunks == 0u && next != 0u) {
                cur = next;
                next = 0u;
                half = 16u;
                chunks = cur >> 16;
            }
            groups = chunks != 0u ? cur & 0xffffu : 0u;
        }
    } while (__any(groups != 0u));
    arg_out = arg;
    best_out = best;
    return !__any(best >= 0x7f800000u || !(fabsf(own_thr) < INFINITY));
}

// One wavefront, one sub-space, the 64 tokens of the tile in x_s: the screen and the exact
// distances of what it marks; the plain search when the screen gives no answer.
template <int d, int C = kCentroids, int DEPTH = 2>
__device__ __forceinline__ void search_tile(const float *x_s, int XS, int ch0, const unsigned char *tab,
                                            const ScreenConsts &k, int lane, int &arg, unsigned &best)
{
    if constexpr (C == kCentroids) {
        if (screen_search<d, DEPTH>(x_s, XS, ch0, tab, k, lane, arg, best)) return;
    } else {
        if (screen_search_shared<d, C>(x_s, XS, ch0, tab, k, lane, arg, best)) return;
    }
    float x[d];
#pragma unroll
    for (int j = 0; j < d; ++j) x[j] = x_s[lane * XS + ch0 + j];
    plain_search<d, C>(x, tab, arg, best);
}

} // namespace

} // namespace vecinfer
