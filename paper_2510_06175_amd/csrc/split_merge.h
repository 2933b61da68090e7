// Log-sum-exp merge of the split partials inside the attention launch: the last workgroup of a
// (sequence, KV head) to finish reads the others' partials and writes the output rows.
//
// The partials, and the arrival word that tells who is last, are written and read by relaxed
// agent-scope atomics only.  On this chip these go through to the memory that all XCDs share by
// themselves, so no fence is needed (a device-scope release writes the XCD's whole L2 back: 4 us per
// workgroup).  What orders them is waiting: a wavefront waits until its partial stores are acknowledged
// (vmcnt 0), the workgroup meets at a barrier, and only then does one thread add 1 to the arrival
// word.  Whoever gets S - 1 back was preceded by all others' adds, hence by all their partials.  Nobody
// waits for another workgroup, so no order of execution can hang.
//
// What it costs: three dependent trips to memory (stores, add, loads).  256 workgroups of 512 threads that
// store a row and end: 2.5 us per launch; with 8 merges of 32 rows by the last arrivers 3.3 us, by a second
// launch 4.9.
//
// Arrival word (one per sequence and KV head, in the workspace, which nobody initialises: behind the new token's
// value, which as a row of fp16 centroids takes half of the D floats that its place has):
//   nonce << 16 | workgroups that have arrived
// The nonce is a launch's own number.  Every workgroup looks at the word when it starts and, if it
// carries another number, swaps it for (nonce, 0) with a compare-and-swap; if that fails another workgroup
// of this launch has done so.  A workgroup's swap is acknowledged before its own add, so no add can
// meet a word that is not set up.  The last one clears the word, so that a captured launch, whose nonce is
// the same at every replay, finds it as it would a fresh one.
#pragma once
#include "common.h"

#include <type_traits>

namespace vecinfer {

namespace {

typedef unsigned long long arrival_t;

template <int D>
__device__ __forceinline__ __half *new_value(const DecodeParams &p, size_t bg)
{
    return reinterpret_cast<__half *>(p.new_v + bg * D);
}

template <int D>
__device__ __forceinline__ arrival_t *arrival_word(const DecodeParams &p, size_t bg)
{
    return reinterpret_cast<arrival_t *>(p.new_v + bg * D + D / 2);
}

__device__ __forceinline__ arrival_t arrival_peek(const arrival_t *word)
{
    return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// (one thread; `seen`: what arrival_peek returned)
__device__ __forceinline__ void arrival_open(arrival_t *word, arrival_t seen, arrival_t nonce)
{
    if (seen >> 16 != nonce)
        __hip_atomic_compare_exchange_strong(word, &seen, nonce << 16, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void shared_store(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ float shared_load(const float *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// (v: an fp16 value, widened)
__device__ __forceinline__ void shared_store_half(__half *p, float v)
{
    __hip_atomic_store(reinterpret_cast<unsigned short *>(p), __half_as_ushort(__float2half(v)), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ float shared_load_half(const __half *p)
{
    return __half2float(__ushort_as_half(
        __hip_atomic_load(reinterpret_cast<const unsigned short *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
}

// Maximum over the wavefront, in every lane, or sum, on the vector ALU (DPP inside the rows of 16 lanes, row swaps
// across them): no trip through the LDS crossbar.  The quads of a row add each other in turned orders, so a sum's last
// bits differ from quad to quad: whoever needs one value takes one lane's.
template <typename Op>
__device__ __forceinline__ float wave_all(float x, Op op)
{
    auto dpp = [](float v, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    x = op(x, dpp(x, std::integral_constant<int, 0xB1>{}));       // quad_perm:[1,0,3,2]
    x = op(x, dpp(x, std::integral_constant<int, 0x4E>{}));       // quad_perm:[2,3,0,1]
    x = op(x, dpp(x, std::integral_constant<int, 0x124>{}));      // row_ror:4
    x = op(x, dpp(x, std::integral_constant<int, 0x128>{}));      // row_ror:8
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto s16 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    x = op(__builtin_bit_cast(float, (unsigned)s16[0]), __builtin_bit_cast(float, (unsigned)s16[1]));
    const unsigned w = __builtin_bit_cast(unsigned, x);
    auto s32 = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    return op(__builtin_bit_cast(float, (unsigned)s32[0]), __builtin_bit_cast(float, (unsigned)s32[1]));
}

constexpr int kMergeSplits = 256;                        // VECINFER_MAX_SPLITS
// LDS that merge_arrived uses, in floats: the flag, the splits' weights, the new token's value, (den, weight of
// the new token) per head.
constexpr int merge_arrived_floats(int D, int KG) { return 4 + kMergeSplits * KG + D + 2 * KG; }

// Called by all BLOCK threads of a workgroup whose partials have been stored (shared_store), and whose
// thread 0 has opened the arrival word.  `lds`: merge_arrived_floats() of scratch that no wavefront uses any
// more once it is here; row0: the first output row.
//   M = max_s m_s,  w_s = 2^(m_s - M),  o = sum_s w_s o_s / sum_s w_s l_s,  L = (M + log2 sum) ln 2
// A wavefront per head works the weights out (a lane per split; the new token's score shares, a lane per
// sub-space, and its partial (m = their sum, l = 1, o = its value) with them), while the partial
// rows of all splits travel to the threads that own their elements.
// (With the maximum, the weights and the sum of the shares in every thread, split after split, this part took
// 1.8 us behind the last load.)
template <int D, int KG, int BLOCK>
__device__ __forceinline__ void merge_arrived(const DecodeParams &p, float *lds, size_t bg, size_t row0, int S, int G,
                                              bool new_tok)
{
    static_assert(KG <= BLOCK / 64, "a wavefront per head");
    constexpr int kElems = (KG * D + BLOCK - 1) / BLOCK;  // output elements per thread
    constexpr int kBatch = 64 / kElems, kStep = 8;        // split partials a thread keeps in flight, by eights
    constexpr int kML = kMergeSplits / 64;
    const int t = threadIdx.x, lane = t & 63, hh_w = __builtin_amdgcn_readfirstlane(t >> 6), GD = G * D;
    arrival_t *const word = arrival_word<D>(p, bg);
    unsigned *const flag = reinterpret_cast<unsigned *>(lds);
    float *const wt_s = lds + 4, *const nv_s = wt_s + kMergeSplits * KG, *const fin_s = nv_s + D;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wavefront's stores (and the word's set-up) are acknowledged
    __syncthreads();
    if (t == 0) {
        const arrival_t before = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag = (int)(before & 0xffffu) == S - 1;
    }
    __syncthreads();
    if (*flag == 0u) return;                             // (the same for the whole workgroup)

    // ---- everything that is needed, requested back to back
    const bool head_wave = hh_w < G;
    float tm[kML], tl[kML], share = 0.f;
    if (head_wave) {
        const float *const pm = p.part_m + bg * S * G + hh_w, *const pl = p.part_l + bg * S * G + hh_w;
#pragma unroll
        for (int i = 0; i < kML; ++i) {
            if (64 * i >= S) break;
            const int at = (lane + 64 * i < S ? lane + 64 * i : S - 1) * G;
            tm[i] = shared_load(pm + at);
            tl[i] = shared_load(pl + at);
        }
        if (new_tok && lane < p.Mk) share = shared_load(p.new_sc + (bg * p.Mk + lane) * G + hh_w);
    }
    float nvv = 0.f;
    if (new_tok && t < D) nvv = shared_load_half(new_value<D>(p, bg) + t);
    float vo[kElems][kBatch];
    auto request = [&](int s0) {
        const float *const po = p.part_o + (bg * S + s0) * GD;
#pragma unroll
        for (int j0 = 0; j0 < kBatch; j0 += kStep) {
            if (s0 + j0 >= S) break;
#pragma unroll
            for (int j = j0; j < j0 + kStep; ++j)
#pragma unroll
                for (int i = 0; i < kElems; ++i) {
                    // (behind the last split: that one again, at weight 0)
                    const int e = t + i * BLOCK < GD ? t + i * BLOCK : 0;
                    vo[i][j] = shared_load(po + (s0 + j < S ? j : S - 1 - s0) * GD + e);
                }
        }
    };
    request(0);

    // ---- weights
    if (t == 0) __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (head_wave) {
        const auto max2 = [](float a, float b) { return fmaxf(a, b); };
        const auto add2 = [](float a, float b) { return a + b; };
        float M = -INFINITY;
#pragma unroll
        for (int i = 0; i < kML; ++i) {
            if (64 * i >= S) break;
            M = fmaxf(M, tm[i]);
        }
        M = wave_all(M, max2);
        // (one lane's: all splits and the new token have to be weighed against the same M)
        const float s_new = new_tok ? __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(wave_all(share, add2)))) : -INFINITY;
        M = fmaxf(M, s_new);
        const float Mc = M > -INFINITY ? M : 0.f;        // nothing to attend to: all weights 0
        const float w_new = __builtin_amdgcn_exp2f(s_new - Mc);
        float den = 0.f;
#pragma unroll
        for (int i = 0; i < kML; ++i) {
            if (64 * i >= S) break;
            const bool in = lane + 64 * i < S;
            const float w = in ? __builtin_amdgcn_exp2f(tm[i] - Mc) : 0.f;
            if (in) den = fmaf(w, tl[i], den);
            wt_s[hh_w * kMergeSplits + lane + 64 * i] = w;
        }
        den = wave_all(den, add2) + w_new;
        if (lane == 0) {
            fin_s[2 * hh_w] = den;
            fin_s[2 * hh_w + 1] = w_new;
            if (p.lse) p.lse[row0 + hh_w] = den > 0.f ? (M + log2f(den)) * kLn2 : -INFINITY;
        }
    }
    if (t < D) nv_s[t] = nvv;
    __syncthreads();

    // ---- the rows
    float acc[kElems];
#pragma unroll
    for (int i = 0; i < kElems; ++i) acc[i] = 0.f;
    for (int s0 = 0;;) {
#pragma unroll
        for (int j0 = 0; j0 < kBatch; j0 += kStep) {
            if (s0 + j0 >= S) break;
#pragma unroll
            for (int i = 0; i < kElems; ++i) {
                const int e = t + i * BLOCK < GD ? t + i * BLOCK : 0;
                const float4 *const w = reinterpret_cast<const float4 *>(wt_s + e / D * kMergeSplits + s0 + j0);
                float wj[kStep];
#pragma unroll
                for (int j = 0; j < kStep; j += 4) {
                    const float4 x = w[j / 4];
                    wj[j] = x.x; wj[j + 1] = x.y; wj[j + 2] = x.z; wj[j + 3] = x.w;
                }
#pragma unroll
                for (int j = 0; j < kStep; ++j) acc[i] = fmaf(wj[j], vo[i][j0 + j], acc[i]);
            }
        }
        s0 += kBatch;
        if (s0 >= S) break;
        request(s0);                                     // more splits than a batch: another trip
    }
#pragma unroll
    for (int i = 0; i < kElems; ++i) {
        const int e = t + i * BLOCK;
        if (e >= GD) continue;
        const int hh = e / D, c = e % D;
        const float den = fin_s[2 * hh];
        const float o = new_tok ? fmaf(fin_s[2 * hh + 1], nv_s[c], acc[i]) : acc[i];
        p.out[(row0 + hh) * D + c] = __float2half(den > 0.f ? o / den : 0.f);
    }
}

} // namespace

} // namespace vecinfer
