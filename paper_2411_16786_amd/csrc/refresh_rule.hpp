// Which pairs a step refreshes, as device code: the elementwise policies (RefreshRule) and the exact top-m selection of tokens.  Shared by
// the kernels that write the mask (refresh.hip) and by the dispatch, which in the layer call forms the mask itself (dispatch.hip).
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace dicemoe {

// Counter-based draw of the "Random" ablation variant: the 32-bit avalanche step of MurmurHash3 (a
// published bit mixer) on seed * 0x9E3779B9 + token, modulo 2^32.
__device__ __forceinline__ uint32_t mix32(uint32_t seed, uint32_t token) {
    uint32_t h = seed * 0x9E3779B9u + token;
    h ^= h >> 16; h *= 0x85EBCA6Bu;
    h ^= h >> 13; h *= 0xC2B2AE35u;
    h ^= h >> 16;
    return h;
}

// Elementwise policies: is pair p refreshed?  kc = columns of the mask (k routed slots, then the shared-expert slots, which are always refreshed).
// kind 1 / 5 / 6: Algorithm 4 with the always-fresh slot being the top-1 slot, the last activated
// slot ("High Score" deprioritised) or a slot drawn per token ("Random"), Section 5.3 ablation.
__device__ __forceinline__ uint8_t simple_mask(const RefreshRule& rule, int p)
{
    const int kc = rule.k + rule.n_shared, k = rule.k;
    const int j = p % kc;
    if (j >= k) return 1;                                   // shared expert: fresh in every step
    if (rule.kind == 0) return 1;                           // every pair
    if (rule.kind == 4) return 0;                           // no pair
    int fresh_slot = 0;                                     // top-1 slot always, others on t mod n == 0
    if (rule.kind == 5) fresh_slot = k - 1;
    else if (rule.kind == 6) fresh_slot = static_cast<int>(mix32(rule.seed, static_cast<uint32_t>(p / kc)) % static_cast<uint32_t>(k));
    return (j == fresh_slot || !rule.off_step) ? 1 : 0;
}

// Selection policies: mask byte of slot j of a token that is (not) selected.
__device__ __forceinline__ uint8_t selected_mask(const RefreshRule& rule, int j, bool sel)
{
    if (j >= rule.k) return 1;                              // shared expert: fresh in every step
    if (rule.token_mode) return sel ? 1 : 0;
    return (j < rule.slot) ? 1 : (j == rule.slot ? (sel ? 1 : 0) : 0);
}

// monotone map from float bits to unsigned: larger float <-> larger key
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;
constexpr int kSelBins = 2048;

// Exact top-m selection by one workgroup of 1024 threads, up to 1024 KPT tokens, keys held in registers (KPT per thread, token
// i = u * 1024 + tid); sel[u]: is that token among them.  A most-significant-digit radix select on (key - smallest key): the digit is the
// top 11 bits of the span the keys still in play cover, so that the 2048 counters are spread over the
// keys' real range (router scores share their sign and most of their exponent bits: fixed bit fields
// would send every key to two or three counters, and LDS atomics on one address serialise).  Round r
// narrows the span by 2^11; it ends early when every key of the threshold digit is admitted, which is
// the usual case after the second round.  Ties at the threshold go to the lower token, by a block-wide
// prefix count in token order.
struct SelectShared {
    uint32_t hist[kSelBins];
    uint32_t wave_a[kSelWaves], wave_b[kSelWaves];
    uint32_t s_bin, s_above, s_cnt;
};

template <int KPT>
__device__ __forceinline__ void select_tokens(const RefreshRule& rule, int T_tok, SelectShared& sh, bool (&selected)[KPT])
{
    uint32_t (&hist)[kSelBins] = sh.hist;
    uint32_t (&wave_a)[kSelWaves] = sh.wave_a;
    uint32_t (&wave_b)[kSelWaves] = sh.wave_b;
    uint32_t &s_bin = sh.s_bin, &s_above = sh.s_above, &s_cnt = sh.s_cnt;
    const float* __restrict__ scores = rule.scores;
    const int kc = rule.k + rule.n_shared, slot = rule.slot, m = rule.m;
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();

    uint32_t key[KPT];
#pragma unroll
    for (int u = 0; u < KPT; ++u) {
        const int i = u * kSelThreads + tid;
        key[u] = order_key(scores[static_cast<size_t>(i < T_tok ? i : T_tok - 1) * kc + slot]);
    }
    const bool need_select = (m > 0 && m < T_tok);
    uint32_t lo = 0, thr = 0;
    int admit_equal = 0;          // > 0: keys equal to thr are admitted in token order, this many of them
    bool ties = false;
    if (need_select) {
        // smallest and largest key
        uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
        for (int u = 0; u < KPT; ++u)
            if (u * kSelThreads + tid < T_tok) { kmin = key[u] < kmin ? key[u] : kmin; kmax = key[u] > kmax ? key[u] : kmax; }
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) {
            const uint32_t a = __shfl_xor(kmin, sh, kWave), b = __shfl_xor(kmax, sh, kWave);
            kmin = a < kmin ? a : kmin;
            kmax = b > kmax ? b : kmax;
        }
        if (lane == 0) { wave_a[wave] = kmin; wave_b[wave] = kmax; }
        __syncthreads();
        kmin = wave_a[lane & (kSelWaves - 1)];
        kmax = wave_b[lane & (kSelWaves - 1)];
#pragma unroll
        for (int sh = kSelWaves / 2; sh >= 1; sh >>= 1) {
            const uint32_t a = __shfl_xor(kmin, sh, kWave), b = __shfl_xor(kmax, sh, kWave);
            kmin = a < kmin ? a : kmin;
            kmax = b > kmax ? b : kmax;
        }
        lo = kmin;
        uint32_t span = kmax - kmin;              // keys in play lie in [lo, lo + span]
        uint32_t remaining = static_cast<uint32_t>(m);
        for (;;) {
            const int shift = span >= kSelBins ? (32 - __builtin_clz(span)) - 11 : 0;     // span >> shift < 2048
            __syncthreads();                      // the previous round's reads of hist / s_* are done
            hist[tid] = 0; hist[tid + kSelThreads] = 0;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < KPT; ++u) {
                const uint32_t rel = key[u] - lo;
                if (u * kSelThreads + tid < T_tok && key[u] >= lo && rel <= span) atomicAdd(&hist[rel >> shift], 1u);
            }
            __syncthreads();
            // keys in digits above each digit: thread t owns digits 2t and 2t+1; suffix sums over the
            // threads of a wave by shuffles, over the waves through LDS
            const uint32_t h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
            uint32_t incl = h0 + h1;              // becomes the sum over lanes >= this one
#pragma unroll
            for (int sh = 1; sh < kWave; sh <<= 1) {
                const uint32_t v = __shfl_down(incl, sh, kWave);
                if (lane + sh < kWave) incl += v;
            }
            if (lane == 0) wave_a[wave] = incl;
            __syncthreads();
            uint32_t higher = 0;
#pragma unroll
            for (int w = 0; w < kSelWaves; ++w) higher += (w > wave) ? wave_a[w] : 0u;
            const uint32_t above1 = higher + incl - (h0 + h1);     // keys in digits above 2t+1
            const uint32_t above0 = above1 + h1;                    // keys in digits above 2t
            if (above1 < remaining && remaining <= above1 + h1) { s_bin = 2 * tid + 1; s_above = above1; s_cnt = h1; }
            if (above0 < remaining && remaining <= above0 + h0) { s_bin = 2 * tid; s_above = above0; s_cnt = h0; }
            __syncthreads();
            const uint32_t bin = s_bin, cnt = s_cnt;
            remaining -= s_above;
            lo += bin << shift;
            if (remaining == cnt) { thr = lo; break; }              // the whole digit is admitted: keys >= lo
            if (shift == 0) { thr = lo; ties = true; admit_equal = static_cast<int>(remaining); break; }
            span = (1u << shift) - 1u;
        }
    }

    int running = 0;
#pragma unroll
    for (int u = 0; u < KPT; ++u) {
        const int i = u * kSelThreads + tid;
        const bool valid = i < T_tok;
        bool sel;
        if (!need_select) {
            sel = (m > 0);
        } else if (!ties) {
            sel = key[u] >= thr;
        } else {
            const bool eq = valid && key[u] == thr;
            const uint64_t b = __ballot(eq);
            __syncthreads();
            if (lane == 0) wave_a[wave] = __popcll(b);
            __syncthreads();
            int before = running + __popcll(b & lanemask_lt());
            int total = 0;
#pragma unroll
            for (int w = 0; w < kSelWaves; ++w) {
                const int c = static_cast<int>(wave_a[w]);
                if (w < wave) before += c;
                total += c;
            }
            running += total;
            sel = key[u] > thr || (eq && before < admit_equal);
        }
        selected[u] = sel;
    }
}

}  // namespace dicemoe
