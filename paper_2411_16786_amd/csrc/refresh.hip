// Conditional Communication decision (supplement, Algorithm 4): which (token, slot) pairs are
// recomputed this step and which reuse the cached expert output.
//
// ALL / NONE / ALG4 are elementwise.  The fraction policies need an exact top-m selection of
// tokens by a float score with ties going to the lower token index; one workgroup does it with a
// most-significant-digit radix select on the score's bit pattern (up to 16384 tokens as select_tokens in refresh_rule.hpp does it,
// beyond that four passes of 8 bits over memory), then resolves ties at the threshold by a block-wide prefix count in index order.
// Everything is integer work on the bit patterns, so the mask is reproducible bit for bit.
#include "refresh_rule.hpp"

namespace dicemoe {

__global__ __launch_bounds__(256) void refresh_simple_kernel(RefreshRule rule, int N)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p == 0) *rule.n_refresh = rule.n_value;
    if (p < N) rule.mask[p] = simple_mask(rule, p);
}

// Selection of any size: keys re-read from memory in every pass.
__global__ __launch_bounds__(kSelThreads) void refresh_select_any_kernel(const float* __restrict__ scores, int T_tok,
                                                                    int kc, int k, int slot, int m, int token_mode,
                                                                    int n_value, uint8_t* __restrict__ mask,
                                                                    int32_t* __restrict__ n_refresh)
{
    __shared__ uint32_t hist[256];
    __shared__ uint32_t sfx[2][256];
    __shared__ uint32_t s_prefix, s_remaining, s_equal;
    __shared__ int wave_cnt[kSelWaves];
    const int tid = threadIdx.x;
    if (tid == 0) { *n_refresh = n_value; s_prefix = 0; s_remaining = static_cast<uint32_t>(m); s_equal = 0; }

    const bool need_select = (m > 0 && m < T_tok);
    if (need_select) {
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            const uint32_t prefix = s_prefix;       // both stable until the end of this pass
            const uint32_t rem = s_remaining;
            for (int i = tid; i < T_tok; i += kSelThreads) {
                const uint32_t key = order_key(scores[static_cast<size_t>(i) * kc + slot]);
                const bool in_play = (pass == 0) || ((key >> (shift + 8)) == (prefix >> (shift + 8)));
                if (in_play) atomicAdd(&hist[(key >> shift) & 255u], 1u);
            }
            __syncthreads();
            // sfx[b] = number of in-play keys whose digit is larger than b (suffix sum, exclusive)
            int cur = 0;
            if (tid < 256) sfx[0][tid] = (tid < 255) ? hist[tid + 1] : 0u;
            __syncthreads();
            for (int step = 1; step < 256; step <<= 1) {
                if (tid < 256) {
                    uint32_t v = sfx[cur][tid];
                    if (tid + step < 256) v += sfx[cur][tid + step];
                    sfx[cur ^ 1][tid] = v;
                }
                cur ^= 1;
                __syncthreads();
            }
            if (tid < 256) {
                const uint32_t above = sfx[cur][tid];
                if (above < rem && rem <= above + hist[tid]) {   // exactly one digit satisfies this
                    s_prefix = prefix | (static_cast<uint32_t>(tid) << shift);
                    s_remaining = rem - above;
                    s_equal = hist[tid];            // after the last pass: the keys equal to the threshold
                }
            }
            __syncthreads();
        }
    }
    __syncthreads();
    const uint32_t thr = s_prefix;
    const int admit_equal = static_cast<int>(s_remaining);  // keys equal to thr to admit, in index order
    // every key equal to the threshold is admitted (no tie straddles the cut, the usual case): no ordering needed
    const bool all_equal_in = need_select && admit_equal == static_cast<int>(s_equal);
    const int wave = tid / kWave;
    int running = 0;
    for (int base = 0; base < T_tok; base += kSelThreads) {
        const int i = base + tid;
        const bool valid = i < T_tok;
        bool sel;
        if (!need_select) {
            sel = (m > 0);
        } else if (all_equal_in) {
            sel = valid && order_key(scores[static_cast<size_t>(i) * kc + slot]) >= thr;
        } else {
            const uint32_t key = valid ? order_key(scores[static_cast<size_t>(i) * kc + slot]) : 0u;
            const bool eq = valid && key == thr;
            const uint64_t b = __ballot(eq);
            if (lane_id() == 0) wave_cnt[wave] = __popcll(b);
            __syncthreads();
            int before = running + __popcll(b & lanemask_lt());
            int total = 0;
            for (int w = 0; w < kSelWaves; ++w) {
                const int c = wave_cnt[w];
                if (w < wave) before += c;
                total += c;
            }
            running += total;
            sel = valid && (key > thr || (eq && before < admit_equal));
            __syncthreads();
        }
        if (valid) {
            for (int j = 0; j < kc; ++j) {
                uint8_t v;
                if (j >= k) v = 1;                                   // shared expert: fresh in every step
                else if (token_mode) v = sel ? 1 : 0;
                else v = (j < slot) ? 1 : (j == slot ? (sel ? 1 : 0) : 0);
                mask[static_cast<size_t>(i) * kc + j] = v;
            }
        }
    }
}

template <int KPT>
__global__ __launch_bounds__(kSelThreads) void refresh_select_kernel(RefreshRule rule, int T_tok)
{
    __shared__ SelectShared sh;
    const int kc = rule.k + rule.n_shared;
    if (threadIdx.x == 0) *rule.n_refresh = rule.n_value;
    bool sel[KPT];
    select_tokens<KPT>(rule, T_tok, sh, sel);
    auto write = [&](auto byte_of) {
#pragma unroll
        for (int u = 0; u < KPT; ++u) {
            const int i = u * kSelThreads + static_cast<int>(threadIdx.x);
            if (i < T_tok)
                for (int j = 0; j < kc; ++j) rule.mask[static_cast<size_t>(i) * kc + j] = byte_of(j, sel[u]);
        }
    };
    if (rule.token_mode) write([&](int j, bool s) -> uint8_t { return s || j >= rule.k ? 1 : 0; });
    else write([&](int j, bool s) { return selected_mask(rule, j, s); });
}

hipError_t launch_refresh(const RefreshRule& rule, int T_tok, hipStream_t stream)
{
    if (!rule.select) {
        const int N = T_tok * (rule.k + rule.n_shared);
        hipLaunchKernelGGL(refresh_simple_kernel, dim3(N > 0 ? (N + 255) / 256 : 1), dim3(256), 0, stream, rule, N);
        return hipGetLastError();
    }
#define DICEMOE_SELECT(KPT_) hipLaunchKernelGGL(refresh_select_kernel<KPT_>, dim3(1), dim3(kSelThreads), 0, stream, rule, T_tok)
    if (T_tok < 1 || T_tok > 16 * kSelThreads)
        hipLaunchKernelGGL(refresh_select_any_kernel, dim3(1), dim3(kSelThreads), 0, stream, rule.scores, T_tok, rule.k + rule.n_shared,
                           rule.k, rule.slot, rule.m, rule.token_mode, rule.n_value, rule.mask, rule.n_refresh);
    else if (T_tok <= kSelThreads) DICEMOE_SELECT(1);
    else if (T_tok <= 2 * kSelThreads) DICEMOE_SELECT(2);
    else if (T_tok <= 4 * kSelThreads) DICEMOE_SELECT(4);
    else if (T_tok <= 8 * kSelThreads) DICEMOE_SELECT(8);
    else DICEMOE_SELECT(16);
#undef DICEMOE_SELECT
    return hipGetLastError();
}

}  // namespace dicemoe
