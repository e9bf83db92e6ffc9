// Host-side launchers of the gfx950 kernels (one per translation unit); the C-ABI in api.hip
// validates arguments and calls these.  Every launcher only enqueues work on `stream`.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ffn_plan.hpp"

namespace dicemoe {

// scores / idx have k + n_shared columns: the k routed slots, then slot k+s = (expert E+s, score 1)
hipError_t launch_gate(bool bf16, const void* x, const void* Wg, const float* bg, int T_tok, int d, int E, int k,
                       int n_shared, int renorm, float* scores, int32_t* idx, float* probs, float* logits,
                       hipStream_t stream);

// What a step refreshes.  Elementwise policies (select 0), by kind: 0 all, 1 / 5 / 6 Algorithm 4 and its ablation variants, 4 none; off_step:
// step_t % stride_n != 0.  Selection (select 1): the exact top-m tokens by scores[i * (k + n_shared) + slot] (descending, ties to the
// lower token); token_mode: selected tokens get all k slots; otherwise slots < slot are all refreshed, slot `slot` follows the selection
// and later slots are not refreshed.  mask has k + n_shared columns; the shared slots are refreshed under every policy.  n_value is
// written to n_refresh (the refreshed pairs, shared slots included).
struct RefreshRule {
    int select, kind, k, n_shared, off_step;
    uint32_t seed;
    int slot, m, token_mode, n_value;
    const float* scores;
    uint8_t* mask;
    int32_t* n_refresh;
};
hipError_t launch_refresh(const RefreshRule& rule, int T_tok, hipStream_t stream);

// scratch: dispatch_scratch_bytes(T_tok * k, E) bytes of device memory (per-workgroup expert counts handed
// from the counting launch to the placing launch); may be null when that size is 0
hipError_t launch_dispatch(bool bf16, const void* x, const int32_t* idx, const uint8_t* mask, int T_tok, int d,
                           int E, int k, void* x_packed, int32_t* counts, int32_t* offsets, int32_t* perm,
                           int32_t* inv, int32_t* scratch, hipStream_t stream, const RefreshRule* rule = nullptr);
// rule: if given, the mask is formed first and written to rule->mask (which `mask` has to be), by the dispatch's own launches
// where they can and by launch_refresh otherwise
size_t dispatch_scratch_bytes(long long n_pairs, int E);
// The library's own scratch for launch_dispatch: a file-scope device array of dispatch_static_scratch_bytes()
// bytes; *out receives its address on the current device (looked up once per device).  No allocation.
size_t dispatch_static_scratch_bytes();
hipError_t dispatch_static_scratch(int32_t** out);

hipError_t launch_combine(bool bf16, const void* h_packed, const int32_t* inv, const float* scores,
                          const uint8_t* mask, int T_tok, int d, int k, int k_cached, void* H_cache,
                          float* S_cache, int use_fresh, void* y, hipStream_t stream);

// Float partial sums that a split second GEMM has left in the workspace for the combine: row r of share i is
// partial[(i * rows + r) * d ..], and h row r = bf16(share 0 + share 1 + ... + bias of its expert).
struct SplitSums { const float* partial = nullptr; int shares = 0, rows = 0; const float* bias = nullptr; };
constexpr int kSumsMaxSlots = 4;
// The combine that adds the shares itself (bf16, k <= kSumsMaxSlots slots per token): every fresh row goes to h_packed (its
// packed row) or, where that is null, to its place in H_cache, as the second pass of the split would have put it, and y, H_cache and
// S_cache receive what launch_combine writes.  idx: segment of every pair, seg_expert: whose weights that segment has.
hipError_t launch_combine_sums(const SplitSums& sums, void* h_packed, const int32_t* inv, const float* scores, const int32_t* idx,
                               const int32_t* seg_expert, const uint8_t* mask, int T_tok, int d, int k, int k_cached, void* H_cache, float* S_cache,
                               int use_fresh, void* y, hipStream_t stream);

// The dispatch of a layer, left to the first GEMM: pairs p of token p / slots with expert expert_idx[p], all of them (rule.mask null) or
// those that an elementwise policy refreshes (where ffn_sorts_pairs says that it can).  Its index outputs and the mask are written as
// launch_dispatch writes them.
struct PairSort {
    const int32_t* expert_idx;
    int n_pairs, experts;
    RefreshRule rule;
    int32_t *counts, *offsets, *perm, *inv;
};

// x_rows is the packed buffer (row_index == nullptr) or the token matrix with row_index[r] / row_div
// naming the row that packed row r reads; the h row of packed row r is written to row r of h_out, or
// to row out_index[r] when out_index is given (scatter into a buffer indexed by pair id)
hipError_t launch_expert_ffn(bool bf16, const void* x_rows, const int32_t* row_index, int row_div,
                             const int32_t* seg_offsets, const int32_t* seg_expert, int n_seg, int n_experts, int max_rows, int d,
                             int F, const void* W1, const float* b1, const void* W2, const float* b2, void* h_out,
                             const int32_t* out_index, void* hidden, void* partial, size_t partial_bytes,
                             int32_t* status, hipStream_t stream, hipEvent_t between = nullptr, SplitSums* sums = nullptr,
                             const PairSort* sort = nullptr);
// sums: if given and the second GEMM is split, its second pass is left to launch_combine_sums and *sums says what to add (h_out and
// out_index are then not used); otherwise sums->shares stays 0
// sort: if given (ffn_sorts_pairs), row_index is its perm and seg_offsets its offsets, which the first GEMM writes
// between: if given, recorded on the stream after the first GEMM has been enqueued (per-GEMM timing)
// status (two int32 on the device, may be null): written by the first GEMM of every call, see
// report_row_overflow in ffn_mfma.hpp.
// Once per device before the first launch_expert_ffn there: raises the dynamic-LDS limit of the wide kernels.
hipError_t prepare_expert_ffn();

// S_buffer[p] = scores[p] for the routed slots (j < k_cached) of every pair with mask[p] != 0 (all if mask is null)
hipError_t launch_commit_scores(const float* scores, const uint8_t* mask, int T_tok, int k, int k_cached,
                                float* S_buffer, hipStream_t stream);

// measurement aids (calibrate.hip): a plain copy of `bytes` (multiple of 16) and a register-resident MFMA loop
// (operands: 16 x 256 x 96 bytes of bf16 bit patterns; flops = workgroups * 4 * iters * 8 * 32768)
hipError_t launch_calibrate_copy(void* dst, const void* src, size_t bytes, int workgroups, hipStream_t stream);
hipError_t launch_calibrate_mfma(const void* operands, float* sink, int iters, int workgroups, hipStream_t stream);

hipError_t launch_ep_segments(const int32_t* recv_counts, int n_seg, int E_loc, int32_t* seg_offsets,
                              int32_t* seg_expert, hipStream_t stream);

}  // namespace dicemoe
