// Router kernel: logits, top-K by logit (ties to the lower expert id), softmax scores.
// Follows Algorithm 1 of the paper ("[s, idx] <- router(x)") with K activated experts per
// token (Conditional Communication figure caption).
//
// gate_mfma_kernel puts the skinny GEMM on the matrix cores, bf16 and float storage alike; gate_few_kernel serves float
// rows of more than 1024 columns with one to four experts, where most of a 16 x 16 block of logits would be padding.
#include <type_traits>
#include "common.hpp"
#include "kernels.hpp"

namespace dicemoe {

// A value of the lane N places away inside the caller's row of 16 lanes (DPP row rotation; N = 1 .. 15
// visits every other lane of the row once).
template <int N>
__device__ __forceinline__ int row_rotate(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xF, 0xF, true);
}
template <int N>
__device__ __forceinline__ float row_rotate(float v) {
    return __builtin_bit_cast(float, row_rotate<N>(__builtin_bit_cast(int, v)));
}
template <int N, typename F>
__device__ __forceinline__ void for_row_rotations(F&& f) {
    if constexpr (N < 16) {
        f(std::integral_constant<int, N>{});
        for_row_rotations<N + 1>(f);
    }
}

// A workgroup owns 16 tokens; logits[16][E] = x[16][d] . Wg[E][d]^T
// is a chain of MFMA steps over k (64 bytes of a row each: one v_mfma_f32_16x16x32_bf16, or four
// v_mfma_f32_16x16x4_f32), split round robin over the 4 wavefronts
// (wavefront w takes k-steps w, w+4, ...).  Operands come straight from global memory in MFMA
// layout: lane l supplies row l%16 (a token for x, an expert for Wg) and the 16 bytes l/16 of
// the step, i.e. one 16-byte load each; all loads of a batch are issued before
// its MFMAs.  Float storage keeps four accumulators per component of those 16 bytes (a step takes the one of its place in the
// batch mod 4), so that a running sum is a sixteenth of a wavefront's share where batches have four steps or twelve, a twelfth with
// three, six or nine, and 3 / 40 with ten: the error of the scores stays that of a butterfly over the lanes.  Accumulator register v of lane l is logits[token 4*(l/16)+v][expert l%16].  The four
// partial sums meet in LDS and are added in wavefront order (fixed, reproducible).  With at most 16
// experts thread (t, e) then finishes logit e of token t: the 16 lanes of a DPP row hold one token and
// rank, maximum and softmax sum come from rotating the row (no further LDS trip, all 16 tokens at once);
// with more experts wavefront w finishes tokens 4w..4w+3 with lane e playing expert e.  Rank is by
// logit, ties to the lower id.
// U = k-steps per batch and wavefront: the launcher picks it so that one batch covers a wavefront's
// whole share of the row (a single round trip to memory) whenever that fits in registers.
template <typename T, int NB, int U>
__global__ __launch_bounds__(256) void gate_mfma_kernel(const T* __restrict__ x, const T* __restrict__ Wg,
                                                        const float* __restrict__ bg, int T_tok, int d, int E,
                                                        int k, int n_shared, int renorm, float* __restrict__ scores,
                                                        int32_t* __restrict__ expert_idx,
                                                        float* __restrict__ probs_all, float* __restrict__ logits)
{
    typedef RowMfma<T> M;
    constexpr int NC = M::kMfma == 1 ? 1 : 4 * M::kMfma;      // accumulators per block of experts
    constexpr int EP = NB * 16;                  // padded expert count
    auto sum_of_waves = [](float a, float b, float c, float d4) { return NC == 1 ? ((a + b) + c) + d4 : (a + b) + (c + d4); };
    __shared__ float part[4][16][EP];
    __shared__ float zfin[16][EP];
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int row = lane & 15, kq = lane >> 4;
    const int tok0 = blockIdx.x * 16;
    int tok = tok0 + row;
    if (tok >= T_tok) tok = T_tok - 1;           // rows past the end repeat the last token; never written
    const u32x4_t* xa = reinterpret_cast<const u32x4_t*>(x + static_cast<size_t>(tok) * d);
    const u32x4_t* wb[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        int e = nb * 16 + row;
        if (e >= E) e = E - 1;                   // padding columns repeat the last expert; ignored later
        wb[nb] = reinterpret_cast<const u32x4_t*>(Wg + static_cast<size_t>(e) * d);
    }
    f32x4_t acc[NB][NC];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[nb][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int nsteps = d / M::kUnit;
    for (int s0 = wave; s0 < nsteps; s0 += 4 * U) {
        u32x4_t av[U], bv[NB][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int sidx = s0 + 4 * u;
            const bool on = sidx < nsteps;
            const int unit = (on ? sidx : s0) * 4 + kq;
            av[u] = xa[unit];
            if (!on) av[u] = u32x4_t{0u, 0u, 0u, 0u};      // a step past the end contributes zero
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                bv[nb][u] = wb[nb][unit];
                if (NC > 1 && !on) bv[nb][u] = u32x4_t{0u, 0u, 0u, 0u};      // (float: an infinite weight times zero would not)
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int c = 0; c < M::kMfma; ++c) {
                    const int to = NC == 1 ? 0 : (u & 3) * M::kMfma + c;
                    acc[nb][to] = M::step(av[u], bv[nb][u], acc[nb][to], c);
                }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float sum = acc[nb][0][v];
            if constexpr (NC == 16) {
                float set[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    set[q] = (acc[nb][4 * q][v] + acc[nb][4 * q + 1][v]) + (acc[nb][4 * q + 2][v] + acc[nb][4 * q + 3][v]);
                sum = (set[0] + set[1]) + (set[2] + set[3]);
            }
            part[wave][4 * kq + v][nb * 16 + row] = sum;
        }
    __syncthreads();
    if (NB == 1) {
        // Up to 16 experts: thread (t, e) = (tid / 16, tid % 16) finishes logit e of token t, so a row of 16
        // lanes is one token and every lane meets the 15 other logits of its token by rotating the row.
        const int t = threadIdx.x >> 4, e = threadIdx.x & 15;
        const bool is_expert = e < E;
        float z = sum_of_waves(part[0][t][e], part[1][t][e], part[2][t][e], part[3][t][e]);      // then the bias
        if (bg && is_expert) z += bg[e];
        const float z_me = is_expert ? z : -INFINITY;       // padding lanes never outrank an expert
        float zmax = z_me;
        int rank = 0;
        for_row_rotations<1>([&](auto n) {
            const float z_o = row_rotate<decltype(n)::value>(z_me);
            const int e_o = row_rotate<decltype(n)::value>(e);
            zmax = fmaxf(zmax, z_o);
            rank += (z_o > z_me || (z_o == z_me && e_o < e)) ? 1 : 0;
        });
        const float q_me = is_expert ? expf(z_me - zmax) : 0.f;
        float denom = q_me;
        for_row_rotations<1>([&](auto n) { denom += row_rotate<decltype(n)::value>(q_me); });
        const float p_me = q_me / denom;
        const bool chosen = is_expert && rank < k;
        float s_me = p_me;
        if (renorm) {
            const float c_me = chosen ? p_me : 0.f;
            float ssum = c_me;
            for_row_rotations<1>([&](auto n) { ssum += row_rotate<decltype(n)::value>(c_me); });
            s_me = p_me / ssum;
        }
        const int tk = tok0 + t;
        if (tk < T_tok) {
            const size_t row = static_cast<size_t>(tk) * (k + n_shared);
            if (chosen) {
                scores[row + rank] = s_me;
                expert_idx[row + rank] = e;
            }
            for (int sh = e; sh < n_shared; sh += 16) {     // shared experts: every token, score 1
                scores[row + k + sh] = 1.0f;
                expert_idx[row + k + sh] = E + sh;
            }
            if (is_expert) {
                if (probs_all) probs_all[static_cast<size_t>(tk) * E + e] = p_me;
                if (logits) logits[static_cast<size_t>(tk) * E + e] = z_me;
            }
        }
        return;
    }
    // logits: the four partial sums in wavefront order, then the bias
    for (int i = threadIdx.x; i < 16 * EP; i += blockDim.x) {
        const int t = i / EP, e = i % EP;
        float z = sum_of_waves(part[0][t][e], part[1][t][e], part[2][t][e], part[3][t][e]);
        if (bg && e < E) z += bg[e];
        zfin[t][e] = z;
    }
    __syncthreads();

    for (int tt = 0; tt < 4; ++tt) {
        const int t = wave * 4 + tt;
        const int tk = tok0 + t;
        if (tk >= T_tok) break;                  // uniform across the wavefront
        const bool is_expert = lane < E;
        const float z_me = is_expert ? zfin[t][lane] : -INFINITY;
        float zmax = -INFINITY;
        for (int e = 0; e < E; ++e) zmax = fmaxf(zmax, zfin[t][e]);
        float denom = 0.f;
        int rank = 0;
        for (int e = 0; e < E; ++e) {
            const float z = zfin[t][e];
            denom += expf(z - zmax);
            rank += (z > z_me || (z == z_me && e < lane)) ? 1 : 0;
        }
        const float p_me = is_expert ? expf(z_me - zmax) / denom : 0.f;
        const bool chosen = is_expert && rank < k;
        float s_me = p_me;
        if (renorm) {
            const float ssum = wave_sum(chosen ? p_me : 0.f);
            s_me = p_me / ssum;
        }
        const size_t row = static_cast<size_t>(tk) * (k + n_shared);
        if (chosen) {
            scores[row + rank] = s_me;
            expert_idx[row + rank] = lane;
        }
        if (lane < n_shared) {                          // shared experts: every token, score 1
            scores[row + k + lane] = 1.0f;
            expert_idx[row + k + lane] = E + lane;
        }
        if (is_expert) {
            if (probs_all) probs_all[static_cast<size_t>(tk) * E + lane] = p_me;
            if (logits) logits[static_cast<size_t>(tk) * E + lane] = z_me;
        }
    }
}

// Float rows, at most four experts.  A wavefront owns TPW tokens: each lane loads its 16-byte slices of all TPW rows (NCH per row,
// whole lines, in flight while the workgroup stages the router matrix in LDS), multiplies them with the matching slices of
// every router row, and the E x TPW sums are reduced over the 64 lanes with a fixed butterfly; then lane e plays expert e.
// Bound by the latency of one round trip to memory where the matrix cores' k-steps are a chain of several.
constexpr int kFewExperts = 4;
template <int NCH, int TPW>
__global__ __launch_bounds__(256) void gate_few_kernel(const float* __restrict__ x, const float* __restrict__ Wg,
                                                       const float* __restrict__ bg, int T_tok, int d, int E, int k,
                                                       int n_shared, int renorm, float* __restrict__ scores,
                                                       int32_t* __restrict__ expert_idx, float* __restrict__ probs_all,
                                                       float* __restrict__ logits)
{
    constexpr int V = Store<float>::kVec;
    extern __shared__ u32x4_t lds_w[];
    const int nvec = d / V;
    const u32x4_t* wsrc = reinterpret_cast<const u32x4_t*>(Wg);
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int tok0 = (blockIdx.x * (blockDim.x / kWave) + wave) * TPW;

    // this lane's slices of the TPW rows (rows past the end repeat the last token; never written)
    u32x4_t xv[TPW][NCH];
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        int tok = tok0 + t;
        if (tok >= T_tok) tok = T_tok - 1;
        const u32x4_t* xr = reinterpret_cast<const u32x4_t*>(x + static_cast<size_t>(tok) * d);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int i = lane + c * kWave;
            xv[t][c] = xr[i < nvec ? i : 0];
        }
    }
    for (int v = threadIdx.x; v < E * nvec; v += blockDim.x) lds_w[v] = wsrc[v];
    __syncthreads();
    if (tok0 >= T_tok) return;

    float acc[TPW][kFewExperts];
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
        for (int e = 0; e < kFewExperts; ++e) acc[t][e] = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int i = lane + c * kWave;
        if (i < nvec) {
            float xf[TPW][V];
#pragma unroll
            for (int t = 0; t < TPW; ++t) Store<float>::unpack(xv[t][c], xf[t]);
#pragma unroll
            for (int e = 0; e < kFewExperts; ++e) {
                if (e < E) {
                    float wf[V];
                    Store<float>::unpack(lds_w[e * nvec + i], wf);
#pragma unroll
                    for (int t = 0; t < TPW; ++t)
#pragma unroll
                        for (int u = 0; u < V; ++u) acc[t][e] = fmaf(xf[t][u], wf[u], acc[t][e]);
                }
            }
        }
    }

#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int tok = tok0 + t;
        if (tok >= T_tok) break;                 // uniform across the wavefront
        float zmax = -INFINITY;
#pragma unroll
        for (int e = 0; e < kFewExperts; ++e) {
            if (e < E) {
                acc[t][e] = wave_sum(acc[t][e]);
                if (bg) acc[t][e] += bg[e];
                zmax = fmaxf(zmax, acc[t][e]);
            }
        }
        // lane e is expert e
        float z_me = -INFINITY;
        float denom = 0.f;
#pragma unroll
        for (int e = 0; e < kFewExperts; ++e) {
            if (e < E) {
                if (lane == e) z_me = acc[t][e];
                denom += expf(acc[t][e] - zmax);
            }
        }
        int rank = 0;
#pragma unroll
        for (int e = 0; e < kFewExperts; ++e)
            if (e < E) rank += (acc[t][e] > z_me || (acc[t][e] == z_me && e < lane)) ? 1 : 0;
        const bool is_expert = lane < E;
        const float p_me = is_expert ? expf(z_me - zmax) / denom : 0.f;
        const bool chosen = is_expert && rank < k;
        float s_me = p_me;
        if (renorm) {
            const float ssum = wave_sum(chosen ? p_me : 0.f);
            s_me = p_me / ssum;
        }
        const size_t row = static_cast<size_t>(tok) * (k + n_shared);
        if (chosen) {
            scores[row + rank] = s_me;
            expert_idx[row + rank] = lane;
        }
        if (lane < n_shared) {                      // shared experts: every token, score 1
            scores[row + k + lane] = 1.0f;
            expert_idx[row + k + lane] = E + lane;
        }
        if (is_expert) {
            if (probs_all) probs_all[static_cast<size_t>(tok) * E + lane] = p_me;
            if (logits) logits[static_cast<size_t>(tok) * E + lane] = z_me;
        }
    }
}

template <int NCH, int TPW>
static hipError_t launch_gate_few(const float* x, const float* Wg, const float* bg, int T_tok, int d, int E, int k, int n_shared,
                                  int renorm, float* scores, int32_t* idx, float* probs, float* logits, hipStream_t stream)
{
    hipLaunchKernelGGL((gate_few_kernel<NCH, TPW>), dim3((T_tok + 4 * TPW - 1) / (4 * TPW)), dim3(256),
                       static_cast<size_t>(E) * d * sizeof(float), stream, x, Wg, bg, T_tok, d, E, k, n_shared, renorm, scores, idx,
                       probs, logits);
    return hipGetLastError();
}

template <typename T, int NB>
static hipError_t launch_gate_mfma_nb(const T* x, const T* Wg, const float* bg, int T_tok, int d, int E, int k,
                                      int n_shared, int renorm, float* scores, int32_t* idx, float* probs, float* logits,
                                      hipStream_t stream)
{
    const int blocks = (T_tok + 15) / 16;
    const int need = (d / RowMfma<T>::kUnit + 3) / 4;      // k-steps per wavefront
    // Float, up to 16 experts: long rows in batches of four.  In batches of sixteen the 18 steps of d = 1152 cost as much as 32; full
    // batches lose too, at the same register count (why was not separated).  us at 500 and 8192 tokens, batches of 16 / of 4: 8 experts
    // of 1152, 11.8 / 7.0 and 20.4 / 11.0; 16 experts of 2048, 13.1 / 10.2 and 26.0 / 18.1.  Up to ten steps one batch is faster
    // (16 experts of 576, 5.2 / 5.9).  The accumulator of a step is its number mod 4 either way: the same bits.
    if constexpr (RowMfma<T>::kMfma > 1 && NB == 1) {
        if (need > 10) {
            hipLaunchKernelGGL((gate_mfma_kernel<T, NB, 4>), dim3(blocks), dim3(256), 0, stream, x, Wg, bg, T_tok, d, E, k, n_shared,
                               renorm, scores, idx, probs, logits);
            return hipGetLastError();
        }
    }
    // registers per lane: 4 * U * (1 + NB) for the operands of a batch
    constexpr int UMAX = NB == 1 ? 16 : (NB == 2 ? 10 : 6);
#define DICEMOE_GATE_U(U_)                                                                                          \
    if (need <= U_ || U_ == UMAX) {                                                                                 \
        hipLaunchKernelGGL((gate_mfma_kernel<T, NB, U_>), dim3(blocks), dim3(256), 0, stream, x, Wg, bg, T_tok, d, E, \
                           k, n_shared, renorm, scores, idx, probs, logits);                                        \
        return hipGetLastError();                                                                                   \
    }
    DICEMOE_GATE_U(3)
    DICEMOE_GATE_U(6)
    if (UMAX >= 9) { DICEMOE_GATE_U((UMAX >= 9 ? 9 : UMAX)) }
    if (UMAX >= 10) { DICEMOE_GATE_U((UMAX >= 10 ? 10 : UMAX)) }
    if (UMAX >= 12) { DICEMOE_GATE_U((UMAX >= 12 ? 12 : UMAX)) }
    if (UMAX >= 16) { DICEMOE_GATE_U((UMAX >= 16 ? 16 : UMAX)) }
#undef DICEMOE_GATE_U
    return hipErrorInvalidValue;                 // not reached: the last case of every NB takes any d
}

template <typename T>
static hipError_t launch_gate_mfma(const void* x, const void* Wg, const float* bg, int T_tok, int d, int E, int k,
                                   int n_shared, int renorm, float* scores, int32_t* idx, float* probs, float* logits,
                                   hipStream_t stream)
{
    const T* xs = static_cast<const T*>(x);
    const T* ws = static_cast<const T*>(Wg);
    // us, few / matrix cores: one expert of 2048 columns, 1024 tokens 4.6 / 8.9, 8192: 13.4 / 14.6; two of 1152: 5.4 / 6.7 and 9.0 / 10.2;
    // four of 4096, 1024 tokens: 11.2 / 13.6, 6000: 39 / 25 (41 with batches of sixteen), 8192: 54 / 28; up to 1024 columns a router of
    // two and more is faster on the matrix cores.
    if constexpr (std::is_same_v<T, float>) {
        if (d > 1024 && d <= 4096 && (E <= 2 || (E <= kFewExperts && T_tok <= 6144))) {
            if (d <= 2048) return launch_gate_few<8, 2>(xs, ws, bg, T_tok, d, E, k, n_shared, renorm, scores, idx, probs, logits, stream);
            return launch_gate_few<16, 1>(xs, ws, bg, T_tok, d, E, k, n_shared, renorm, scores, idx, probs, logits, stream);
        }
    }
    if (E <= 16) return launch_gate_mfma_nb<T, 1>(xs, ws, bg, T_tok, d, E, k, n_shared, renorm, scores, idx, probs, logits, stream);
    if (E <= 32) return launch_gate_mfma_nb<T, 2>(xs, ws, bg, T_tok, d, E, k, n_shared, renorm, scores, idx, probs, logits, stream);
    return launch_gate_mfma_nb<T, 4>(xs, ws, bg, T_tok, d, E, k, n_shared, renorm, scores, idx, probs, logits, stream);
}

hipError_t launch_gate(bool bf16, const void* x, const void* Wg, const float* bg, int T_tok, int d, int E, int k,
                       int n_shared, int renorm, float* scores, int32_t* idx, float* probs, float* logits, hipStream_t stream)
{
    if (bf16) return launch_gate_mfma<bf16_t>(x, Wg, bg, T_tok, d, E, k, n_shared, renorm, scores, idx, probs, logits, stream);
    return launch_gate_mfma<float>(x, Wg, bg, T_tok, d, E, k, n_shared, renorm, scores, idx, probs, logits, stream);
}

}  // namespace dicemoe
