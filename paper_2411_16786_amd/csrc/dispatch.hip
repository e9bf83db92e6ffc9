// Dispatch on one device (Algorithm 1, "x_d <- all2all_dispatch(x, idx)"): group the refreshed
// (token, slot) pairs by destination expert with a stable counting sort, then gather the token
// rows into the expert-contiguous buffer.
//
// Index kernels (count, then place; no workgroup waits for another).  Workgroup b owns the
// contiguous pair ids [b*256*S, (b+1)*256*S), wave w of it a contiguous quarter, and a wave walks
// its range in steps of 64, so "workgroup, wave, step, lane" is ascending pair id and the sort is
// stable by construction.
//   dispatch_count_kernel: per-workgroup, per-expert counts of refreshed pairs -> scratch[b][e].
//   dispatch_place_kernel: every workgroup sums the scratch table into the experts' totals and
//     into the counts of the workgroups before it (grids beyond 256 workgroups: dispatch_scan_kernel
//     has done that once for all of them), scans the totals into the experts' offsets,
//     ranks its own pairs (lanes that hold the same expert find each other with one ballot per bit
//     of the expert id; per-wave, per-expert running counts in LDS), and writes perm / inv.
//     Up to 4096 pairs one workgroup of 1024 threads places them all: no table and no count launch.
// All integer work; the only atomics are integer adds in LDS: the result is unique.
//
// dispatch_gather_kernel: one wavefront per token reads the row once (16 bytes per lane per
// pass) and stores it to each of its refreshed slots' packed rows; bound by HBM traffic
// T*d*b read + R*d*b written.
#include <mutex>
#include <type_traits>

#include "pair_sort.hpp"

namespace dicemoe {

constexpr int kIdxThreads = 256;
constexpr int kIdxWaves = kIdxThreads / kWave;
// Pairs that one workgroup sorts alone.  One call of 28 in a graph, us, alone / counting and placing over many workgroups: 8 experts,
// 2049 pairs 3.8 / 4.8, 4096: 4.7 / 4.9, 4097: 5.5 / 4.9, 8192: 7.4 / 5.0; 64 experts, 4096: 5.6 / 6.2, 4097: 6.6 / 6.6, 8192: 9.1 / 7.7.
// (Durations of a kernel trace mislead here: about 2 us of each are a launch's own, which in a row of launches overlap.)  Up to 256
// pairs four wavefronts do it: fewer to wait for at the barriers.
constexpr int kAlonePairs = 4096;
constexpr int kNoScratchPairs = 2048;         // (a promise of moe_dispatch: up to these the workspace may be null)

// Where the dispatch takes the mask from: an array (or none: every pair), an elementwise policy, or a selection of tokens
// made by this workgroup (`bits`: one bit per token, in LDS).  The mask of the last two is written out by the way.
enum MaskSource { kMaskArray, kMaskSimple, kMaskSelect };
struct NoRule {};
template <int SOURCE> using Rule = std::conditional_t<SOURCE == kMaskArray, NoRule, RefreshRule>;

// Expert ids of this wave's S steps, -1 where the pair is past the end, not refreshed or carries a
// bad id.  The loads are unconditional (index clamped) so that all of them are in flight at once.
template <int S, int SOURCE>
__device__ __forceinline__ void load_steps(const int32_t* __restrict__ expert_idx, const uint8_t* __restrict__ mask,
                                           int p0, int lane, int N, int E, const Rule<SOURCE>& rule, const uint32_t* bits, int (&ev)[S]) {
    uint8_t mv[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int p = p0 + u * kWave + lane;
        ev[u] = expert_idx[p < N ? p : N - 1];
    }
    if constexpr (SOURCE == kMaskSimple) {
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const int p = p0 + u * kWave + lane;
            mv[u] = simple_mask(rule, p);
            if (p < N) rule.mask[p] = mv[u];
        }
    } else if constexpr (SOURCE == kMaskSelect) {
        const int kc = rule.k + rule.n_shared;
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const int p = p0 + u * kWave + lane;
            const int tok = (p < N ? p : N - 1) / kc;
            mv[u] = selected_mask(rule, p - tok * kc, (bits[tok >> 5] >> (tok & 31)) & 1u);
            if (p < N) rule.mask[p] = mv[u];
        }
    } else if (mask != nullptr) {
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const int p = p0 + u * kWave + lane;
            mv[u] = mask[p < N ? p : N - 1];
        }
    } else {
#pragma unroll
        for (int u = 0; u < S; ++u) mv[u] = 1;
    }
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int p = p0 + u * kWave + lane;
        ev[u] = has_row(p, N, ev[u], E) && mv[u] != 0 ? ev[u] : -1;
    }
}

template <int S, int SOURCE>
__global__ __launch_bounds__(kIdxThreads) void dispatch_count_kernel(const int32_t* __restrict__ expert_idx,
                                                                    const uint8_t* __restrict__ mask, int N, int E,
                                                                    int32_t* __restrict__ block_counts, Rule<SOURCE> rule)
{
    if constexpr (SOURCE == kMaskSimple)
        if (blockIdx.x == 0 && threadIdx.x == 0) *rule.n_refresh = rule.n_value;
    __shared__ int cnt[kMaxExperts];
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();
    const int nbits = E > 1 ? 32 - __builtin_clz(static_cast<unsigned>(E - 1)) : 0;
    if (tid < kMaxExperts) cnt[tid] = 0;
    __syncthreads();
    const int p0 = (static_cast<int>(blockIdx.x) * kIdxWaves + wave) * kWave * S;
    if (p0 < N) {                                           // wave-uniform
        int ev[S];
        load_steps<S, SOURCE>(expert_idx, mask, p0, lane, N, E, rule, nullptr, ev);
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const bool live = ev[u] >= 0;
            const int e = live ? ev[u] : 0;
            const uint64_t peers = same_expert_peers(live, e, nbits);
            if (live && (peers & lanemask_lt()) == 0) atomicAdd(&cnt[e], __popcll(peers));   // one add per expert and step
        }
    }
    __syncthreads();
    if (tid < E) block_counts[static_cast<size_t>(blockIdx.x) * E + tid] = cnt[tid];
}

// Grids beyond 256 workgroups: one workgroup turns the table of per-workgroup counts into exclusive
// prefixes over the workgroups (row b: pairs of each expert in the workgroups before b) and appends the
// totals as row n_blocks, so that every placing workgroup reads two rows instead of the whole table.
// Wave w takes experts w, w + 16, ...; lane l of it owns a contiguous run of workgroups.
__global__ __launch_bounds__(1024) void dispatch_scan_kernel(int32_t* __restrict__ block_counts, int n_blocks, int E)
{
    const int wave = threadIdx.x / kWave;
    const int lane = lane_id();
    const int per_lane = (n_blocks + kWave - 1) / kWave;
    const int b_lo = lane * per_lane;
    const int b_hi = (b_lo + per_lane < n_blocks) ? b_lo + per_lane : n_blocks;
    for (int e = wave; e < E; e += 1024 / kWave) {
        int run = 0;
        for (int bb = b_lo; bb < b_hi; ++bb) run += block_counts[static_cast<size_t>(bb) * E + e];
        const int incl = wave_scan(run);
        int prefix = incl - run;
        for (int bb = b_lo; bb < b_hi; ++bb) {
            const int c = block_counts[static_cast<size_t>(bb) * E + e];
            block_counts[static_cast<size_t>(bb) * E + e] = prefix;
            prefix += c;
        }
        if (lane == kWave - 1) block_counts[static_cast<size_t>(n_blocks) * E + e] = incl;
    }
}

// SOURCE other than the array: one workgroup alone, which forms the mask (the selection: of up to 1024 S tokens)
template <int S, int THREADS, int SOURCE>
__global__ __launch_bounds__(THREADS) void dispatch_place_kernel(const int32_t* __restrict__ expert_idx,
                                                                    const uint8_t* __restrict__ mask, int N, int E,
                                                                    const int32_t* __restrict__ block_counts,
                                                                    int prefix_ready, int32_t* __restrict__ counts,
                                                                    int32_t* __restrict__ offsets,
                                                                    int32_t* __restrict__ perm,
                                                                    int32_t* __restrict__ inv, Rule<SOURCE> rule)
{
    constexpr int WAVES = THREADS / kWave;
    static_assert(SOURCE != kMaskSelect || THREADS == kSelThreads, "the selection is made by 1024 threads");
    __shared__ uint32_t sel_bits[SOURCE == kMaskSelect ? 32 * S : 1];
    __shared__ int wave_run[WAVES][kMaxExperts];       // running count of a wave's pairs per expert; then the pairs of the waves before it
    __shared__ int s_tot[kMaxExperts];                 // pairs per expert over all workgroups
    __shared__ int s_pre[kMaxExperts];                 // pairs per expert in the workgroups before this one
    __shared__ int s_off[kMaxExperts + 1];
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = lane_id();
    const int b = blockIdx.x;
    const int n_blocks = gridDim.x;
    const int nbits = E > 1 ? 32 - __builtin_clz(static_cast<unsigned>(E - 1)) : 0;
    wave_run[tid / kMaxExperts][tid % kMaxExperts] = 0;   // the threads cover the WAVES x 64 table
    if (tid < kMaxExperts) { s_tot[tid] = 0; s_pre[tid] = 0; }
    if constexpr (SOURCE != kMaskArray)
        if (tid == 0) *rule.n_refresh = rule.n_value;
    if constexpr (SOURCE == kMaskSelect) {
        __shared__ SelectShared sel_shared;
        bool sel[S];
        select_tokens<S>(rule, N / (rule.k + rule.n_shared), sel_shared, sel);
#pragma unroll
        for (int u = 0; u < S; ++u) {                      // token u * 1024 + tid
            const uint64_t b = __ballot(sel[u]);
            if (lane < 2) sel_bits[(u * WAVES + wave) * 2 + lane] = static_cast<uint32_t>(b >> (32 * lane));
        }
    }
    __syncthreads();

    // the table of the other workgroups' counts: totals, and the part that precedes this workgroup.  Large
    // grids (prefix_ready) find both already summed by dispatch_scan_kernel: row b holds the counts of the
    // workgroups before b, row n_blocks the totals.
    if (n_blocks > 1 && prefix_ready) {
        if (tid < E) {
            s_pre[tid] = block_counts[static_cast<size_t>(b) * E + tid];
            s_tot[tid] = block_counts[static_cast<size_t>(n_blocks) * E + tid];
        }
    } else if (n_blocks > 1) {
        for (int i = tid; i < n_blocks * E; i += THREADS) {
            const int c = block_counts[i];
            const int bb = i / E, e = i - bb * E;
            if (c != 0) {
                atomicAdd(&s_tot[e], c);
                if (bb < b) atomicAdd(&s_pre[e], c);
            }
        }
    }

    // rank of each of this wave's pairs among the wave's pairs of the same expert
    const int p0 = (b * WAVES + wave) * kWave * S;
    int ev[S], rank[S];
    if (p0 < N) {                                           // wave-uniform
        load_steps<S, SOURCE>(expert_idx, mask, p0, lane, N, E, rule, sel_bits, ev);
#pragma unroll
        for (int u = 0; u < S; ++u) rank[u] = rank_step(ev[u], nbits, wave_run[wave]);
    } else {
#pragma unroll
        for (int u = 0; u < S; ++u) { ev[u] = -1; rank[u] = 0; }
    }
    __syncthreads();
    if (tid < E) {
        const int t = counts_to_prefixes<WAVES>(wave_run[0], tid);
        if (n_blocks == 1) s_tot[tid] = t;
    }
    __syncthreads();
    // exclusive scan over the experts: lane e of the first wave holds expert e's total
    if (wave == 0) {
        const int mine = lane < E ? s_tot[lane] : 0;
        const int incl = wave_scan(mine);
        if (lane < E) {
            s_off[lane] = incl - mine;
            if (b == 0) { counts[lane] = mine; offsets[lane] = incl - mine; }
        }
        if (lane == E - 1) {
            s_off[E] = incl;
            if (b == 0) offsets[E] = incl;
        }
    }
    __syncthreads();
    const int R = s_off[E];

    if (p0 < N) {
#pragma unroll
        for (int u = 0; u < S; ++u) {
            const int p = p0 + u * kWave + lane;
            const int e = ev[u];
            leave_index(p, N, e >= 0, [&] { return s_off[e] + s_pre[e] + wave_run[wave][e] + rank[u]; }, R, perm, inv);
        }
    }
}

// NP > 0: a row is at most NP passes of 64 lanes x 16 bytes; all passes are loaded before the first
// store (one memory round trip per token); NP == 0: any row length, pass by pass.
template <typename T, int NP>
__global__ __launch_bounds__(256) void dispatch_gather_kernel(const T* __restrict__ x, const int32_t* __restrict__ inv,
                                                              int T_tok, int d, int k, int all_pairs, T* __restrict__ x_packed)
{
    constexpr int V = Store<T>::kVec;
    const int tok = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (tok >= T_tok) return;
    const int lane = lane_id();
    const int nvec = d / V;
    const int32_t* rows = inv + static_cast<size_t>(tok) * k;
    const u32x4_t* src = reinterpret_cast<const u32x4_t*>(x + static_cast<size_t>(tok) * d);
    u32x4_t* dst = reinterpret_cast<u32x4_t*>(x_packed);
    if (NP > 0 && all_pairs) {
        // every pair is refreshed: the row is needed whatever inv says, so its loads go out together with
        // the loads of the destinations instead of behind them
        constexpr int NPN = NP > 0 ? NP : 1;
        u32x4_t v[NPN];
#pragma unroll
        for (int p = 0; p < NPN; ++p) {
            const int c = lane + p * kWave;
            v[p] = c < nvec ? src[c] : u32x4_t{0u, 0u, 0u, 0u};
        }
        for (int j = 0; j < k; ++j) {
            const int r = rows[j];
            if (r < 0) continue;
#pragma unroll
            for (int p = 0; p < NPN; ++p) {
                const int c = lane + p * kWave;
                if (c < nvec) dst[static_cast<size_t>(r) * nvec + c] = v[p];
            }
        }
        return;
    }
    bool any = false;
    for (int j = 0; j < k; ++j) any |= rows[j] >= 0;
    if (!any) return;
    if (NP > 0) {
        constexpr int NPN = NP > 0 ? NP : 1;
        u32x4_t v[NPN];
#pragma unroll
        for (int p = 0; p < NPN; ++p) {
            const int c = lane + p * kWave;
            v[p] = c < nvec ? src[c] : u32x4_t{0u, 0u, 0u, 0u};
        }
        for (int j = 0; j < k; ++j) {
            const int r = rows[j];
            if (r < 0) continue;
#pragma unroll
            for (int p = 0; p < NPN; ++p) {
                const int c = lane + p * kWave;
                if (c < nvec) dst[static_cast<size_t>(r) * nvec + c] = v[p];
            }
        }
    } else {
        for (int c = lane; c < nvec; c += kWave) {
            const u32x4_t v = src[c];
            for (int j = 0; j < k; ++j) {
                const int r = rows[j];
                if (r >= 0) dst[static_cast<size_t>(r) * nvec + c] = v;
            }
        }
    }
}

// Steps per wave and workgroups of the counting and placing kernels for N pairs: the fewest steps (1, 2, 4, 8) that keep the grid
// at 256 workgroups or fewer; beyond 2^19 pairs the grid grows instead.
static void dispatch_plan(long long N, int& steps, int& blocks)
{
    steps = 1;
    while (steps < 8 && (N + static_cast<long long>(kIdxThreads) * steps - 1) / (kIdxThreads * steps) > 256) steps *= 2;
    blocks = static_cast<int>((N + static_cast<long long>(kIdxThreads) * steps - 1) / (kIdxThreads * steps));
}

// Scratch that the entry points ask their callers for: a row per workgroup, and the totals.  None up to kNoScratchPairs; between those and
// kAlonePairs it is asked for as ever, but not used.
size_t dispatch_scratch_bytes(long long n_pairs, int E)
{
    if (n_pairs <= kNoScratchPairs) return 0;
    int steps, blocks;
    dispatch_plan(n_pairs, steps, blocks);
    return static_cast<size_t>(blocks + 1) * E * sizeof(int32_t);
}

template <int S>
static void launch_dispatch_index(const int32_t* idx, const uint8_t* mask, int N, int E, int blocks, int32_t* scratch,
                                  int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv, const RefreshRule* rule, hipStream_t stream)
{
    const int scan = blocks > 256 ? 1 : 0;      // small grids: every placing workgroup sums the table itself
    if (rule)
        hipLaunchKernelGGL((dispatch_count_kernel<S, kMaskSimple>), dim3(blocks), dim3(kIdxThreads), 0, stream, idx, mask, N, E, scratch, *rule);
    else
        hipLaunchKernelGGL((dispatch_count_kernel<S, kMaskArray>), dim3(blocks), dim3(kIdxThreads), 0, stream, idx, mask, N, E, scratch, NoRule{});
    if (scan)
        hipLaunchKernelGGL(dispatch_scan_kernel, dim3(1), dim3(1024), 0, stream, scratch, blocks, E);
    hipLaunchKernelGGL((dispatch_place_kernel<S, kIdxThreads, kMaskArray>), dim3(blocks), dim3(kIdxThreads), 0, stream, idx, mask, N, E, scratch,
                       scan, counts, offsets, perm, inv, NoRule{});
}

// One workgroup for all pairs, no counting launch and no table
template <int S, int THREADS>
static void launch_dispatch_alone(const int32_t* idx, const uint8_t* mask, int N, int E, int32_t* counts, int32_t* offsets,
                                  int32_t* perm, int32_t* inv, const RefreshRule* rule, hipStream_t stream)
{
    if constexpr (THREADS == kSelThreads) {
        if (rule && rule->select) {
            hipLaunchKernelGGL((dispatch_place_kernel<S, THREADS, kMaskSelect>), dim3(1), dim3(THREADS), 0, stream, idx, mask, N, E,
                               static_cast<const int32_t*>(nullptr), 0, counts, offsets, perm, inv, *rule);
            return;
        }
    }
    if (rule)
        hipLaunchKernelGGL((dispatch_place_kernel<S, THREADS, kMaskSimple>), dim3(1), dim3(THREADS), 0, stream, idx, mask, N, E,
                           static_cast<const int32_t*>(nullptr), 0, counts, offsets, perm, inv, *rule);
    else
        hipLaunchKernelGGL((dispatch_place_kernel<S, THREADS, kMaskArray>), dim3(1), dim3(THREADS), 0, stream, idx, mask, N, E,
                           static_cast<const int32_t*>(nullptr), 0, counts, offsets, perm, inv, NoRule{});
}

hipError_t launch_dispatch(bool bf16, const void* x, const int32_t* idx, const uint8_t* mask, int T_tok, int d,
                           int E, int k, void* x_packed, int32_t* counts, int32_t* offsets, int32_t* perm,
                           int32_t* inv, int32_t* scratch, hipStream_t stream, const RefreshRule* rule)
{
    const int N = T_tok * k;
    if (N > kNoScratchPairs && scratch == nullptr) return hipErrorInvalidValue;
    // Elementwise masks are formed by whoever reads the expert ids first, a selection of tokens by the workgroup that sorts alone;
    // beyond that the selection is a launch of its own.
    if (rule && (N == 0 || (rule->select && N > kAlonePairs))) {
        if (hipError_t err = launch_refresh(*rule, T_tok, stream); err != hipSuccess) return err;
        rule = nullptr;
    }
    int steps, blocks;
    dispatch_plan(N, steps, blocks);
    if (N <= kIdxThreads && !(rule && rule->select)) launch_dispatch_alone<1, kIdxThreads>(idx, mask, N, E, counts, offsets, perm, inv, rule, stream);
    else if (N <= 1024) launch_dispatch_alone<1, 1024>(idx, mask, N, E, counts, offsets, perm, inv, rule, stream);
    else if (N <= 2048) launch_dispatch_alone<2, 1024>(idx, mask, N, E, counts, offsets, perm, inv, rule, stream);
    else if (N <= kAlonePairs) launch_dispatch_alone<4, 1024>(idx, mask, N, E, counts, offsets, perm, inv, rule, stream);
    else switch (steps) {
    case 1: launch_dispatch_index<1>(idx, mask, N, E, blocks, scratch, counts, offsets, perm, inv, rule, stream); break;
    case 2: launch_dispatch_index<2>(idx, mask, N, E, blocks, scratch, counts, offsets, perm, inv, rule, stream); break;
    case 4: launch_dispatch_index<4>(idx, mask, N, E, blocks, scratch, counts, offsets, perm, inv, rule, stream); break;
    default: launch_dispatch_index<8>(idx, mask, N, E, blocks, scratch, counts, offsets, perm, inv, rule, stream); break;
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || T_tok == 0 || x_packed == nullptr) return err;   // no packed buffer: index only
    const int gblocks = (T_tok + 3) / 4;
    const int passes = (d / (bf16 ? 8 : 4) + kWave - 1) / kWave;
#define DICEMOE_GATHER(T_, NP_)                                                                                      \
    hipLaunchKernelGGL((dispatch_gather_kernel<T_, NP_>), dim3(gblocks), dim3(256), 0, stream, static_cast<const T_*>(x), \
                       inv, T_tok, d, k, mask == nullptr ? 1 : 0, static_cast<T_*>(x_packed))
    if (bf16) {
        if (passes == 1) DICEMOE_GATHER(bf16_t, 1);
        else if (passes == 2) DICEMOE_GATHER(bf16_t, 2);
        else if (passes == 3) DICEMOE_GATHER(bf16_t, 3);
        else if (passes == 4) DICEMOE_GATHER(bf16_t, 4);
        else DICEMOE_GATHER(bf16_t, 0);
    } else {
        if (passes == 1) DICEMOE_GATHER(float, 1);
        else if (passes == 2) DICEMOE_GATHER(float, 2);
        else if (passes <= 4) DICEMOE_GATHER(float, 4);
        else DICEMOE_GATHER(float, 0);
    }
#undef DICEMOE_GATHER
    return hipGetLastError();
}

// ---- scratch for callers that cannot hand over a workspace (moe_dispatch_noalloc)
// One array per device, held until the process ends.  Host code never uses the array's name as an
// address: the device address is looked up once per device and kept.
constexpr size_t kStaticScratchBytes = 64 * 1024;
static __device__ __align__(256) int32_t scratch[kStaticScratchBytes / sizeof(int32_t)];

constexpr int kMaxDevices = 64;
static int32_t* g_scratch_ptr[kMaxDevices];        // device address of `scratch` on each device, null until looked up
static std::mutex g_scratch_lock;

size_t dispatch_static_scratch_bytes() { return kStaticScratchBytes; }

hipError_t dispatch_static_scratch(int32_t** out)
{
    int device = -1;
    hipError_t err = hipGetDevice(&device);
    if (err != hipSuccess) return err;
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(g_scratch_lock);
    if (g_scratch_ptr[device] == nullptr) {
        void* ptr = nullptr;
        err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));      // the current device's copy of the array
        if (err != hipSuccess) return err;
        if (ptr == nullptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = static_cast<int32_t*>(ptr);
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

__global__ void ep_segments_kernel(const int32_t* __restrict__ recv_counts, int n_seg, int E_loc,
                                   int32_t* __restrict__ seg_offsets, int32_t* __restrict__ seg_expert)
{
    // tiny table (at most 1024 entries): one wavefront scans it 64 entries at a time.  (One thread walking it waited for
    // memory entry by entry: 5.7 us for 16 segments.)
    const int lane = lane_id();
    int run = 0;
    for (int g0 = 0; g0 < n_seg; g0 += kWave) {
        const int g = g0 + lane;
        const int mine = g < n_seg ? recv_counts[g] : 0;
        const int incl = wave_scan(mine);
        if (g < n_seg) {
            seg_offsets[g] = run + incl - mine;
            seg_expert[g] = g % E_loc;
        }
        run += __shfl(incl, kWave - 1, kWave);
    }
    if (lane == 0) seg_offsets[n_seg] = run;
}

hipError_t launch_ep_segments(const int32_t* recv_counts, int n_seg, int E_loc, int32_t* seg_offsets,
                              int32_t* seg_expert, hipStream_t stream)
{
    hipLaunchKernelGGL(ep_segments_kernel, dim3(1), dim3(64), 0, stream, recv_counts, n_seg, E_loc, seg_offsets,
                       seg_expert);
    return hipGetLastError();
}

}  // namespace dicemoe
