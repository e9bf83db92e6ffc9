// The stable sort of refreshed pairs by expert inside one workgroup, for kernels that use its result themselves: the first GEMM of a
// small layer does its own dispatch, which takes the dispatch's launch out of the chain (every workgroup sorts, the first one leaves
// the index arrays for the kernels behind).
#pragma once
#include "refresh_rule.hpp"

namespace dicemoe {

// order this wavefront's LDS accesses: reads before the point complete before writes after it
// are issued, and the compiler keeps them on their side
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// lanes of this wave that are live and hold the same expert id as the calling lane; nbits = number of
// bits an expert id can have (ballots are scalar work)
__device__ __forceinline__ uint64_t same_expert_peers(bool live, int e, int nbits) {
    uint64_t peers = __ballot(live);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        if (b < nbits) {                          // uniform
            const bool bit = (e >> b) & 1;
            const uint64_t bb = __ballot(bit);
            peers &= bit ? bb : ~bb;
        }
    }
    return peers;
}

// ---- one pair of the sort, the same for every kernel that sorts (these two, and the dispatch's own)

// Does pair p with expert id e have a row, if it is refreshed?  Not past the end, and not with a bad id.
__device__ __forceinline__ bool has_row(int p, int N, int e, int E)
{
    return p < N && static_cast<unsigned>(e) < static_cast<unsigned>(E);
}

// Rank of each lane's pair among this wavefront's pairs of the same expert so far (e < 0: none), in lane order; run: their counts
__device__ __forceinline__ int rank_step(int e, int nbits, int* run)
{
    const bool live = e >= 0;
    e = live ? e : 0;
    const uint64_t peers = same_expert_peers(live, e, nbits);
    const int before = __popcll(peers & lanemask_lt());
    const int so_far = run[e];                               // every peer reads the same running count ...
    wave_sync();
    if (live && before == 0) run[e] = so_far + __popcll(peers);      // ... then the first updates it
    wave_sync();
    return so_far + before;
}

// run[WAVES][kMaxExperts]: the wavefronts' counts of expert e become those of the wavefronts before each; returns the sum
template <int WAVES>
__device__ __forceinline__ int counts_to_prefixes(int* run, int e)
{
    int cnt[WAVES], total = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) cnt[w] = run[w * kMaxExperts + e];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { run[w * kMaxExperts + e] = total; total += cnt[w]; }
    return total;
}

// Index entries of pair p (its row(), if it has one) and of packed row p (that there is none, if there are only R)
template <typename Fn>
__device__ __forceinline__ void leave_index(int p, int N, bool has, Fn row, int R, int32_t* __restrict__ perm, int32_t* __restrict__ inv)
{
    int r = -1;
    if (has) {
        r = row();
        perm[r] = p;
    }
    if (p < N) {
        inv[p] = r;
        if (p >= R) perm[p] = -1;
    }
}

constexpr int own_sort_ints(int waves) { return waves * kMaxExperts + kMaxExperts + 4; }      // scratch beside the row list

// off[0 .. E]: offsets of the experts' rows; row[r]: pair of packed row r.  scratch: own_sort_ints(WAVES) ints of LDS, of which `off` is the
// part behind the first WAVES * kMaxExperts.  All threads of the workgroup, behind whose last barrier the results can be read.
template <int WAVES>
__device__ __forceinline__ const int* sort_pairs(const PairSort& s, bool writer, int* scratch, uint16_t* row)
{
    constexpr int S = kOwnSortPairs / (WAVES * kWave);      // steps of a wavefront at most
    int* const run = scratch;                               // [WAVES][kMaxExperts]
    int* const off = scratch + WAVES * kMaxExperts;
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int N = s.n_pairs, E = s.experts;
    const int steps = (N + WAVES * kWave - 1) / (WAVES * kWave);
    const int nbits = E > 1 ? 32 - __builtin_clz(static_cast<unsigned>(E - 1)) : 0;
    const int p0 = wave * steps * kWave + lane;
    int ev[S], rank[S];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int p = p0 + u * kWave;
        ev[u] = s.expert_idx[p < N ? p : N - 1];
    }
    run[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < S; ++u) {
        const int p = p0 + u * kWave;
        rank[u] = 0;
        if (u >= steps) { ev[u] = -1; continue; }           // (uniform)
        bool ok = has_row(p, N, ev[u], E);
        if (s.rule.mask) {
            const uint8_t m = simple_mask(s.rule, p);
            if (writer && p < N) s.rule.mask[p] = m;
            ok = ok && m != 0;
        }
        if (!ok) ev[u] = -1;
        rank[u] = rank_step(ev[u], nbits, run + wave * kMaxExperts);
    }
    __syncthreads();
    if (wave == 0) {                                         // lane e is expert e
        const int total = counts_to_prefixes<WAVES>(run, lane), incl = wave_scan(total);
        if (lane == 0) off[0] = 0;
        off[lane + 1] = incl;                                // (experts from E on have no pairs)
        if (writer) {
            if (lane < E) { s.counts[lane] = total; s.offsets[lane] = incl - total; }
            if (lane == E - 1) s.offsets[E] = incl;
            if (s.rule.mask && lane == 0) *s.rule.n_refresh = s.rule.n_value;
        }
    }
    __syncthreads();
    const int R = off[E];
#pragma unroll
    for (int u = 0; u < S; ++u) {
        if (u >= steps) break;                               // (uniform)
        const int p = p0 + u * kWave;
        int r = -1;
        if (ev[u] >= 0) {
            r = off[ev[u]] + run[wave * kMaxExperts + ev[u]] + rank[u];
            row[r] = static_cast<uint16_t>(p);
        }
        if (writer) leave_index(p, N, r >= 0, [&] { return r; }, R, s.perm, s.inv);
    }
    __syncthreads();
    return off;
}

// The rows of single experts out of up to kStreamSortPairs pairs, for a workgroup that computes a few tiles of a large sort: every workgroup counts all
// pairs, but ranks only those that it computes.  The loops stay rolled: counts in
// registers and loops unrolled took 4 us a layer more (613 us below; code that runs once and is long has to be fetched first, which was not
// measured by itself).  DiT-MoE-S, 2048 tokens x 12 layers, us: dispatched 585,
// every workgroup ranking all pairs 572, this 561.
template <int WAVES>
struct CountedPairs {
    static constexpr int kGroups = kStreamSortPairs / (WAVES * kWave * 4);
    static constexpr int kBytes = WAVES * kMaxExperts * 4 + WAVES * kGroups * kWave * 4;

    uint32_t* key;              // LDS: experts of four pairs of a lane (255: none)
    int groups, wave, rows;     // groups of 4 x 64 pairs of a wavefront; all rows
    int begin, end;             // lane e: the rows of expert e
    int first, count;           // ... the first of them that is a pair of this wavefront, and how many are

    // lds: kBytes.  Writes the mask, inv of pairs that have no row, perm beyond the rows, counts and offsets, each workgroup of the grid a part;
    // perm and inv of the rows are left to those who ask for them.
    __device__ __forceinline__ void form(const PairSort& s, char* lds)
    {
        int* const run = reinterpret_cast<int*>(lds);        // [WAVES][kMaxExperts]
        key = reinterpret_cast<uint32_t*>(lds + WAVES * kMaxExperts * 4);
        const int tid = threadIdx.x, lane = lane_id();
        wave = __builtin_amdgcn_readfirstlane(tid / kWave);
        const int N = s.n_pairs, E = s.experts;
        groups = (N + WAVES * kWave * 4 - 1) / (WAVES * kWave * 4);
        run[tid] = 0;
        wave_sync();                                         // (a wavefront's own counts)
        const int base = wave * groups * 4 * kWave;
        static_assert(kGroups == 2, "loads of both groups in flight");
        int ev[4], later[4];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int p = base + u * kWave + lane;
            (u < 4 ? ev[u & 3] : later[u & 3]) = s.expert_idx[p < N ? p : N - 1];
        }
#pragma unroll 1
        for (int g = 0; g < groups; ++g) {
            uint32_t word = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = base + (g * 4 + u) * kWave + lane;
                const bool mine = (p >> 6) == static_cast<int>(blockIdx.x) && p < N;
                bool ok = has_row(p, N, ev[u], E);
                if (s.rule.mask) {
                    const uint8_t m = simple_mask(s.rule, p);
                    if (mine) s.rule.mask[p] = m;
                    ok = ok && m != 0;
                }
                if (mine && !ok) s.inv[p] = -1;
                word |= static_cast<uint32_t>(ok ? ev[u] : 255) << (8 * u);
                if (ok) __hip_atomic_fetch_add(&run[wave * kMaxExperts + ev[u]], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            key[(wave * groups + g) * kWave + lane] = word;
#pragma unroll
            for (int u = 0; u < 4; ++u) ev[u] = later[u];
        }
        wave_sync();
        count = run[wave * kMaxExperts + lane];
        __syncthreads();
        int total = 0, before = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const int c = run[w * kMaxExperts + lane];
            before += w < wave ? c : 0;
            total += c;
        }
        const int incl = wave_scan(total);
        begin = incl - total;
        end = incl;
        first = begin + before;
        rows = __builtin_amdgcn_readlane(incl, kWave - 1);
        if (wave == 0) {
            const int p = blockIdx.x * kWave + lane;
            if (p < N && p >= rows) s.perm[p] = -1;          // packed rows beyond the refreshed ones
            if (blockIdx.x == 0) {
                if (lane < E) { s.counts[lane] = total; s.offsets[lane] = begin; }
                if (lane == E - 1) s.offsets[E] = incl;
                if (s.rule.mask && lane == 0) *s.rule.n_refresh = s.rule.n_value;
            }
        }
    }

    // fn(row, pair) for the rows lo .. hi - 1 of expert e (uniform) that are pairs of this wavefront
    template <typename Fn>
    __device__ __forceinline__ void each(int e, int lo, int hi, Fn fn) const
    {
        int r0 = __builtin_amdgcn_readlane(first, e);
        const int past = r0 + __builtin_amdgcn_readlane(count, e);
        if (r0 >= hi || past <= lo) return;
        const int lane = lane_id();
        const int stop = past < hi ? past : hi;
        for (int g = 0; g < groups && r0 < stop; ++g) {
            const uint32_t word = key[(wave * groups + g) * kWave + lane];
#pragma unroll 1
            for (int u = 0; u < 4; ++u) {
                const bool hit = ((word >> (8 * u)) & 255u) == static_cast<uint32_t>(e);
                const uint64_t hits = __ballot(hit);
                const int r = r0 + __popcll(hits & lanemask_lt());
                if (hit && r >= lo && r < hi) fn(r, ((wave * groups + g) * 4 + u) * kWave + lane);
                r0 += __popcll(hits);
            }
        }
    }
};

}  // namespace dicemoe
