// Persistent grouped bf16 GEMM of the expert FFN (Algorithm 1, "x_e <- expert(x_d)"): 256 workgroups of eight
// wavefronts, one per compute unit, each walking a list of 256-row output tiles without a pause in its load
// stream.
//
// What bounds a grouped GEMM here.  On random operands a loop of nothing but MFMAs holds 1.72 PFLOP/s (power: the clock falls as more
// pipes are busy) and the main loop of a 256-row tile 1.5 (1.06 us per 64-deep step of 256 x 192 on every compute unit), so
// that loop is near what the machine gives; what a workgroup per tile loses lies between the tiles: 1.7 us of turnover, 2.5 us of tile
// lookup and row indices, 2 us until the first stage is in LDS, the epilogue, and a last round in which most compute
// units idle.  Hence
//   * the stage rings run on across tiles: the refills of a tile's last steps fetch the first stages of the next
//     tile, whose place, bias and row indices were looked up a tile earlier, so the matrix pipes wait for nothing but the
//     epilogue (first GEMM at 8192 rows of the DiT-MoE-XL widths: 117 us with a workgroup per 128 x 192 tile,
//     two per compute unit; 103 here);
//   * the tiles left over after the whole rounds are cut into halves (128 rows) or quarters (128 rows and half of the
//     columns) when the pieces fit one round.  A few workgroups alone are bound by the latency of their loads, not by
//     the matrix pipes (a half tile on the whole tile's rings takes 0.9 us a step), so the pieces use the LDS they no
//     longer need for deeper rings (0.5 - 0.7 us a step).  Expert-parallel shard (16384 rows, d = 2048, F = 8192), second
//     GEMM: 3.1 rounds of 192 columns run as four in 575 us; 2 rounds and a quarter round of 256 columns in 480.
// Cutting the leftover reductions instead (float sums through memory, the last part adds them up) is as fast, but ties
// the rounding of a row to where its tile happens to lie in the list; here every row has the same bits in any layout.
//
// Tile shapes (rows x columns, stages of activations + stages of weights in 160 KB of LDS): whole 256 x 192 (2 + 4) and
// 256 x 256 (2 + 3), halves 128 x 192 (4 + 4) and 128 x 256 (3 + 3), quarters 128 x 128 (5 + 5).  The wide one moves 15 %
// fewer bytes per flop and has fewer epilogues; which one wins is mostly a matter of how the tile count meets 32
// compute units per XCD: stream_cost on the host's estimate of it, stream_columns on the real count.
#pragma once
#include <type_traits>
#include "ffn_mfma.hpp"
#include "ffn_plan.hpp"
#include "ffn_ring.hpp"
#include "ffn_wide.hpp"

namespace dicemoe {

constexpr int kStreamThreads = 512;
constexpr int kStreamLds = 160 * 1024;
using StreamPairs = CountedPairs<kStreamThreads / kWave>;
constexpr int kStreamOwnRows = 2 * 256;                    // the rows of a workgroup's first two tiles
constexpr int kStreamSortBytes = kStreamOwnRows * 2 + StreamPairs::kBytes;

// The tiles of one grouped GEMM dealt to the eight XCDs by expert, as find_tile_by_expert does for a workgroup per tile
// (home XCD = expert mod 8, an XCD keeps at most cap = ceil(total / 8) tiles of its own list and takes overflow of
// the others in XCD order; inside a segment bands of GROUP_M row tiles, row tile fastest).
// n_seg <= 64: lane g of every wavefront holds segment g, lane i < 8 the lengths of XCD i's list, so that looking a
// tile up is a ballot and a few readlanes.
struct XcdTiles {
    int begin, end, expert, row_tiles, first;   // lane g: rows, expert, row tiles of segment g; its first tile's place in its home's list
    int over, over_first;                       // lane i < 8: tiles of XCD i beyond the cap, and their place in the overflow list
    int n_seg, n_tiles_n, bm, bn, xcd, cap;
    int kept, spare_before, count;              // this XCD: own tiles it keeps, spare slots of the XCDs before it, length of its list

    __device__ __forceinline__ void deal(const int32_t* __restrict__ seg_offsets, const int32_t* __restrict__ seg_expert,
                                         int n_seg_, int bm_, int bn_, int n_tiles_n_, int xcd_, int max_rows)
    {
        const int lane = threadIdx.x & 63;
        int b = 0, e = 0, x = 8;                             // (a home that is nobody's)
        if (lane < n_seg_) { b = seg_offsets[lane]; e = seg_offsets[lane + 1]; x = seg_expert[lane]; }
        set(b, e, x, n_seg_, bm_, max_rows);
        deal_columns(bn_, n_tiles_n_, xcd_);
    }

    // each lane's entry of seg_expert
    static __device__ __forceinline__ int expert_of(const int32_t* __restrict__ seg_expert, int n_seg)
    {
        const int lane = threadIdx.x & 63;
        return lane < n_seg ? seg_expert[lane] : 8;          // (a home that is nobody's)
    }

    __device__ __forceinline__ void load(const int32_t* seg_offsets, int expert_, int n_seg_, int bm_, int max_rows)
    {
        const int lane = threadIdx.x & 63;
        set(lane < n_seg_ ? seg_offsets[lane] : 0, lane < n_seg_ ? seg_offsets[lane + 1] : 0, expert_, n_seg_, bm_, max_rows);
    }

    // each lane's segment
    __device__ __forceinline__ void set(int begin_, int end_, int expert_, int n_seg_, int bm_, int max_rows)
    {
        n_seg = n_seg_; bm = bm_;
        end = end_ < max_rows ? end_ : max_rows;            // (a table that holds more rows than the caller said)
        begin = begin_ < end ? begin_ : end;
        expert = expert_;
        row_tiles = (end - begin + bm - 1) / bm;
    }

    __device__ __forceinline__ int all_row_tiles() const
    {
        int sum = 0;
        for (int g = 0; g < n_seg; ++g) sum += __builtin_amdgcn_readlane(row_tiles, g);
        return sum;
    }

    __device__ __forceinline__ void deal_columns(int bn_, int n_tiles_n_, int xcd_)
    {
        const int lane = threadIdx.x & 63;
        bn = bn_; n_tiles_n = n_tiles_n_; xcd = xcd_;
        const int home = lane < n_seg ? expert & 7 : 8;
        first = 0;
        int own = 0;
        for (int g = 0; g < n_seg; ++g) {
            const int tiles = __builtin_amdgcn_readlane(row_tiles, g) * n_tiles_n;
            const int h = __builtin_amdgcn_readlane(home, g);
            first += (home == h && g < lane) ? tiles : 0;
            own += lane == h ? tiles : 0;
        }
        int total = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) total += __builtin_amdgcn_readlane(own, i);
        cap = (total + 7) >> 3;
        over = own > cap ? own - cap : 0;
        const int spare = own < cap ? cap - own : 0;
        over_first = 0;
        spare_before = 0;
        int over_total = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            over_first += i < lane ? __builtin_amdgcn_readlane(over, i) : 0;
            spare_before += i < xcd ? __builtin_amdgcn_readlane(spare, i) : 0;
            over_total += __builtin_amdgcn_readlane(over, i);
        }
        const int my_spare = __builtin_amdgcn_readlane(spare, xcd);
        kept = cap - my_spare;
        int taken = over_total - spare_before;
        taken = taken < 0 ? 0 : taken;
        count = kept + (taken < my_spare ? taken : my_spare);
    }

    // Row range, first column and expert of tile `idx` (< count) of this XCD's list, another idx in every lane
    __device__ __forceinline__ void locate_each(int idx, int& row0, int& row_end, int& col0, int& e) const
    {
        constexpr int GROUP_M = 8;
        int list = xcd;
        const int pos = spare_before + idx - kept;
        const bool spilled = idx >= kept;       // overflow of another XCD
        if (__ballot(spilled) != 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int o = pos - __builtin_amdgcn_readlane(over_first, i);
                if (spilled && o >= 0 && o < __builtin_amdgcn_readlane(over, i)) { list = i; idx = cap + o; }
            }
        }
        int local = 0, nt = 1;
        row0 = row_end = e = 0;
        for (int g = 0; g < n_seg; ++g) {
            const int t = __builtin_amdgcn_readlane(row_tiles, g), ge = __builtin_amdgcn_readlane(expert, g);
            const int o = idx - __builtin_amdgcn_readlane(first, g);
            if ((ge & 7) == list && o >= 0 && o < t * n_tiles_n) {
                local = o; nt = t; e = ge;
                row0 = __builtin_amdgcn_readlane(begin, g);
                row_end = __builtin_amdgcn_readlane(end, g);
            }
        }
        const int band = local / (GROUP_M * n_tiles_n), in_band = local - band * (GROUP_M * n_tiles_n);
        const int left = nt - band * GROUP_M;
        const int rows_here = left < GROUP_M ? left : GROUP_M;
        const int tile_n = in_band / rows_here;
        row0 += (band * GROUP_M + in_band - tile_n * rows_here) * bm;
        col0 = tile_n * bn;
    }

    // the same for one tile
    __device__ __forceinline__ void locate(int idx, int& row0, int& row_end, int& col0, int& e) const
    {
        constexpr int GROUP_M = 8;
        int list = xcd;
        if (idx >= kept) {                      // overflow of another XCD
            const int pos = spare_before + idx - kept;
            const uint64_t hit = __ballot(pos >= over_first && pos < over_first + over);
            list = __builtin_ctzll(hit);
            idx = cap + pos - __builtin_amdgcn_readlane(over_first, list);
        }
        const uint64_t hit = __ballot((expert & 7) == list && idx >= first && idx < first + row_tiles * n_tiles_n);
        const int g = __builtin_ctzll(hit);
        idx -= __builtin_amdgcn_readlane(first, g);
        const int nt = __builtin_amdgcn_readlane(row_tiles, g);
        const int band = idx / (GROUP_M * n_tiles_n), in_band = idx - band * (GROUP_M * n_tiles_n);
        const int left = nt - band * GROUP_M;
        const int rows_here = left < GROUP_M ? left : GROUP_M;
        const int tile_n = in_band / rows_here;
        col0 = tile_n * bn;
        row0 = __builtin_amdgcn_readlane(begin, g) + (band * GROUP_M + in_band - tile_n * rows_here) * bm;
        row_end = __builtin_amdgcn_readlane(end, g);
        e = __builtin_amdgcn_readlane(expert, g);
    }
};

// bias of column `col` of this wavefront's columns, held by lane col % 64 of register col / 64
template <int NB>
__device__ __forceinline__ float lane_held(const float (&reg)[NB], int block, int lane_bytes)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(lane_bytes, __builtin_bit_cast(int, reg[block])));
}

// Epilogue of a wavefront's block: bias, GELU, rounding, stores.  After the swap of register pairs between the
// half-wavefronts (v_permlane32_swap) every lane holds 8 consecutive columns of one row and stores 16 bytes.  Buffer
// stores: rows and columns that do not exist get an offset beyond the buffer and are dropped by the hardware, so every
// wavefront issues the same number of store instructions whatever its tile looks like (the main loop counts them).
// dst[i]: row of C for row (lane % 32) of slab i, or -1.  bias_reg: lane c % 64 of register c / 64 holds column c's.
template <int TM, int TN, bool GELU, int NB>
__device__ __forceinline__ void store_block(const f32x16_v (&sums)[TM][TN], const float (&bias_reg)[NB], __amdgpu_buffer_rsrc_t rs,
                                            int N, int col_end, const int (&dst)[TM], int col_first, int lane)
{
    const int h = lane >> 5;
    float b[2][8];                                       // bias of this group of 16 columns, and of the next one
    auto bias_of = [&](int grp, float (&v)[8]) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int c = 16 * grp + 8 * (t / 4) + t % 4;
            v[t] = lane_held<NB>(bias_reg, c / 64, ((c & 63) + 4 * h) * 4);
        }
    };
    bias_of(0, b[0]);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
            DICEMOE_SCHED_FENCE();
            const int grp = 2 * j + gp;
            if (grp + 1 < 2 * TN) bias_of(grp + 1, b[(grp + 1) & 1]);
            DICEMOE_SCHED_FENCE();
            const int n = col_first + j * 32 + 16 * gp + 8 * h;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                DICEMOE_SCHED_FENCE();
                uint2 packed[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int g = 2 * gp + q;
                    float v[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        v[t] = sums[i][j][4 * g + t] + b[grp & 1][4 * q + t];
                        if (GELU) v[t] = gelu_erf_fast(v[t]);
                    }
                    packed[q] = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                }
                const auto sx = __builtin_amdgcn_permlane32_swap(packed[0].x, packed[1].x, false, false);
                const auto sy = __builtin_amdgcn_permlane32_swap(packed[0].y, packed[1].y, false, false);
                const uint32_t off = (dst[i] >= 0 && n < col_end) ? (static_cast<uint32_t>(dst[i]) * static_cast<uint32_t>(N) + static_cast<uint32_t>(n)) * 2u : kBeyondBuffer;
                __builtin_amdgcn_raw_buffer_store_b128(u32x4_v{sx[0], sy[0], sx[1], sy[1]}, rs, static_cast<int>(off), 0, 0);
            }
        }
}

// One code path for whole tiles and for the pieces of a leftover round.
struct Place { int row0, row_end, col0, col_end, e; };      // rows and columns of one item, its expert

struct StreamArgs {
    const bf16_t* A; const bf16_t* W; const float* bias; bf16_t* C;
    int N, K;
    const int32_t* row_index; int row_div; const int32_t* out_index;
};

// The items first, place(1) .. place(n_items - 1) of this workgroup, each a (32 TM WGM) x (32 TN WGN) tile or part of one.
// OWN: own_rows is the row index of the first two items, 256 each, in the LDS of the activations' ring.
template <int TM, int TN, int SPREAD, int AST, int WST, bool GELU, bool GATHER, bool OWN, int WGM, int WGN, typename PlaceFn>
__device__ __forceinline__ void stream_tiles(const StreamArgs& g, char* smem, int n_items, Place first, PlaceFn place, const uint16_t* own_rows = nullptr)
{
    constexpr int NW = WGM * WGN;
    constexpr int BM = 32 * TM * WGM, BN = 32 * TN * WGN;
    constexpr int WM = 32 * TM, WN = 32 * TN;
    constexpr int CH = 8;
    constexpr int QA = BM / (8 * NW), QB = BN / (8 * NW);
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "every wavefront loads whole groups of eight rows");
    constexpr int QW = QA + QB;
    constexpr int ABYTES = BM * 128, WBYTES = BN * 128;
    constexpr int NFRAG = TM + TN;
    constexpr int NMFMA = TM * TN;
    constexpr int FPER = (NFRAG + NMFMA - 1) / NMFMA;
    constexpr int DEPTH = AST > WST ? AST : WST;
    constexpr int NB = (WN + 63) / 64;
    constexpr int NSTORE = TM * TN * 2;                  // store instructions of a wavefront's epilogue
    static_assert(SPREAD >= 1 && SPREAD <= 4, "a refill is issued within the four slices before it is needed");
    static_assert(!OWN || kStreamSortBytes <= AST * ABYTES, "the sorted rows fit the activations' ring");
    char* const a_lds = smem;
    char* const w_lds = smem + AST * ABYTES;
    const bf16_t* const A = g.A;
    const bf16_t* const W = g.W;
    const float* const bias = g.bias;
    bf16_t* const C = g.C;
    const int N = g.N, K = g.K, row_div = g.row_div;
    const int32_t* const row_index = g.row_index;
    const int32_t* const out_index = g.out_index;
    const int nk = K / 64;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    Place p = first;

    // ---- sources.  Load q of an operand fills tile rows 8q .. 8q+7; lane l lands at LDS slot (row 8q + l/8, l%8) and
    // therefore fetches the chunk that the swizzle assigns to that slot.  Rows of A come through the row index when
    // there is one.  Weight rows beyond the matrix read as zero (bounds of the buffer).
    const __amdgpu_buffer_rsrc_t a_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(A), 0, static_cast<int>(kBeyondBuffer), kBufferFlags);
    // Behind the last item: no rows and no columns, so that the stages asked for there cost no memory access
    auto nowhere = [](Place pl) { return Place{pl.row0, pl.row0, pl.col0, pl.col0, pl.e}; };
    auto w_buffer = [&](const Place& pl) {
        const int rows = pl.col_end - pl.col0;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(W + (static_cast<size_t>(pl.e) * N + pl.col0) * K), 0, rows * K * 2, kBufferFlags);
    };
    uint32_t w_off[QB];
#pragma unroll
    for (int i = 0; i < QB; ++i) {
        const int row = (wave * QB + i) * 8 + (lane >> 3);
        w_off[i] = static_cast<uint32_t>(row) * static_cast<uint32_t>(K) * 2u + ((lane & 7) ^ chunk_swizzle<CH>(row)) * 16;
    }
    // Rows beyond the item's get an offset beyond the buffer: they read as zero and cost no memory access.
    auto fetch_own_rows = [&](const Place& pl, int (&rows)[QA], const uint16_t* list) {
#pragma unroll
        for (int i = 0; i < QA; ++i) {
            int r = (wave * QA + i) * 8 + (lane >> 3);
            const int here = pl.row_end - pl.row0;
            r = r < here ? r : here - 1;
            rows[i] = list[r > 0 ? r : 0];
        }
    };
    auto fetch_rows = [&](const Place& pl, int (&rows)[QA]) {
#pragma unroll
        for (int i = 0; i < QA; ++i) {
            int r = pl.row0 + (wave * QA + i) * 8 + (lane >> 3);
            if (GATHER) {
                r = r < pl.row_end ? r : pl.row_end - 1;
                rows[i] = row_index[r > 0 ? r : 0];
            } else {
                rows[i] = r;
            }
        }
    };
    auto row_offsets = [&](const Place& pl, const int (&rows)[QA], uint32_t (&off)[QA]) {
#pragma unroll
        for (int i = 0; i < QA; ++i) {
            const int row = (wave * QA + i) * 8 + (lane >> 3);
            const uint32_t r = GATHER ? static_cast<uint32_t>(rows[i]) / static_cast<uint32_t>(row_div) : static_cast<uint32_t>(rows[i]);
            off[i] = pl.row0 + row < pl.row_end ? r * static_cast<uint32_t>(K) * 2u + ((lane & 7) ^ chunk_swizzle<CH>(row)) * 16 : kBeyondBuffer;
        }
    };
    auto dma_a = [&](int i, uint32_t off, int sa, int kt) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rs, DICEMOE_LDS_PTR(a_lds + sa * ABYTES + (wave * QA + i) * 1024), 16, static_cast<int>(off), kt * 128, 0, 0);
    };
    auto dma_w = [&](int i, __amdgpu_buffer_rsrc_t rs, int sw, int kt) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, DICEMOE_LDS_PTR(w_lds + sw * WBYTES + (wave * QB + i) * 1024), 16, static_cast<int>(w_off[i]), kt * 128, 0, 0);
    };

    int a_off[4], b_off[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int chunk = kk * 2 + (lane >> 5);
        const int ra = wm * WM + (lane & 31), rb = wn * WN + (lane & 31);
        a_off[kk] = (ra * CH + (chunk ^ chunk_swizzle<CH>(ra))) * 16;
        b_off[kk] = (rb * CH + (chunk ^ chunk_swizzle<CH>(rb))) * 16;
    }

    f32x16_v acc[TM][TN];
    bf16x8_v fr[2][NFRAG];
    auto read_frag = [&](int set, int f, const char* sta, const char* stw, int kk) {
        const char* q = f < TM ? sta + a_off[kk] + f * 4096 : stw + b_off[kk] + (f - TM) * 4096;
        const u32x4_v v = *reinterpret_cast<const u32x4_v*>(q);
        fr[set][f] = *reinterpret_cast<const bf16x8_v*>(&v);
    };
    auto mfma = [&](int set, int m) {
        const int i = m / TN, j = m % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[set][TM + j], fr[set][i], acc[i][j], 0, 0, 0);
    };

    constexpr int PART = (QW + SPREAD - 1) / SPREAD;
    constexpr int PER = (PART + NMFMA - 1) / NMFMA;
    // loads of the stage that the first step of an item waits for have all been issued before the previous item's epilogue
    constexpr bool EARLY = (AST > 2 || QA <= PART) && (WST > 2 || QW <= PART);
    constexpr int PEND = ring_pending(AST, WST, QA, QB, 8 * DEPTH, 4 * DEPTH);
    constexpr int FIRST = GATHER && !OWN ? ring_first_pending(QA, PART) : 0;
    static_assert(ring_waits_hold(AST, WST, QA, QB, PART, FIRST, PEND, EARLY ? NSTORE : 0) && ring_waits_hold(AST, WST, QA, QB, PART, FIRST, PEND, 0),
                  "every stage has landed before it is read, whether the item before left stores behind or not");
    int sa = 0, sw = 0;
    uint32_t a_cur[QA], a_nxt[QA];
    int rows[QA];
    float bias_reg[NB];
    __amdgpu_buffer_rsrc_t w_cur = w_buffer(p), w_nxt = w_cur;

    // One 64-deep step.  REM = steps of this item after it (exact in the last DEPTH steps, else DEPTH): the refill of
    // a slot takes the stage AST (A) or WST (W) steps ahead, which lies in the next item when fewer steps than that
    // are left.  mid() runs behind the barrier.
    auto step = [&](auto live_tag, int kt, int nk, auto rem_tag, bool stores_behind, auto mid) {
        constexpr bool LIVE = decltype(live_tag)::value;
        constexpr int REM = decltype(rem_tag)::value;
        const int sa_nxt = (sa + 1 == AST) ? 0 : sa + 1, sw_nxt = (sw + 1 == WST) ? 0 : sw + 1;
        const int sa_prev = (sa == 0) ? AST - 1 : sa - 1, sw_prev = (sw == 0) ? WST - 1 : sw - 1;
        const char* cur_a = a_lds + sa * ABYTES;
        const char* cur_w = w_lds + sw * WBYTES;
        const char* nxt_a = a_lds + sa_nxt * ABYTES;
        const char* nxt_w = w_lds + sw_nxt * WBYTES;
        constexpr bool CAN = REM + 1 < AST, CWN = REM + 1 < WST;      // the carried part of the previous refill is the next item's
        constexpr bool RAN = REM < AST, RWN = REM < WST;
        const int a_carry = CAN ? kt - 1 + AST - nk : kt - 1 + AST;
        const int w_carry = CWN ? kt - 1 + WST - nk : kt - 1 + WST;
        const int a_refill = RAN ? kt + AST - nk : kt + AST;
        const int w_refill = RWN ? kt + WST - nk : kt + WST;
#pragma unroll
        for (int kk = 0; kk < 3; ++kk) {
            const int set = kk & 1;
            DICEMOE_SCHED_FENCE();
#pragma unroll
            for (int m = 0; m < NMFMA; ++m) {
                if (LIVE) mfma(set, m);
                DICEMOE_SCHED_FENCE();
#pragma unroll
                for (int q = 0; q < FPER; ++q)
                    if (LIVE && m * FPER + q < NFRAG) { read_frag(set ^ 1, m * FPER + q, cur_a, cur_w, kk + 1); DICEMOE_SCHED_FENCE(); }
                if (kk + 1 < SPREAD) {
#pragma unroll
                    for (int j = 0; j < PER; ++j) {
                        const int i = (kk + 1) * PART + m * PER + j;
                        if (m * PER + j < PART && i < QW) {
                            if (i < QA) dma_a(i, CAN ? a_nxt[i] : a_cur[i], sa_prev, a_carry);
                            else dma_w(i - QA, CWN ? w_nxt : w_cur, sw_prev, w_carry);
                            DICEMOE_SCHED_FENCE();
                        }
                    }
                }
            }
        }
        DICEMOE_SCHED_FENCE();
        wait_lgkmcnt<0>();                                 // every fragment of this stage has been read
        // my loads of the next stage have landed (the stores of an epilogue that ran just before this step are younger)
        if (EARLY && stores_behind) wait_vmcnt<PEND + NSTORE>();
        else wait_vmcnt<PEND>();
        block_barrier();
        DICEMOE_SCHED_FENCE();
        mid();
        DICEMOE_SCHED_FENCE();
#pragma unroll
        for (int m = 0; m < NMFMA; ++m) {
            if (LIVE) mfma(1, m);
            DICEMOE_SCHED_FENCE();
#pragma unroll
            for (int q = 0; q < FPER; ++q)
                if ((LIVE || REM == 0) && m * FPER + q < NFRAG) { read_frag(0, m * FPER + q, nxt_a, nxt_w, 0); DICEMOE_SCHED_FENCE(); }
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const int i = m * PER + j;
                if (i < PART && i < QW) {
                    if (i < QA) dma_a(i, RAN ? a_nxt[i] : a_cur[i], sa, a_refill);
                    else dma_w(i - QA, RWN ? w_nxt : w_cur, sw, w_refill);
                    DICEMOE_SCHED_FENCE();
                }
            }
        }
        sa = sa_nxt;
        sw = sw_nxt;
    };
    auto nothing = [] {};

    // ---- first item: fill the rings (what is left out here, step 0 issues as the carried part of a refill).  All row indices are asked for
    // before the first weight load, so that the wait for them is not one for the weights (with one of them moved behind these, first
    // products 5.9 us after the start instead of 4.6)
    auto fetch_bias = [&](const Place& pl) {
        const int c = pl.col0 + wn * WN;
        load_bias_columns<WN>(bias ? bias + static_cast<size_t>(pl.e) * N + c : nullptr, N - c, lane, bias_reg);
    };
    Place q;
    if constexpr (OWN) fetch_own_rows(p, rows, own_rows);
    else fetch_rows(p, rows);
    DICEMOE_SCHED_FENCE();
#pragma unroll
    for (int s = 0; s < WST; ++s)
#pragma unroll
        for (int i = 0; i < QB; ++i) if (s < WST - 1 || QA + i < PART) dma_w(i, w_cur, s, s);
    row_offsets(p, rows, a_cur);
    if constexpr (OWN) {                             // (the second item's too, then stages can take their place)
        q = n_items > 1 ? place(1) : nowhere(p);
        fetch_own_rows(q, rows, own_rows + 256);
        asm volatile("" ::: "memory");
        wait_lgkmcnt<0>();
        block_barrier();
    }
#pragma unroll
    for (int s = 0; s < AST; ++s)
#pragma unroll
        for (int i = 0; i < QA; ++i) if (s < AST - 1 || i < PART) dma_a(i, a_cur[i], s, s);
    fetch_bias(p);
    DICEMOE_SCHED_FENCE();
    if constexpr (!OWN) {
        q = n_items > 1 ? place(1) : nowhere(p);
        fetch_rows(q, rows);
    }
    DICEMOE_SCHED_FENCE();
    wait_vmcnt<FIRST>();                             // (the second item's row indices, where it has any, need not be here yet)
    block_barrier();
#pragma unroll
    for (int f = 0; f < NFRAG; ++f) read_frag(0, f, a_lds, w_lds, 0);
    const __amdgpu_buffer_rsrc_t c_rs = __builtin_amdgcn_make_buffer_rsrc(C, 0, static_cast<int>(kBeyondBuffer), kBufferFlags);
    bool stores_behind = false;

    for (int it = 0; it < n_items; ++it) {
        w_nxt = w_buffer(q);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
        const bool live = p.row0 + wm * WM < p.row_end && p.col0 + wn * WN < p.col_end;
        auto run = [&](auto live_tag) {
            // behind the barrier of the first step the loads asked for before the last epilogue have arrived
            step(live_tag, 0, nk, std::integral_constant<int, DEPTH>{}, stores_behind, [&] { row_offsets(q, rows, a_nxt); });
            int kt = 1;
            for (; kt + DEPTH < nk; ++kt) step(live_tag, kt, nk, std::integral_constant<int, DEPTH>{}, false, nothing);
#pragma unroll
            for (int b = 0; b < NB; ++b) asm volatile("" : "+v"(bias_reg[b]));      // (asked for behind the stores of the last epilogue)
            auto tail = [&](auto self, auto r) {
                constexpr int REM = decltype(r)::value;
                if constexpr (REM >= 0) {
                    step(live_tag, kt, nk, r, false, nothing);
                    ++kt;
                    self(self, std::integral_constant<int, REM - 1>{});
                }
            };
            tail(tail, std::integral_constant<int, DEPTH - 1>{});
        };
        if (live) run(std::true_type{});
        else run(std::false_type{});

        // ---- bias, then what the next items need from memory, then the stores
        const int col_first = p.col0 + wn * WN;
        int dst[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int r = p.row0 + wm * WM + i * 32 + (lane & 31);
            dst[i] = r < p.row_end ? r : -1;
            if (!GELU && out_index) dst[i] = r < p.row_end ? out_index[r] : -1;
        }
        const Place after = it + 2 < n_items ? place(it + 2) : nowhere(q);
        fetch_rows(after, rows);
        asm volatile("" ::: "memory");                   // (these loads before the stores below: see stores_behind)
        DICEMOE_SCHED_FENCE();
        if (live) store_block<TM, TN, GELU, NB>(acc, bias_reg, c_rs, N, p.col_end, dst, col_first, lane);
        DICEMOE_SCHED_FENCE();
        asm volatile("" ::: "memory");
        fetch_bias(q);
        stores_behind = live;
        p = q;
        q = after;
        w_cur = w_nxt;
#pragma unroll
        for (int i = 0; i < QA; ++i) a_cur[i] = a_nxt[i];
    }
    wait_vmcnt<0>();                                 // the stages fetched beyond the last item must not land in what uses this LDS next
    block_barrier();
}

// All items of a workgroup on tiles of 256 x 64 TN
// OWN: the row index comes from `pairs`, before anything is loaded: into LDS for the first two items, and where the kernels behind read it for
// what a workgroup comes to after its LDS has been taken by stages.  That is the piece behind whole tiles: ffn_sorts_pairs lets in as many tiles as
// compute units by its estimate, of which there are half as many again at most, so that nobody has a third whole one.  Workgroups with
// an item's first columns leave its rows there in any case (who writes the same place writes the same).
template <int TN, bool GELU, bool GATHER, bool OWN>
__device__ __forceinline__ void stream_items(const StreamArgs& g, char* smem, XcdTiles& tiles, const StreamPairs* pairs = nullptr, const PairSort* sort = nullptr)
{
    constexpr int BM = 256, BN = 64 * TN;
    const int N = g.N;
    const int lane = threadIdx.x & 63;
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, n_slots = gridDim.x >> 3;
    tiles.deal_columns(BN, (N + BN - 1) / BN, xcd);
    const int rounds = tiles.count / n_slots;
    const int left = tiles.count - rounds * n_slots;
    const int pieces = leftover_pieces(BN, left, n_slots);
    const int n_whole = rounds + (pieces == 1 && slot < left ? 1 : 0);
    uint16_t* const own_rows = reinterpret_cast<uint16_t*>(smem);
    auto columns = [&](Place& p, int width) { p.col_end = p.col0 + width < N ? p.col0 + width : N; };
    auto locate_piece = [&](Place& p) {
        if (pieces == 1 || slot >= left * pieces) return false;
        const int tile = slot / pieces, piece = slot - tile * pieces;
        tiles.locate(rounds * n_slots + tile, p.row0, p.row_end, p.col0, p.e);
        p.row0 += (piece & 1) * (BM / 2);
        if (p.row_end > p.row0 + BM / 2) p.row_end = p.row0 + BM / 2;
        p.col0 += (piece >> 1) * (BN / 2);
        columns(p, pieces == 4 ? BN / 2 : BN);
        return p.row0 < p.row_end && p.col0 < p.col_end;       // else a piece without rows or columns
    };
    if constexpr (OWN) {
        Place p;
        const int n_items = n_whole + (locate_piece(p) ? 1 : 0);
        if (n_items == 0) return;
#pragma unroll 1
        for (int i = 0; i < n_items; ++i) {
            Place at = p;
            if (i < n_whole) {
                tiles.locate(slot + i * n_slots, at.row0, at.row_end, at.col0, at.e);
                if (at.row_end > at.row0 + BM) at.row_end = at.row0 + BM;
            }
            const int keep = i == n_whole && i > 0 ? 2 : i;        // (a piece behind whole tiles finds its rows in memory)
            const int seg = __builtin_ctzll(__ballot(at.row0 >= pairs->begin && at.row0 < pairs->end));
            pairs->each(seg, at.row0, at.row_end, [&](int r, int pair) {
                if (keep < 2) own_rows[keep * 256 + r - at.row0] = static_cast<uint16_t>(pair);
                if (keep >= 2 || at.col0 == 0) sort->perm[r] = pair;
                if (at.col0 == 0) sort->inv[pair] = r;
            });
        }
        asm volatile("" ::: "memory");                   // the rows are in LDS (stores to memory may be on their way)
        wait_lgkmcnt<0>();
        block_barrier();
    }
    if (n_whole > 0) {
        Place first;
        tiles.locate(slot, first.row0, first.row_end, first.col0, first.e);
        columns(first, BN);
        // Places of up to 64 items, item 64 w + l in lane l
        Place window;
        auto fill_window = [&](int w) {
            int i = w * 64 + lane;
            if (i > n_whole - 1) i = n_whole - 1;
            tiles.locate_each(slot + i * n_slots, window.row0, window.row_end, window.col0, window.e);
        };
        auto place = [&](int i) {
            if (i == 1 || (i & 63) == 0) fill_window(i >> 6);
            Place q;
            q.row0 = __builtin_amdgcn_readlane(window.row0, i & 63);
            q.row_end = __builtin_amdgcn_readlane(window.row_end, i & 63);
            q.col0 = __builtin_amdgcn_readlane(window.col0, i & 63);
            q.e = __builtin_amdgcn_readlane(window.e, i & 63);
            columns(q, BN);
            return q;
        };
        // 256 columns without GELU: wavefronts of 128 x 64 (2048 x 8192, 4 x 2048 rows, second GEMM: 1.42 - 1.55 us a step against 1.51 - 1.57
        // of 64 x 128, epilogue 2.7 - 2.9 against 3.1; with GELU, whose stores are the more, 1.69 against 1.59 at DiT-MoE-XL widths)
        if constexpr (TN == 4 && !GELU) stream_tiles<4, 2, 2, 2, 3, GELU, GATHER, OWN, 2, 4>(g, smem, n_whole, first, place, own_rows);
        else stream_tiles<2, TN, 2, 2, TN == 3 ? 4 : 3, GELU, GATHER, OWN, 4, 2>(g, smem, n_whole, first, place, own_rows);
    }
    Place p;
    if (locate_piece(p)) {
        auto same = [&](int) { return p; };
        auto run = [&](auto own) {
            constexpr bool O = decltype(own)::value;
            if constexpr (TN == 3) stream_tiles<1, 3, 2, 4, 4, GELU, GATHER, O, 4, 2>(g, smem, 1, p, same, own_rows);
            else if (pieces == 4) stream_tiles<1, 2, 2, 5, 5, GELU, GATHER, O, 4, 2>(g, smem, 1, p, same, own_rows);
            else stream_tiles<1, 4, 2, 3, 3, GELU, GATHER, O, 4, 2>(g, smem, 1, p, same, own_rows);
        };
        if constexpr (OWN) {
            if (n_whole == 0) {
                run(std::true_type{});
                return;
            }
        }
        run(std::false_type{});
    }
}

// Both widths: `planned` unless the table says the other one
struct StreamWidths { int planned; StreamCost c192, c256; };

// TN: 3 or 4, 192 or 256 columns, or 0: as StreamWidths says.  OWN: the workgroup sorts the pairs itself (ffn_sorts_pairs).
template <int TN, bool GELU, bool GATHER, bool OWN>
__global__ __launch_bounds__(512, 1) void ffn_gemm_bf16_stream_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, const float* __restrict__ bias,
    bf16_t* __restrict__ C, int N, int K, const int32_t* __restrict__ seg_offsets,
    const int32_t* __restrict__ seg_expert, int n_seg,
    const int32_t* __restrict__ row_index, int row_div, const int32_t* __restrict__ out_index,
    int max_rows, int32_t* __restrict__ status, std::conditional_t<TN == 0, StreamWidths, NoMore> widths, OwnSort<OWN> sort)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    XcdTiles tiles;
    StreamArgs g = {A, W, bias, C, N, K, row_index, row_div, out_index};
    const int expert = XcdTiles::expert_of(seg_expert, n_seg);
    StreamPairs pairs;
    const PairSort* own = nullptr;
    if constexpr (OWN) {
        static_assert((kStreamOwnRows & 255) == 0 && kStreamGrid * kWave >= kStreamSortPairs, "every 64 pairs have a workgroup");
        pairs.form(sort, smem + kStreamOwnRows * 2);
        own = &sort;
        g.row_index = sort.perm;                            // (written here: not through the argument that nobody writes)
        report_rows(status, pairs.rows, max_rows);
        tiles.set(pairs.begin, pairs.end, expert, n_seg, 256, max_rows);
        if (pairs.rows > max_rows)                          // rows that no tile has
            for (int e = blockIdx.x; e < n_seg; e += gridDim.x) {
                const int lo = __builtin_amdgcn_readlane(pairs.begin, e), hi = __builtin_amdgcn_readlane(pairs.end, e);
                pairs.each(e, lo > max_rows ? lo : max_rows, hi, [&](int r, int p) { sort.perm[r] = p; sort.inv[p] = r; });
            }
    } else {
        report_row_overflow(status, seg_offsets, n_seg, max_rows);
        tiles.load(seg_offsets, expert, n_seg, 256, max_rows);
    }
    auto items = [&](auto tn) { stream_items<decltype(tn)::value, GELU, GATHER, OWN>(g, smem, tiles, &pairs, own); };
    if constexpr (TN == 0) {
        if (stream_columns(widths.planned, widths.c192, widths.c256, tiles.all_row_tiles()) == 192) items(std::integral_constant<int, 3>{});
        else items(std::integral_constant<int, 4>{});
    } else {
        items(std::integral_constant<int, TN>{});
    }
}

template <bool GELU>
static hipError_t configure_gemm_bf16_stream()
{
    hipError_t err = hipSuccess;
    auto raise = [&](auto kern) {
        if (err == hipSuccess) err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kStreamLds);
    };
    raise(&ffn_gemm_bf16_stream_kernel<0, GELU, false, false>);
    raise(&ffn_gemm_bf16_stream_kernel<3, GELU, false, false>);
    raise(&ffn_gemm_bf16_stream_kernel<4, GELU, false, false>);
    if constexpr (GELU) {
        raise(&ffn_gemm_bf16_stream_kernel<0, GELU, true, false>);
        raise(&ffn_gemm_bf16_stream_kernel<3, GELU, true, false>);
        raise(&ffn_gemm_bf16_stream_kernel<4, GELU, true, false>);
        raise(&ffn_gemm_bf16_stream_kernel<0, GELU, true, true>);
        raise(&ffn_gemm_bf16_stream_kernel<3, GELU, true, true>);
        raise(&ffn_gemm_bf16_stream_kernel<4, GELU, true, true>);
    }
    return err;
}

template <int TN, bool GELU, typename Widths>
static hipError_t launch_gemm_bf16_stream_kernel(const void* A, const void* W, const float* bias, void* C, int N, int K,
                                                 const int32_t* seg_offsets, const int32_t* seg_expert, int n_seg, int max_rows,
                                                 hipStream_t stream, const int32_t* row_index, int row_div,
                                                 const int32_t* out_index, int32_t* status, const PairSort* sort, Widths widths)
{
    auto launch = [&](auto kern, auto own) {
        hipLaunchKernelGGL(kern, dim3(kStreamGrid), dim3(kStreamThreads), kStreamLds, stream, static_cast<const bf16_t*>(A),
                           static_cast<const bf16_t*>(W), bias, static_cast<bf16_t*>(C), N, K, seg_offsets, seg_expert, n_seg,
                           row_index, row_div, out_index, max_rows, status, widths, own);
        return hipGetLastError();
    };
    if constexpr (GELU) {
        if (sort) return launch(&ffn_gemm_bf16_stream_kernel<TN, true, true, true>, *sort);
        if (row_index) return launch(&ffn_gemm_bf16_stream_kernel<TN, true, true, false>, NoMore{});
    }
    return launch(&ffn_gemm_bf16_stream_kernel<TN, GELU, false, false>, NoMore{});
}

// columns: 192 or 256, as planned on the host's estimate
template <bool GELU>
static hipError_t launch_gemm_bf16_stream(int columns, const void* A, const void* W, const float* bias, void* C, int N, int K,
                                          const int32_t* seg_offsets, const int32_t* seg_expert, int n_seg, int max_rows,
                                          hipStream_t stream, const int32_t* row_index, int row_div,
                                          const int32_t* out_index, int32_t* status, const PairSort* sort = nullptr)
{
    // every ring needs one step more than it is deep; only the first GEMM gathers its rows
    if (n_seg > 64 || K / 64 < 6 || (!GELU && row_index) || (sort && (!row_index || sort->n_pairs > kStreamSortPairs))) return hipErrorInvalidValue;
#define DICEMOE_STREAM(TN, widths) \
    return launch_gemm_bf16_stream_kernel<TN, GELU>(A, W, bias, C, N, K, seg_offsets, seg_expert, n_seg, max_rows, stream, row_index, row_div, out_index, status, sort, widths)
    if (stream_looks(columns, N, K, GELU, max_rows, n_seg)) {
        const StreamWidths widths = {columns, stream_cost_192(N, K, GELU), stream_cost_256(N, K, GELU)};
        DICEMOE_STREAM(0, widths);
    }
    if (columns == 192) DICEMOE_STREAM(3, NoMore{});
    DICEMOE_STREAM(4, NoMore{});
#undef DICEMOE_STREAM
}

}  // namespace dicemoe
