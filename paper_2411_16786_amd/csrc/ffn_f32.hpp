// Grouped GEMM of the expert FFN for float storage, on the matrix cores: small tiles whose reduction is shared by the
// wavefronts of a workgroup, larger ones once they fill the chip.
//
// What bounds it.  Float workloads here are small (a few hundred rows, 16 experts): a 64 x 64 tile on the vector units
// walked all of K = 1536 in 96 barrier-separated steps of LDS stores and reads, and the second GEMM has too few such tiles for
// the chip.  Hence
//   * a workgroup's four wavefronts each take a contiguous quarter of K for the same tile; they meet once, in LDS,
//     where the partial sums are added in wavefront order (the same bits in every run, for a row wherever it lies, and on
//     either tile).  No barrier and no LDS in the main loop;
//   * operands come from global memory in MFMA layout (RowMfma): a 64-byte unit of a 16-row block is one 16-byte load per
//     lane.  32 x 32 tiles have three units in flight per wavefront, sixteen wavefronts per compute unit; 64 x 64 tiles, which
//     move half the bytes per flop, one unit and eight wavefronts (with two and three units 5 - 20 % slower).
// Both GEMMs, graph of ten calls, against 64 x 64 tiles on the vector units: DiT-MoE-S widths, 500 tokens top-2: 137 -> 56 us; 100
// tokens 127 -> 28; 64 x 256, 4 experts, 64 tokens 28 -> 10, all on 32 x 32 tiles.  On those alone many rows lose what few
// gain: 16384 rows of the DiT-MoE-S widths 577 us on the vector units, 595 on 32 x 32 tiles, 493 on 64 x 64; 8192 of DiT-MoE-XL 2422, 2604
// and 1769.  Which of these sizes the ring kernel below has taken over since: f32_tile.
#pragma once
#include "ffn_mfma.hpp"
#include "ffn_plan.hpp"
#include "ffn_stream.hpp"
#include "kernels.hpp"

namespace dicemoe {

constexpr int kDirectShares = 4;                         // wavefronts sharing K
constexpr long long kDirectGrid = 1 << 20;

// find_row_tile for a whole wavefront: 64 segments at a time, one per lane, instead of a chain of dependent loads.  A table of 1024 is
// walked by every workgroup of a grid four times as fine as that of 64 x 64 tiles (64 x 256, 64 experts in 1024 segments, 4096 rows, both
// GEMMs: 2727 us segment by segment, 166 so; 64 x 64 tiles on the vector units, segment by segment, 625).
__device__ __forceinline__ bool find_row_tile_by_lanes(const int32_t* __restrict__ seg_offsets, int n_seg, int BM, int tile, int& seg,
                                                       int& row0, int& row_end)
{
    const int lane = threadIdx.x & 63;
    for (int g0 = 0; g0 < n_seg; g0 += 64) {
        const int g = g0 + lane;
        const int begin = g < n_seg ? seg_offsets[g] : 0, end = g < n_seg ? seg_offsets[g + 1] : 0;
        const int nt = (end - begin + BM - 1) / BM;
        const int incl = wave_scan(nt);
        const uint64_t hit = __ballot(tile < incl);          // the first lane's segment holds the tile
        if (hit != 0) {
            const int l = __builtin_ctzll(hit);
            seg = g0 + l;
            row0 = __builtin_amdgcn_readlane(begin, l) + (tile - __builtin_amdgcn_readlane(incl - nt, l)) * BM;
            row_end = __builtin_amdgcn_readlane(end, l);
            return true;
        }
        tile -= __builtin_amdgcn_readlane(incl, 63);
    }
    return false;
}

// TM, TN: 16-row blocks of a tile, rows and columns; U: units in flight; MANY: more segments than a wavefront has lanes (a kernel of
// its own: with both ways of finding a tile in one, 500 tokens of the DiT-MoE-S widths take 2 us more)
template <bool GELU, int TM, int TN, int U, bool MANY, bool SELF>
__global__ __launch_bounds__(64 * kDirectShares, TM * TN > 4 ? 2 : 4) void ffn_gemm_f32_kernel(
    const float* __restrict__ A, const float* __restrict__ W, const float* __restrict__ bias, float* __restrict__ C, int N, int K,
    const int32_t* __restrict__ seg_offsets, const int32_t* __restrict__ seg_expert, int n_seg, int n_tiles_n,
    const int32_t* __restrict__ row_index, int row_div, const int32_t* __restrict__ out_index, int max_rows,
    int32_t* __restrict__ status, OwnSort<SELF> sort)
{
    typedef RowMfma<float> M;
    constexpr int KS = kDirectShares;
    static_assert(!(SELF && MANY), "a workgroup that sorts the pairs itself knows 64 experts at most");
    constexpr int BM = 16 * TM, BN = 16 * TN, BLOCKS = TM * TN;
    constexpr int CH = 4;                                // 16-byte chunks per unit
    __shared__ __attribute__((aligned(16))) f32x4_t part[KS][BLOCKS][64];
    const int32_t* seg_table = seg_offsets;
    const uint16_t* own_rows = nullptr;
    if constexpr (SELF) {                                // this workgroup's own dispatch
        __shared__ int scratch[own_sort_ints(KS)];
        __shared__ uint16_t rows_lds[kOwnSortPairs];
        seg_table = sort_pairs<KS>(sort, blockIdx.x == 0, scratch, rows_lds);
        own_rows = rows_lds;
    }
    report_row_overflow(status, seg_table, n_seg, max_rows);

    // ---- place: the tiles of an expert on one XCD (its weights and rows stay in that XCD's L2) while the segment table
    // fits a wavefront, else in segment order
    XcdTiles tiles;
    if constexpr (!MANY) tiles.deal(seg_table, seg_expert, n_seg, BM, BN, n_tiles_n, blockIdx.x & 7, max_rows);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = lane & 15, quarter = lane >> 4;

    // ---- this wavefront's share of K
    const int units = K / M::kUnit;
    const int u0 = units * wave / KS, n = units * (wave + 1) / KS - u0;
    const int last = n > 0 ? n - 1 : 0;                  // (a share may be empty; u0 < units all the same)

    // one tile per workgroup unless that would be a grid beyond what a launch takes
    for (int id = blockIdx.x;; id += gridDim.x) {
        int row0, row_end, n0, e;
        if constexpr (!MANY) {
            const int slot = id >> 3;
            if (slot >= tiles.count) return;
            tiles.locate(slot, row0, row_end, n0, e);
        } else {
            const int tile_m = id / n_tiles_n;
            int seg;
            if (!find_row_tile_by_lanes(seg_offsets, n_seg, BM, tile_m, seg, row0, row_end)) return;
            row_end = row_end < max_rows ? row_end : max_rows;
            if (row0 >= row_end) return;                     // (rows of the tiles behind it are further out still)
            e = seg_expert[seg];
            n0 = (id - tile_m * n_tiles_n) * BN;
        }
        const u32x4_t* a_src[TM];
        const u32x4_t* w_src[TN];
        const float* We = W + static_cast<size_t>(e) * N * K;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            int c = n0 + 16 * j + sub;
            c = c < N ? c : N - 1;                           // columns that do not exist repeat the last one; never stored
            w_src[j] = reinterpret_cast<const u32x4_t*>(We + static_cast<size_t>(c) * K) + u0 * CH + quarter;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            int r = row0 + 16 * i + sub;
            r = r < row_end ? r : row_end - 1;               // rows past the segment repeat its last one; never stored
            if constexpr (SELF) r = own_rows[r] / row_div;
            else if (row_index) r = row_index[r] / row_div;
            a_src[i] = reinterpret_cast<const u32x4_t*>(A + static_cast<size_t>(r) * K) + u0 * CH + quarter;
        }
        f32x4_t acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

        u32x4_t av[U][TM], wv[U][TN];
        auto load = [&](int s, int u) {
#pragma unroll
            for (int j = 0; j < TN; ++j) wv[s][j] = w_src[j][u * CH];
#pragma unroll
            for (int i = 0; i < TM; ++i) av[s][i] = a_src[i][u * CH];
        };
        auto multiply = [&](int s) {
#pragma unroll
            for (int t = 0; t < M::kMfma; ++t)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = M::step(wv[s][j], av[s][i], acc[i][j], t);
        };
        // U units in flight.  Loads are unconditional (past the share they repeat its last unit) and fenced between the
        // multiplications, so that the compiler keeps them there and waits for the oldest unit alone.
#pragma unroll
        for (int s = 0; s < U; ++s) {
            DICEMOE_SCHED_FENCE();
            load(s, s < last ? s : last);
        }
        int u = 0;
        for (; u + U < n; u += U) {
#pragma unroll
            for (int s = 0; s < U; ++s) {
                DICEMOE_SCHED_FENCE();
                multiply(s);
                DICEMOE_SCHED_FENCE();
                load(s, u + U + s < last ? u + U + s : last);
            }
        }
#pragma unroll
        for (int s = 0; s < U; ++s) {
            DICEMOE_SCHED_FENCE();
            if (u + s < n) multiply(s);
        }

        // ---- the partial sums meet; wavefront w finishes blocks w, w + KS, ...
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) part[wave][i * TN + j][lane] = acc[i][j];
        __syncthreads();
        for (int b = wave; b < BLOCKS; b += KS) {
            const int i = b / TN, j = b - i * TN;
            f32x4_t sum = part[0][b][lane];
#pragma unroll
            for (int w = 1; w < KS; ++w) sum += part[w][b][lane];
            // operands swapped: lane (sub, quarter) holds columns 4 quarter .. + 3 of row sub
            const int r = row0 + 16 * i + sub, c = n0 + 16 * j + 4 * quarter;
            if (r >= row_end || c >= N) continue;
            const int dst = out_index ? out_index[r] : r;
            if (dst < 0) continue;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                sum[t] += bias ? bias[static_cast<size_t>(e) * N + c + t] : 0.f;
                if (GELU) sum[t] = gelu_erf(sum[t]);
            }
            *reinterpret_cast<f32x4_t*>(C + static_cast<size_t>(dst) * N + c) = sum;
        }
        __syncthreads();                                 // the partial sums have been read
    }
}

template <bool GELU, int TM, int TN, int U>
static hipError_t launch_gemm_f32_tile(const float* A, const float* W, const float* bias, float* C, int N, int K,
                                       const int32_t* seg_offsets, const int32_t* seg_expert, int n_seg, int max_rows,
                                       hipStream_t stream, const int32_t* row_index, int row_div, const int32_t* out_index,
                                       int32_t* status, const PairSort* sort = nullptr)
{
    constexpr int BM = 16 * TM, BN = 16 * TN;
    const int n_tiles_n = (N + BN - 1) / BN;
    const long long tiles = (static_cast<long long>(max_rows) + BM - 1) / BM * n_tiles_n + static_cast<long long>(n_seg) * n_tiles_n;
    const long long blocks = (tiles + 7) / 8 * 8;        // every XCD gets room for ceil(tiles / 8)
    const dim3 grid(static_cast<unsigned>(blocks < kDirectGrid ? blocks : kDirectGrid));
    if constexpr (GELU && TM * TN <= 4) {
        if (sort) {
            hipLaunchKernelGGL((ffn_gemm_f32_kernel<GELU, TM, TN, U, false, true>), grid, dim3(64 * kDirectShares), 0, stream, A, W, bias, C, N, K,
                               seg_offsets, seg_expert, n_seg, n_tiles_n, row_index, row_div, out_index, max_rows, status, *sort);
            return hipGetLastError();
        }
    }
    const auto kern = n_seg > 64 ? &ffn_gemm_f32_kernel<GELU, TM, TN, U, true, false> : &ffn_gemm_f32_kernel<GELU, TM, TN, U, false, false>;
    hipLaunchKernelGGL(kern, grid, dim3(64 * kDirectShares), 0, stream, A, W, bias, C, N, K, seg_offsets, seg_expert, n_seg, n_tiles_n, row_index,
                       row_div, out_index, max_rows, status, NoMore{});
    return hipGetLastError();
}

// The ring kernel.  What bounds the kernel above at some tens of rows per expert (DiT-MoE-S widths, 500 tokens: time stamps per workgroup):
// loads into registers hold a line of the 32 KB vector cache each while they are in flight, so that a compute unit has 32 KB of cold
// weights on their way at most, and every workgroup waits for segment table, row indices and first loads in turn (8 of its 17 us).  Here
//   * operands go to LDS directly (a row's whole 128-byte line per eight lanes), into a ring of D stages that each wavefront has to
//     itself: no barrier in the main loop, because no wavefront reads what another one loaded;
//   * a wavefront still has a quarter of K, and the quarters meet in LDS in wavefront order: the same bits as above;
//   * the workgroups that fit the chip walk a list of tiles each, and the rings run on across tiles: row indices, biases and output
//     rows come through LDS as well, so that no load into a register makes the wavefront wait for the loads behind it.
// 32 x 32 tiles, two stages, two workgroups per compute unit (one multiplies while the other one's sums meet): three or four stages and one
// workgroup are slower, also with 32 x 64 tiles (500 tokens of DiT-MoE-S, both GEMMs: 66.6 us above; 55.1; 66.5 four stages; 57.2
// 32 x 64 in three).  64 x 64 tiles, two stages, one workgroup, move half the bytes per flop: ring_wide says where that is better.
// What bounds it now is the way into LDS: 10 TB/s of stage loads where L2 misses keep 64 to 128 KB per compute unit in flight for
// about 2 us, as in the bf16 kernels.  Both GEMMs, us, above / here: DiT-MoE-S, 18 tokens top-3 30.5 / 26.8, 2000 tokens 179 / 139, 8192: 508 / 480;
// DiT-MoE-XL, 100 tokens 157 / 103, 2000: 984 / 880; 2048 x 8192, 4 experts, 200 tokens 458 / 309.
// K is a multiple of 128 (equal shares of whole stages) and at least kRingMinK (two stages a share).
constexpr int ring_lds(int tm, int tn, int d, bool self = false)
{
    return kDirectShares * (d * 16 * (tm + tn) * 128 + (kDirectShares - 1) * 1024 + (self ? 512 : 768)) + (self ? kOwnSortPairs * 2 : 0);
}
template <bool GELU, int TM, int TN, int D, bool SELF>
__global__ __launch_bounds__(64 * kDirectShares, ring_lds(TM, TN, D, SELF) <= 80 * 1024 ? 2 : 1) void ffn_gemm_f32_ring_kernel(
    const float* __restrict__ A, const float* __restrict__ W, const float* __restrict__ bias, float* __restrict__ C, int N, int K,
    const int32_t* __restrict__ seg_offsets, const int32_t* __restrict__ seg_expert, int n_seg, int n_tiles_n,
    const int32_t* __restrict__ row_index, int row_div, const int32_t* __restrict__ out_index, int max_rows,
    int32_t* __restrict__ status, OwnSort<SELF> sort)
{
    typedef RowMfma<float> M;
    constexpr int KS = kDirectShares;
    constexpr int BM = 16 * TM, BN = 16 * TN;
    constexpr int QA = BM / 8, QB = BN / 8, Q = QA + QB;  // loads of a stage: eight rows each
    constexpr int STAGE = (BM + BN) * 128;
    constexpr int CH = 8;
    static_assert(32 * KS * D <= kRingMinK, "a share of K has D stages at least: what is asked for a tile ahead has landed by then");
    static_assert(TM * TN % KS == 0 && BN <= 64 && BM <= 64, "blocks for every wavefront; a lane each for a tile's columns and rows");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = lane & 15, quarter = lane >> 4;
    char* const ring = smem + wave * D * STAGE;
    f32x4_t* const meet = reinterpret_cast<f32x4_t*>(smem + KS * D * STAGE);      // [KS][KS - 1][64]
    char* const behind = smem + KS * D * STAGE + KS * (KS - 1) * 1024;
    char* const aux = behind + wave * (SELF ? 512 : 768);
    int32_t* const dst_lds = reinterpret_cast<int32_t*>(aux);                     // output rows and biases of the tile that is multiplied
    float* const bias_lds = reinterpret_cast<float*>(aux + 256);
    int32_t* const rows_lds = reinterpret_cast<int32_t*>(aux + 512);              // row indices of the tile that the ring goes on to
    uint16_t* const own_rows = reinterpret_cast<uint16_t*>(behind + KS * 512);    // SELF: all of them, sorted by this workgroup

    const int32_t* seg_table = seg_offsets;
    if constexpr (SELF) {
        static_assert(own_sort_ints(KS) * 4 <= KS * (KS - 1) * 1024, "the sort's scratch fits the place where the sums meet");
        seg_table = sort_pairs<KS>(sort, blockIdx.x == 0, reinterpret_cast<int*>(meet), own_rows);
    }
    report_row_overflow(status, seg_table, n_seg, max_rows);
    XcdTiles tiles;
    tiles.deal(seg_table, seg_expert, n_seg, BM, BN, n_tiles_n, blockIdx.x & 7, max_rows);
    if constexpr (SELF) __syncthreads();                 // every wavefront has the table: sums can meet where it was
    const int slot = blockIdx.x >> 3, n_slots = gridDim.x >> 3;
    const int n_items = tiles.count > slot ? (tiles.count - slot + n_slots - 1) / n_slots : 0;
    if (n_items == 0) return;

    // ---- this wavefront's stages of K, 32 values each
    const int n = K / (32 * KS), s0 = n * wave;

    struct Item { int row0, row_end, n0, e; };
    auto locate = [&](int i) {
        Item t;
        tiles.locate(slot + i * n_slots, t.row0, t.row_end, t.n0, t.e);
        return t;
    };
    // 64 values of an array to LDS, lane l's from index `at` of its own
    auto to_lds = [&](const void* array, int at, void* lds) {
        __builtin_amdgcn_global_load_lds(DICEMOE_GLOBAL_PTR(reinterpret_cast<const char*>(array) + static_cast<size_t>(at) * 4), DICEMOE_LDS_PTR(lds), 4, 0, 0);
    };
    auto row_of = [&](const Item& t, int i) { return t.row0 + i < t.row_end ? t.row0 + i : t.row_end - 1; };      // (rows past the end repeat the last one)
    auto ask_rows = [&](const Item& t) {
        if (!SELF && row_index) to_lds(row_index, row_of(t, lane), rows_lds);
    };
    // Load q of a stage fills rows 8q .. 8q + 7; lane l lands at LDS slot (row 8q + l / 8, l % 8) and fetches the chunk that the swizzle
    // assigns to it.
    const char* a_src[QA];
    const char* w_src[QB];
    auto sources = [&](const Item& t) {                  // its row indices have landed
#pragma unroll
        for (int q = 0; q < QA; ++q) {
            const int i = 8 * q + (lane >> 3);
            const int r = SELF ? own_rows[row_of(t, i)] / row_div : row_index ? rows_lds[i] / row_div : row_of(t, i);
            a_src[q] = reinterpret_cast<const char*>(A + static_cast<size_t>(r) * K + s0 * 32) + ((lane & 7) ^ chunk_swizzle<CH>(i)) * 16;
        }
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            const int i = 8 * q + (lane >> 3);
            const int c = t.n0 + i < N ? t.n0 + i : N - 1;
            w_src[q] = reinterpret_cast<const char*>(W + (static_cast<size_t>(t.e) * N + c) * K + s0 * 32) + ((lane & 7) ^ chunk_swizzle<CH>(i)) * 16;
        }
    };
    auto load = [&](int q, int to, int s) {              // load q of stage s of this wavefront's share
        const char* src = (q < QA ? a_src[q < QA ? q : 0] : w_src[q < QA ? 0 : q - QA]) + s * 128;
        __builtin_amdgcn_global_load_lds(DICEMOE_GLOBAL_PTR(src), DICEMOE_LDS_PTR(ring + to * STAGE + q * 1024), 16, 0, 0);
    };
    int f_off[2];                                        // of 16-row block 0 in a stage; blocks are 2 KB apart (same swizzle)
#pragma unroll
    for (int h = 0; h < 2; ++h) f_off[h] = (sub * CH + ((4 * h + quarter) ^ chunk_swizzle<CH>(sub))) * 16;
    u32x4_t fr[2][TM + TN];
    auto read = [&](int h, int from) {
#pragma unroll
        for (int f = 0; f < TM + TN; ++f) fr[h][f] = *reinterpret_cast<const u32x4_t*>(ring + from * STAGE + f * 2048 + f_off[h]);
    };

    // ---- the ring's end: stage `is` of item `ii`; `ahead` is the item behind it, whose row indices have been asked for
    auto landed = [] {                                   // (LDS is read behind the wait, not before it)
        asm volatile("" ::: "memory");
        DICEMOE_SCHED_FENCE();
    };
    const int total = n_items * n;
    int is = 0, ii = 0, issued = 0;
    Item cur = locate(0), nxt = n_items > 1 ? locate(1) : cur, ahead = nxt;
    ask_rows(cur);
    wait_vmcnt<0>();
    landed();
    sources(cur);
    wait_lgkmcnt<0>();
    ask_rows(ahead);
    auto issued_one = [&] {                              // behind the loads of stage `is`
        ++issued;
        if (++is == n) {
            // (n - 1) Q loads were issued behind the row indices before the last wait for a stage, which left (D - 1) Q
            is = 0;
            ++ii;
            sources(ahead);
            wait_lgkmcnt<0>();
            if (ii + 1 < n_items) ahead = locate(ii + 1);
            ask_rows(ahead);
        }
    };
#pragma unroll
    for (int s = 0; s < D; ++s) {
        if (issued < total) {
#pragma unroll
            for (int q = 0; q < Q; ++q) load(q, s, is);
            if (is == n - 1) { wait_vmcnt<0>(); landed(); }      // (the row indices of the next tile: no wait for a stage so far)
            issued_one();
        }
    }
    int at = 0, seq = 0;
    if (issued == D) wait_vmcnt<(D - 1) * Q>(); else wait_vmcnt<0>();
    landed();
    read(0, 0);
    wait_lgkmcnt<0>();
    for (int it = 0; it < n_items; ++it) {
        f32x4_t acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (out_index) to_lds(out_index, row_of(cur, lane), dst_lds);
        if (bias) to_lds(bias, cur.e * N + (cur.n0 + lane < N ? cur.n0 + lane : N - 1), bias_lds);
        const int live = (cur.row_end - cur.row0 + 15) / 16;      // 16-row blocks that have rows
        auto multiply = [&](int h) {                     // products of half h of a stage
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (i == 0 || i < live) {
#pragma unroll
                    for (int t = 0; t < M::kMfma; ++t)
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[i][j] = M::step(fr[h][TM + j], fr[h][i], acc[i][j], t);
                }
            }
        };
        for (int s = 0; s < n; ++s) {
            DICEMOE_SCHED_FENCE();
            read(1, at);
            DICEMOE_SCHED_FENCE();
            multiply(0);
            DICEMOE_SCHED_FENCE();
            wait_lgkmcnt<0>();                           // this stage is in registers: its slot can be filled again
            const int here = at;
            at = at + 1 == D ? 0 : at + 1;
            ++seq;
            // (all loads of the refill at once: spread over the products of the second half they cost 5 - 9 us of 55)
            if (issued < total) {
#pragma unroll
                for (int q = 0; q < Q; ++q) load(q, here, is);
                issued_one();
            }
            if (issued - seq >= D) wait_vmcnt<(D - 1) * Q>(); else wait_vmcnt<0>();      // the next stage has landed
            landed();
            if (seq < total) read(0, at);
            DICEMOE_SCHED_FENCE();
            multiply(1);
            DICEMOE_SCHED_FENCE();
            wait_lgkmcnt<0>();
        }
        // ---- the partial sums meet, KS blocks at a time; wavefront w finishes the w-th of them.  Biases and output rows have landed: they
        // were asked for n stages ago
#pragma unroll
        for (int b0 = 0; b0 < TM * TN; b0 += KS) {
            f32x4_t own = acc[b0 / TN][b0 % TN];
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                const int b = b0 + j;
                if (j == wave) own = acc[b / TN][b % TN];
                else meet[(wave * (KS - 1) + (j > wave ? j - 1 : j)) * 64 + lane] = acc[b / TN][b % TN];
            }
            wait_lgkmcnt<0>();
            block_barrier();
            f32x4_t part[KS];                            // (this wavefront's own share never went through LDS; some other one is read in its place)
#pragma unroll
            for (int w = 0; w < KS; ++w) part[w] = meet[(w * (KS - 1) + (wave > w ? wave - 1 : (wave < w ? wave : 0))) * 64 + lane];
            f32x4_t sum = wave == 0 ? own : part[0];
#pragma unroll
            for (int w = 1; w < KS; ++w) sum += wave == w ? own : part[w];
            const int i = (b0 + wave) / TN, c_in = 16 * ((b0 + wave) % TN) + 4 * quarter, c = cur.n0 + c_in;
            f32x4_t b = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (bias) b = *reinterpret_cast<const f32x4_t*>(bias_lds + c_in);
            const int r = cur.row0 + 16 * i + sub;
            const int dst = r < cur.row_end ? (out_index ? dst_lds[16 * i + sub] : r) : -1;
            wait_lgkmcnt<0>();
            block_barrier();
            if (dst >= 0 && c < N) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    sum[t] += b[t];
                    if (GELU) sum[t] = gelu_erf(sum[t]);
                }
                *reinterpret_cast<f32x4_t*>(C + static_cast<size_t>(dst) * N + c) = sum;
            }
        }
        cur = nxt;
        if (it + 2 < n_items) nxt = locate(it + 2);
    }
}

template <bool GELU, int TM, int TN, int D, bool SELF = false>
static hipError_t configure_gemm_f32_ring()
{
    return hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_gemm_f32_ring_kernel<GELU, TM, TN, D, SELF>), hipFuncAttributeMaxDynamicSharedMemorySize, ring_lds(TM, TN, D, SELF));
}

template <bool GELU, int TM, int TN, int D, bool SELF = false>
static hipError_t launch_gemm_f32_ring(const float* A, const float* W, const float* bias, float* C, int N, int K,
                                       const int32_t* seg_offsets, const int32_t* seg_expert, int n_seg, int max_rows,
                                       hipStream_t stream, const int32_t* row_index, int row_div, const int32_t* out_index,
                                       int32_t* status, OwnSort<SELF> sort = {})
{
    constexpr int BN = 16 * TN, smem = ring_lds(TM, TN, D, SELF);
    static_assert(smem <= 160 * 1024, "the rings and the meeting place fit a compute unit's LDS");
    hipLaunchKernelGGL((ffn_gemm_f32_ring_kernel<GELU, TM, TN, D, SELF>), dim3(kStreamGrid * (smem <= 80 * 1024 ? 2 : 1)), dim3(64 * kDirectShares), smem, stream, A, W, bias, C, N, K,
                       seg_offsets, seg_expert, n_seg, (N + BN - 1) / BN, row_index, row_div, out_index, max_rows, status, sort);
    return hipGetLastError();
}

template <bool GELU>
static hipError_t launch_gemm_f32(const void* A, const void* W, const float* bias, void* C, int N, int K,
                                  const int32_t* seg_offsets, const int32_t* seg_expert, int n_seg, int max_rows,
                                  hipStream_t stream, const int32_t* row_index = nullptr, int row_div = 1,
                                  const int32_t* out_index = nullptr, int32_t* status = nullptr, const PairSort* sort = nullptr)
{
    const float *a = static_cast<const float*>(A), *w = static_cast<const float*>(W);
    float* c = static_cast<float*>(C);
#define DICEMOE_F32(fn, ...) return fn<GELU, __VA_ARGS__>(a, w, bias, c, N, K, seg_offsets, seg_expert, n_seg, max_rows, stream, row_index, row_div, out_index, status
    switch (f32_tile(N, K, max_rows, n_seg)) {
    case F32Tile::Ring64:
        if (sort) break;                                 // (ffn_sorts_pairs)
        DICEMOE_F32(launch_gemm_f32_ring, 4, 4, 2));
    case F32Tile::Ring32:
        if constexpr (GELU) {
            if (sort) DICEMOE_F32(launch_gemm_f32_ring, 2, 2, 2, true), *sort);
        }
        DICEMOE_F32(launch_gemm_f32_ring, 2, 2, 2));
    case F32Tile::Direct64:
        if (sort) break;
        DICEMOE_F32(launch_gemm_f32_tile, 4, 4, 1));
    case F32Tile::Direct32: DICEMOE_F32(launch_gemm_f32_tile, 2, 2, 3), sort);
    }
#undef DICEMOE_F32
    return hipErrorInvalidValue;
}

}  // namespace dicemoe
