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
// and 1769.  What bounds the small tiles now was not separated: 33 us and 28 us at 500 tokens (kernel trace) move 185 MB each
// into the compute units, 38 MB of them cold weights; the matrix pipes need 8 us each.
#pragma once
#include "ffn_mfma.hpp"
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
        int incl = nt;
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) {
            const int v = __shfl_up(incl, sh, 64);
            if (lane >= sh) incl += v;
        }
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
template <bool GELU, int TM, int TN, int U, bool MANY>
__global__ __launch_bounds__(64 * kDirectShares, TM * TN > 4 ? 2 : 4) void ffn_gemm_f32_kernel(
    const float* __restrict__ A, const float* __restrict__ W, const float* __restrict__ bias, float* __restrict__ C, int N, int K,
    const int32_t* __restrict__ seg_offsets, const int32_t* __restrict__ seg_expert, int n_seg, int n_tiles_n,
    const int32_t* __restrict__ row_index, int row_div, const int32_t* __restrict__ out_index, int max_rows,
    int32_t* __restrict__ status)
{
    typedef RowMfma<float> M;
    constexpr int KS = kDirectShares;
    constexpr int BM = 16 * TM, BN = 16 * TN, BLOCKS = TM * TN;
    constexpr int CH = 4;                                // 16-byte chunks per unit
    __shared__ __attribute__((aligned(16))) f32x4_t part[KS][BLOCKS][64];
    report_row_overflow(status, seg_offsets, n_seg, max_rows);

    // ---- place: the tiles of an expert on one XCD (its weights and rows stay in that XCD's L2) while the segment table
    // fits a wavefront, else in segment order
    XcdTiles tiles;
    if constexpr (!MANY) tiles.deal(seg_offsets, seg_expert, n_seg, BM, BN, n_tiles_n, blockIdx.x & 7, max_rows);
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
            if (row_index) r = row_index[r] / row_div;
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
                                       int32_t* status)
{
    constexpr int BM = 16 * TM, BN = 16 * TN;
    const int n_tiles_n = (N + BN - 1) / BN;
    const long long tiles = (static_cast<long long>(max_rows) + BM - 1) / BM * n_tiles_n + static_cast<long long>(n_seg) * n_tiles_n;
    const long long blocks = (tiles + 7) / 8 * 8;        // every XCD gets room for ceil(tiles / 8)
    const auto kern = n_seg > 64 ? &ffn_gemm_f32_kernel<GELU, TM, TN, U, true> : &ffn_gemm_f32_kernel<GELU, TM, TN, U, false>;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(blocks < kDirectGrid ? blocks : kDirectGrid)),
                       dim3(64 * kDirectShares), 0, stream, A, W, bias, C, N, K, seg_offsets, seg_expert, n_seg, n_tiles_n, row_index,
                       row_div, out_index, max_rows, status);
    return hipGetLastError();
}

// 64 x 64 tiles once they fill two and a half rounds of the 256 compute units and the experts have rows for one and a half of them
// (a segment ends in half a tile on average).  One GEMM, us, 32 x 32 tiles / what 64 x 64 change: second GEMM of DiT-MoE-S, 330 tiles
// + 5, 612: - 4, 798: - 42, 1584: - 126; 2048 x 8192, 4 experts, 576 tiles + 10; first GEMM of DiT-MoE-S, 94 rows an expert + 5,
// 125 rows, 940 tiles - 3, 375 rows - 21; 512 x 2048, 64 experts, 31 rows an expert, 2048 tiles + 10, 128 rows - 69.
template <bool GELU>
static hipError_t launch_gemm_f32(const void* A, const void* W, const float* bias, void* C, int N, int K,
                                  const int32_t* seg_offsets, const int32_t* seg_expert, int n_seg, int max_rows,
                                  hipStream_t stream, const int32_t* row_index = nullptr, int row_div = 1,
                                  const int32_t* out_index = nullptr, int32_t* status = nullptr)
{
    const float *a = static_cast<const float*>(A), *w = static_cast<const float*>(W);
    float* c = static_cast<float*>(C);
    const long long tiles = (max_rows / 64 + n_seg / 2ll) * ((N + 63) / 64);
    if (tiles >= 640 && max_rows >= 96ll * n_seg)
        return launch_gemm_f32_tile<GELU, 4, 4, 1>(a, w, bias, c, N, K, seg_offsets, seg_expert, n_seg, max_rows, stream, row_index, row_div, out_index, status);
    return launch_gemm_f32_tile<GELU, 2, 2, 3>(a, w, bias, c, N, K, seg_offsets, seg_expert, n_seg, max_rows, stream, row_index, row_div, out_index, status);
}

}  // namespace dicemoe
