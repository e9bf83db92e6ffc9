// Which kernel and tile one bf16 grouped GEMM of the expert FFN runs on: the rule on sizes, in plain C++, so that it can be
// evaluated without a GPU.
#pragma once
#include <cstddef>

namespace dicemoe {

constexpr int kComputeUnits = 256;
constexpr int kStreamGrid = kComputeUnits, kStreamSlots = kStreamGrid / 8;      // persistent workgroups, and workgroups per XCD

enum class FfnTile {
    Stream192,      // persistent kernel, 256 rows x 192 columns
    Stream256,      // persistent kernel, 256 x 256
    Small64,        // a workgroup per tile from here on: 64 x 128, three stages, two workgroups per compute unit
    Small128,       // 128 x 128, three stages
    Mid192Deep,     // 128 x 192, three stages, one workgroup per compute unit
    Mid192,         // 128 x 192, two stages, two workgroups per compute unit
    Wide192W4,      // 256 x 192, eight wavefronts, two stages of activations and four of weights
    Wide192W3,      // the same with three stages of weights
    Wide192,        // 256 x 192, four wavefronts, two stages
    Staged128,      // 128 x 128 through registers, three workgroups per compute unit
};

// bytes of float partial sums that the split reduction of the second GEMM may use (beyond `hidden`)
// (at most about 270 workgroups of 128 x 192 float tiles)
constexpr size_t kSplitKBytes = static_cast<size_t>(288) * 128 * 192 * sizeof(float);

// shares > 1: that many workgroups per tile, each on a share of K, and a second pass that adds their float sums
struct FfnPlan { FfnTile tile; int shares; };

// Pieces that each of `left` leftover tiles of an XCD is cut into by the persistent kernel.
constexpr int leftover_pieces(int bn, int left, int slots)
{
    return left == 0 ? 1 : (bn == 256 && 4 * left <= slots ? 4 : (2 * left <= slots ? 2 : 1));
}

// Expected time (us) of one grouped GEMM on 256 x bn tiles.  The segment sizes live on the device; a segment ends in half a
// row tile on average, and the count is averaged over the row tiles around that.  Measured on the DiT-MoE-XL, DiT-MoE-G
// and expert-parallel widths: 1.06 (192 columns) and 1.42 us (256) per 64-deep step with all compute units busy,
// 0.68 / 0.8 for a round of halves and 0.6 for quarters, epilogues 4.3 / 5.5 us with GELU and 2.6 / 4.2 without.
inline float stream_cost(int bn, int N, int K, bool gelu, int rows, int n_seg)
{
    const float step[5] = {0.f, bn == 192 ? 1.06f : 1.42f, bn == 192 ? 0.68f : 0.8f, 0.f, 0.6f};      // by pieces
    const float epilogue = gelu ? (bn == 192 ? 4.3f : 5.5f) : (bn == 192 ? 2.6f : 4.2f);
    const int nk = K / 64, cols = (N + bn - 1) / bn;
    float sum = 0.f;
    for (int d = -2; d <= 2; ++d) {
        int bands = (rows + 255) / 256 + n_seg / 2 + d;
        bands = bands < 1 ? 1 : bands;
        const int per_xcd = (bands * cols + 7) / 8;
        const int rounds = per_xcd / kStreamSlots, left = per_xcd % kStreamSlots;
        const int pieces = leftover_pieces(bn, left, kStreamSlots);
        sum += rounds * (nk * step[1] + epilogue);
        if (left > 0) sum += nk * step[pieces] + epilogue + (pieces > 1 ? 3.f : 0.f);      // (a piece fills its rings anew)
    }
    return sum * 0.2f;
}

// Tile shape for one bf16 grouped GEMM.  With at most 64 segments and enough tiles the persistent kernel of
// ffn_stream.hpp, 192 or 256 columns, whichever its cost model expects to be faster.  The line for the first GEMM: 96 tiles
// of 256 x 192 and 128 rows per expert.  For the second, more tiles of 256 x 192 than compute units: with one tile per
// workgroup there is nothing to run on into, and the wide kernel starts sooner (kernel trace, DiT-MoE-XL widths: 8192 rows,
// 240 tiles, 90 us against 94 - 98; 4096 rows, 120 tiles, 61 against 66; 16384 rows with two shared experts, 384
// tiles, 160 against 145 on the persistent kernel).
// Otherwise the wide kernel, a workgroup per tile, hand-scheduled wavefronts:
//   256 x 192, one workgroup of eight wavefronts (4 x 2, each a 64 x 96 block; two per SIMD cover each
//     other's waits, +1 % over four wavefronts of 128 x 96) per compute unit, two stages of activations
//     and four of weights (all 160 KB of LDS; three with short reductions): the GEMM with the plain
//     epilogue, when that grid covers most of the 256 compute units.
//     The weights stream from HBM exactly once, and a barrier waits for the slowest of a step's loads:
//     every weight stage more gives those loads another step of flight (DiT-MoE-XL shape, GEMM2, same
//     box: 98 us with two weight stages, 86 - 91 with three, 82 - 86 with four);
//   128 x 192, two stages (80 KB of LDS), two workgroups per compute unit: the GEMM whose epilogue
//     evaluates GELU (one workgroup's MFMAs cover the other's epilogue arithmetic), and GEMMs between
//     one and two 256-wide rounds;
//   128 x 192, three stages, one workgroup per compute unit: grids of a quarter to one workgroup per
//     compute unit (few refreshed rows, or narrow outputs).  Alone on a compute unit a workgroup has nobody to hide its load
//     latency, and the third stage gives every load two steps of flight instead of one
//     (57 us instead of 78 us for GEMM2 at 4096 rows of the DiT-MoE-XL widths).
// Tiny problems stay on the 128 x 128 kernel, three workgroups per compute unit.
//
// Segments: up to 64, the tiles are dealt to the XCDs by expert (one L2 per XCD: an expert's weight slabs are then fetched by one
// XCD); beyond, in bands of row tiles.
inline FfnPlan plan_ffn_gemm(bool gelu, int N, int K, int max_rows, int n_seg, size_t partial_bytes)
{
    const bool by_expert = n_seg <= 64;
    // expected tiles: every segment ends in a partial row tile, half a tile on average
    auto tiles = [&](int bm, int bn) {
        const long long m_tiles = (static_cast<long long>(max_rows) + static_cast<long long>(n_seg) * bm / 2 + bm - 1) / bm;
        return m_tiles * ((N + bn - 1) / bn);
    };
    const bool fits_192 = (N + 191) / 192 * 192 * 8 <= N * 9;          // at most 1/8 of the columns computed in vain
    const bool fits_128 = (N + 127) / 128 * 128 * 8 <= N * 9;
    const bool full_rows = max_rows >= 128 * n_seg;                    // (row tiles half full on average)
    if (by_expert && K >= 384 && (fits_192 || N % 256 == 0) && full_rows && tiles(256, 192) >= (gelu ? 96 : kComputeUnits + 1)) {
        const bool wide = !fits_192 || stream_cost(256, N, K, gelu, max_rows, n_seg) < stream_cost(192, N, K, gelu, max_rows, n_seg);
        return {wide ? FfnTile::Stream256 : FfnTile::Stream192, 1};
    }
    const long long t64 = tiles(64, 128), t128 = tiles(128, 128), t192 = tiles(128, 192);
    // Few rows and a long reduction (the second GEMM after a small refresh fraction or for a small batch):
    // the 128 x 192 tiles do not fill the chip and each walks all of K.  With two or three workgroups per
    // tile, each on a share of K (float partial sums in the workspace, added by a second pass in a fixed
    // order), more compute units stream the weights at once: 54 -> 47 us at 2048 rows of the DiT-MoE-XL
    // widths.  Not worth it once the tiles fill the chip by themselves (57 vs 66 us at 4096 rows), nor when a
    // share is left with fewer than sixteen steps (DiT-MoE-S widths, K = 1536, 4096 rows: 32 us split in
    // three, 23 in two, 20 unsplit on three-stage tiles): the second pass then costs more than the split saves.
    int shares = 1;                      // the deepest split whose shares still fill the chip at most once
    if (!gelu && by_expert && fits_192)
        for (int s = 3; s >= 2 && shares == 1; --s)
            if (t192 * s * 20 <= kComputeUnits * 21 && K / 64 / s >= 16 &&
                static_cast<size_t>(s) * max_rows * N * sizeof(float) <= partial_bytes)
                shares = s;
    // Few rows per expert, or few tiles altogether: 64 x 128 tiles, three stages in 72 KB of LDS, so that two workgroups share
    // a compute unit and cover each other's waits, and a 64-row tile of a small expert is not half padding.
    // First GEMM (us, 128-row tiles / 64-row tiles): up to 72 rows per expert, above that a second row tile
    // reads the weights again (DiT-MoE-XL, 75 rows an expert 26 / 29.5, 88: 25.5 / 30): DiT-MoE-S, 38: 15 / 12, 69: 16 / 14;
    // DiT-MoE-G, 16: 116 / 90, 64: 122 / 105; and up to 96 rows where the 128 x 192 tiles would take more than one round: DiT-MoE-G, 88:
    // 121 / 116, 112: 123 / 129; expert-parallel widths, 88: 170 / 145.
    // Second GEMM: while there is at most one tile per compute unit (128 x 192 tiles, K in two or three shares / 64-row tiles: DiT-MoE-XL,
    // 900 rows 48 / 29.5, 1400 rows 42 / 34; DiT-MoE-S, 2000 rows 27 / 16; DiT-MoE-G, 256 rows 109 / 84); then 128 x 128 tiles
    // up to seven eighths of that (a count beyond 256 is a second round: DiT-MoE-G, 1024 rows, 224 tiles 110 / 99; 1200 rows, 252 tiles
    // 110 / 138), unless two shares of K on 128 x 192 tiles fill the chip (DiT-MoE-XL, 2000 rows: 45 split, 49 on 128 x 128).
    if (by_expert && fits_128 && K >= 256) {
        // (not for a long reduction that 128 x 192 tiles do in one round: those have 120 KB of loads in flight per compute unit, which
        // cold weights need: whole layer, DiT-MoE-XL widths, 256 tokens, other weights in every pass, 72.6 us against 74.1)
        const bool one_round = t192 <= kComputeUnits && K >= 1024;
        const bool small_experts = (max_rows <= 72 * n_seg && !one_round) || (max_rows <= 96 * n_seg && t192 > kComputeUnits);
        if (gelu && (small_experts || (full_rows && t64 <= 2 * kComputeUnits))) return {FfnTile::Small64, 1};
        // (the same for the second GEMM in three shares of K on one 128-row tile per expert)
        const bool three_shares = shares == 3 && max_rows <= 100 * n_seg;
        if (!gelu && !three_shares && t64 <= kComputeUnits) return {FfnTile::Small64, 1};
        if (!gelu && shares == 1 && 8 * t128 <= 7 * kComputeUnits) return {FfnTile::Small128, 1};
    }
    if (shares > 1) return {FfnTile::Mid192Deep, shares};
    if (!gelu && fits_192 && tiles(256, 192) * 10 >= kComputeUnits * 6) {
        if (K >= 320) return {FfnTile::Wide192W4, 1};      // (four weight stages: three steps of flight for the cold weight stream)
        return {K >= 256 ? FfnTile::Wide192W3 : FfnTile::Wide192, 1};
    }
    if (fits_192 && K >= 256 && t192 <= kComputeUnits && t192 * 4 >= kComputeUnits) return {FfnTile::Mid192Deep, 1};
    if (fits_192 && t192 * 2 >= kComputeUnits) return {FfnTile::Mid192, 1};
    return {FfnTile::Staged128, 1};
}

}  // namespace dicemoe
