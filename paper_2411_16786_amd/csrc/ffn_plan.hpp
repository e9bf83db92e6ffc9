// Which kernel and tile one grouped GEMM of the expert FFN runs on: the rules on sizes, in plain C++, so that they can be
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
    Mid192Deep,     // 128 x 192, three stages, one workgroup per compute unit (with GELU eight wavefronts, without four)
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

// One round of workgroups per XCD?  By the times below an XCD's workgroups, those that find no tile among them, go to four groups of eight
// compute units in turn: of the `tiles` first workgroups of every `slots` that a share of the grid gives to an XCD, no group may get more
// than eight.  (128 x 128 tiles in three shares, K = 3072, both GEMMs: 27 workgroups an XCD in three times 12 slots, nine of them in one group,
// 49.8 us where 24 take 39.6; in three times 14 slots, eight at most, 41.4; 30 in three times 15 slots, eight at most, 40.0, in three times 16 52.6.)
constexpr bool one_round_of_shares(int tiles, int shares, int slots)
{
    for (int group = 0; group < 4; ++group) {
        int here = 0;
        for (int s = 0; s < shares; ++s)
            for (int i = 0; i < tiles; ++i) here += (s * slots + i) % 4 == group ? 1 : 0;
        if (here > kStreamSlots / 4) return false;
    }
    return true;
}

// Pieces that each of `left` leftover tiles of an XCD is cut into by the persistent kernel.
constexpr int leftover_pieces(int bn, int left, int slots)
{
    return left == 0 ? 1 : (bn == 256 && 4 * left <= slots ? 4 : (2 * left <= slots ? 2 : 1));
}

// Expected time (us) of one grouped GEMM of the persistent kernel on 256 x bn tiles: what a round of whole tiles, of halves and of quarters costs.
// Measured on the DiT-MoE-XL, DiT-MoE-G and expert-parallel widths: 1.06 (192 columns) and 1.42 us (256) per 64-deep step with all
// compute units busy, 0.68 / 0.8 for a round of halves and 0.6 for quarters, epilogues 4.3 / 5.5 us with GELU and 2.6 / 4.2 without.
struct StreamCost { int bn, cols; float whole, halves, quarters; };

constexpr StreamCost stream_cost_of(int bn, int N, int K, bool gelu, float step_192 = 1.06f)
{
    const int nk = K / 64;
    const float epilogue = gelu ? (bn == 192 ? 4.3f : 5.5f) : (bn == 192 ? 2.6f : 4.2f);
    return {bn, (N + bn - 1) / bn, nk * (bn == 192 ? step_192 : 1.42f) + epilogue,
            nk * (bn == 192 ? 0.68f : 0.8f) + epilogue + 3.f, nk * 0.6f + epilogue + 3.f};      // (a piece fills its rings anew)
}

// ... and of `bands` row tiles
constexpr float stream_cost_of_bands(const StreamCost& c, int bands)
{
    const int per_xcd = (bands * c.cols + 7) / 8;
    const int rounds = per_xcd / kStreamSlots, left = per_xcd % kStreamSlots;
    const int pieces = leftover_pieces(c.bn, left, kStreamSlots);
    return rounds * c.whole + (left == 0 ? 0.f : pieces == 1 ? c.whole : pieces == 2 ? c.halves : c.quarters);
}

// The same where the segment sizes are not known (they live on the device): a segment ends in half a row tile on average, and the
// cost is averaged over the row tiles around that.
inline float stream_cost(int bn, int N, int K, bool gelu, int rows, int n_seg)
{
    const StreamCost c = stream_cost_of(bn, N, K, gelu);
    float sum = 0.f;
    for (int d = -2; d <= 2; ++d) {
        const int bands = (rows + 255) / 256 + n_seg / 2 + d;
        sum += stream_cost_of_bands(c, bands < 1 ? 1 : bands);
    }
    return sum * 0.2f;
}

// at most 1/8 of the columns computed in vain by tiles of 192
constexpr bool stream_fits_192(int N) { return (N + 191) / 192 * 192 * 8 <= N * 9; }

// Columns of the persistent kernel's tiles once the segment table is known: those that the host planned on its estimate of the row tiles,
// unless the other width is expected to be faster by more than the model is off (8 us) on the real ones.  Weights from memory make a step of
// 192 columns 1.11 us where the host's 1.06 were measured warm.  Whole layer, us, with the planned width / with this rule: second GEMM of
// DiT-MoE-G, 4096 tokens, 504 / 483 (192 -> 256); first of DiT-MoE-XL, 3000 tokens, 174 / 167 (192 -> 256), 5000 tokens 243 / 230; expert-parallel widths,
// 4000 tokens, 592 / 568 (192 -> 256); DiT-MoE-XL with two shared experts, 4096 tokens, 298 / 291 to 296.
constexpr int stream_columns(int planned, const StreamCost& c192, const StreamCost& c256, int bands)
{
    const float t192 = stream_cost_of_bands(c192, bands), t256 = stream_cost_of_bands(c256, bands);
    if (planned == 192) return t192 - t256 > 8.f ? 256 : 192;
    return t256 - t192 > 8.f ? 192 : 256;
}
constexpr StreamCost stream_cost_192(int N, int K, bool gelu) { return stream_cost_of(192, N, K, gelu, 1.11f); }
constexpr StreamCost stream_cost_256(int N, int K, bool gelu) { return stream_cost_of(256, N, K, gelu); }

// Can the table say so?  A kernel that holds both widths costs 0.5 - 1 us (DiT-MoE-S, 2048 tokens x 12 layers 584 / 587 us, DiT-MoE-XL, 4096 tokens
// 198.2 / 199.0): it runs only where the row tiles that these rows can come to, all in one segment or an empty tile in each, allow
// either answer and the estimate is not far from where it changes.
inline bool stream_looks(int planned, int N, int K, bool gelu, int rows, int n_seg)
{
    if (!stream_fits_192(N)) return false;
    const StreamCost c192 = stream_cost_192(N, K, gelu), c256 = stream_cost_256(N, K, gelu);
    const int least = (rows + 255) / 256, expected = least + n_seg / 2;
    for (int bands = expected - 3; bands <= expected + 3; ++bands)
        if (bands >= least && bands <= least + n_seg && stream_columns(planned, c192, c256, bands) != planned) return true;
    return false;
}

// Tile shape for one bf16 grouped GEMM.  With at most 64 segments and enough tiles the persistent kernel of
// ffn_stream.hpp, 192 or 256 columns, whichever its cost model expects to be faster.  The line for the first GEMM: 96 tiles
// of 256 x 192 and 128 rows per expert.  For the second, more tiles of 256 x 192 than compute units: with one tile per
// workgroup there is nothing to run on into, and the wide kernel starts sooner (kernel trace, DiT-MoE-XL widths: 8192 rows,
// 216 tiles, 90 us against 94 - 98; 4096 rows, 120 tiles, 61 against 66; 12288 rows with two shared experts, 318
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
// and below that the small tiles as said beside their lines.  What fits none of them stays on the register-staged 128 x 128 kernel,
// three workgroups per compute unit.
//
// Segments: up to 64, the tiles are dealt to the XCDs by expert (one L2 per XCD: an expert's weight slabs are then fetched by one
// XCD); beyond, in bands of row tiles.  n_experts: distinct weights at most.
//
// The lines between the tiles up to 128 rows were drawn from 2641 combinations of nine widths, 2 to 64 experts, 1 to 8 segments per
// expert and 8 to 2048 rows per segment (graphs of calls with weights from memory, every tile that can run timed for either GEMM);
// figures beside them are us, or % of the FFN.
// sums: the caller's combine adds the shares of a split reduction (no second pass)
inline FfnPlan plan_ffn_gemm(bool gelu, int N, int K, int max_rows, int n_seg, int n_experts, size_t partial_bytes, bool sums = false)
{
    const bool by_expert = n_seg <= 64;
    const long long rows = max_rows, segs = n_seg;
    // expected tiles: every segment ends in a partial row tile, half a tile on average ...
    auto row_tiles = [&](int bm) { return (rows + segs * bm / 2 + bm - 1) / bm; };
    auto tiles = [&](int bm, int bn) { return row_tiles(bm) * ((N + bn - 1) / bn); };
    // ... and, however few its rows, has one
    auto all_tiles = [&](int bm, int bn) { return (row_tiles(bm) > segs ? row_tiles(bm) : segs) * ((N + bn - 1) / bn); };
    const bool fits_192 = stream_fits_192(N);
    const bool fits_128 = (N + 127) / 128 * 128 * 8 <= N * 9;
    const bool full_rows = rows >= 128 * segs;                         // (row tiles half full on average)
    if (by_expert && K >= 384 && (fits_192 || N % 256 == 0) && full_rows && tiles(256, 192) >= (gelu ? 96 : kComputeUnits + 1)) {
        const bool wide = !fits_192 || stream_cost(256, N, K, gelu, max_rows, n_seg) < stream_cost(192, N, K, gelu, max_rows, n_seg);
        return {wide ? FfnTile::Stream256 : FfnTile::Stream192, 1};
    }
    const long long t192 = tiles(128, 192);
    if (gelu && by_expert && fits_128 && K >= 256) {
        // Few rows per expert: 64 x 128 tiles, three stages in 72 KB of LDS, so that two workgroups share a compute unit and cover each
        // other's waits, and a 64-row tile of a small expert is not half padding (128-row tiles / 64-row tiles: DiT-MoE-S, 38 rows an
        // expert 15 / 12, 69: 16 / 14).  In one round of two per compute unit (a little more by the estimate: 384 x 1536, 32 experts, 528
        // tiles - 12 %, 576 tiles + 11 %), but not for a long reduction that 128 x 192 tiles do in one round: those have 120 KB of loads
        // in flight per compute unit, which cold weights need (DiT-MoE-XL, 256 tokens, whole layer 72.6 against 74.1).
        const long long t64 = all_tiles(64, 128);
        const bool one_round = t192 <= kComputeUnits && K >= 1024;
        if (t64 <= 560 && rows <= 72 * segs && !one_round) return {FfnTile::Small64, 1};
        // With so few rows that every segment has one tile also in two rounds that they nearly fill (1024 tiles: 512 x 2048, 64 experts - 8 %,
        // 1024 x 4096, 32 segments - 5 %; 768 tiles: 384 x 1536, 64 experts + 6 %; in four and more, 1152 x 4608, 8 experts in 64 segments + 5 %).
        if (t64 <= 1024 && 8 * t64 >= 7 * 1024 && rows <= 24 * segs && !one_round) return {FfnTile::Small64, 1};
        // In several rounds where the weights are what the time goes to: 128 MB of them, at most K / 16 rows for each expert's, and few
        // tiles altogether (DiT-MoE-G, 64 rows an expert: - 7 %, 96: - 1 %, 128: + 7 %; 1024 x 4096, 32 experts, 48: - 10 %, 96: 0; four
        // experts of 1152 x 4608 in 16 or 32 segments + 2 to + 15 % at any number of rows).
        const long long weights = (n_experts < n_seg ? n_experts : n_seg) * static_cast<long long>(K);      // x N
        if (weights * N >= (1 << 26) && 16 * rows <= weights && rows * N <= 12 * (1 << 20) && rows <= 96 * segs && t64 >= 640 &&
            t192 > kComputeUnits)
            return {FfnTile::Small64, 1};
        if (full_rows && tiles(64, 128) <= 2 * kComputeUnits) return {FfnTile::Small64, 1};
    }
    // Few rows and a long reduction (the second GEMM after a small refresh fraction or for a small batch):
    // the 128 x 192 tiles do not fill the chip and each walks all of K.  With two or three workgroups per
    // tile, each on a share of K (float partial sums in the workspace, added by a second pass in a fixed
    // order), more compute units stream the weights at once: 54 -> 47 us at 2048 rows of the DiT-MoE-XL
    // widths.  Not worth it once the tiles fill the chip by themselves (57 vs 66 us at 4096 rows), nor when a
    // share is left with fewer than sixteen steps (DiT-MoE-S widths, K = 1536, 4096 rows: 32 us split in
    // three, 23 in two, 20 unsplit on three-stage tiles): the second pass then costs more than the split saves.
    // Three shares of experts with more than 100 rows: only if they run in one round even when every segment ends in an empty tile
    // and the second pass has little to add (two experts of 2048 x 8192, 500 rows, 64 x 128 / three shares 101 / 85; of 1152 x 4608,
    // 968 rows 57 / 53, 1219 rows 64 / 73; DiT-MoE-XL, 900 rows 29.5 / 48).
    // Where the combine adds the shares, a share more costs its part of that traffic and no launch.  Long reductions (the weights are what the
    // time goes to): 128 x 128 tiles in as many shares, of sixteen steps at least, as one round has room for, with a row tile to spare
    // once segments are likely to need a second one (whole layer, 128 x 192 in three shares / so: DiT-MoE-XL, 48 tokens 57.2 / 53.7 us, 138:
    // 63.4 / 59.9; 500 tokens, in two, 85.5 / 81.9, 700 rows 77.0 / 73.8, 575 rows 75.6 / 76.2; where it would be a second round, 267 rows of nine
    // experts, 11 tiles an XCD, 68.2 / 76.4 in three; 1280 x 5120, 8 experts, 48 to 384 rows, 10 tiles an XCD, 55 - 68 / 65 - 79).  Short ones:
    // 64 x 128 tiles in three shares while these fill three quarters of the chip at most (DiT-MoE-S, 60 tokens 30.9 / 27.9, 170: 31.0 / 28.2, 400:
    // 32.4 / 30.5; 800 tokens top-3, 150 tiles, 36.5 / 38.4; four shares of six steps 1 us behind three).
    if (sums && !gelu && by_expert && fits_128) {
        auto room = [&](int s) { return static_cast<size_t>(s) * max_rows * N * sizeof(float) <= partial_bytes; };
        const int steps = K / 64;
        if (steps < 48) {
            if (steps >= 24 && rows <= 64 * segs && 4 * all_tiles(64, 128) <= kComputeUnits && room(3)) return {FfnTile::Small64, 3};
        } else {
            const int cols = (N + 127) / 128;
            const long long expected = all_tiles(128, 128), t = expected + (rows > 48 * segs ? cols : 0);
            const int bands = static_cast<int>(((rows + 127) / 128 + segs + 7) / 8);      // of eight row tiles, as the launcher's grid has them
            auto fits = [&](int s) {
                return steps / s >= 16 && (t + 7) / 8 * s <= kStreamSlots && room(s) &&
                       one_round_of_shares(static_cast<int>((expected + 7) / 8), s, bands * cols);
            };
            if (fits(3)) return {FfnTile::Small128, 3};
            if (rows > 80 * segs && fits(2)) return {FfnTile::Small128, 2};
        }
    }
    int shares = 1;
    if (!gelu && by_expert && fits_192) {
        auto can = [&](int s, long long t) {
            return t * s * 20 <= kComputeUnits * 21 && K / 64 / s >= 16 && static_cast<size_t>(s) * max_rows * N * sizeof(float) <= partial_bytes;
        };
        const long long worst = (rows + 128 * segs + 127) / 128 * ((N + 191) / 192);
        if (can(3, t192) && (rows <= 100 * segs || (can(3, worst) && rows * N <= 1150000))) shares = 3;
        else if (can(2, all_tiles(128, 192))) shares = 2;
    }
    if (!gelu && by_expert && fits_128 && K >= 256) {
        // 64 x 128 tiles while there is at most one per compute unit (128 x 192 tiles, K in two shares / 64-row tiles: DiT-MoE-XL, 1400
        // rows 42 / 34; DiT-MoE-S, 2000 rows 27 / 16; DiT-MoE-G, 256 rows 109 / 84); then 128 x 128 up to seven eighths of that (a count
        // beyond 256 is a second round: DiT-MoE-G, 1024 rows, 224 tiles 110 / 99; 1200 rows, 252 tiles 110 / 138), unless two shares of K
        // on 128 x 192 tiles fill the chip (DiT-MoE-XL, 2000 rows: 45 split, 49 on 128 x 128).
        // Counted with a tile for every segment, except where 128 x 192 tiles do not fit the columns (640 x 2560, 8 experts in 64 segments
        // of 12 rows, 320 tiles 79 us, register-staged 128 x 128 103) and, for the small ones, two of which share a compute unit, where
        // segments share weights (1152 x 4608, 4 experts in 32 segments, 288 tiles 101, 128 x 192 104; with 32 experts 159 and 144).
        const long long t64 = fits_192 && n_experts >= n_seg ? all_tiles(64, 128) : tiles(64, 128);
        if (shares != 3 && t64 <= kComputeUnits) return {FfnTile::Small64, 1};
        const long long t128 = fits_192 ? all_tiles(128, 128) : tiles(128, 128);
        if (shares == 1 && 8 * tiles(128, 128) <= 7 * kComputeUnits && t128 <= kComputeUnits) return {FfnTile::Small128, 1};
    }
    if (shares > 1) return {FfnTile::Mid192Deep, shares};
    // (many experts with few rows, one round of 128-row tiles: 1152 x 4608, 32 experts of 30 rows, 64 x 128 tiles 173, 256 x 192 160, these 146)
    if (!gelu && fits_192 && K >= 256 && rows <= 48 * segs && all_tiles(128, 192) <= kComputeUnits && t192 * 4 >= kComputeUnits)
        return {FfnTile::Mid192Deep, 1};
    if (!gelu && fits_192 && tiles(256, 192) * 10 >= kComputeUnits * 6) {
        if (K >= 320) return {FfnTile::Wide192W4, 1};      // (four weight stages: three steps of flight for the cold weight stream)
        return {K >= 256 ? FfnTile::Wide192W3 : FfnTile::Wide192, 1};
    }
    if (fits_192 && K >= 256 && t192 <= kComputeUnits && t192 * 4 >= kComputeUnits) return {FfnTile::Mid192Deep, 1};
    if (fits_192 && t192 * 2 >= kComputeUnits) return {FfnTile::Mid192, 1};
    return {FfnTile::Staged128, 1};
}

// ---- float storage: which kernel of ffn_f32.hpp, and its tile
enum class F32Tile { Ring32, Ring64, Direct32, Direct64 };
constexpr int kRingMinK = 256;

// 64 x 64 tiles on the ring kernel, one workgroup per compute unit, in place of 32 x 32?  They move half the bytes per flop, but the last round is
// as long as a full one, half a tile of rows at the end of a segment is twice as many, and short reductions spend their time elsewhere.
// One GEMM (weights from memory), what 64 x 64 change, in us of the whole FFN:
//   K from 1536 on: one round nearly full with 112 rows a segment (K = 1536, 234 tiles, 125 rows: - 6 of 95, 252: - 6 of 87; 2048, 208: - 8 of 97; 3072, 228:
//     - 12 of 154), or five sixths of the rounds' tiles (four fifths from K = 3072 on) with 128 rows (2048, 888 tiles: - 8 of 340; 4608, 432: - 19 of 359,
//     756: - 56 of 596; 8192, 416: - 27 of 573; but 1536, 276 tiles: + 20 of 89; 2048, 544: + 10 of 216; 3072, 312: + 20 of 181, 816: 0; and 2048, 64 experts of 38
//     rows, 560 tiles: + 15 of 186, with one hot expert + 22; 3072, 32 experts of 16 rows: + 6 to + 36 of 148);
//   K from 768 on: nine tenths of them, 700 tiles and 240 rows a segment (768, 1680 tiles, 250 rows: - 10 of 260, 1248 tiles, 181 rows: - 3 to + 12 of 181; 1024,
//     732 tiles: - 9 of 170, 868: 0; 1152, 2520 tiles, 250 rows: - 23 of 520, 1872 tiles, 181 rows: - 5 to + 1);
//   below, nowhere (256, 1056 tiles: + 7 of 70; 384, 1632: + 5 of 135; 512, 64 experts, 1024 tiles and more: + 2 to + 28).
inline bool ring_wide(int N, int K, int max_rows, int n_seg)
{
    const long long rows = max_rows, segs = n_seg;
    const long long tiles = (rows / 64 + segs / 2) * ((N + 63) / 64);
    const long long full = (tiles + kStreamGrid - 1) / kStreamGrid * kStreamGrid;      // tiles of so many full rounds
    if (K < 768) return false;
    if (K < 1536) return rows >= 240 * segs && tiles >= 700 && 10 * tiles >= 9 * full;
    if (tiles <= kStreamGrid) return tiles >= 200 && rows >= 112 * segs;
    return rows >= 128 * segs && (K >= 3072 ? 5 * tiles >= 4 * full : 6 * tiles >= 5 * full);
}

// The direct kernel takes other reductions and longer tables: 64 x 64 tiles once they fill two and a half rounds of the 256 compute units and the experts have rows for one and a half of them
// (a segment ends in half a tile on average).  One GEMM, us, 32 x 32 tiles / what 64 x 64 change: second GEMM of DiT-MoE-S, 330 tiles
// + 5, 612: - 4, 798: - 42, 1584: - 126; 2048 x 8192, 4 experts, 576 tiles + 10; first GEMM of DiT-MoE-S, 94 rows an expert + 5,
// 125 rows, 940 tiles - 3, 375 rows - 21; 512 x 2048, 64 experts, 31 rows an expert, 2048 tiles + 10, 128 rows - 69.
// Short reductions leave the ring at either end: two stages a share in a quarter of a round (K = 256, us of the FFN, direct 32 x 32 against the ring: 16
// to 56 tiles - 0.2 to - 0.5 of 12, 240: - 0.2 of 14, 400: + 1 of 17), and very many rows, where few loads of a tile are first ones (direct 64 x 64:
// K = 256, 2928 tiles - 9 of 170; 4896: - 17 of 277; 384, 4440: - 6 of 339; 512, 3552: - 8 of 340, 9856: - 35 of 919; 640, 7400: - 19 of 836; but 512, 32 experts of
// 362 rows, 6304 tiles + 10 of 585).
inline F32Tile f32_tile(int N, int K, int max_rows, int n_seg)
{
    const long long rows = max_rows, segs = n_seg;
    const long long tiles = (rows / 64 + segs / 2) * ((N + 63) / 64);
    if (n_seg <= 64 && K % 128 == 0 && K >= kRingMinK) {
        if (ring_wide(N, K, max_rows, n_seg)) return F32Tile::Ring64;
        if (K < 768 && tiles >= 3500 && rows >= 700 * segs) return F32Tile::Direct64;
        if (K < 384 && (rows / 32 + segs / 2) * ((N + 31) / 32) <= kComputeUnits) return F32Tile::Direct32;
        return F32Tile::Ring32;
    }
    return tiles >= 640 && rows >= 96 * segs ? F32Tile::Direct64 : F32Tile::Direct32;
}

// ---- the dispatch of a layer, left to the first GEMM (pair_sort.hpp)
// Pairs that a workgroup of it sorts for itself.  What it costs there is about what the loads of the segment table and of the row
// indices, one behind the other, cost otherwise; what it saves is a launch.
constexpr int kOwnSortPairs = 1024;
// ... and a workgroup of the persistent kernel, which ranks no more than it computes
constexpr int kStreamSortPairs = 4096;

// Where the first GEMM's workgroups run in about one round: each sorts once, while the loads it saves would have taken as long.  In several
// rounds the sort comes again with every workgroup (whole layers, us, dispatch / own sort: 64 x 256 float, 64 tokens 28.4 / 24.8; DiT-MoE-S, 60
// tokens 28.2 / 25.4, 500 tokens 33.9 / 32.1; DiT-MoE-XL, 138 tokens 61.2 / 59.4, 256 tokens 69.4 / 67.5; but DiT-MoE-G, 132 tokens with a shared expert,
// 952 tiles, 214.3 / 215.5; DiT-MoE-XL, 500 tokens, 720 tiles, 82.0 / 82.1).  The persistent kernel, dispatch / own sort: DiT-MoE-S, 1200 tokens
// 36.9 / 35.3, 2048 tokens 42.9 / 40.9; DiT-MoE-XL, 1000 tokens 93.2 / 92.6; with more tiles than compute units nothing or a loss (DiT-MoE-XL, 1500 tokens
// 122.1 / 122.9), and more than 4096 pairs take longer here than in a dispatch on many compute units (DiT-MoE-S, 8192 tokens 93 / 98).
inline bool ffn_sorts_pairs(bool bf16, int n_pairs, int n_seg, int n_experts, int max_rows, int d, int F)
{
    if (n_pairs < 1 || n_pairs > kStreamSortPairs || n_seg != n_experts || max_rows < 1) return false;
    auto tiles = [&](int bm, int bn) {
        const int row_tiles = max_rows / bm + n_seg / 2;
        return static_cast<long long>(row_tiles > n_seg ? row_tiles : n_seg) * ((F + bn - 1) / bn);
    };
    if (bf16) {
        const FfnTile tile = plan_ffn_gemm(true, F, d, max_rows, n_seg, n_experts, 0).tile;
        if (tile == FfnTile::Stream192) return tiles(256, 192) <= kComputeUnits;
        if (tile == FfnTile::Stream256) return tiles(256, 256) <= kComputeUnits;
        return n_pairs <= kOwnSortPairs && ((tile == FfnTile::Small64 && tiles(64, 128) <= 2 * kComputeUnits) || (tile == FfnTile::Mid192Deep && tiles(128, 192) <= kComputeUnits));
    }
    if (n_pairs > kOwnSortPairs) return false;
    const F32Tile tile = f32_tile(F, d, max_rows, n_seg);
    return tile == F32Tile::Ring32 || (tile == F32Tile::Direct32 && tiles(32, 32) <= 4 * kComputeUnits);
}

}  // namespace dicemoe
