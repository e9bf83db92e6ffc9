"""The tile rule of the expert FFN (csrc/ffn_plan.hpp, compiled here as plain C++) and, in Python, what the persistent kernel makes of
a segment table: the pieces that its leftover tiles are cut into.  Needs no GPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_16786_amd", "csrc")

# in the order of the enumeration FfnTile; "/2", "/3" behind a name: that many shares of K
TILES = ["stream192", "stream256", "64x128", "128x128", "128x192deep", "128x192", "256x192w4", "256x192w3", "256x192", "staged"]
SHIM = """#include "ffn_plan.hpp"
extern "C" void plan(int gelu, int N, int K, int rows, int n_seg, int n_experts, int sums, int* out) {
    const dicemoe::FfnPlan p = dicemoe::plan_ffn_gemm(gelu != 0, N, K, rows, n_seg, n_experts, gelu ? 0 : dicemoe::kSplitKBytes, sums != 0);
    out[0] = static_cast<int>(p.tile);
    out[1] = p.shares;
}
extern "C" int columns(int planned, int N, int K, int gelu, int rows, int n_seg, int bands) {
    return dicemoe::stream_looks(planned, N, K, gelu != 0, rows, n_seg) ? dicemoe::stream_columns(planned, dicemoe::stream_cost_192(N, K, gelu != 0), dicemoe::stream_cost_256(N, K, gelu != 0), bands) : planned;
}
extern "C" int f32_tile(int N, int K, int rows, int n_seg) { return static_cast<int>(dicemoe::f32_tile(N, K, rows, n_seg)); }
extern "C" int sorts_pairs(int bf16, int n_pairs, int n_seg, int n_experts, int rows, int d, int F) {
    return dicemoe::ffn_sorts_pairs(bf16 != 0, n_pairs, n_seg, n_experts, rows, d, F) ? 1 : 0;
}
extern "C" int pieces(int bn, int left, int slots) { return dicemoe::leftover_pieces(bn, left, slots); }
"""


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory(prefix="ffn_plan_") as folder:
        src, out = os.path.join(folder, "plan.cpp"), os.path.join(folder, "plan.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", out], check=True)
        return ctypes.CDLL(out)


def plan(gelu, N, K, rows, n_seg, n_experts=None, sums=False):
    """sums: inside the layer call, whose combine adds the shares of a split reduction"""
    out = (ctypes.c_int * 2)()
    _lib().plan(int(gelu), N, K, rows, n_seg, n_seg if n_experts is None else n_experts, int(sums), out)
    return TILES[out[0]] + (f"/{out[1]}" if out[1] > 1 else "")


def ffn_plans(rows, n_seg, d, F, n_experts=None):
    """Tiles of the first and of the second GEMM (n_experts: as many as segments unless given)."""
    return plan(True, F, d, rows, n_seg, n_experts), plan(False, d, F, rows, n_seg, n_experts)


# in the order of the enumeration F32Tile
F32_TILES = ["ring32", "ring64", "direct32", "direct64"]


def f32_plans(rows, n_seg, d, F):
    """Kernel and tile of the first and of the second float GEMM."""
    return F32_TILES[_lib().f32_tile(F, d, rows, n_seg)], F32_TILES[_lib().f32_tile(d, F, rows, n_seg)]


def sorts_pairs(dtype, T, slots, experts, d, F, rows=None):
    """Does the first GEMM of a layer call (gather fused, elementwise policy or none) sort the pairs itself?  rows: refreshed pairs (default: all)."""
    return bool(_lib().sorts_pairs(int(dtype == "bf16"), T * slots, experts, experts, T * slots if rows is None else rows, d, F))


def stream_tiles(seg_rows, seg_expert, N, bn):
    """Per XCD the (rows, columns) of its 256 x bn tiles in the order the persistent kernel takes them: its own experts' tiles up to
    the cap, then its share of what is beyond the cap elsewhere."""
    own = [[] for _ in range(8)]
    n_cols = -(-N // bn)
    for rows, expert in zip(seg_rows, seg_expert):
        row_tiles = -(-rows // 256)
        for band in range(0, row_tiles, 8):
            for col in range(n_cols):
                for t in range(band, min(band + 8, row_tiles)):
                    own[expert % 8].append((min(256, rows - 256 * t), min(bn, N - bn * col)))
    cap = -(-sum(map(len, own)) // 8)
    spilled = [t for o in own for t in o[cap:]]
    lists = []
    for o in own:
        spare = max(0, cap - len(o))
        lists.append(o[:cap] + spilled[:spare])
        spilled = spilled[spare:]
    assert not spilled
    return lists


def stream_items(seg_rows, seg_expert, N, bn):
    """What the persistent kernel runs: "whole" rounds of whole tiles, "leftover" tiles run whole, "halves" / "quarters" of them, "rowless" /
    "columnless" if some of these pieces have nothing to do, "many" for more than 64 whole tiles per workgroup."""
    kinds, slots = set(), 32
    for tiles in stream_tiles(seg_rows, seg_expert, N, bn):
        rounds, left = divmod(len(tiles), slots)
        pieces = _lib().pieces(bn, left, slots)
        if rounds:
            kinds.add("whole")
        if rounds > 64:
            kinds.add("many")
        if left and pieces == 1:
            kinds.add("leftover")
        if left and pieces > 1:
            kinds.add("halves" if pieces == 2 else "quarters")
            rest = tiles[rounds * slots:]
            if any(rows <= 128 for rows, _ in rest):
                kinds.add("rowless")
            if pieces == 4 and any(cols <= bn // 2 for _, cols in rest):
                kinds.add("columnless")
    return kinds


def describe(seg_rows, seg_expert, d, F):
    """Tile of either GEMM, and for the persistent kernel what it runs, as one line each."""
    lines = []
    bands = sum(-(-n // 256) for n in seg_rows)
    for tile, N, K, gelu in zip(ffn_plans(sum(seg_rows), len(seg_rows), d, F), (F, d), (d, F), (1, 0)):
        if tile.startswith("stream"):                    # the kernel takes the other width if the table says so
            tile = f"stream{_lib().columns(int(tile[6:]), N, K, gelu, sum(seg_rows), len(seg_rows), bands)}"
        items = stream_items(seg_rows, seg_expert, N, int(tile[6:])) if tile.startswith("stream") else ()
        lines.append(" ".join([tile] + sorted(items)))
    return tuple(lines)
