"""Wait counts of the persistent GEMM (csrc/ffn_ring.hpp, compiled here as plain C++): every ring it uses is sound on the stage loads alone, and
the model that says so at compile time sees a count that is one too large.  Needs no GPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

import pytest

from plan_util import CSRC

SHIM = """#include "ffn_ring.hpp"
extern "C" int pending(int ast, int wst, int qa, int qb) { const int d = ast > wst ? ast : wst; return dicemoe::ring_pending(ast, wst, qa, qb, 8 * d, 4 * d); }
extern "C" int first_pending(int qa, int part) { return dicemoe::ring_first_pending(qa, part); }
extern "C" int holds(int ast, int wst, int qa, int qb, int part, int first, int pending, int stores) {
    return dicemoe::ring_waits_hold(ast, wst, qa, qb, part, first, pending, stores) ? 1 : 0;
}
"""

RINGS = [
    # (TM, TN, SPREAD, AST, WST, WGM, WGN): whole tiles of 192 and 256 columns, halves and quarters of either
    (2, 3, 2, 2, 4, 4, 2), (2, 4, 2, 2, 3, 4, 2), (4, 2, 2, 2, 3, 2, 4), (1, 3, 2, 4, 4, 4, 2), (1, 4, 2, 3, 3, 4, 2), (1, 2, 2, 5, 5, 4, 2),
]


@functools.lru_cache(None)
def lib():
    with tempfile.TemporaryDirectory(prefix="ffn_ring_") as folder:
        src, out = os.path.join(folder, "ring.cpp"), os.path.join(folder, "ring.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", out], check=True)
        return ctypes.CDLL(out)


@pytest.mark.parametrize("ring", RINGS)
def test_stage_loads_alone_are_enough(ring):
    tm, tn, spread, ast, wst, wgm, wgn = ring
    waves = wgm * wgn
    qa, qb = 32 * tm * wgm // (8 * waves), 32 * tn * wgn // (8 * waves)
    part, stores = -(-(qa + qb) // spread), 2 * tm * tn
    pending, first = lib().pending(ast, wst, qa, qb), lib().first_pending(qa, part)
    for f in (0, first):
        for s in (0, stores):
            assert lib().holds(ast, wst, qa, qb, part, f, pending, s)
    # one load more in flight and a stage is read too early (deep rings: the whole first stage of the activations)
    assert not lib().holds(ast, wst, qa, qb, part, first + 1 if ast == 2 else (ast - 1) * qa + first, pending, 0)
    assert not lib().holds(ast, wst, qa, qb, part, 0, pending + 1, 0)
