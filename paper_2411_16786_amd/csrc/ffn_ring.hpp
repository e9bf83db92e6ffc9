// Wait counts of the persistent GEMM's stage rings (ffn_stream.hpp), in plain C++: they are compile-time constants that no test on a GPU can
// prove, so that a model of the issue order checks each set of them where it is used.
//
// Issue order of one wavefront (loads return in order): prologue W0 .. W(WST-1), A0 .. A(AST-1); refill of step j: A(j + AST), then W(j + WST),
// its first `part` loads behind the barrier of step j, the others (the carried ones) in step j + 1 ahead of that step's wait.  The last
// stage of either operand in the prologue leaves out the loads that step 0 issues as carried ones.
#pragma once

namespace dicemoe {

// Loads of one wavefront that may still be in flight at the barrier of step kt: those issued after the last load of stage kt + 1.
constexpr int ring_pending(int ast, int wst, int qa, int qb, int nk, int kt)
{
    int younger = 0;
    auto load = [&](bool is_next, int n) { if (is_next) younger = 0; else younger += n; };
    for (int s = 0; s < wst && s < nk; ++s) load(s == kt + 1, qb);
    for (int s = 0; s < ast && s < nk; ++s) load(s == kt + 1, qa);
    for (int j = 0; j < kt; ++j) {
        if (j + ast < nk) load(j + ast == kt + 1, qa);
        if (j + wst < nk) load(j + wst == kt + 1, qb);
    }
    return younger;
}

// ... and at the barrier before step 0, which reads stage 0: the activations' last stage, as far as the prologue asks for it.  It counts on
// stage loads alone: loads of row indices and biases that are younger still make the wait longer, and need not be there.
constexpr int ring_first_pending(int qa, int part) { return qa < part ? qa : part; }

// Has every stage landed at the barrier behind which it is read, with `first` loads left in flight ahead of step 0, `pending` at the barrier of a
// step, and `pending` + `stores` at that of an item's first step if the item before it issued that many stores (0: that wait does not
// count them)?  Only what is sure to be issued is counted: the stage loads, and the stores.
constexpr bool ring_waits_hold(int ast, int wst, int qa, int qb, int part, int first, int pending, int stores)
{
    constexpr int nk = 8, steps = 3 * nk, room = steps + 16;
    int a_last[room] = {}, w_last[room] = {}, a_count[room] = {}, w_count[room] = {};
    int seq = 0, landed = 0;
    auto load_a = [&](int s) { a_last[s] = ++seq; ++a_count[s]; };
    auto load_w = [&](int s) { w_last[s] = ++seq; ++w_count[s]; };
    auto wait = [&](int left) { if (seq - left > landed) landed = seq - left; };
    auto here = [&](int s) { return a_count[s] == qa && w_count[s] == qb && a_last[s] <= landed && w_last[s] <= landed; };
    auto refill = [&](int j, int from, int to) {
        for (int i = from; i < to; ++i) {
            if (i < qa) load_a(j + ast);
            else load_w(j + wst);
        }
    };
    for (int s = 0; s < wst; ++s)
        for (int i = 0; i < qb; ++i)
            if (s < wst - 1 || qa + i < part) load_w(s);
    for (int s = 0; s < ast; ++s)
        for (int i = 0; i < qa; ++i)
            if (s < ast - 1 || i < part) load_a(s);
    wait(first);
    if (!here(0)) return false;
    for (int g = 0; g < steps; ++g) {
        refill(g - 1, part, qa + qb);
        wait(pending + (g > 0 && g % nk == 0 ? stores : 0));
        if (!here(g + 1)) return false;
        refill(g, 0, part < qa + qb ? part : qa + qb);
        if (g % nk == nk - 1) seq += stores;
    }
    return true;
}

}  // namespace dicemoe
