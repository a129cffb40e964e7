// Replay plan of captured step graphs, shared by the single and batched
// forms; host logic free of HIP types (a host-only test compiles it with a
// plain C++ compiler).
//
// A graph of glen steps (graph_steps rounded up to even, so the buffer read
// at its start is always buffer 0) replays only from a time that is a
// multiple of glen; other steps are plain launches.  The fused diagnostics
// then run at exactly the steps t with (t + 1) % diag_every == 0, graph or
// not: either diag_every divides glen (one graph, diagnostics at those of its
// steps) or glen divides diag_every (a graph without diagnostics and one with
// them at its last step, chosen per replay).  Other pairs are refused.
#pragma once

#include <cstdint>

namespace mclbm {

struct GraphPlan {
    int glen = 0;  // 0: no graphs
    int diag_every = 0;
    bool two = false;
};

// Fills g; returns false when graph_steps and diag_every do not divide one
// another (after rounding graph_steps up to even).
inline bool graph_plan(int graph_steps, int diag_every, GraphPlan &g) {
    g = GraphPlan{};
    if (graph_steps <= 0) return true;
    g.glen = (graph_steps + 1) / 2 * 2;
    g.diag_every = diag_every > 0 ? diag_every : 0;
    if (g.diag_every > 0 && g.glen % g.diag_every != 0) {
        if (g.diag_every % g.glen != 0) return false;
        g.two = true;
    }
    return true;
}
inline int graph_variants(const GraphPlan &g) { return g.glen ? (g.two ? 2 : 1) : 0; }
// does step s (0-based) of graph variant v run the diagnostics?
inline bool graph_diag(const GraphPlan &g, int v, int s) {
    if (g.diag_every <= 0) return false;
    if (!g.two) return (s + 1) % g.diag_every == 0;
    return v == 1 && s == g.glen - 1;
}
// the variant that replays from time t (a multiple of glen)
inline int graph_variant(const GraphPlan &g, int64_t t) {
    return g.two && (t + g.glen) % g.diag_every == 0 ? 1 : 0;
}
// plain launch at time t: does it run the diagnostics?
inline bool plain_diag(int diag_every, int64_t t) { return diag_every > 0 && (t + 1) % diag_every == 0; }
// What a step loop launches at time t with n steps left: a graph variant
// (>= 0, glen steps) or -1 for one plain step.
inline int next_launch(const GraphPlan &g, int64_t t, int64_t n) {
    return g.glen > 0 && t % g.glen == 0 && n >= g.glen ? graph_variant(g, t) : -1;
}

// Plain steps from time t with n left that may be fused: those before the next
// diagnostic step and before the next time a graph replays from.
inline int64_t plain_stretch(const GraphPlan &g, int diag_every, int64_t t, int64_t n) {
    int64_t m = n;
    if (diag_every > 0) {
        const int64_t d = diag_every - 1 - t % diag_every;  // steps before the diagnostic one
        m = d < m ? d : m;
    }
    if (g.glen > 0) {
        const int64_t a = (g.glen - t % g.glen) % g.glen;  // steps to the next multiple of glen
        if (a > 0 && n - a >= g.glen && a < m) m = a;
    }
    return m;
}
// Pairs of steps fused out of a stretch of m.  Every launch swaps the buffers,
// and a pair advances the time by two: where the buffer read must follow the
// parity of the time (keep), pairs go in twos.
inline int64_t sweep_pairs(int64_t m, bool keep) { return keep ? m / 4 * 2 : m / 2; }

// Where a simulation stands.  keep: launches exist outside the step loop that
// read a fixed buffer (the graphs, which replay from buffer 0 at multiples of
// their length, and code that the caller has captured, steps or fields passes,
// from the buffer of that time).  From then on the buffer changes with the
// parity of the time only: any even number of steps, and a state set at a time
// of the same parity, leave the state where those launches look for it.
struct StepState {
    int64_t t = 0;
    int cur = 0;  // population buffer that holds the state at time t
    bool keep = false;
};
// The buffer that takes a state set at time step.
inline int buffer_for(const StepState &s, int64_t step) { return (int)((s.cur ^ s.t ^ step) & 1); }

// Advances by n steps: replay(v) runs graph variant v, pair(cur) two steps and
// single(cur, diag) one step from buffer cur into the other.  replay returns 0,
// or a code that ends the loop and is returned.
template <typename Replay, typename Pair, typename Single>
int run_steps(const GraphPlan &g, int diag_every, bool fuse, StepState &s, int64_t n, Replay replay, Pair pair, Single single) {
    while (n > 0) {
        const int v = next_launch(g, s.t, n);
        if (v >= 0) {
            if (const int rc = replay(v)) return rc;
            s.t += g.glen;
            n -= g.glen;
            continue;
        }
        for (int64_t p = fuse ? sweep_pairs(plain_stretch(g, diag_every, s.t, n), s.keep) : 0; p > 0; --p) {
            pair(s.cur);
            s.cur ^= 1;
            s.t += 2;
            n -= 2;
        }
        if (n == 0 || next_launch(g, s.t, n) >= 0) continue;
        single(s.cur, plain_diag(diag_every, s.t));
        s.cur ^= 1;
        s.t += 1;
        n -= 1;
    }
    return 0;
}

}  // namespace mclbm
