// Host-only check of the pairs that the step loop fuses: for every accepted
// pair (graph_steps, diag_every) up to 24 and random sequences of step calls,
// every step runs once, no pair holds a diagnostic step or the start of a
// graph replay, replays find the state in buffer 0, and where the buffer has to
// stay the parity of the time (graphs, captured code) it does.
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2009_12584_amd/csrc/lbm_plan.hpp"

using namespace mclbm;

int main() {
    std::mt19937 rng(11);
    long pairs_run = 0;
    for (int gs = 0; gs <= 24; ++gs)
        for (int de = 0; de <= 24; ++de) {
            GraphPlan g;
            if (!graph_plan(gs, de, g)) continue;
            for (int rep = 0; rep < 20; ++rep) {
                const int64_t T = 300;
                const bool keep = g.glen > 0 || rep % 2;
                std::vector<int> ran(T, 0);
                int64_t t = 0;
                int cur = 0;
                while (t < T) {
                    int64_t n = 1 + (int64_t)(rng() % 70);
                    if (t + n > T) n = T - t;
                    while (n > 0) {
                        if (next_launch(g, t, n) >= 0) {
                            if (cur != 0) return std::printf("replay from buffer 1 at %lld\n", (long long)t), 1;
                            for (int s = 0; s < g.glen; ++s) ran[t + s] += 1;
                            t += g.glen;
                            n -= g.glen;
                            continue;
                        }
                        for (int64_t p = sweep_pairs(plain_stretch(g, de, t, n), keep); p > 0; --p, t += 2, n -= 2, cur ^= 1) {
                            ++pairs_run;
                            for (int64_t s = t; s < t + 2; ++s) {
                                ran[s] += 1;
                                if (plain_diag(de, s)) return std::printf("diagnostic step %lld in a pair\n", (long long)s), 1;
                            }
                            if (next_launch(g, t + 1, n - 1) >= 0) return std::printf("replay inside a pair\n"), 1;
                        }
                        if (n == 0 || next_launch(g, t, n) >= 0) continue;
                        ran[t] += 1;
                        t += 1;
                        n -= 1;
                        cur ^= 1;
                    }
                    if (keep && cur != (t & 1)) return std::printf("buffer %d at %lld\n", cur, (long long)t), 1;
                }
                for (int64_t k = 0; k < T; ++k)
                    if (ran[k] != 1) return std::printf("graph %d diag %d: step %lld ran %d times\n", gs, de, (long long)k, ran[k]), 1;
            }
        }
    std::printf("ok %ld pairs\n", pairs_run);
    return pairs_run > 0 ? 0 : 1;
}
