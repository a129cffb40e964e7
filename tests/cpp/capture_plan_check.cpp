// Host-only check of the step loop mixed with launches that the caller has
// captured: over random sequences of plain steps, captures of steps and of
// fields passes, replays at times of the parity they were captured at, and
// states set at other times, no launch reads a buffer that does not hold the
// state.  A buffer is modelled by the number of steps that its contents have
// seen.
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2009_12584_amd/csrc/lbm_plan.hpp"

using namespace mclbm;

struct Launch {
    int cur, steps;  // 0 steps: a fields pass
};
struct Captured {
    int64_t parity;
    std::vector<Launch> list;
};

int main() {
    std::mt19937 rng(23);
    long replays = 0, pairs_run = 0;
    for (int diag = 0; diag <= 7; ++diag)
        for (int rep = 0; rep < 400; ++rep) {
            GraphPlan g;  // no graphs of the library's own: those always keep the parity
            StepState s;
            int64_t seen[2] = {0, -1000000}, truth = 0;
            std::vector<Captured> graphs;
            auto run = [&](const Launch &l) {
                if (seen[l.cur] != truth) return false;
                if (l.steps) {
                    truth += l.steps;
                    seen[l.cur ^ 1] = truth;
                }
                return true;
            };
            for (int op = 0; op < 60; ++op) {
                const int kind = (int)(rng() % 6);
                bool ok = true;
                if (kind <= 1) {  // plain steps
                    run_steps(g, diag, true, s, 1 + (int64_t)(rng() % 11), [](int) { return 0; },
                              [&](int cur) { ok = run({cur, 2}) && ok; ++pairs_run; },
                              [&](int cur, bool) { ok = run({cur, 1}) && ok; });
                } else if (kind == 2) {  // an even number of steps, or a fields pass, captured
                    Captured c{s.t & 1, {}};
                    s.keep = true;
                    if (rng() % 3 == 0)
                        c.list.push_back({s.cur, 0});
                    else
                        run_steps(g, diag, true, s, 2 * (1 + (int64_t)(rng() % 6)), [](int) { return 0; },
                                  [&](int cur) { c.list.push_back({cur, 2}); }, [&](int cur, bool) { c.list.push_back({cur, 1}); });
                    graphs.push_back(c);
                } else if (kind == 3) {  // a state set at another time
                    const int64_t step = (int64_t)(rng() % 50);
                    s.cur = buffer_for(s, step);
                    s.t = step;
                    truth += 1000;
                    seen[s.cur] = truth;
                } else if (!graphs.empty()) {
                    const Captured &c = graphs[rng() % graphs.size()];
                    if (c.parity != (s.t & 1)) continue;
                    for (const Launch &l : c.list) ok = run(l) && ok;
                    ++replays;
                }
                if (!ok || seen[s.cur] != truth)
                    return std::printf("diag %d, sequence %d, operation %d (kind %d): the state is not where it is read\n", diag, rep, op, kind), 1;
            }
        }
    std::printf("ok %ld replays, %ld pairs\n", replays, pairs_run);
    return 0;
}
