// Host-only check of the sweep's plan.  Segments: on random masks, for every
// length, they hold each fluid node once, begin and end on rows with fluid, are
// as many as counted, and the walled ones are those that reach a solid.  Choice
// between sweeps and tile steps: as timed on grids and lists where one of them
// is clearly faster, edge tiles counted from the mask.
#include <cstdio>
#include <functional>
#include <random>
#include <string>

#include "../../paper_2009_12584_amd/csrc/lbm_sweep_plan.hpp"

using namespace mclbm;

struct Grid {
    int nx, ny;
    std::vector<uint8_t> m;
    Grid(int w, int h, const std::function<bool(int, int)> &solid, bool closed) : nx(w), ny(h), m((size_t)w * h) {
        for (int y = 0; y < ny; ++y)
            for (int x = 0; x < nx; ++x)
                m[(size_t)y * nx + x] = solid(x, y) || (closed && (x == 0 || y == 0 || x == nx - 1 || y == ny - 1));
    }
    bool solid(int x, int y) const { return x < 0 || y < 0 || x >= nx || y >= ny || m[(size_t)y * nx + x]; }
    bool next_to_solid(int x, int y) const {
        if (solid(x, y)) return false;
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx)
                if (solid(x + dx, y + dy)) return true;
        return false;
    }
};

static int check_segments() {
    std::mt19937 rng(3);
    for (int rep = 0; rep < 60; ++rep) {
        const int nx = 64 + (int)(rng() % 180), ny = 32 + (int)(rng() % 70), fill = (int)(rng() % 3);
        const Grid g(nx, ny, [&](int, int) { return fill == 0 ? rng() % 40 == 0 : (fill == 1 ? rng() % 3 > 0 : rng() % 300 > 0); }, rng() % 2);
        const std::vector<uint8_t> f = sweep_strips(g.m.data(), nx, ny);
        int count[SWEEP_LENGTHS];
        sweep_counts(f, nx, ny, count);
        for (int k = 0; k < SWEEP_LENGTHS; ++k) {
            const int R = SWEEP_MIN_ROWS + 2 * k, h = segment_rows(ny, R);
            std::vector<SweepTask> seg;
            const int walled = sweep_segments(f, nx, ny, R, 7, seg);
            std::vector<uint8_t> seen(g.m.size(), 0);
            int reach = 0;
            for (const SweepTask &t : seg) {
                const int x0 = t.x0w & 0xfffff, w = (t.x0w >> 20) & 127, c0 = t.y0 / h * h;
                if (t.inst != 7 || t.y1 > std::min(c0 + h, ny) || t.y0 >= t.y1) return std::printf("bad rows\n"), 1;
                if (((t.x0w & SWEEP_DOWN) != 0) != (t.y0 / h % 2 != 0)) return std::printf("bad direction\n"), 1;
                bool first = false, last = false, near = false;
                for (int x = x0; x < x0 + w; ++x) {
                    first |= !g.solid(x, t.y0);
                    last |= !g.solid(x, t.y1 - 1);
                    for (int y = t.y0; y < t.y1; ++y) seen[(size_t)y * nx + x] += 1;
                    for (int y = std::max(c0 - 1, 0); y < std::min(c0 + h + 1, ny); ++y) near |= g.solid(x, y);
                }
                if (!first || !last) return std::printf("solid rows at a segment's end\n"), 1;
                reach += near;
            }
            for (size_t q = 0; q < g.m.size(); ++q)
                if (seen[q] > 1 || (!g.m[q] && seen[q] != 1)) return std::printf("node %zu swept %d times\n", q, seen[q]), 1;
            if ((int)seg.size() != count[k] || reach != walled) return std::printf("%zu segments, counted %d; %d walled, %d\n", seg.size(), count[k], reach, walled), 1;
        }
    }
    return 0;
}

// n instances of a grid, in the improved scheme or another rule
static bool sweeps(const Grid &g, int n, bool improved, SweepKind kind, bool f16) {
    const int ty = f16 && kind != SWEEP_SC1 ? 16 : 8;
    SweepLoad w;
    for (int y0 = 0; y0 < g.ny; y0 += ty)
        for (int x0 = 0; x0 < g.nx; x0 += 64) {
            bool any = false;
            for (int y = y0; y < std::min(y0 + ty, g.ny); ++y)
                for (int x = x0; x < std::min(x0 + 64, g.nx); ++x) any |= !g.solid(x, y);
            w.tiles += any ? n : 0;
        }
    w.improved_tiles = improved ? w.tiles : 0;
    for (uint8_t v : g.m) w.fluid += v ? 0 : n;
    if (improved)
        for (int y0 = 0; y0 < g.ny; y0 += 14)
            for (int x0 = 0; x0 < g.nx; x0 += 16) {
                bool any = false;
                for (int y = y0 - 2; y < y0 + 16 && !any; ++y)
                    for (int x = x0 - 2; x < x0 + 18 && !any; ++x) any = g.next_to_solid(x, y);
                w.edge += any ? n : 0;
            }
    const std::vector<uint8_t> f = sweep_strips(g.m.data(), g.nx, g.ny);
    w.strip_rows = n * strip_rows_with_fluid(f);
    int count[SWEEP_LENGTHS];
    sweep_counts(f, g.nx, g.ny, count);
    for (int &c : count) c *= n;
    const int rows = sweep_rows(count, f16 || kind == SWEEP_SC1 ? 4 : 3, w.edge);
    std::vector<SweepTask> seg;
    for (int k = 0; k < n; ++k) {
        const size_t from = seg.size();
        const int walled = sweep_segments(f, g.nx, g.ny, rows, k, seg);
        add_segments(w, seg, from, improved ? 0 : walled);
    }
    const double per_node = (kind == SWEEP_SC1 ? 1 : 2) * (f16 ? 20.0 : 36.0);
    const bool nt = 2.0 * n * g.ny * ((g.nx + 63) / 64 * 64) * per_node > 192.0 * (1 << 20);
    return sweep_pays(w, kind, f16, nt);
}

static int check_choice() {
    const auto open = [](int, int) { return false; };
    const auto disks = [](int x, int y) { return (x % 32 - 16) * (x % 32 - 16) + (y % 32 - 16) * (y % 32 - 16) <= 64; };
    const auto channels = [](int, int y) { return y % 16 < 4; };
    struct Case {
        const char *name;
        Grid g;
        int n;
        bool improved;
        SweepKind kind;
        int f32, f16;  // 1: sweeps, 0: tile steps, -1: no clear difference
    };
    const Case cases[] = {
        {"periodic 2048 x 1536", Grid(2048, 1536, open, false), 1, false, SWEEP_SINGLE, 1, 1},
        {"box 2048 x 1536, improved", Grid(2048, 1536, open, true), 1, true, SWEEP_SINGLE, 1, 1},
        {"disk 1024 x 1024, improved", Grid(1024, 1024, [](int x, int y) { return (x - 512) * (x - 512) + (y - 512) * (y - 512) <= 90000; }, true),
         1, true, SWEEP_SINGLE, 1, -1},
        {"plane 2801 x 1999", Grid(2801, 1999, [](int x, int y) { return y <= 0.58 * (x - 1400) + 800; }, true), 1, false, SWEEP_SINGLE, 1, 1},
        {"disks 2048 x 1536, improved", Grid(2048, 1536, disks, true), 1, true, SWEEP_SINGLE, 0, 0},
        {"channels 700 x 500, improved", Grid(700, 500, channels, true), 1, true, SWEEP_SINGLE, 0, 0},
        {"box 64 x 8001, improved", Grid(64, 8001, open, true), 1, true, SWEEP_SINGLE, 0, 0},
        {"single component, plane 2800 x 2000", Grid(2800, 2000, [](int x, int y) { return y <= 0.47 * (x - 1400) + 800; }, true), 1, false, SWEEP_SC1, 1, 1},
        {"single component, channels 1400 x 1001", Grid(1400, 1001, channels, true), 1, false, SWEEP_SC1, 0, -1},
        {"64 boxes 300 x 200", Grid(300, 200, open, true), 64, false, SWEEP_LIST, 1, 1},
        {"500 boxes 64 x 64, improved", Grid(64, 64, open, true), 500, true, SWEEP_LIST, 0, 0},
        {"256 boxes 64 x 32, improved", Grid(64, 32, open, true), 256, true, SWEEP_LIST, 0, 0},
        {"64 grids of disks 100 x 100, improved", Grid(100, 100, disks, true), 64, true, SWEEP_LIST, 0, 0},
    };
    int bad = 0;
    for (const Case &c : cases)
        for (int f16 = 0; f16 < 2; ++f16) {
            const int want = f16 ? c.f16 : c.f32;
            if (want < 0) continue;
            if (sweeps(c.g, c.n, c.improved, c.kind, f16) != (want == 1)) {
                std::printf("%s %s: %s\n", c.name, f16 ? "FP16" : "FP32", want ? "tile steps" : "sweeps");
                ++bad;
            }
        }
    return bad;
}

int main() {
    if (check_segments() || check_choice()) return 1;
    std::printf("ok\n");
    return 0;
}
