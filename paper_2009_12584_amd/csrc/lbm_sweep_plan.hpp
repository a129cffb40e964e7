// Host side of the two-step sweeps: strip segments, their length, and whether
// sweeps are faster than tile steps for a grid or a list of grids.  Free of
// HIP types (a host-only test compiles it with a plain C++ compiler).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

namespace mclbm {

// Columns a strip writes.  58 would leave the least waste, but then the runs
// written per direction start and end inside 64-byte blocks: with 56 every FP32
// run is whole blocks, and the 5600 x 4000 mixture takes 343 us per step instead
// of 401 (48 columns, whole 128-byte lines: 358).
constexpr int SWEEP_OUT = 56;
constexpr int SWEEP_WAVES = 4;  // wavefronts (strips) per workgroup

// One strip segment: columns [x0, x0 + width), rows [y0, y1) of instance inst,
// swept upwards or downwards.
struct SweepTask {
    int inst, x0w, y0, y1;  // x0w = x0 | width << 20 | SWEEP_DOWN (grids are below 2^18 columns)
};
constexpr int SWEEP_DOWN = 1 << 30;

// Is one of n bytes set?  Eight at a time.
inline bool any_set(const uint8_t *m, int n) {
    uint64_t any = 0, v;
    for (; n >= 8; n -= 8, m += 8) {
        std::memcpy(&v, m, 8);
        any |= v;
    }
    for (; n > 0; --n, ++m) any |= *m;
    return any != 0;
}

// What the strips of a grid hold, a byte per row and strip (row after row):
// whether the strip's part of the row has a fluid node, and whether it has a
// solid one.
enum : uint8_t { STRIP_FLUID = 1, STRIP_SOLID = 2 };
inline int strips_of(int nx) { return (nx + SWEEP_OUT - 1) / SWEEP_OUT; }
inline std::vector<uint8_t> sweep_strips(const uint8_t *mask, int nx, int ny) {
    const int ns = strips_of(nx);
    std::vector<uint8_t> f((size_t)ns * ny);
    for (int y = 0; y < ny; ++y)
        for (int s = 0; s < ns; ++s) {
            const uint8_t *m = mask + (size_t)y * nx + s * SWEEP_OUT;
            const int w = std::min(SWEEP_OUT, nx - s * SWEEP_OUT);
            f[(size_t)y * ns + s] = !any_set(m, w) ? STRIP_FLUID : STRIP_SOLID | (std::memchr(m, 0, w) ? STRIP_FLUID : 0);
        }
    return f;
}

// Rows that a strip is cut into for segments of at most `rows` rows.
inline int segment_rows(int ny, int rows) {
    const int n = (ny + rows - 1) / rows;
    return (ny + n - 1) / n;
}
// Appends the segments of a grid: rows [y0, y0 + h) of each strip that hold
// fluid, without the solid rows at either end; every other row of segments is
// swept downwards.  Neighbouring strips of the same rows follow one another.
// Returns how many reach a solid (their rows take the slower walled row step).
inline int sweep_segments(const std::vector<uint8_t> &f, int nx, int ny, int rows, int inst, std::vector<SweepTask> &out) {
    const int ns = strips_of(nx), h = segment_rows(ny, rows);
    int walled = 0;
    for (int y0 = 0; y0 < ny; y0 += h)
        for (int s = 0; s < ns; ++s) {
            int a = y0, b = std::min(y0 + h, ny);
            uint8_t near = 0;
            for (int y = std::max(a - 1, 0); y < std::min(b + 1, ny); ++y) near |= f[(size_t)y * ns + s];
            while (a < b && !(f[(size_t)a * ns + s] & STRIP_FLUID)) ++a;
            while (b > a && !(f[(size_t)(b - 1) * ns + s] & STRIP_FLUID)) --b;
            if (a == b) continue;
            const int x0 = s * SWEEP_OUT;
            out.push_back(SweepTask{inst, x0 | std::min(SWEEP_OUT, nx - x0) << 20 | (y0 / h % 2 ? SWEEP_DOWN : 0), a, b});
            walled += near & STRIP_SOLID ? 1 : 0;
        }
    return walled;
}

// Rows per segment.  A segment of R rows runs R + 6 row steps (the rows that
// only feed it), so long segments waste less; but the launch should put the
// same number of wavefronts on every SIMD.  A row step takes SWEEP_ROW_US where
// a SIMD holds 1, 2, 3 (4) wavefronts (a lone one issues an instruction every
// 5 cycles).  Edge tiles, which come last and mostly wait for their barriers,
// count EDGE_ROWS row steps each in FP32, where they take a third of a CU's
// slots, and nothing in FP16.  The rows are chosen for the least time of this
// model: on 22 measured grids (700 x 500 to 2801 x 1999, both storages, periodic,
// planes and disks, with and without edge tiles; 8 lengths each) within 1.2% of
// the best length in FP32 and 7% in FP16.  With a time of 19 us per round of edge
// tiles instead it was off by 9% in both: 1024 x 1024 disk FP32 20.9 us for 19.1,
// 2801 x 1999 plane FP16 52.6 for 48.2.  Beyond 20 rows nothing was gained.
constexpr int SWEEP_MIN_ROWS = 4, SWEEP_MAX_ROWS = 20, SWEEP_LENGTHS = (SWEEP_MAX_ROWS - SWEEP_MIN_ROWS) / 2 + 1;
constexpr double SWEEP_ROW_US[2][4] = {{1.5, 2.0, 2.7, 0.0}, {1.65, 2.1, 2.9, 3.5}}, EDGE_ROWS[2] = {2.0, 0.0};  // 3 and 4 per SIMD
// Time of the row steps of `groups` workgroups (one wavefront per SIMD each) with
// `steps` row steps: full rounds of cap workgroups per CU, and a last one.
inline double row_steps_us(double groups, double steps, int cap) {
    const double *us = SWEEP_ROW_US[cap == 4], per_cu = std::max(1.0, groups / 256.0);
    const int full = (int)std::ceil(per_cu / cap) - 1, last = (int)std::ceil(per_cu - full * cap);
    return steps * (full * us[cap - 1] + us[last - 1]);
}
// Segments of a grid for each length (SWEEP_MIN_ROWS + 2 k).
inline void sweep_counts(const std::vector<uint8_t> &f, int nx, int ny, int count[SWEEP_LENGTHS]) {
    const int ns = strips_of(nx);
    std::vector<uint8_t> any(ns);
    for (int k = 0; k < SWEEP_LENGTHS; ++k) {
        const int h = segment_rows(ny, SWEEP_MIN_ROWS + 2 * k);
        count[k] = 0;
        for (int y0 = 0; y0 < ny; y0 += h) {
            std::fill(any.begin(), any.end(), 0);
            for (int y = y0; y < std::min(y0 + h, ny); ++y)
                for (int s = 0; s < ns; ++s) any[s] |= f[(size_t)y * ns + s];
            for (int s = 0; s < ns; ++s) count[k] += any[s] & STRIP_FLUID;
        }
    }
}
inline int sweep_rows(const int count[SWEEP_LENGTHS], int cap, int nedge) {
    int best = SWEEP_MIN_ROWS;
    double least = INFINITY;
    for (int k = 0; k < SWEEP_LENGTHS; ++k) {
        const int R = SWEEP_MIN_ROWS + 2 * k, groups = (count[k] + SWEEP_WAVES - 1) / SWEEP_WAVES;
        const double cost = row_steps_us(groups + nedge * EDGE_ROWS[cap == 4] / (R + 6), R + 6, cap);
        if (cost < least) {
            least = cost;
            best = R;
        }
    }
    return best;
}

// Sweep or tile steps?  Sweeps lose where most nodes lie near a wall of the
// improved scheme (an edge tile computes 30 x 28 densities to store at most
// 16 x 14 nodes), where strips are narrow (64 columns take two strips of 56) or
// hold little fluid, and in batches of such grids.  Both are estimated:
//   two tile steps   2 x (fixed + rounds of 256 tiles + strip rows with fluid
//                    + fluid nodes / 64 + the improved scheme's share)
//   a pair           row steps (row_steps_us, and at full throughput), more with
//                    walls in the segments, + edge tiles beyond those that hide
//                    behind the row steps
// with coefficients per kind, storage and stores (plain, streaming), fitted
// without negative ones to both forms' times on 1,300 grids and batches: 64 x 2000 to
// 2801 x 1999, periodic, boxes, planes, disks, channels and obstacles from 8 to
// 200 nodes apart (standard deviation 2 to 9% for tile steps, 4 to 8% for pairs).
// A pair must be estimated sweep_margin of two tile steps or less.  us per step,
// tile steps / sweeps, on grids that now take tile steps: 2048 x 1536 with disks
// of radius 8 every 32 nodes, improved, FP32 98 / 170, FP16 68 / 133; 64 x 8001 box,
// improved, FP32 17.8 / 26.0; 500 instances of 64 x 64, improved, FP32 63 / 102.  On
// grids that sweep: 1024 x 1024 disk, improved, FP32 22.9 / 19.8; 2801 x 1999
// plane, FP16 68 / 51; 64 instances of 128 to 768 columns, FP32 113 / 83, FP16 79 / 71.
// Timed again with this rule, nothing on 1,550 grids and batches of those kinds was
// more than 5% slower than tile steps but FP16 grids of channels between solid
// rows (28 wide, 1400 x 1001: 24.0 / 25.5 us; a batch of them 12 wide, 500 x 400:
// 27 / 30); gains of up to 12% in FP32 and 24% in FP16 are left to tile steps.
struct SweepLoad {
    int tiles = 0;           // a tile step's tiles that hold fluid
    int improved_tiles = 0;  // those of the improved scheme
    int64_t fluid = 0;       // fluid nodes
    int64_t strip_rows = 0;  // rows of strips that hold fluid
    int segments = 0, rows = 0, walled = 0;  // segments, the longest one's rows, those of other rules that reach a solid
    int64_t row_steps = 0;                   // of all segments, feeding rows included
    int edge = 0;                            // edge tiles
};
enum SweepKind { SWEEP_SINGLE, SWEEP_SC1, SWEEP_LIST };  // one simulation, of the single-component model, batches and pools
struct SweepFit {
    double tile[6], pair[4], hidden;  // hidden: edge tiles per CU that hide behind a us of row steps
};
constexpr SweepFit SWEEP_FIT[3][2][2] = {  // kind, FP16, streaming stores
    {{{{4.187, 1.065, 0.022, 0.181, 0.815, 0.304}, {1.01, 0.22, 0.08, 3.58}, 0.03},
      {{5.372, 0.0, 0.190, 0.236, 0.647, 0.289}, {0.55, 0.99, 0.18, 3.82}, 0.01}},
     {{{5.850, 1.901, 0.043, 0.067, 2.764, 0.340}, {0.79, 0.42, 0.12, 3.23}, 0.01},
      {{8.587, 0.0, 0.145, 0.110, 1.187, 0.302}, {1.22, 0.0, 0.22, 3.43}, 0.02}}},
    {{{{1.250, 0.783, 0.049, 0.085, 0.0, 0.0}, {0.61, 0.39, 0.11, 0.0}, 0.0},
      {{4.461, 0.193, 0.115, 0.100, 0.0, 0.0}, {0.0, 1.0, 0.05, 0.0}, 0.0}},
     {{{5.890, 0.369, 0.090, 0.010, 0.0, 0.0}, {0.91, 0.08, 0.14, 0.0}, 0.0},
      {{9.611, 0.390, 0.127, 0.0, 0.0, 0.0}, {0.88, 0.05, 0.18, 0.0}, 0.0}}},
    {{{{5.377, 1.195, 0.021, 0.269, 0.750, 0.0}, {0.68, 0.66, 0.10, 3.25}, 0.0},
      {{6.470, 0.465, 0.031, 0.348, 0.086, 0.228}, {0.33, 1.22, 0.02, 3.35}, 0.0}},
     {{{4.066, 2.118, 0.003, 0.205, 1.081, 0.0}, {0.98, 0.28, 0.09, 2.96}, 0.01},
      {{15.641, 0.0, 0.203, 0.002, 0.334, 0.152}, {1.31, 0.0, 0.03, 3.01}, 0.05}}}};
// Closer estimates need no margin: the single-component model's (2 to 5%; 1776 x
// 1615 channel in FP16, 34.7 / 31.3 us, is estimated at 0.97) and streaming FP16 batches
// and pools (tile steps to 2%; 64 instances, 79 / 71 us, at 0.98).  Other FP16 lists
// err by 9%, and without a margin 200 instances of 64 x 64 would take 24.1 us for 22.4.
constexpr double SWEEP_MARGIN = 0.95;
inline double sweep_margin(SweepKind kind, bool f16, bool nt) {
    return kind == SWEEP_SC1 || (kind == SWEEP_LIST && f16 && nt) ? 1.0 : SWEEP_MARGIN;
}

inline double tile_steps_us(const SweepLoad &w, SweepKind kind, bool f16, bool nt) {
    const double *c = SWEEP_FIT[kind][f16][nt].tile;
    const double improved = kind == SWEEP_LIST ? w.improved_tiles / 256.0 : w.improved_tiles > 0;
    return 2.0 * (c[0] + c[1] * ((w.tiles + 255) / 256) + c[2] * (double)w.strip_rows / 256.0 + c[3] * (double)w.fluid / (64.0 * 256.0) +
                  c[4] * improved + c[5] * w.edge / 256.0);
}
inline double sweep_pair_us(const SweepLoad &w, SweepKind kind, bool f16, bool nt) {
    const SweepFit &c = SWEEP_FIT[kind][f16][nt];
    const int cap = f16 ? 4 : 3;
    const double rounds = row_steps_us((w.segments + SWEEP_WAVES - 1) / SWEEP_WAVES, w.rows + 6, cap);
    const double through = (double)w.row_steps / SWEEP_WAVES / 256.0 * SWEEP_ROW_US[f16][cap - 1] / cap;
    return c.pair[0] * rounds + c.pair[1] * through + c.pair[2] * rounds * w.walled / w.segments +
           c.pair[3] * std::max(0.0, w.edge / 256.0 - c.hidden * rounds);
}
inline bool sweep_pays(const SweepLoad &w, SweepKind kind, bool f16, bool nt) {
    if (!w.segments) return false;
    return sweep_pair_us(w, kind, f16, nt) <= sweep_margin(kind, f16, nt) * tile_steps_us(w, kind, f16, nt);
}
// The load's part that its segments give.
inline void add_segments(SweepLoad &w, const std::vector<SweepTask> &seg, size_t from, int walled) {
    for (size_t k = from; k < seg.size(); ++k) {
        w.rows = std::max(w.rows, seg[k].y1 - seg[k].y0);
        w.row_steps += seg[k].y1 - seg[k].y0 + 6;
    }
    w.segments = (int)seg.size();
    w.walled += walled;
}
inline int64_t strip_rows_with_fluid(const std::vector<uint8_t> &f) {
    int64_t n = 0;
    for (uint8_t v : f) n += v & STRIP_FLUID;
    return n;
}

}  // namespace mclbm
