// Two time steps in one pass over the populations: a wavefront sweeps a strip
// of the lattice row by row and carries both steps in registers.
//
// A step reads and writes every population once, so on grids beyond the
// caches a launch per step is bound by HBM.  Here the populations of time t
// are read once and those of t + 2 written once per pair of steps; the ones
// of t + 1 never leave the registers.  A strip is 64 columns, one per lane,
// of which the middle SWEEP_OUT are written (each step needs one column for
// the pull and one for the density stencil on either side, the first step's
// pull straight from memory).  At row r the wavefront
//   A  sums the densities of row r at t from its pulled populations,
//   B  collides row r - 1 (its density stencil is now complete) and issues
//      the loads of row r + 1,
//   C  completes the populations of row r - 2 at t + 1 from the collided rows
//      r - 3, r - 2, r - 1, sums its densities,
//   D  collides row r - 3 at t + 1 and stores it as time t + 2.
// Neighbours in x come from the next lane (DPP wavefront shifts), neighbours
// in y from registers, so there is no LDS, no barrier and no halo frame, and
// a row's loads are in flight while the rows before it are computed.
//
// Every value is computed by the same expressions in the same order as the
// tile step's (node_state, node_collide, grad9), stored populations rounded
// to storage between the two steps, so the result is bit for bit that of two
// tile steps.
#pragma once

#include "lbm_device.hpp"

namespace mclbm {

constexpr int SWEEP_OUT = 58;   // columns a strip writes
constexpr int SWEEP_HALO = 3;   // columns either side that only feed them
constexpr int SWEEP_WAVES = 4;  // wavefronts (strips) per workgroup

// One strip segment: columns [x0, x0 + width), rows [y0, y1) of instance inst.
struct SweepTask {
    int inst, x0w, y0, y1;  // x0w = x0 | width << 20 (grids are below 2^18 columns)
};

// Value of the lane to the left (x - 1) and to the right (x + 1).
__device__ __forceinline__ float lane_left(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_right(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}

// The element of direction i of a node's populations (Incoming<S>::D), as one
// to two words: how many words hold it.
template <typename S> constexpr int elem_words(int i) { return sizeof(S) == 4 || i == 0 ? 2 : 1; }

// Neighbour values of one density plane from its rows y - 1, y, y + 1.
__device__ __forceinline__ void row_stencil(float m, float c, float p, float &sx, float &sy) {
    float v[9];
    v[0] = c;
    v[1] = lane_right(c);
    v[2] = p;
    v[3] = lane_left(c);
    v[4] = m;
    v[5] = lane_right(p);
    v[6] = lane_left(p);
    v[7] = lane_left(m);
    v[8] = lane_right(m);
    grad9(v, sx, sy);
}

// Populations of a row at the uniform byte offsets row[] of the rows below,
// at and above it, for lanes none of which has a solid neighbour.
template <typename S>
__device__ __forceinline__ void pull_open(const char *fin, const uint32_t row[3], const uint32_t col[3],
                                          typename Incoming<S>::D &d) {
    using P = typename Store<S>::P;
    constexpr uint32_t pb = slot_bytes<S, 2>();
    const char *b = fin + row[1];
    if constexpr (sizeof(S) == 4) {
        const float2 v = *(const float2 *)(b + col[1]);
        d[0][0] = v.x;
        d[1][0] = v.y;
    } else {
        d[0][0] = *(const float *)(b + col[1]);
        d[1][0] = *(const float *)(b + 9u * pb + col[1]);
    }
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        const P v = *(const P *)(fin + row[1 - CY[i]] + (uint32_t)i * pb + col[1 - CX[i]]);
        if constexpr (sizeof(S) == 4) {
            d[0][i] = v.x;
            d[1][i] = v.y;
        } else {
            d[0][i] = __builtin_bit_cast(float, v);
        }
    }
}

// Two steps of instance I over columns [x0, x0 + width), rows [y0, y1), from
// fin to fout.  BC_IMPROVED: only for strips whose nodes have no solid node
// within reach of a virtual density (their adhesion is zero).
template <typename S, int BC, bool NT>
__device__ __forceinline__ void sweep_pair(const Inst &I, const typename Store<S>::P *__restrict__ fin_,
                                           typename Store<S>::P *__restrict__ fout, int x0, int width, int y0, int y1) {
#pragma clang fp contract(off)
    using In = Incoming<S>;
    using D = typename In::D;
    constexpr float SC = Store<S>::SC;
    constexpr uint32_t pb = slot_bytes<S, 2>();
    const char *fin = (const char *)fin_;
    const int lane = threadIdx.x & 63;
    const int gx = x0 - SWEEP_HALO + lane;
    const bool perx = I.periodic & 1u, pery = I.periodic & 2u;
    const bool inside = perx || (unsigned)gx < (unsigned)I.nx;
    const int wx = keep_in(gx, I.nx, perx, false);
    uint32_t col[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) col[j] = col_off<S, 2>(keep_in(gx - 1 + j, I.nx, perx, false));
    const bool mine = lane >= SWEEP_HALO && lane < SWEEP_HALO + width;
    const float rref[2] = {I.rrefA, I.rrefB};

    // node word of row y: solid beyond a closed border
    auto word = [&](int y) -> uint32_t {
        const bool in = inside && (pery || (unsigned)y < (unsigned)I.ny);
        const uint32_t v = I.node[__umul24((uint32_t)keep_in(y, I.ny, pery, false), (uint32_t)I.pitch) + (uint32_t)wx];
        return in ? v : (uint32_t)NW_SOLID;
    };
    auto any_wall = [&](uint32_t w) { return __any((w & (NW_SOLID | 0xffu)) != 0u) != 0; };
    // pull of row y; solid lanes read values that are not used
    auto pull = [&](int y, uint32_t w, bool wall, D &d) {
        uint32_t row[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) row[j] = row_off<S, 2>(I, keep_in(y - 1 + j, I.ny, pery, false));
        if (!wall) {
            pull_open<S>(fin, row, col, d);
        } else {
            Around a;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                a.row[j] = row[j];
                a.col[j] = col[j];
            }
            In::pull(fin_, pb, a, w, d);
        }
    };

    D d[2];               // populations at t: rows r and r - 1 alternate
    D e[2];               // populations at t + 1: rows r - 2 and r - 3 alternate
    D ep;                 // populations at t + 1 of row r - 1, directions of rows r - 2 and r - 1
    D up;                 // collided row r - 2: directions 2, 5, 6 (going up)
    float sd[2][2];       // deviation sums at t of rows r, r - 1
    float se[2][2];       // and at t + 1 of rows r - 2, r - 3
    float p1[2][3] = {};  // densities at t of rows r - 2, r - 1, r
    float p2[2][3] = {};  // densities at t + 1 of rows r - 4, r - 3, r - 2
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 9; ++i) d[0][c][i] = d[1][c][i] = e[0][c][i] = e[1][c][i] = ep[c][i] = up[c][i] = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c) sd[0][c] = sd[1][c] = se[0][c] = se[1][c] = 0.f;
    uint32_t w0 = NW_SOLID, w1 = NW_SOLID, w2 = NW_SOLID, w3 = NW_SOLID;  // words of rows r, r - 1, r - 2, r - 3
    bool f0, f1 = true, f2 = true, f3 = true;                             // any_wall of them

    const int last = y1 + 2;
    w0 = word(y0 - 3);
    f0 = any_wall(w0);
    pull(y0 - 3, w0, f0, d[0]);
    uint32_t wn = word(y0 - 2);

    // one row; K alternates the two-row arrays
    auto row_step = [&](int r, D &dr, D &dq, float(&sr)[2], float(&sq)[2], D &er, D &eq, float(&ser)[2], float(&seq)[2]) {
        // ---- A: densities of row r at t
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            sr[c] = In::sum(dr, c);
            p1[c][0] = p1[c][1];
            p1[c][1] = p1[c][2];
            p1[c][2] = rref[c] + sr[c] * (1.f / SC);
            if (f0) p1[c][2] = (w0 & NW_SOLID) ? 0.f : p1[c][2];
        }
        // ---- B: collision of row r - 1 at t
        D q;
        if (r >= y0 - 1) {
            float sax, say, sbx, sby, nxs = 0.f, nys = 0.f;
            row_stencil(p1[0][0], p1[0][1], p1[0][2], sax, say);
            row_stencil(p1[1][0], p1[1][1], p1[1][2], sbx, sby);
            NodeState n;
            if (BC != BC_IMPROVED && f1) {
                float vn[9];
#pragma unroll
                for (int i = 1; i < 9; ++i) vn[i] = ((w1 >> (i - 1)) & 1u) ? 1.f : 0.f;
                grad9(vn, nxs, nys);
                n = node_state<S, BC, true>(I, dq, p1[0][1], p1[1][1], sax, say, sbx, sby, nxs, nys, 0.f, 0.f, 0.f, 0.f);
            } else {
                n = node_state<S, BC, false>(I, dq, p1[0][1], p1[1][1], sax, say, sbx, sby, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f);
            }
            const float2 rest = node_collide<S>(I, dq, sq, p1[0][1], p1[1][1], n, [&](int i, auto v) {
                if constexpr (sizeof(S) == 4) {
                    q[0][i] = v.x;
                    q[1][i] = v.y;
                } else {
                    q[0][i] = __builtin_bit_cast(float, v);
                }
            });
            q[0][0] = rest.x;
            q[1][0] = rest.y;
        }
        const uint32_t wc = wn;
        const bool fc = any_wall(wc);
        if (r < last) {
            pull(r + 1, wc, fc, dq);
            wn = word(r + 2);
        }
        if (r >= y0 - 1) {
            // ---- C: row r - 2 at t + 1: its directions from above (row r - 1);
            // a solid neighbour returns the node's own opposite population
#pragma unroll
            for (int i = 0; i < 9; ++i)
#pragma unroll
                for (int c = 0; c < elem_words<S>(i); ++c) {
                    if (CY[i] == -1) {
                        float v = CX[i] == 0 ? q[c][i] : (CX[i] == 1 ? lane_left(q[c][i]) : lane_right(q[c][i]));
                        if (f2) v = ((w2 >> (OPP[i] - 1)) & 1u) ? up[c][OPP[i]] : v;
                        er[c][i] = v;
                    } else {
                        er[c][i] = ep[c][i];
                    }
                }
            // row r - 1: its directions from below (row r - 2) and its own
#pragma unroll
            for (int i = 0; i < 9; ++i)
#pragma unroll
                for (int c = 0; c < elem_words<S>(i); ++c) {
                    if (CY[i] == -1) continue;
                    const float s = CY[i] == 1 ? up[c][i] : q[c][i];
                    float v = CX[i] == 0 ? s : (CX[i] == 1 ? lane_left(s) : lane_right(s));
                    if (i > 0 && f1) v = ((w1 >> (OPP[i] - 1)) & 1u) ? q[c][OPP[i]] : v;
                    ep[c][i] = v;
                }
#pragma unroll
            for (int i = 1; i < 9; ++i)
#pragma unroll
                for (int c = 0; c < elem_words<S>(i); ++c)
                    if (CY[i] == 1) up[c][i] = q[c][i];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                ser[c] = In::sum(er, c);
                p2[c][0] = p2[c][1];
                p2[c][1] = p2[c][2];
                p2[c][2] = rref[c] + ser[c] * (1.f / SC);
                if (f2) p2[c][2] = (w2 & NW_SOLID) ? 0.f : p2[c][2];
            }
        }
        // ---- D: collision of row r - 3 at t + 1
        if (r >= y0 + 3) {
            float sax, say, sbx, sby, nxs = 0.f, nys = 0.f;
            row_stencil(p2[0][0], p2[0][1], p2[0][2], sax, say);
            row_stencil(p2[1][0], p2[1][1], p2[1][2], sbx, sby);
            NodeState n;
            if (BC != BC_IMPROVED && f3) {
                float vn[9];
#pragma unroll
                for (int i = 1; i < 9; ++i) vn[i] = ((w3 >> (i - 1)) & 1u) ? 1.f : 0.f;
                grad9(vn, nxs, nys);
                n = node_state<S, BC, true>(I, eq, p2[0][1], p2[1][1], sax, say, sbx, sby, nxs, nys, 0.f, 0.f, 0.f, 0.f);
            } else {
                n = node_state<S, BC, false>(I, eq, p2[0][1], p2[1][1], sax, say, sbx, sby, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f);
            }
            char *o = (char *)fout + row_off<S, 2>(I, r - 3);
            if (mine && !(w3 & NW_SOLID)) {
                const float2 rest = node_collide<S>(I, eq, seq, p2[0][1], p2[1][1], n, [&](int i, auto v) {
                    auto *a = (typename Store<S>::P *)(o + (uint32_t)i * pb + col[1]);
                    if constexpr (NT)
                        Store<S>::put2nt(a, v);
                    else
                        Store<S>::put2(a, v);
                });
                put_rest<S>((typename Store<S>::P *)o, pb, col[1], rest.x, rest.y, NT);
            }
        }
        w3 = w2;
        w2 = w1;
        w1 = w0;
        w0 = wc;
        f3 = f2;
        f2 = f1;
        f1 = f0;
        f0 = fc;
    };
    for (int r = y0 - 3; r <= last; r += 2) {
        row_step(r, d[0], d[1], sd[0], sd[1], e[0], e[1], se[0], se[1]);
        if (r + 1 > last) break;
        row_step(r + 1, d[1], d[0], sd[1], sd[0], e[1], e[0], se[1], se[0]);
    }
}

}  // namespace mclbm
