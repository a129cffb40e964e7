// Two time steps in one pass over the populations: a wavefront sweeps a strip
// of the lattice row by row and carries both steps in registers.
//
// A step reads and writes every population once, so on grids beyond the
// caches a launch per step is bound by HBM.  Here the populations of time t
// are read once and those of t + 2 written once per pair of steps; the ones
// of t + 1 never leave the chip.  A strip is 64 columns, one per lane, of
// which the middle SWEEP_OUT are written (each step needs one column for the
// pull and one for the density stencil on either side, the first step's pull
// straight from memory).  At row r the wavefront
//   A  sums the densities of row r at t from its pulled populations,
//   B  collides row r - 1 (its density stencil is now complete) and issues
//      the loads of row r + 1,
//   C  completes the populations of row r - 2 at t + 1 from the collided rows
//      r - 3, r - 2, r - 1, sums its densities,
//   D  collides row r - 3 at t + 1 and stores it as time t + 2.
// Neighbours in x come from the next lane (DPP wavefront shifts), neighbours
// in y from registers, so there is no barrier and no halo frame, and a row's
// loads are in flight while the rows before it are computed.  Rows that wait
// (r for B, r - 2 for D) are parked in the wavefront's own LDS: with them in
// registers the FP32 sweep needs 218 VGPRs (2 wavefronts per SIMD), without
// 168 (3; FP16 124, 4).  Rows without a solid in reach of the strip skip the
// bounce-back selects and the wall forces (a wave-uniform branch), and their
// loads need no address arithmetic (a uniform row pointer, a column offset
// kept per lane, the direction as an immediate).
//
// 5600 x 4000 mixture, per step, against the tile step: FP32 640 -> 343 us
// (then 4.3 GB of cache-to-memory traffic per pair at 6.1 TB/s: bound by
// memory), FP16 382 -> 270 us (bound by instruction issue: the mixed-precision
// operations run at half and quarter rate).
//
// Every value is computed by the same expressions in the same order as the
// tile step's (node_state, node_collide, grad9), stored populations rounded
// to storage between the two steps, so the result is bit for bit that of two
// tile steps.
#pragma once

#include <type_traits>

#include "lbm_device.hpp"

namespace mclbm {

// Columns a strip writes.  58 would leave the least waste, but then the runs
// written per direction start and end inside 64-byte blocks: with 56 every FP32
// run is whole blocks, and the 5600 x 4000 mixture takes 343 us per step instead
// of 401 (48 columns, whole 128-byte lines: 358).
constexpr int SWEEP_OUT = 56;
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

// Words that hold direction i of a node's populations (Incoming<S>::D).
template <typename S> constexpr int elem_words(int i) { return sizeof(S) == 4 || i == 0 ? 2 : 1; }

// Rows that wait for the next row's densities are parked in LDS, so that the
// registers hold one row of loads in flight and one row at work: each lane
// keeps its own words, four (16 bytes) per lane and access.
template <typename S> constexpr int row_words() { return sizeof(S) == 4 ? 18 : 10; }
template <typename S> constexpr int park_groups() { return (row_words<S>() + 3) / 4; }
template <typename S> struct SweepPark {
    float4 at[2][park_groups<S>()][64];  // rows at t and at t + 1
};
template <typename S> __device__ __forceinline__ float &row_word(typename Incoming<S>::D &d, int k) {
    if constexpr (sizeof(S) == 4) return d[k & 1][k >> 1];
    return k < 2 ? d[k][0] : d[0][k - 1];
}
template <typename S>
__device__ __forceinline__ void park_put(SweepPark<S> &pk, int which, int lane, typename Incoming<S>::D &d) {
#pragma unroll
    for (int g = 0; g < park_groups<S>(); ++g) {
        float4 v = make_float4(row_word<S>(d, 4 * g), row_word<S>(d, 4 * g + 1), 0.f, 0.f);
        if (4 * g + 2 < row_words<S>()) {
            v.z = row_word<S>(d, 4 * g + 2);
            v.w = row_word<S>(d, 4 * g + 3);
            pk.at[which][g][lane] = v;
        } else {
            *(float2 *)&pk.at[which][g][lane] = make_float2(v.x, v.y);
        }
    }
}
template <typename S>
__device__ __forceinline__ void park_get(SweepPark<S> &pk, int which, int lane, typename Incoming<S>::D &d) {
#pragma unroll
    for (int g = 0; g < park_groups<S>(); ++g) {
        if (4 * g + 2 < row_words<S>()) {
            const float4 v = pk.at[which][g][lane];
            row_word<S>(d, 4 * g) = v.x;
            row_word<S>(d, 4 * g + 1) = v.y;
            row_word<S>(d, 4 * g + 2) = v.z;
            row_word<S>(d, 4 * g + 3) = v.w;
        } else {
            const float2 v = *(const float2 *)&pk.at[which][g][lane];
            row_word<S>(d, 4 * g) = v.x;
            row_word<S>(d, 4 * g + 1) = v.y;
        }
    }
}
// Parked values are read back from LDS, not kept in registers by the compiler.
__device__ __forceinline__ void park_fence() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

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
                                           typename Store<S>::P *__restrict__ fout, int x0, int width, int y0, int y1,
                                           SweepPark<S> &pk) {
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

    D d;                  // populations at t of row r, then of r + 1 in flight
    D ep;                 // populations at t + 1 of row r - 1, directions of rows r - 2 and r - 1
    D up;                 // collided row r - 2: directions 2, 5, 6 (going up)
    float sd[2] = {};     // deviation sums at t of row r - 1
    float se[2] = {};     // and at t + 1 of row r - 3
    float p1[2][3] = {};  // densities at t of rows r - 2, r - 1, r
    float p2[2][3] = {};  // densities at t + 1 of rows r - 4, r - 3, r - 2
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 9; ++i) ep[c][i] = up[c][i] = 0.f;
    uint32_t w0 = word(y0 - 3), w1 = NW_SOLID, w2 = NW_SOLID, w3 = NW_SOLID;  // words of rows r, r - 1, r - 2, r - 3
    bool f0 = any_wall(w0), f1 = true, f2 = true, f3 = true;                 // any_wall of them
    pull(y0 - 3, w0, f0, d);
    uint32_t wn = word(y0 - 2);

    // Collision of a node of this lane: densities around it, its word and
    // whether any lane of the row touches a wall.
    auto collide = [&](const D &f, const float(&sf)[2], const float(&p)[2][3], uint32_t w, bool wall, auto put) -> float2 {
        float sax, say, sbx, sby;
        row_stencil(p[0][0], p[0][1], p[0][2], sax, say);
        row_stencil(p[1][0], p[1][1], p[1][2], sbx, sby);
        NodeState n;
        if (BC != BC_IMPROVED && wall) {
            float vn[9], nxs, nys;
#pragma unroll
            for (int i = 1; i < 9; ++i) vn[i] = ((w >> (i - 1)) & 1u) ? 1.f : 0.f;
            grad9(vn, nxs, nys);
            n = node_state<S, BC, true>(I, f, p[0][1], p[1][1], sax, say, sbx, sby, nxs, nys, 0.f, 0.f, 0.f, 0.f);
        } else {
            n = node_state<S, BC, false>(I, f, p[0][1], p[1][1], sax, say, sbx, sby, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f);
        }
        return node_collide<S>(I, f, sf, p[0][1], p[1][1], n, put);
    };
    auto shifted = [](int i, float v) { return CX[i] == 0 ? v : (CX[i] == 1 ? lane_left(v) : lane_right(v)); };

    // Row r; PH says how far the pipeline is filled: 0 A only, 1 + collision of
    // row r - 1, 2 + row r - 2 at t + 1, 3 + collision and store of row r - 3.
    auto row_step = [&](auto ph, int r) {
        constexpr int PH = decltype(ph)::value;
        // ---- A: densities of row r at t
        D dq;
        if constexpr (PH >= 1) park_get<S>(pk, 0, lane, dq);
        const float sq[2] = {sd[0], sd[1]};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            sd[c] = In::sum(d, c);
            p1[c][0] = p1[c][1];
            p1[c][1] = p1[c][2];
            p1[c][2] = rref[c] + sd[c] * (1.f / SC);
        }
        if (f0) {
#pragma unroll
            for (int c = 0; c < 2; ++c) p1[c][2] = (w0 & NW_SOLID) ? 0.f : p1[c][2];
        }
        park_put<S>(pk, 0, lane, d);
        park_fence();
        // ---- B: collision of row r - 1 at t
        D q;
        if constexpr (PH >= 1) {
            const float2 rest = collide(dq, sq, p1, w1, f1, [&](int i, auto v) {
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
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t wc = wn;
        const bool fc = any_wall(wc);
        pull(r + 1, wc, fc, d);
        wn = word(r + 2);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (PH >= 1) {
            // ---- C: row r - 2 at t + 1 takes its directions from above (row
            // r - 1); row r - 1 those from below (row r - 2) and its own
            D nu, er;
#pragma unroll
            for (int i = 0; i < 9; ++i)
#pragma unroll
                for (int c = 0; c < elem_words<S>(i); ++c) {
                    if (CY[i] == -1) ep[c][i] = shifted(i, q[c][i]);
                    else nu[c][i] = shifted(i, CY[i] == 1 ? up[c][i] : q[c][i]);
                }
            if (f1 || f2) {
                // a solid neighbour returns the node's own opposite population
#pragma unroll
                for (int i = 1; i < 9; ++i)
#pragma unroll
                    for (int c = 0; c < elem_words<S>(i); ++c) {
                        if (CY[i] == -1) ep[c][i] = ((w2 >> (OPP[i] - 1)) & 1u) ? up[c][OPP[i]] : ep[c][i];
                        else nu[c][i] = ((w1 >> (OPP[i] - 1)) & 1u) ? q[c][OPP[i]] : nu[c][i];
                    }
            }
#pragma unroll
            for (int i = 0; i < 9; ++i)
#pragma unroll
                for (int c = 0; c < elem_words<S>(i); ++c) {
                    er[c][i] = ep[c][i];
                    if (CY[i] != -1) ep[c][i] = nu[c][i];
                    if (CY[i] == 1) up[c][i] = q[c][i];
                }
            if constexpr (PH >= 2) {
                __builtin_amdgcn_sched_barrier(0);
                float ser[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    ser[c] = In::sum(er, c);
                    p2[c][0] = p2[c][1];
                    p2[c][1] = p2[c][2];
                    p2[c][2] = rref[c] + ser[c] * (1.f / SC);
                }
                if (f2) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) p2[c][2] = (w2 & NW_SOLID) ? 0.f : p2[c][2];
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (PH >= 3) park_get<S>(pk, 1, lane, dq);
                park_put<S>(pk, 1, lane, er);
                park_fence();
                // ---- D: collision of row r - 3 at t + 1
                if constexpr (PH >= 3) {
                    char *o = (char *)fout + row_off<S, 2>(I, r - 3);
                    const bool st = mine && !(w3 & NW_SOLID);
                    const float2 rest = collide(dq, se, p2, w3, f3, [&](int i, auto v) {
                        auto *a = (typename Store<S>::P *)(o + (uint32_t)i * pb + col[1]);
                        if (st) {
                            if constexpr (NT)
                                Store<S>::put2nt(a, v);
                            else
                                Store<S>::put2(a, v);
                        }
                    });
                    if (st) put_rest<S>((typename Store<S>::P *)o, pb, col[1], rest.x, rest.y, NT);
                }
                se[0] = ser[0];
                se[1] = ser[1];
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
    row_step(std::integral_constant<int, 0>{}, y0 - 3);
    row_step(std::integral_constant<int, 0>{}, y0 - 2);
    row_step(std::integral_constant<int, 1>{}, y0 - 1);
    row_step(std::integral_constant<int, 1>{}, y0);
    row_step(std::integral_constant<int, 2>{}, y0 + 1);
    row_step(std::integral_constant<int, 2>{}, y0 + 2);
    for (int r = y0 + 3; r <= y1 + 2; ++r) row_step(std::integral_constant<int, 3>{}, r);
}

}  // namespace mclbm
