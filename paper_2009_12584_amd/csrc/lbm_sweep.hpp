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
//   A  sums the densities of row r at t from its pulled populations and
//      issues the loads of row r + 1,
//   B  collides row r - 1 (its density stencil is now complete),
//   C  completes the populations of row r - 2 at t + 1 from the collided rows
//      r - 3, r - 2, r - 1, sums its densities,
//   D  collides row r - 3 at t + 1 and stores it as time t + 2.
// Neighbours in x come from the next lane (DPP wavefront shifts), neighbours
// in y from registers, so there is no barrier and no halo frame, and a row's
// loads are in flight while the rows before it are computed.  Rows that wait
// (r for B, r - 2 for D) are parked in the wavefront's own LDS: with them in
// registers the FP32 sweep needs 218 VGPRs (2 wavefronts per SIMD), without
// 163 (3; FP16 114, 4).  Rows without a solid in reach of the strip skip the
// bounce-back selects and the wall forces (a wave-uniform branch), and their
// loads need no address arithmetic.
//
// 5600 x 4000 mixture, per step, against the tile step: FP32 640 -> 334 us (a
// pair reads 2.16 GB, a third of it twice because segments and strips overlap,
// and writes 1.64 GB: 5.7 TB/s, where a copy reaches 6.1: bound by memory), FP16
// 382 -> 259 us (1.29 and 1.00 GB, 4.4 TB/s: bound by the issue of the mixed-
// precision operations, which run at half and quarter rate, and by what a
// wavefront's one row of loads in flight covers of memory's latency; neither
// 30 fewer register moves per row of about 490 instructions nor one wavefront
// more per SIMD changed it).  In the caches, where the wait for a row's loads
// shows: 1024 x 1024 periodic 24.7 -> 17.6 us (a us more while the stores sat in
// a branch, so that this wait was for them too; 0.5 more with the loads issued
// after B).
//
// Beyond the caches (streaming stores) the four wavefronts of a workgroup, which
// sweep neighbouring strips, meet once per row: the lines at their borders
// are then read once and written whole.  5600 x 4000: FP32 341 -> 335 us, FP16
// 264 -> 258; 2800 x 2000 single component 39.5 -> 38.1.  In the caches the wait
// costs more than it gives (1024 x 1024 with a disk: 20.4 -> 21.4).  Wavefronts
// with fewer rows have ended, and the barrier counts only those that run.
//
// Every value is computed by the same expressions in the same order as the
// tile step's (node_state, node_collide, grad9), stored populations rounded
// to storage between the two steps, so the result is bit for bit that of two
// tile steps.
#pragma once

#include <type_traits>

#include "lbm_sc1.hpp"
#include "lbm_sweep_plan.hpp"

namespace mclbm {

constexpr int SWEEP_HALO = 3;  // columns either side of a strip's own that only feed them

// Value of the lane to the left (x - 1) and to the right (x + 1).
__device__ __forceinline__ float lane_left(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_right(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}

// Rows that wait for the next row's densities are parked in LDS, so that the
// registers hold one row of loads in flight and one row at work: each lane
// keeps its own words, four (16 bytes) per lane and access.
template <typename M> constexpr int park_groups() { return (M::ROW_WORDS + 3) / 4; }
template <typename M> struct SweepPark {
    float4 at[2][park_groups<M>()][64];  // rows at t and at t + 1
};
template <typename M> __device__ __forceinline__ void park_put(SweepPark<M> &pk, int which, int lane, typename M::D &d) {
#pragma unroll
    for (int g = 0; g < park_groups<M>(); ++g) {
        float4 v = make_float4(M::word(d, 4 * g), M::word(d, 4 * g + 1), 0.f, 0.f);
        if (4 * g + 2 < M::ROW_WORDS) {
            v.z = M::word(d, 4 * g + 2);
            v.w = M::word(d, 4 * g + 3);
            pk.at[which][g][lane] = v;
        } else {
            *(float2 *)&pk.at[which][g][lane] = make_float2(v.x, v.y);
        }
    }
}
template <typename M> __device__ __forceinline__ void park_get(SweepPark<M> &pk, int which, int lane, typename M::D &d) {
#pragma unroll
    for (int g = 0; g < park_groups<M>(); ++g) {
        if (4 * g + 2 < M::ROW_WORDS) {
            const float4 v = pk.at[which][g][lane];
            M::word(d, 4 * g) = v.x;
            M::word(d, 4 * g + 1) = v.y;
            M::word(d, 4 * g + 2) = v.z;
            M::word(d, 4 * g + 3) = v.w;
        } else {
            const float2 v = *(const float2 *)&pk.at[which][g][lane];
            M::word(d, 4 * g) = v.x;
            M::word(d, 4 * g + 1) = v.y;
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

// Wall normal sum w phi c of Eq. 6 from a node word.
__device__ __forceinline__ void wall_normal(uint32_t w, float &nx, float &ny) {
    float v[9];
#pragma unroll
    for (int i = 1; i < 9; ++i) v[i] = ((w >> (i - 1)) & 1u) ? 1.f : 0.f;
    grad9(v, nx, ny);
}

// Buffer access: a uniform descriptor and row offset, a 32-bit offset per lane
// and the slot as an immediate, so that addresses cost no vector arithmetic.
// The hardware drops a store whose lane offset lies beyond the descriptor's
// size, which is how lanes that own no node are left out: every row step then
// issues the same loads and stores, and a wait for a row's loads need not
// wait for the stores that follow them.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t SWEEP_NO_STORE = 0xffff0000u;  // plus any slot still beyond every buffer that sweeps
constexpr int BUF_WORD3 = 0x00020000;             // raw 32-bit data
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, BUF_WORD3);
}
__device__ __forceinline__ float ld32(__amdgpu_buffer_rsrc_t b, uint32_t lane_off, uint32_t row_off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, lane_off, row_off, 0));
}
template <int AUX> __device__ __forceinline__ void st32(float v, __amdgpu_buffer_rsrc_t b, uint32_t lane_off, uint32_t row_off) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), b, lane_off, row_off, AUX);
}

// What a sweep does with the populations of a node.  A row's populations D
// are words: direction i takes WORDS(i) of them, d[0][i], d[1][i]; a row has
// ROW_WORDS (even; word(d, k) is the k-th).  ld issues the loads of direction
// i from a lane's and a row's offset (slot included); sum is the deviation sum
// of a component, field the quantity whose stencil the forces take, collide
// the collision (put(i, v) takes the moving populations, put_rest the rest),
// keep and store what put does with a population of a collided row: into
// words, or to memory.
template <typename S> struct TwoPop {  // the two-component model
    using Storage = S;
    using In = Incoming<S>;
    using D = typename In::D;
    static constexpr int NC = 2, ROW_WORDS = sizeof(S) == 4 ? 18 : 10;
    static constexpr int words(int i) { return sizeof(S) == 4 || i == 0 ? 2 : 1; }
    static __device__ __forceinline__ float &word(D &d, int k) {
        if constexpr (sizeof(S) == 4) return d[k & 1][k >> 1];
        return k < 2 ? d[k][0] : d[0][k - 1];
    }
    static __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t b, int i, uint32_t lane_off, uint32_t row_off, D &d) {
        if constexpr (sizeof(S) == 4) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(b, lane_off, row_off, 0);
            const uint32_t a = v.x, c = v.y;  // scalars first: a vector element's bit cast takes element 0
            d[0][i] = __builtin_bit_cast(float, a);
            d[1][i] = __builtin_bit_cast(float, c);
        } else {
            d[0][i] = ld32(b, lane_off, row_off);
            if (i == 0) d[1][0] = ld32(b, lane_off + 9u * slot_bytes<S, 2>(), row_off);  // slots 0 and 9: FP32 rest populations
        }
    }
    static __device__ __forceinline__ float sum(const D &d, int c) { return In::sum(d, c); }
    static __device__ __forceinline__ float field(const Inst &, float rho) { return rho; }
    static __device__ __forceinline__ void keep(D &q, int i, typename Store<S>::P v) {
        if constexpr (sizeof(S) == 4) {
            q[0][i] = v.x;
            q[1][i] = v.y;
        } else {
            q[0][i] = __builtin_bit_cast(float, v);
        }
    }
    static __device__ __forceinline__ void keep_rest(D &q, float2 r) {
        q[0][0] = r.x;
        q[1][0] = r.y;
    }
    template <int AUX>
    static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t b, int i, typename Store<S>::P v, uint32_t at, uint32_t ro) {
        const uint32_t o = at + (uint32_t)i * slot_bytes<S, 2>();
        if constexpr (sizeof(S) == 4)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, o, ro, AUX);
        else
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), b, o, ro, AUX);
    }
    template <int AUX> static __device__ __forceinline__ void store_rest(__amdgpu_buffer_rsrc_t b, float2 r, uint32_t at, uint32_t ro) {
        if constexpr (sizeof(S) == 4) {
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, r), b, at, ro, AUX);
        } else {
            st32<AUX>(r.x, b, at, ro);
            st32<AUX>(r.y, b, at + 9u * slot_bytes<S, 2>(), ro);
        }
    }
    // p: the field on the rows below, at and above the node; w its word, wall whether the row touches a solid
    template <typename Put, typename Rest>
    static __device__ __forceinline__ void collide(const Inst &I, const D &f, const float (&sf)[2], const float (&p)[2][3], uint32_t w,
                                                   bool wall, Put put, Rest put_rest) {
        float sax, say, sbx, sby;
        row_stencil(p[0][0], p[0][1], p[0][2], sax, say);
        row_stencil(p[1][0], p[1][1], p[1][2], sbx, sby);
        const float ra = p[0][1], rb = p[1][1];
        NodeState n;
        if (wall && I.bc != BC_IMPROVED) {
            float nxs, nys;
            wall_normal(w, nxs, nys);
            if (I.bc == BC_MC)
                n = node_state<S, BC_MC, true>(I, f, ra, rb, sax, say, sbx, sby, nxs, nys, 0.f, 0.f, 0.f, 0.f);
            else
                n = node_state<S, BC_LLKC, true>(I, f, ra, rb, sax, say, sbx, sby, nxs, nys, 0.f, 0.f, 0.f, 0.f);
        } else {
            n = node_state<S, BC_MC, false>(I, f, ra, rb, sax, say, sbx, sby, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f);
        }
        put_rest(node_collide<S>(I, f, sf, ra, rb, n, put));
    }
};

template <typename S> struct OnePop {  // the single-component model
    using Storage = S;
    using D = float[2][9];  // FP16: raw halves, the rest's upper 16 bits in d[0][0] and its lower ones in d[1][0]
    static constexpr int NC = 1, ROW_WORDS = 10;
    static constexpr int words(int i) { return sizeof(S) == 2 && i == 0 ? 2 : 1; }
    static __device__ __forceinline__ float &word(D &d, int k) { return k < 9 ? d[0][k] : d[1][0]; }
    static __device__ __forceinline__ float ld16(__amdgpu_buffer_rsrc_t b, uint32_t lane_off, uint32_t row_off) {
        return __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(b, lane_off, row_off, 0));
    }
    static __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t b, int i, uint32_t lane_off, uint32_t row_off, D &d) {
        if constexpr (sizeof(S) == 4) {
            d[0][i] = ld32(b, lane_off, row_off);
            if (i == 0) d[1][0] = 0.f;  // unused, but a parked row is an even number of words
        } else {
            d[0][i] = ld16(b, lane_off, row_off);
            if (i == 0) d[1][0] = ld16(b, lane_off + 9u * slot_bytes<S, 1>(), row_off);
        }
    }
    static __device__ __forceinline__ uint32_t bits(float v) { return __builtin_bit_cast(uint32_t, v); }
    static __device__ __forceinline__ void values(const D &d, float v[9]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if constexpr (sizeof(S) == 4)
                v[i] = d[0][i];
            else
                v[i] = i == 0 ? __builtin_bit_cast(float, bits(d[0][0]) << 16 | bits(d[1][0]))
                              : __half2float(__builtin_bit_cast(__half, (uint16_t)bits(d[0][i])));
        }
    }
    static __device__ __forceinline__ float sum(const D &d, int) {
        float v[9];
        values(d, v);
        return fsum9(v);
    }
    static __device__ __forceinline__ float field(const Inst &I, float rho) { return psi_of(rho, I.psi0); }
    static __device__ __forceinline__ void keep(D &q, int i, S v) {
        if constexpr (sizeof(S) == 4)
            q[0][i] = v;
        else
            q[0][i] = __builtin_bit_cast(float, (uint32_t)__builtin_bit_cast(uint16_t, v));
    }
    static __device__ __forceinline__ void keep_rest(D &q, float r) {
        q[0][0] = sizeof(S) == 4 ? r : __builtin_bit_cast(float, bits(r) >> 16);
        q[1][0] = sizeof(S) == 4 ? 0.f : __builtin_bit_cast(float, bits(r) & 0xffffu);
    }
    template <int AUX> static __device__ __forceinline__ void st16(uint32_t v, __amdgpu_buffer_rsrc_t b, uint32_t at, uint32_t ro) {
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)v, b, at, ro, AUX);
    }
    template <int AUX> static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t b, int i, S v, uint32_t at, uint32_t ro) {
        const uint32_t o = at + (uint32_t)i * slot_bytes<S, 1>();
        if constexpr (sizeof(S) == 4)
            st32<AUX>(v, b, o, ro);
        else
            st16<AUX>(__builtin_bit_cast(uint16_t, v), b, o, ro);
    }
    template <int AUX> static __device__ __forceinline__ void store_rest(__amdgpu_buffer_rsrc_t b, float r, uint32_t at, uint32_t ro) {
        if constexpr (sizeof(S) == 4) {
            st32<AUX>(r, b, at, ro);
        } else {
            st16<AUX>(bits(r) >> 16, b, at, ro);
            st16<AUX>(bits(r) & 0xffffu, b, at + 9u * slot_bytes<S, 1>(), ro);
        }
    }
    template <typename Put, typename Rest>
    static __device__ __forceinline__ void collide(const Inst &I, const D &f, const float (&sf)[1], const float (&p)[1][3], uint32_t w,
                                                   bool wall, Put put, Rest put_rest) {
#pragma clang fp contract(off)
        float v[9], sx, sy;
        values(f, v);
        row_stencil(p[0][0], p[0][1], p[0][2], sx, sy);
        const float ra = I.rrefA + sf[0] * (1.f / Store1<S>::SC);
        NodeState1 n;
        if (wall) {
            float nxs, nys;
            wall_normal(w, nxs, nys);
            n = I.bc == BC_MC ? node_state1<S, BC_MC, true>(I, v, ra, p[0][1], sx, sy, nxs, nys)
                              : node_state1<S, BC_LLKC, true>(I, v, ra, p[0][1], sx, sy, nxs, nys);
        } else {
            n = node_state1<S, BC_MC, false>(I, v, ra, p[0][1], sx, sy, 0.f, 0.f);
        }
        put_rest(node_collide1<S>(I, v, sf[0], ra, n, put));
    }
};

// Two steps of instance I over the task's columns and rows, from fin to fout.
// The rule is the instance's: it only matters in rows next to a wall.  In the
// improved scheme the adhesion is left out and the nodes that it reaches
// within the two steps (NW_EDGE) are not stored: their virtual densities average
// over 5 x 5 nodes, three rows ahead of the sweep, so edge tiles advance them
// (pair_tile).  DIR is the direction of the sweep, 1 up, -1 down; "row r + 1"
// is the next row in that direction.
template <typename M, bool NT, int DIR>
__device__ __forceinline__ void sweep_pair_dir(const Inst &I, const void *fin, void *fout, const SweepTask &task, SweepPark<M> &pk) {
#pragma clang fp contract(off)
    using S = typename M::Storage;
    using D = typename M::D;
    constexpr int NC = M::NC;
    constexpr float SC = Store<S>::SC;
    constexpr uint32_t pb = slot_bytes<S, NC>();
    constexpr int AUX = NT ? 2 : 0;  // streaming stores
    const int x0 = task.x0w & 0xfffff, width = (task.x0w >> 20) & 127, y0 = task.y0, y1 = task.y1;
    auto row_at = [&](int k) -> int { return DIR > 0 ? y0 + k : y1 - 1 - k; };  // the k-th row of the segment
    const int lane = threadIdx.x & 63;
    const int gx = x0 - SWEEP_HALO + lane;
    const bool perx = I.periodic & 1u, pery = I.periodic & 2u;
    const uint32_t off_x = perx || (unsigned)gx < (unsigned)I.nx ? 0u : (uint32_t)NW_SOLID;
    const uint32_t wcol = 2u * (uint32_t)keep_in(gx, I.nx, perx, false);
    uint32_t col[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) col[j] = col_off<S, NC>(keep_in(gx - 1 + j, I.nx, perx, false));
    const bool mine = lane >= SWEEP_HALO && lane < SWEEP_HALO + width;
    const float rref[2] = {I.rrefA, I.rrefB};
    const uint32_t rb = row_bytes<S, NC>(I);
    const __amdgpu_buffer_rsrc_t bin = buffer_of(fin, (uint32_t)I.ny * rb), bout = buffer_of(fout, (uint32_t)I.ny * rb),
                                 bw = buffer_of(I.node, (uint32_t)(2 * I.plane));

    // Row y inside the lattice (wrapped, or clamped at a closed border), its
    // node words as stored, and what is added to them: solid beyond a closed
    // border.  (Added where the word is used; at the load it would wait.)
    auto row_in = [&](int y) -> int {
        const int lo = pery ? y + I.ny : 0, hi = pery ? y - I.ny : I.ny - 1;
        return y < 0 ? lo : (y >= I.ny ? hi : y);
    };
    auto word = [&](int yin) -> uint16_t {
        return __builtin_amdgcn_raw_buffer_load_b16(bw, wcol, 2u * (uint32_t)yin * (uint32_t)I.pitch, 0);
    };
    auto off = [&](int y) -> uint32_t { return off_x | (pery || (unsigned)y < (unsigned)I.ny ? 0u : (uint32_t)NW_SOLID); };
    auto any_wall = [&](uint32_t w) { return __any((w & (NW_SOLID | 0xffu)) != 0u) != 0; };
    // pull from the rows at byte offsets row[] (before, at, after); solid lanes read values that are not used
    auto pull = [&](const uint32_t row[3], uint32_t w, bool wall, D &d) {
        if (!wall) {
#pragma unroll
            for (int i = 0; i < 9; ++i) M::ld(bin, i, col[1 - CX[i]] + (uint32_t)i * pb, row[1 - DIR * CY[i]], d);
            asm volatile("; open row");  // the two kinds of row keep their own loads
        } else {
            Around a;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                a.row[j] = row[1 + DIR * (j - 1)];
                a.col[j] = col[j];
            }
            const uint32_t own = row[1] + col[1];
            M::ld(bin, 0, own, 0, d);
#pragma unroll
            for (int i = 1; i < 9; ++i) M::ld(bin, i, pull_off(i, pb, a, own, w), 0, d);
            asm volatile("; walled row");
        }
    };

    D d;                  // populations at t of row r, then of r + 1 in flight
    D ep;                 // populations at t + 1 of row r - 1, directions of rows r - 2 and r - 1
    D up;                 // collided row r - 2: the three directions that go to row r - 1
    float sd[NC] = {};     // deviation sums at t of row r - 1
    float se[NC] = {};     // and at t + 1 of row r - 3
    float p1[NC][3] = {};  // field at t of rows r - 2, r - 1, r
    float p2[NC][3] = {};  // field at t + 1 of rows r - 4, r - 3, r - 2
#pragma unroll
    for (int i = 0; i < 9; ++i)
#pragma unroll
        for (int c = 0; c < M::words(i); ++c) ep[c][i] = up[c][i] = 0.f;
    uint32_t row[3];  // offsets of rows r - 1, r, r + 1
#pragma unroll
    for (int j = 0; j < 3; ++j) row[j] = (uint32_t)row_in(row_at(j - 4)) * rb;
    // words of rows r, r - 1, r - 2, r - 3, and any_wall of them
    uint32_t w0 = word(row_in(row_at(-3))) | off(row_at(-3)), w1 = NW_SOLID, w2 = NW_SOLID, w3 = NW_SOLID;
    bool f0 = any_wall(w0), f1 = true, f2 = true, f3 = true;
    uint16_t wn = word(row_in(row_at(-2)));
    pull(row, w0, f0, d);

    auto shifted = [](int i, float v) { return CX[i] == 0 ? v : (CX[i] == 1 ? lane_left(v) : lane_right(v)); };

    // three rows of a field, from below to above
    auto ordered = [](const float (&p)[NC][3], float (&o)[NC][3]) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 3; ++j) o[c][j] = p[c][1 + DIR * (j - 1)];
    };
    // Row r, the k-th of the segment; PH says how far the pipeline is filled:
    // 0 A only, 1 + collision of row r - 1, 2 + row r - 2 at t + 1, 3 + collision
    // and store of row r - 3.
    auto row_step = [&](auto ph, int k) {
        constexpr int PH = decltype(ph)::value;
        if constexpr (NT) __builtin_amdgcn_s_barrier();  // neighbouring strips stay in step (above)
        // ---- A: densities of row r at t
        D dq;
        if constexpr (PH >= 1) park_get<M>(pk, 0, lane, dq);
        float sq[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) sq[c] = sd[c];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            sd[c] = M::sum(d, c);
            p1[c][0] = p1[c][1];
            p1[c][1] = p1[c][2];
            p1[c][2] = M::field(I, rref[c] + sd[c] * (1.f / SC));
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) p1[c][2] = (w0 & NW_SOLID) ? 0.f : p1[c][2];
        park_put<M>(pk, 0, lane, d);
        park_fence();
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t wc = (uint32_t)wn | off(row_at(k + 1));
        const bool fc = any_wall(wc);
        const int y2 = row_in(row_at(k + 2));
        row[0] = row[1];
        row[1] = row[2];
        row[2] = (uint32_t)y2 * rb;
        wn = word(y2);
        pull(row, wc, fc, d);
        __builtin_amdgcn_sched_barrier(0);
        // ---- B: collision of row r - 1 at t
        D q;
        float po[NC][3];
        ordered(p1, po);
        if constexpr (PH >= 1)
            M::collide(I, dq, sq, po, w1, f1, [&](int i, auto v) { M::keep(q, i, v); }, [&](auto v) { M::keep_rest(q, v); });
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (PH >= 1) {
            // ---- C: row r - 2 at t + 1 takes its directions from row r - 1; row
            // r - 1 those from row r - 2 and its own
            D nu, er;
#pragma unroll
            for (int i = 0; i < 9; ++i)
#pragma unroll
                for (int c = 0; c < M::words(i); ++c) {
                    if (CY[i] == -DIR) ep[c][i] = shifted(i, q[c][i]);
                    else nu[c][i] = shifted(i, CY[i] == DIR ? up[c][i] : q[c][i]);
                }
            if (f1 || f2) {
                // a solid neighbour returns the node's own opposite population
#pragma unroll
                for (int i = 1; i < 9; ++i)
#pragma unroll
                    for (int c = 0; c < M::words(i); ++c) {
                        if (CY[i] == -DIR) ep[c][i] = ((w2 >> (OPP[i] - 1)) & 1u) ? up[c][OPP[i]] : ep[c][i];
                        else nu[c][i] = ((w1 >> (OPP[i] - 1)) & 1u) ? q[c][OPP[i]] : nu[c][i];
                    }
            }
#pragma unroll
            for (int i = 0; i < 9; ++i)
#pragma unroll
                for (int c = 0; c < M::words(i); ++c) {
                    er[c][i] = ep[c][i];
                    if (CY[i] != -DIR) ep[c][i] = nu[c][i];
                    if (CY[i] == DIR) up[c][i] = q[c][i];
                }
            if constexpr (PH >= 2) {
                __builtin_amdgcn_sched_barrier(0);
                float ser[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    ser[c] = M::sum(er, c);
                    p2[c][0] = p2[c][1];
                    p2[c][1] = p2[c][2];
                    p2[c][2] = M::field(I, rref[c] + ser[c] * (1.f / SC));
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) p2[c][2] = (w2 & NW_SOLID) ? 0.f : p2[c][2];
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (PH >= 3) park_get<M>(pk, 1, lane, dq);
                park_put<M>(pk, 1, lane, er);
                park_fence();
                // ---- D: collision of row r - 3 at t + 1
                if constexpr (PH >= 3) {
                    ordered(p2, po);
                    const uint32_t ro = (uint32_t)row_at(k - 3) * rb;
                    const uint32_t at = mine && !(w3 & (NW_SOLID | NW_EDGE)) ? col[1] : SWEEP_NO_STORE;
                    M::collide(
                        I, dq, se, po, w3, f3, [&](int i, auto v) { M::template store<AUX>(bout, i, v, at, ro); },
                        [&](auto v) { M::template store_rest<AUX>(bout, v, at, ro); });
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) se[c] = ser[c];
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
    row_step(std::integral_constant<int, 0>{}, -3);
    row_step(std::integral_constant<int, 0>{}, -2);
    row_step(std::integral_constant<int, 1>{}, -1);
    row_step(std::integral_constant<int, 1>{}, 0);
    row_step(std::integral_constant<int, 2>{}, 1);
    row_step(std::integral_constant<int, 2>{}, 2);
    for (int k = 3, e = y1 - y0 + 2; k <= e; ++k) row_step(std::integral_constant<int, 3>{}, k);
}
// The segments of a strip are swept in turn upwards and downwards, so that the
// rows which two of them both read are read at about the same time.  In FP32
// (5600 x 4000 mixture) that is 4% fewer reads from the caches' memory side and
// 347 -> 341 us per step; FP16 gained nothing there (264 us both) and its
// batches lost to the second copy of the code (64 instances of 240 x 160 to 400 x
// 320: 63.9 -> 66 us), so FP16 sweeps upwards only.
template <typename M, bool NT>
__device__ __forceinline__ void sweep_pair(const Inst &I, const void *fin, void *fout, const SweepTask &task, SweepPark<M> &pk) {
    if (sizeof(typename M::Storage) == 4 && (task.x0w & SWEEP_DOWN))
        sweep_pair_dir<M, NT, -1>(I, fin, fout, task, pk);
    else
        sweep_pair_dir<M, NT, 1>(I, fin, fout, task, pk);
}

// Two steps of one small tile, held in LDS.  Each step widens what a node
// depends on: by 2 (the density of a neighbour, one more for its pull), or in
// the improved scheme next to a wall (DEEP) by 4 (the virtual density of a
// neighbouring solid averages densities up to three nodes away).  So the tile
// computes the densities at t with a halo HD, collides with a halo HC into
// LDS, takes the densities at t + 1 with a halo H2 from there and stores its
// own nodes.  Beyond the first ring of either step only densities within reach
// of an interface solid are needed.
template <int W_, int H_, int T_, bool DEEP_> struct PairTile {
    static constexpr int W = W_, H = H_, T = T_;  // nodes, threads
    static constexpr bool DEEP = DEEP_;
    static constexpr int HC = DEEP ? 4 : 2, HD = DEEP ? 7 : 3, H2 = DEEP ? 3 : 1, HV = DEEP ? 5 : 0;
    template <int R> static constexpr int w() { return W + 2 * R; }
    template <int R> static constexpr int n() { return w<R>() * (H + 2 * R); }
    // index of position (x, y) in an array with halo R, and back
    template <int R> static __device__ __forceinline__ int at(int x, int y) { return (y + R) * w<R>() + x + R; }
    template <int R> static __device__ __forceinline__ void pos(int k, int &x, int &y) {
        x = k % w<R>() - R;
        y = k / w<R>() - R;
    }
    // position k of the frame between halos RI and RO: the rows above, the rows below, the columns left and right
    template <int RI, int RO> static __device__ __forceinline__ void frame(int k, int &x, int &y) {
        constexpr int F = RO - RI, FW = w<RO>(), B = F * FW;
        if (k < 2 * B) {
            const int r = k / FW;
            x = k % FW - RO;
            y = r < F ? r - RO : H + RI + r - F;
        } else {
            const int c = (k - 2 * B) % (2 * F);
            y = (k - 2 * B) / (2 * F) - RI;
            x = c < F ? c - RO : W + RI + c - F;
        }
    }
    static __device__ __forceinline__ int ring(int x, int y) { return max(max(-x, x - (W - 1)), max(-y, y - (H - 1))); }
};
template <typename S, typename G> struct PairTileSmem {
    float rho[2][G::template n<G::HD>()];               // densities, at t and then at t + 1
    float rt[2][G::DEEP ? G::template n<G::HV>() : 1];  // virtual densities of the interface solids, likewise
    uint16_t w[G::template n<G::HD>()];                 // node words
    typename Store<S>::P mv[8][G::template n<G::HC>()]; // populations after the first collision
    float2 rest[G::template n<G::HC>()];
};

// The edge nodes of a sweep (improved scheme): a small tile keeps the halo's
// waste to the wall.  16 x 14 is the most whose LDS (51 KB in FP32) leaves room
// for three workgroups per CU.
constexpr int EDGE_W = 16, EDGE_H = 14;
using EdgeTile = PairTile<EDGE_W, EDGE_H, 64 * SWEEP_WAVES, true>;

// Two steps of the tile at (tx0, ty0) of instance I, from fin to fout; stores
// the fluid nodes whose word has the bits `need`.
template <typename G, typename S, bool NT>
__device__ __forceinline__ void pair_tile(const Inst &I, const void *fin, void *fout, int tx0, int ty0, uint32_t need,
                                          PairTileSmem<S, G> &sm) {
#pragma clang fp contract(off)
    using In = Incoming<S>;
    using D = typename In::D;
    using P = typename Store<S>::P;
    constexpr float SC = Store<S>::SC;
    constexpr uint32_t pb = slot_bytes<S, 2>();
    constexpr int T = G::T, HC = G::HC, HD = G::HD, H2 = G::H2, HV = G::HV, NC = G::template n<HC>(), ND = G::template n<HD>(),
                  NO = G::W * G::H, WD = G::template w<HD>(), WC = G::template w<HC>(), WV = G::template w<HV>(),
                  NS = (NC + T - 1) / T;
    const int tid = threadIdx.x;
    const float rref[2] = {I.rrefA, I.rrefB}, chi[2] = {I.chiA, I.chiB};

    for (int k = tid; k < ND; k += T) {
        int x, y;
        G::template pos<HD>(k, x, y);
        sm.w[k] = (uint16_t)node_word(I, tx0 + x, ty0 + y);
    }
    __syncthreads();

    // ---- densities at t; the populations of the inner nodes stay in registers
    D d[NS];
    float sd[NS][2];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int k = tid + s * T;
        int x, y;
        G::template pos<HC>(k, x, y);
        const uint32_t w = k < NC ? sm.w[G::template at<HD>(x, y)] : (uint32_t)NW_SOLID;
        if (!(w & NW_SOLID))
            In::pull((const P *)fin, pb, around<S>(I, tx0 + x, ty0 + y, true), w, d[s]);
        else
#pragma unroll
            for (int i = 0; i < 9; ++i) d[s][0][i] = d[s][1][i] = 0.f;
    }
#pragma unroll
    for (int s = 0; s < (ND - NC + T - 1) / T; ++s) {
        int x, y;
        G::template frame<HC, HD>(tid + s * T, x, y);
        if (tid + s * T >= ND - NC) break;
        const int ring = G::ring(x, y), k = G::template at<HD>(x, y);
        const uint32_t w = sm.w[k];
        float r[2] = {0.f, 0.f};
        if (!(w & NW_SOLID) && (ring == HC + 1 || (w & NW_NEAR))) {
            D f;
            In::pull((const P *)fin, pb, around<S>(I, tx0 + x, ty0 + y, true), w, f);
#pragma unroll
            for (int c = 0; c < 2; ++c) r[c] = rref[c] + In::sum(f, c) * (1.f / SC);
        }
        sm.rho[0][k] = r[0];
        sm.rho[1][k] = r[1];
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int k = tid + s * T;
        if (k >= NC) break;
        int x, y;
        G::template pos<HC>(k, x, y);
        const int q = G::template at<HD>(x, y);
        const bool solid = sm.w[q] & NW_SOLID;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            sd[s][c] = In::sum(d[s], c);
            sm.rho[c][q] = solid ? 0.f : rref[c] + sd[s][c] * (1.f / SC);
        }
    }
    __syncthreads();

    // Eq. 7 on the interface solids of the tile with halo R
    auto virtual_densities = [&](auto halo) {
        constexpr int R = decltype(halo)::value;
        for (int k = tid; k < G::template n<R>(); k += T) {
            int x, y;
            G::template pos<R>(k, x, y);
            const int q = G::template at<HD>(x, y), v = G::template at<HV>(x, y);
            float r[2] = {0.f, 0.f};
            if (sm.w[q] & NW_IFACE) {
                const int gx = keep_in(tx0 + x, I.nx, I.periodic & 1u, false), gy = keep_in(ty0 + y, I.ny, I.periodic & 2u, false);
                const float rden = I.den7[__umul24((uint32_t)gy, (uint32_t)I.pitch) + (uint32_t)gx];
#pragma unroll
                for (int c = 0; c < 2; ++c) r[c] = chi[c] * eq7_sum<WD>(&sm.rho[c][q], I.avg) * rden;
            }
            sm.rt[0][v] = r[0];
            sm.rt[1][v] = r[1];
        }
    };
    // collision of the node at (x, y) with word w
    auto collide = [&](int x, int y, uint32_t w, const D &f, const float(&sf)[2], auto put) -> float2 {
        const int q = G::template at<HD>(x, y);
        float g[4][2];  // stencil sums of rho A, B and rho~ A, B
        float nxs = 0.f, nys = 0.f;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            float a[9];
#pragma unroll
            for (int i = 1; i < 9; ++i) a[i] = sm.rho[c][q + CY[i] * WD + CX[i]];
            grad9(a, g[c][0], g[c][1]);
            if constexpr (G::DEEP) {
                const int v = G::template at<HV>(x, y);
#pragma unroll
                for (int i = 1; i < 9; ++i) a[i] = sm.rt[c][v + CY[i] * WV + CX[i]];
                grad9(a, g[2 + c][0], g[2 + c][1]);
            } else {
                g[2 + c][0] = g[2 + c][1] = 0.f;
            }
        }
        const float ra = sm.rho[0][q], rb = sm.rho[1][q];
        auto state = [&](auto bc, auto wall) {
            return node_state<S, decltype(bc)::value, decltype(wall)::value>(I, f, ra, rb, g[0][0], g[0][1], g[1][0], g[1][1], nxs,
                                                                             nys, g[2][0], g[2][1], g[3][0], g[3][1]);
        };
        using std::integral_constant;
        NodeState n;
        if constexpr (G::DEEP) {
            n = state(integral_constant<int, BC_IMPROVED>{}, std::true_type{});
        } else if (I.bc == BC_IMPROVED) {  // no wall in reach
            n = state(integral_constant<int, BC_MC>{}, std::false_type{});
        } else {
            float vn[9];
#pragma unroll
            for (int i = 1; i < 9; ++i) vn[i] = ((w >> (i - 1)) & 1u) ? 1.f : 0.f;
            grad9(vn, nxs, nys);
            n = I.bc == BC_MC ? state(integral_constant<int, BC_MC>{}, std::true_type{})
                              : state(integral_constant<int, BC_LLKC>{}, std::true_type{});
        }
        return node_collide<S>(I, f, sf, ra, rb, n, put);
    };
    if constexpr (G::DEEP) {
        virtual_densities(std::integral_constant<int, HV>{});
        __syncthreads();
    }

    // ---- first collision
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int k = tid + s * T;
        if (k >= NC) break;
        int x, y;
        G::template pos<HC>(k, x, y);
        const uint32_t w = sm.w[G::template at<HD>(x, y)];
        if (w & NW_SOLID) continue;
        sm.rest[k] = collide(x, y, w, d[s], sd[s], [&](int i, auto v) { sm.mv[i - 1][k] = v; });
    }
    __syncthreads();

    // ---- densities at t + 1
    auto pull2 = [&](int x, int y, uint32_t w, D &f) {
        const int k = G::template at<HC>(x, y);
        const float2 r = sm.rest[k];
        f[0][0] = r.x;
        f[1][0] = r.y;
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const bool bb = (w >> (OPP[i] - 1)) & 1u;
            const P v = bb ? sm.mv[OPP[i] - 1][k] : sm.mv[i - 1][k - CY[i] * WC - CX[i]];
            if constexpr (sizeof(S) == 4) {
                f[0][i] = v.x;
                f[1][i] = v.y;
            } else {
                f[0][i] = __builtin_bit_cast(float, v);
            }
        }
    };
    constexpr int NF = G::template n<H2>() - NO;
    static_assert(NF <= T && NO <= T, "one position per thread");
    constexpr int F0 = NO + NF <= T ? NO : 0;  // first thread of the frame: the threads after the tile's own where they suffice
    const int ex = tid % G::W, ey = tid / G::W;
    const uint32_t we = tid < NO ? sm.w[G::template at<HD>(ex, ey)] : (uint32_t)NW_SOLID;
    D e;
    float se[2] = {0.f, 0.f};
    if (!(we & NW_SOLID)) {
        pull2(ex, ey, we, e);
        se[0] = In::sum(e, 0);
        se[1] = In::sum(e, 1);
    }
    if (tid < NO) {
        const int q = G::template at<HD>(ex, ey);
        const bool solid = we & NW_SOLID;
#pragma unroll
        for (int c = 0; c < 2; ++c) sm.rho[c][q] = solid ? 0.f : rref[c] + se[c] * (1.f / SC);
    }
    if (tid >= F0 && tid < F0 + NF) {
        int x, y;
        G::template frame<0, H2>(tid - F0, x, y);
        const int ring = G::ring(x, y), q = G::template at<HD>(x, y);
        const uint32_t w = sm.w[q];
        float r[2] = {0.f, 0.f};
        if (!(w & NW_SOLID) && (ring == 1 || (w & NW_NEAR))) {
            D f;
            pull2(x, y, w, f);
#pragma unroll
            for (int c = 0; c < 2; ++c) r[c] = rref[c] + In::sum(f, c) * (1.f / SC);
        }
        sm.rho[0][q] = r[0];
        sm.rho[1][q] = r[1];
    }
    __syncthreads();
    if constexpr (G::DEEP) {
        virtual_densities(std::integral_constant<int, 1>{});
        __syncthreads();
    }

    // ---- second collision
    if (!(we & NW_SOLID) && (we & need) == need && tx0 + ex < I.nx && ty0 + ey < I.ny) {
        const uint32_t own = row_off<S, 2>(I, ty0 + ey) + col_off<S, 2>(tx0 + ex);
        const float2 rest = collide(ex, ey, we, e, se, [&](int i, auto v) {
            if constexpr (NT)
                Store<S>::put2nt(at((P *)fout, own + (uint32_t)i * pb), v);
            else
                Store<S>::put2(at((P *)fout, own + (uint32_t)i * pb), v);
        });
        put_rest<S>((P *)fout, pb, own, rest.x, rest.y, NT);
    }
}

// LDS of a workgroup: four wavefronts' parks, or an edge tile.
template <typename S> union SweepSmem {
    SweepPark<TwoPop<S>> park[SWEEP_WAVES];
    PairTileSmem<S, EdgeTile> edge;
};
template <typename S> constexpr int sweep_occupancy() { return sizeof(S) == 4 ? 3 : 4; }  // wavefronts per SIMD
// Blocks that sweep n segments, a multiple of 8 so that the edge tiles start on XCD 0 too.
MCLBM_HD int sweep_blocks(int n) { return ((n + SWEEP_WAVES - 1) / SWEEP_WAVES + 7) & ~7; }

// Small grids, where a sweep leaves most of the chip idle: every fluid node in
// pair tiles of 14 x 14, one thread per node with its halo of 4 (22 x 22), so that
// a tile's time is one chain of latencies (launch, words, pulls, and per step
// densities, Eq. 7, collision, each behind a barrier).  Listed tiles with
// TILE_DEEP reach a wall in the improved scheme.  Per step against the tile
// step, FP32 (FP16): 64 x 64 channel 4.8 -> 3.8 us (8.3 -> 3.9), 512 x 256
// improved plane 7.3 -> 5.9 (13.1 -> 5.9); the plain launches of the 64 x 64 one
// 5.9 -> 3.8, half as many.  Up to SMALL_MAX_TILES, three workgroups per CU:
// with 841 tiles (400 x 400 channel) it takes 7.7 us, tiles 7.3, a sweep 7.2.
// In FP32 up to SMALL_ROUND_TILES, two per CU, where a tile step needs no more
// than one workgroup per CU: 64 x 2000 (250 tiles, 715 pair tiles) improved box
// 8.1 us by tile steps, 8.7 in pairs, Martys-Chen channels 12 wide 5.1 / 5.5.
constexpr int SMALL_MAX_TILES = 768, SMALL_ROUND_TILES = 512;
constexpr int SMALL_W = 14, SMALL_H = 14, SMALL_T = 512;
constexpr int TILE_DEEP = (int)(1u << 31);
using SmallDeep = PairTile<SMALL_W, SMALL_H, SMALL_T, true>;
using SmallFlat = PairTile<SMALL_W, SMALL_H, SMALL_T, false>;
template <typename S> union SmallSmem {
    PairTileSmem<S, SmallDeep> deep;
    PairTileSmem<S, SmallFlat> flat;
};

}  // namespace mclbm
