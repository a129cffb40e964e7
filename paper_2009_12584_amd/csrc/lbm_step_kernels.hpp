// Step kernels of one simulation (one-lane, two-lane and single-component
// tile bodies) and their dispatch over the template parameters, instantiated
// once per storage type in lbm_step_f32.hip and lbm_step_f16.hip.
#pragma once

#include "lbm_common.hpp"
#include "lbm_sweep.hpp"

namespace mclbm {

// Tile of block b: a step launch covers the listed tiles (those that hold a
// fluid node, so that every XCD's band of blocks gets an equal share of the
// work), whose coordinates the list holds packed; a fields pass covers every
// logical tile.
template <int MODE> __device__ __forceinline__ void block_tile(const Inst &I, int &tx, int &ty) {
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    if (MODE == MODE_STEP && I.steps_tiles)
        unpack_tile(I.steps_tiles[b], tx, ty);
    else
        tile_coords(b, I.tiles_x, I.tiles_y, I.tg, tx, ty);
}

template <typename S, int TY, int BC, int MODE, bool DIAG, bool NT>
__global__ __launch_bounds__(threads_for(TY)) void k_step(Inst I, int parity, Fields fo, double *partials) {
    __shared__ Smem<TY> sm;
    int tx, ty;
    block_tile<MODE>(I, tx, ty);
    DiagAcc acc;
    process_tile<S, TY, BC, MODE, DIAG, NT>(I, tx, ty, parity, sm, acc, fo);
    if (DIAG) diag_partial<TY>(sm, acc, partials, blockIdx.x);
}

// The same step with two lanes per node (lbm_pair.hpp); bit-identical results.
template <typename S, int TY, int BC, int MODE, bool DIAG, bool NT>
__global__ __launch_bounds__(ls_threads(TY)) void k_step_ls(Inst I, int parity, Fields fo, double *partials) {
    __shared__ SmemLS<TY> sm;
    int tx, ty;
    block_tile<MODE>(I, tx, ty);
    DiagAcc acc;
    process_tile_ls<S, TY, BC, MODE, DIAG, NT>(I, tx, ty, parity, sm, acc, fo);
    if (DIAG) diag_partial_ls<TY>(sm, acc, partials, blockIdx.x);
}

template <typename S, int TY, int BC, int MODE, bool DIAG, bool NT>
__global__ __launch_bounds__(threads_for(TY)) void k_step_sc1(Inst I, int parity, Fields fo, double *partials) {
    __shared__ Smem<TY> sm;
    int tx, ty;
    block_tile<MODE>(I, tx, ty);
    DiagAcc acc;
    process_tile_sc1<S, TY, BC, MODE, DIAG, NT>(I, tx, ty, parity, sm, acc, fo);
    if (DIAG) diag_partial<TY>(sm, acc, partials, blockIdx.x);
}

// Two steps of one simulation: the first blocks sweep its strip segments, one
// wavefront each (the blocks of an XCD take neighbouring segments, whose halo
// columns then meet in its L2); the others advance the edge tiles of the
// improved scheme.  In one launch, so that the edge tiles, which wait through a
// chain of barriers, hide behind the sweep.
template <typename S, bool NT>
__global__ __launch_bounds__(64 * SWEEP_WAVES, sweep_occupancy<S>()) void k_sweep(Inst I, const SweepTask *__restrict__ tasks,
                                                                                  int n, const int2 *__restrict__ edge,
                                                                                  int nedge, int parity) {
    __shared__ SweepSmem<S> u;
    const int groups = sweep_blocks(n);
    if ((int)blockIdx.x >= groups) {
        int tx, ty;
        unpack_tile(edge[xcd_tile(blockIdx.x - groups, nedge)].y, tx, ty);
        pair_tile<EdgeTile, S, NT>(I, I.buf[parity], I.buf[parity ^ 1], tx * EDGE_W, ty * EDGE_H, NW_EDGE, u.edge);
        return;
    }
    const int t = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, groups) * SWEEP_WAVES + (int)(threadIdx.x >> 6));
    if (t >= n) return;
    const SweepTask k = tasks[t];
    sweep_pair<TwoPop<S>, NT>(I, I.buf[parity], I.buf[parity ^ 1], k, u.park[threadIdx.x >> 6]);
}

// Two steps of one single-component simulation (no edge tiles: its rules reach
// one node).
template <typename S, bool NT>
__global__ __launch_bounds__(64 * SWEEP_WAVES, 4) void k_sweep_sc1(Inst I, const SweepTask *__restrict__ tasks, int n, int parity) {
    __shared__ SweepPark<OnePop<S>> park[SWEEP_WAVES];
    const int t = __builtin_amdgcn_readfirstlane(xcd_tile(blockIdx.x, gridDim.x) * SWEEP_WAVES + (int)(threadIdx.x >> 6));
    if (t >= n) return;
    const SweepTask k = tasks[t];
    sweep_pair<OnePop<S>, NT>(I, I.buf[parity], I.buf[parity ^ 1], k, park[threadIdx.x >> 6]);
}

// Two steps of one small simulation, a listed pair tile per block.
template <typename S>
__global__ __launch_bounds__(SMALL_T, 6) void k_pair_tiles(Inst I, const int *__restrict__ tiles, int parity) {
    __shared__ SmallSmem<S> u;
    const int t = tiles[xcd_tile(blockIdx.x, gridDim.x)];
    int tx, ty;
    unpack_tile(t & ~TILE_DEEP, tx, ty);
    if (t & TILE_DEEP)
        pair_tile<SmallDeep, S, false>(I, I.buf[parity], I.buf[parity ^ 1], tx * SMALL_W, ty * SMALL_H, 0u, u.deep);
    else
        pair_tile<SmallFlat, S, false>(I, I.buf[parity], I.buf[parity ^ 1], tx * SMALL_W, ty * SMALL_H, 0u, u.flat);
}

template <typename S>
inline void launch_sweep_storage(const Launch &L, hipStream_t s, const Inst &I, const SweepPlan &W, int parity) {
    if (W.nsmall) {
        hipLaunchKernelGGL((k_pair_tiles<S>), dim3((unsigned)W.nsmall), dim3(SMALL_T), 0, s, I, W.small, parity);
        return;
    }
    const dim3 g((unsigned)(sweep_blocks(W.n) + W.nedge)), b(64 * SWEEP_WAVES);
    if (L.model == LBM_MODEL_SC1) {
        if (L.nt)
            hipLaunchKernelGGL((k_sweep_sc1<S, true>), g, b, 0, s, I, W.tasks, W.n, parity);
        else
            hipLaunchKernelGGL((k_sweep_sc1<S, false>), g, b, 0, s, I, W.tasks, W.n, parity);
        return;
    }
    if (L.nt)
        hipLaunchKernelGGL((k_sweep<S, true>), g, b, 0, s, I, W.tasks, W.n, W.edge, W.nedge, parity);
    else
        hipLaunchKernelGGL((k_sweep<S, false>), g, b, 0, s, I, W.tasks, W.n, W.edge, W.nedge, parity);
}

// A step of kernel family K at (storage, tile rows, rule): fields passes
// (no population stores), steps with or without the fused diagnostics, with
// streaming or plain stores.
#define MCLBM_DISPATCH(K, B)                                                                          \
    do {                                                                                              \
        if (L.mode == MODE_FIELDS)                                                                    \
            hipLaunchKernelGGL((K<S, TY, BC, MODE_FIELDS, true, false>), g, B, 0, s, I, parity, fo, partials); \
        else if (L.diag && L.nt)                                                                      \
            hipLaunchKernelGGL((K<S, TY, BC, MODE_STEP, true, true>), g, B, 0, s, I, parity, fo, partials); \
        else if (L.diag)                                                                              \
            hipLaunchKernelGGL((K<S, TY, BC, MODE_STEP, true, false>), g, B, 0, s, I, parity, fo, partials); \
        else if (L.nt)                                                                                \
            hipLaunchKernelGGL((K<S, TY, BC, MODE_STEP, false, true>), g, B, 0, s, I, parity, fo, partials); \
        else                                                                                          \
            hipLaunchKernelGGL((K<S, TY, BC, MODE_STEP, false, false>), g, B, 0, s, I, parity, fo, partials); \
    } while (0)

template <typename S, int TY, int BC>
inline void launch3(const Launch &L, dim3 g, hipStream_t s, const Inst &I, int parity, const Fields &fo,
                    double *partials) {
    if (L.model == LBM_MODEL_SC1) {
        if constexpr (BC == BC_MC || BC == BC_LLKC) MCLBM_DISPATCH(k_step_sc1, dim3(threads_for(TY)));
        return;
    }
    if (L.lanes == 2)
        MCLBM_DISPATCH(k_step_ls, dim3(ls_threads(TY)));
    else
        MCLBM_DISPATCH(k_step, dim3(threads_for(TY)));
}

#undef MCLBM_DISPATCH

template <typename S, int TY>
inline void launch2(const Launch &L, dim3 g, hipStream_t s, const Inst &I, int parity, const Fields &fo,
                    double *partials) {
    switch (L.bc) {
    case BC_MC: launch3<S, TY, BC_MC>(L, g, s, I, parity, fo, partials); break;
    case BC_LLKC: launch3<S, TY, BC_LLKC>(L, g, s, I, parity, fo, partials); break;
    default: launch3<S, TY, BC_IMPROVED>(L, g, s, I, parity, fo, partials); break;
    }
}

template <typename S>
inline void launch_storage(const Launch &L, dim3 g, hipStream_t s, const Inst &I, int parity, const Fields &fo,
                    double *partials) {
    switch (L.ty) {
    case 4: launch2<S, 4>(L, g, s, I, parity, fo, partials); break;
    case 16: launch2<S, 16>(L, g, s, I, parity, fo, partials); break;
    case 32: launch2<S, 32>(L, g, s, I, parity, fo, partials); break;
    default: launch2<S, 8>(L, g, s, I, parity, fo, partials); break;
    }
}

}  // namespace mclbm
