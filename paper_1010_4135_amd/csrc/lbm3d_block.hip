// The untiled time step (lbm3d_block.h): its launches.
#include "lbm3d_block.h"

#include <hip/hip_ext.h>

namespace lbm3d {

template <int MODE, bool U2, bool PM>
static void launch(const Grid& g, const FaceBC& bc, const Model<double>& md, const Model<float>& mf,
                   const double (*inflow)[5], const void* f, void* fn, uint32_t* health, hipStream_t s, hipEvent_t e0,
                   hipEvent_t e1)
{
    BlockArgs K;
    K.g = g;
    K.bc = bc;
    x_fixed_states(inflow, K.xin);
    K.md = md;
    K.mf = mf;
    K.bg = block_grid(g);
    K.f = f;
    K.fn = fn;
    K.health = health;
    const dim3 grid(K.bg.count), block(BLOCK_T);
    if (e0 || e1)
        hipExtLaunchKernelGGL(k_step_block<MODE, U2, PM>, grid, block, 0, s, e0, e1, 0, K);
    else
        k_step_block<MODE, U2, PM><<<grid, block, 0, s>>>(K);
}

template <int MODE, typename... T>
static void launch_as(bool upwind2, const Grid& g, T... a)
{
    if (upwind2) {
        if (g.plane_major) launch<MODE, true, true>(g, a...);
        else launch<MODE, true, false>(g, a...);
    } else {
        if (g.plane_major) launch<MODE, false, true>(g, a...);
        else launch<MODE, false, false>(g, a...);
    }
}

void launch_block(int mode, const Grid& g, const FaceBC& bc, const Model<double>& md, const Model<float>& mf,
                  const double (*inflow)[5], const void* f, void* fn, uint32_t* health, hipStream_t s, bool upwind2,
                  hipEvent_t e0, hipEvent_t e1)
{
    if (mode == MODE_FP64)
        launch_as<MODE_FP64>(upwind2, g, bc, md, mf, inflow, f, fn, health, s, e0, e1);
    else if (mode == MODE_FP32)
        launch_as<MODE_FP32>(upwind2, g, bc, md, mf, inflow, f, fn, health, s, e0, e1);
    else
        launch_as<MODE_FP32_T64>(upwind2, g, bc, md, mf, inflow, f, fn, health, s, e0, e1);
}

void launch_batch_blocks(int mode, int nblocks, const BatchSolve* solves, const BatchTile* entries,
                         const BatchQueue* queue, int parity, const BatchCount* counts, hipStream_t s)
{
    const dim3 grid((unsigned)nblocks), block(BLOCK_T);
    if (mode == MODE_FP64)
        k_batch_block<MODE_FP64><<<grid, block, 0, s>>>(solves, entries, queue, parity, counts);
    else if (mode == MODE_FP32)
        k_batch_block<MODE_FP32><<<grid, block, 0, s>>>(solves, entries, queue, parity, counts);
    else
        k_batch_block<MODE_FP32_T64><<<grid, block, 0, s>>>(solves, entries, queue, parity, counts);
}

}  // namespace lbm3d
