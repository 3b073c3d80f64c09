// The untiled time step (lbm3d_block.h): its launches.
#include "lbm3d_block.h"

#include <hip/hip_ext.h>

namespace lbm3d {

// Block rows of a strip: the smallest power of two that gives a strip at
// least STRIP_BLOCKS blocks per plane.  An XCD runs about 128 blocks at a
// time; in plane order on a wide grid those span less than the five planes
// the z stencil reads, whose lines then leave its 4 MiB L2 before their
// next use, while a narrow strip keeps several planes of it there.  128^3
// FP32, 4 block rows against whole planes (16): 52.5 against 62.3 us a
// step; 298x78x78 FP32 with FP64 moments, 2 against 10: 60.5 against 73.0;
// 256x128x128 FP32, 2 against 16: 151 against 178.  Grids of a few hundred
// thousand nodes, whose levels the L2s hold, move by 3% either way.
constexpr uint32_t STRIP_BLOCKS = 16;

static BlockGrid block_grid(const Grid& g)
{
    BlockGrid b;
    const uint32_t nty = (uint32_t)((g.ny + BLOCK_Y - 1) / BLOCK_Y);
    b.ntx = (uint32_t)((g.nx + BLOCK_X - 1) / BLOCK_X);
    uint32_t ys = 1;
    while (ys < nty && b.ntx * ys < STRIP_BLOCKS) ys *= 2;
    b.ys = ys < nty ? ys : nty;
    b.full = nty / b.ys;
    b.last = nty % b.ys;
    b.strip = b.ntx * b.ys * (uint32_t)g.nz;
    b.xmagic = div_magic(b.ntx);
    b.smagic = div_magic(b.strip);
    b.pmagic = div_magic(b.ntx * b.ys);
    b.lmagic = div_magic(b.ntx * b.last);
    return b;
}

template <int MODE, bool U2, bool PM>
static void launch(const Grid& g, const FaceBC& bc, const Model<double>& md, const Model<float>& mf,
                   const double (*inflow)[5], const void* f, void* fn, uint32_t* health, hipStream_t s, hipEvent_t e0,
                   hipEvent_t e1)
{
    using S = typename Types<MODE>::S;
    BlockArgs<MODE> K;
    K.A.g = g;
    K.A.bc = bc;
    K.A.f = (const S*)f;
    K.A.fn = (S*)fn;
    K.A.health = health;
    x_fixed_states(inflow, K.A.xin);
    K.bg = block_grid(g);
    K.md = md;
    K.mf = mf;
    const dim3 grid(K.bg.ntx * (K.bg.full * K.bg.ys + K.bg.last) * (unsigned)g.nz), block(BLOCK_T);
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

}  // namespace lbm3d
