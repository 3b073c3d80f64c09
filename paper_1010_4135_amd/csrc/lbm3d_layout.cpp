// Host-side layout decisions of the lbm3d library: where each node's
// distributions sit in memory, which kernels and tile shapes take a solve,
// which boundary layers the kernels leave to memory.
#include "lbm3d_api_impl.h"
#include "lbm3d_model.h"

#include <algorithm>
#include <mutex>
#include <vector>

namespace lbm3d {

size_t elem_size(int precision) { return precision == LBM3D_FP64 ? 8 : 4; }

// Padded layout: each x row holds `ox` leading elements (the two boundary
// layers sit just before interior x = 0, which starts on a 128-byte line),
// the nx interior nodes and two boundary layers, rounded up to whole lines.
Grid make_grid(const lbm3d_params* p)
{
    Grid g;
    const int64_t es = (int64_t)elem_size(p->precision);
    const int64_t line = 128 / es;
    g.nx = p->nx;
    g.ny = p->ny;
    g.nz = p->nz;
    const bool dense = dense_rows(p->nx);
    // dense rows: the interior only, rows start on a line (nx is a multiple
    // of 64 elements); otherwise the x layers pad the rows
    const int64_t ox = dense ? 0 : line;
    // one cache line of padding per row, holding the two right layer nodes
    // of the row (its first elements) and the two left layer nodes of the
    // next row (its last elements); interior rows start on a line
    const int64_t mxp = (p->nx + line - 1) / line * line + line;
    const int64_t mx = dense ? p->nx : mxp;
    const int64_t my = p->ny + 2 * NG;
    const int64_t mz = p->nz + 2 * NG;
    const int64_t plane = mx * my;
    const int64_t xrows = dense ? 4 * my : 0;  // x layers of one plane's rows (dense rows)
    const int64_t sinkn = (int64_t)SINK_ROWS * TILE_X;
    g.my = (int32_t)my;
    g.sy = mx;
    // an odd number of 256-byte blocks holding at least n elements
    const int64_t blk = 256 / es;
    auto odd_blocks = [&](int64_t n) {
        int64_t b = (n + blk - 1) / blk;
        if ((b & 1) == 0) b += 1;
        return b * blk;
    };
    // The sink region of the tiled step's stores from lanes outside the grid
    // sits after one spare line past the last plane (the right layer nodes
    // of the last row of a padded plane reach two elements past it), at the
    // same offset from every velocity's base.
    const bool velocity_major = (p->flags & LBM3D_VELOCITY_MAJOR) != 0;
    if (!velocity_major) {
        const int64_t sv = odd_blocks(plane + xrows);
        const int64_t sz = NV * sv;
        const int64_t sink = sz * mz + line;
        const int64_t len = (NV - 1) * sv + sink + sinkn + line;
        if (len * es < ((int64_t)1 << 31)) {
            g.plane_major = 1;
            g.sv = sv;
            g.sz = sz;
            g.sink = sink;
            g.xg = dense ? plane : 0;
            g.xgz = sz;
            g.len = len;
            g.org = NG * g.sz + NG * g.sy + ox;
            return g;
        }
    }
    g.plane_major = 0;
    g.sz = plane;
    g.sink = g.sz * mz + line;
    const int64_t sink_end = g.sink + sinkn;
    // dense rows: the x layers of every row (4 nodes) after the sink region
    g.xg = dense ? sink_end + line : 0;
    g.xgz = xrows;
    const int64_t end = dense ? g.xg + xrows * mz : sink_end + line;
    g.sv = odd_blocks(end);
    g.len = NV * g.sv;
    g.org = NG * g.sz + NG * g.sy + ox;
    return g;
}

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

// floor(2^32 / d) (2^32 - 1 for d <= 1)
static uint32_t div_magic(uint32_t d) { return d <= 1 ? 0xffffffffu : (uint32_t)(((uint64_t)1 << 32) / d); }

BlockGrid block_grid(const Grid& g)
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
    b.count = b.ntx * nty * (uint32_t)g.nz;
    b.xmagic = div_magic(b.ntx);
    b.smagic = div_magic(b.strip);
    b.pmagic = div_magic(b.ntx * b.ys);
    b.lmagic = div_magic(b.ntx * b.last);
    return b;
}

size_t f_bytes(const Grid& g, int precision) { return (size_t)g.len * elem_size(precision); }


bool tiled_fits(int mode, const Grid& g)
{
    // the tiled kernels reach everything from a velocity's base (its sink
    // region included) with 32-bit byte offsets: the whole level when it is
    // plane-major, one velocity block when it is velocity-major
    const int64_t es = mode == MODE_FP64 ? 8 : 4;
    return (g.plane_major ? g.len : g.sv) * es < ((int64_t)1 << 31);
}

int device_cus()
{
    static std::mutex mu;
    static std::vector<int> cache;  // per device, 0 until looked up
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) {
        (void)hipGetLastError();
        return 256;
    }
    std::lock_guard<std::mutex> lk(mu);
    if ((size_t)dev >= cache.size()) cache.resize((size_t)dev + 1, 0);
    if (!cache[(size_t)dev]) {
        int cus = 256;
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
            cus = prop.multiProcessorCount;
        cache[(size_t)dev] = cus;
    }
    return cache[(size_t)dev];
}

bool stream_rows(const Grid& g, int mode)
{
    const int64_t bytes = 2 * (int64_t)f_bytes(g, mode);
    return bytes > STREAM_MIN_BYTES && (dense_rows(g.nx) || (mode == MODE_FP64 && bytes <= 2 * STREAM_MIN_BYTES));
}

// The launch shape of a solve that is not tuned, from a model of the two
// kernels (256 compute units, us a step; the autotuner remains the way to the
// best shape).
//
// Tiled, 64 x BY columns (BY = 8 in the FP32 modes, 4 in FP64, the rows that
// fit two wavefronts per SIMD) of `d` planes, every chunk count whose d is 8
// or more: the tiles run in rounds of one per compute unit, and a tile takes
// time in proportion to its planes plus the four its z ring loads first; one
// of its planes takes 2.4 us in the FP32 modes while both levels stay in the
// 256 MB memory-side cache (2.33 - 2.46 over 10 grids) and 2.8 beyond (2.67 -
// 2.92 over 6), 2.95 in FP64 (2.78 - 3.1 over 14).  The cheapest d wins, in
// FP64 as it is; in the FP32 modes, whose tiles lean more on the caches, the
// deepest within an eighth of it: a round more means more halo planes read
// again (FP32 200x200x100: two rounds of 20 planes 159 us, one of 50 150;
// 300x150x100 167 and 152).  Against depths of powers of two only: FP32
// 160^3 157 -> 123 us, 192x128x128 93.9 -> 83.7; FP64 250x120x33 101 -> 60.
//
// Untiled, per 1000 nodes of its 32 x 8 blocks: 25 ns (24 - 27) in the FP32
// modes and 60 in FP64 in that cache, 39 and 77 beyond.  Its small blocks
// spread over all units whatever the grid, so it wins where the tiles fill
// their rounds badly: FP32 150x100x70 31 us (tiles of 12 planes 38),
// 384x96x50 44.6 (49.2), FP64 100x61x50 29 (34).  Where the tiles fill 95%
// of their rounds the two models are mostly within their own error (FP32
// 128^3 52 and 52, 512x64x48 38.6 tiled and 39.3, 128x128x64 29.5 and 27.0)
// and the tiles stay.  96x64x64 FP64 pays for this line: 34.4 us tiled and
// 27.8 untiled periodic, 43.1 and 30.7 with walls.  So do grids just beyond
// the cache with walls along y or z, whose tiled step takes a layer launch of
// 6 us more that this model leaves out: 298x78x78 FP32 with FP64 moments (274
// MB) 67.5 us tiled and 58.6 untiled with walls, 52.5 and 52.1 periodic.
constexpr int64_t CACHED_BYTES = (int64_t)256 << 20;

TileCfg default_tile(int mode, const Grid& g)
{
    TileCfg t;
    t.by = 0;
    t.tz = 1;
    if (!tiled_fits(mode, g)) return t;
    t.stream = stream_rows(g, mode);
    const bool fp64 = mode == MODE_FP64;
    const bool cached = 2 * (int64_t)f_bytes(g, mode) <= CACHED_BYTES;
    const int by = fp64 ? 4 : 8;
    const int64_t cus = device_cus();
    const int64_t cols = (int64_t)((g.nx + TILE_X - 1) / TILE_X) * ((g.ny + by - 1) / by);
    const auto tiles_at = [&](int64_t d) { return cols * ((g.nz + d - 1) / d); };
    const auto cost_at = [&](int64_t d) { return (tiles_at(d) + cus - 1) / cus * (d + 4); };
    // depths from the deepest; chunks of equal depth but for the last
    const int64_t shortest = std::min<int64_t>(8, g.nz);
    int64_t cheapest = cost_at(g.nz);
    for (int64_t d = shortest; d < g.nz; d++) cheapest = std::min(cheapest, cost_at(d));
    const int64_t limit = fp64 ? cheapest : cheapest + cheapest / 8;
    int64_t depth = g.nz;
    for (int64_t c = 1; cost_at(depth) > limit; c++) depth = std::max(shortest, (g.nz + c - 1) / c);
    const int64_t tiles = tiles_at(depth), rounds = (tiles + cus - 1) / cus;
    if (20 * tiles < 19 * rounds * cus) {
        const double plane = fp64 ? 2.95 : cached ? 2.4 : 2.8;
        const double node = (fp64 ? (cached ? 0.060 : 0.077) : (cached ? 0.025 : 0.039)) * 256.0 / cus;
        const double untiled = node * 1e-3 * BLOCK_T * block_grid(g).count;
        if (untiled < plane * (double)(rounds * (depth + 4))) return t;
    }
    t.by = by;
    t.tz = (int)depth;
    return t;
}

bool tile_supported(int mode, const Grid& g, const TileCfg& t)
{
    if (t.tz < 1) return false;
    if (t.by == 0) return true;
    if (!tiled_fits(mode, g)) return false;
    if (t.by == 2 || t.by == 4) return true;
    return t.by == 8 && mode != MODE_FP64;
}

uint32_t ghost_faces(const Grid& g, const FaceBC& bc, bool tiled)
{
    uint32_t m = 0;
    if (!tiled) return m;
    for (int face = 0; face < 6; face++) {
        const int kind = bc.kind[face];
        if (kind == BC_INFLOW) continue;
        // the tiles form the -x layers, and the +x layers unless the last
        // tile holds a single column (see x_forms)
        if (face == 0) continue;
        if (face == 1 && g.nx % TILE_X != 1) continue;
        if (kind == BC_PERIODIC) continue;
        m |= 1u << face;
    }
    return m;
}

void x_fixed_states(const double (*inflow)[5], double (&xin)[2][5])
{
    for (int s = 0; s < 2; s++) {
        const double* st = inflow[s];
        xin[s][0] = st[0];
        xin[s][1] = st[1];
        xin[s][2] = st[2];
        xin[s][3] = st[3];
        xin[s][4] = st[0] > 0.0 ? st[4] / st[0] : 0.0;  // T = p / rho
    }
}

int conserved_blocks(const Grid& g)
{
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    return (int)std::min<int64_t>(1024, std::max<int64_t>(1, (n + RB - 1) / RB));
}

}  // namespace lbm3d
