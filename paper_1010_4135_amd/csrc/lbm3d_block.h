// The fused FD-LB time step without a z march (the "untiled" launch shape),
// for grids too small to give every compute unit a tile of the tiled kernel.
//
// One workgroup updates 32 x 8 nodes of one plane, a node per thread.  What
// bounds such grids is latency (launches, dependent memory accesses, the
// length of one wavefront's instruction stream) and the loads per node that
// go through L1, not HBM: the levels sit in the L2s and the memory-side
// cache.  Hence
//  - every load is issued at the start: the node's own values, one halo
//    node per thread, the z neighbours (40 of the 70); x and y neighbours
//    then come from LDS;
//  - 32 x 8 nodes: a smaller halo than 64 x 4 and whole 128-byte rows.
//    Measured per step against 16 x 16 blocks: 64^3 FP32 10.1 / 12.1 us,
//    96x64x64 bubble FP32 with FP64 moments 17.5 / 20.1 (before the face
//    blocks were spread over the shader engines: 16.7), 32^3 5.1 / 5.4;
//  - the z terms are reduced to a difference and a Laplacian part per
//    velocity before the moments, which keeps the FP32 modes at four
//    wavefronts per SIMD without a spill (FP64: two; capping it at three
//    spills, and scratch made it 1.4 times slower);
//  - boundary layers need neither memory nor a launch of their own: periodic
//    neighbours are addressed on the other side, fixed states are read (they
//    never change), and the layers of extrapolating and reflecting faces are
//    formed from the moments of the two nodes next to the face, with
//    layer_line's operations, so results are bitwise those of layers kept in
//    memory: those of z faces by each thread for its column, those of x and
//    y faces once a block, by wavefronts 0 (low y), 1 (high y) and 3 (x),
//    which leave them in the LDS halo.  Blocks away from such faces skip
//    that code.
// Time per step, before (one node per thread with every neighbour from
// global memory, and a boundary-layer launch of 4 - 6 us) and now, replayed
// from graphs: 32^3 periodic FP32 with FP64 moments 10.9 / 5.1 us; 64^3
// periodic FP32 15.6 / 10.1; 96x64x64 bubble FP32 with FP64 moments 24.4 /
// 16.7; 48x32x32 bubble FP64 14.4 / 9.4; 256x4x4 tube FP64 12.6 / 7.3.  An
// empty kernel of the same grid takes 1.8 - 2.2 us.
#pragma once

#include "lbm3d_tile.h"

namespace lbm3d {

// BX x BY nodes of one plane in LDS, all 15 velocities, with the halo the x and y
// stencils reach: two rows (BX wide) and two columns (BY tall) beyond each
// side.  Per velocity the rows -2 .. BY + 1 come first, one after the other
// (a y neighbour is at a fixed distance), then the halo columns -2, -1, BX,
// BX + 1.  The velocity stride is a multiple of 64 elements, so that one
// LDS instruction reads the same place of two velocities.
template <typename S>
struct BlockPlane {
    static constexpr int BX = BLOCK_X, BY = BLOCK_Y;
    static constexpr int COLS = (BY + 4) * BX;
    static constexpr int HALO = 4 * (BX + BY);
    static constexpr int VS = (COLS + 4 * BY + 63) / 64 * 64;
    S v[NV][VS];
    // place of the node at column lx, row ly (one of them inside the block)
    static __device__ __forceinline__ int at(int lx, int ly)
    {
        const int row = (ly + 2) * BX + lx, col = COLS + (lx < 0 ? lx + 2 : lx - BX + 2) * BY + ly;
        return (unsigned)lx < (unsigned)BX ? row : col;
    }
};

// a / d and a % d for d with magic = floor(2^32 / d): the product's high word
// is the quotient or one less.
__device__ __forceinline__ uint32_t div_rem(uint32_t a, uint32_t d, uint32_t magic, uint32_t& rem)
{
    uint32_t q = __umulhi(a, magic);
    uint32_t r = a - q * d;
    if (r >= d) {
        q += 1;
        r -= d;
    }
    rem = r;
    return q;
}

// Access at a uniform base and a per-lane byte offset.
template <typename S>
__device__ __forceinline__ S ld_lane(const S* base, uint32_t off)
{
    using GP = const __attribute__((address_space(1))) S*;
    return *reinterpret_cast<GP>(reinterpret_cast<uint64_t>(base) + (uint64_t)off);
}
template <typename S>
__device__ __forceinline__ void st_lane(S* base, uint32_t off, S v)
{
    using GP = __attribute__((address_space(1))) S*;
    *reinterpret_cast<GP>(reinterpret_cast<uint64_t>(base) + (uint64_t)off) = v;
}

// NND (or upwind) difference D of velocity I along axis AX and the axis'
// part of its Laplacian, as node_update takes them.  fm2 is read for v > 0
// only, fp2 for v < 0 only.
template <int I, int AX, bool U2, typename C>
__device__ __forceinline__ void axis_diff(C f0, C fm2, C fm1, C fp1, C fp2, C& D, C& lap)
{
    constexpr int S = vsign(I, AX), G = vgroup(I);
    if constexpr (S > 0) {
        const C e0 = f0 - fm1, e1 = fp1 - f0;
        D = U2 ? up2_pos(fm1 - fm2, e0) : nnd_pos(fm1 - fm2, e0, e1);
        lap = e1 - e0;
    } else if constexpr (S < 0) {
        const C e0 = f0 - fm1, e1 = fp1 - f0;
        D = U2 ? up2_neg(e1, fp2 - fp1) : nnd_neg(e0, e1, fp2 - fp1);
        lap = e1 - e0;
    } else if constexpr (G <= 1) {
        lap = fm1 + fp1;
    }
}

template <typename M>
__device__ __forceinline__ Macro<M> pick_macro(bool first, const Macro<M>& a, const Macro<M>& b)
{
    Macro<M> q;
    q.rho = first ? a.rho : b.rho;
    q.ux = first ? a.ux : b.ux;
    q.uy = first ? a.uy : b.uy;
    q.uz = first ? a.uz : b.uz;
    q.T = first ? a.T : b.T;
    return q;
}

// What the step of a solve is described by, in the kernel's argument segment
// (a member of a batch: its entry of the solve table).
struct BlockArgs {
    Grid g;
    FaceBC bc;
    double xin[2][5];
    Model<double> md;
    Model<float> mf;
    BlockGrid bg;
    const void* f;
    void* fn;
    uint32_t* health;
};
__device__ __forceinline__ constexpr bool formed(int kind) { return kind == BC_OUTFLOW || kind == BC_REFLECT; }

// Moments of a block's nodes next to its x and y faces, by face side, the
// node's distance from the face (0, 1) and line.
template <typename M>
struct FaceNodes {
    Macro<M> x[2][2][BLOCK_Y], y[2][2][BLOCK_X];
};

// Boundary layers of the x and y faces a block's stencils reach, formed in
// its LDS plane: the threads of the nodes next to a face leave their moments
// in Q, then one thread per (line, layer) forms a layer node, a wavefront
// for each y face and one for the x faces.  (Each wavefront forming the x
// layers of its own rows instead, without these barriers, costs every
// wavefront of the block the 150 instructions: an extrapolating x face then
// adds 1.7 us to a 64^3 step instead of 1.4.)  Of a pair of nodes split between two
// blocks the other block's node is in this one's halo, from which its
// moments are computed.  The fixed x layers are formed here too where they
// are out of reach in memory (xmem false).
template <int MODE, typename D>
__device__ __forceinline__ void block_layers(const D& K, BlockPlane<typename Types<MODE>::S>& P,
                                             FaceNodes<typename Types<MODE>::M>& Q, int x0, int y0, bool xmem,
                                             const Macro<typename Types<MODE>::M>& mac)
{
    using S = typename Types<MODE>::S;
    using C = typename Types<MODE>::C;
    using M = typename Types<MODE>::M;
    using Plane = BlockPlane<S>;
    constexpr int BX = Plane::BX, BY = Plane::BY;
    static_assert(2 * BX == 64 && 4 * BY <= 64 && BLOCK_T == 256, "a wavefront per y face, one for both x faces");
    const Model<C>& mc = pick<C>(K.md, K.mf);
    const Model<M>& mm = pick<M>(K.md, K.mf);
    const int kx0 = K.bc.kind[0], kx1 = K.bc.kind[1], ky0 = K.bc.kind[2], ky1 = K.bc.kind[3];
    // columns and rows from the block's first to the high faces
    const int xr = K.g.nx - x0, yr = K.g.ny - y0;
    const int tid = (int)threadIdx.x, tx = tid % BX, ty = tid / BX;
    const bool fx0 = x0 == 0, fx1 = xr <= BX + 1, fy0 = y0 == 0, fy1 = yr <= BY + 1;
    if (fx0 && tx < 2) Q.x[0][tx][ty] = mac;
    if (fx1 && (unsigned)(xr - 1 - tx) < 2u) Q.x[1][xr - 1 - tx][ty] = mac;
    if (fy0 && ty < 2) Q.y[0][ty][tx] = mac;
    if (fy1 && (unsigned)(yr - 1 - ty) < 2u) Q.y[1][yr - 1 - ty][tx] = mac;
    lds_barrier();
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid & 63;
    const bool isx = wave == 3;
    const bool high = isx ? lane >= 2 * BY : wave == 1;
    const int kind = isx ? (high ? kx1 : kx0) : (high ? ky1 : ky0);
    const bool face = isx ? lane < 4 * BY && (high ? fx1 : fx0) : wave < 2 && (high ? fy1 : fy0);
    if (face && (formed(kind) || (isx && kind == BC_INFLOW && !xmem))) {
        const int k = isx ? lane % (2 * BY) : lane, len = isx ? BY : BX;
        const int layer = k >= len ? 2 : 1, line = k >= len ? k - len : k;
        const int a = high ? (isx ? xr : yr) - 1 : 0, d = high ? 1 : -1;  // the node next to the face, outwards
        auto at = [&](int p) { return Plane::at(isx ? p : line, isx ? line : p); };
        auto halo_node = [&](int p) {
            C b[NV];
            const int pp = at(p);
#pragma unroll
            for (int i = 0; i < NV; i++) b[i] = static_cast<C>(P.v[i][pp]);
            return moments<M, C>(b, mm);
        };
        const Macro<M>* q = isx ? &Q.x[high ? 1 : 0][0][line] : &Q.y[high ? 1 : 0][0][line];
        Macro<M> q0 = q[0], q1 = q[len];
        const int size = isx ? BX : BY;
        if (a == size) q0 = halo_node(a);
        if (high && a == 0) q1 = halo_node(-1);
        q1 = pick_macro(kind == BC_OUTFLOW, q1, q0);
        M c = M(0), m = M(1);
        if (kind != BC_INFLOW) layer_coefs(kind, layer, c, m);
        Macro<M> s = layer_state(q0, q1, c, M(1), 2);
        s.ux = isx ? m * s.ux : s.ux;
        s.uy = isx ? s.uy : m * s.uy;
        if (kind == BC_INFLOW) {
            // (selects: a per-lane index would put the argument in private
            // memory)
            s.rho = static_cast<M>(high ? K.xin[1][0] : K.xin[0][0]);
            s.ux = static_cast<M>(high ? K.xin[1][1] : K.xin[0][1]);
            s.uy = static_cast<M>(high ? K.xin[1][2] : K.xin[0][2]);
            s.uz = static_cast<M>(high ? K.xin[1][3] : K.xin[0][3]);
            s.T = static_cast<M>(high ? K.xin[1][4] : K.xin[0][4]);
        }
        C lf[NV];
        equilibrium<C, M>(s, mm, mc, lf);
        const int to = a + layer * d;
        if (to < size + 2) {  // (a block one short of the face reads its first layer only)
            const int pt = at(to);
#pragma unroll
            for (int i = 0; i < NV; i++) P.v[i][pt] = static_cast<S>(lf[i]);
        }
    }
}

// Layers of the z faces, formed by each thread for its own column into its
// z neighbours (the plane is the block's own, so the branches are uniform).
template <int MODE, typename D>
__device__ __forceinline__ void block_z_layers(uint64_t args, int z, const typename Types<MODE>::C (&f0)[NV],
                                               typename Types<MODE>::C (&zm2)[NV], typename Types<MODE>::C (&zm1)[NV],
                                               typename Types<MODE>::C (&zp1)[NV], typename Types<MODE>::C (&zp2)[NV])
{
    using C = typename Types<MODE>::C;
    using M = typename Types<MODE>::M;
    const D& K = again<D>(args);
    const Model<C>& mc = pick<C>(K.md, K.mf);
    const Model<M>& mm = pick<M>(K.md, K.mf);
    const Macro<M> mac = moments<M, C>(f0, mm);
#pragma unroll 1
    for (int side = 0; side < 2; side++) {
        const int kind = side ? K.bc.kind[5] : K.bc.kind[4];
        const int d = side ? K.g.nz - 1 - z : z;
        if (!formed(kind) || d > 1) continue;
        // the other node of the pair next to the face: one further in
        // (d = 0) or out (d = 1)
        const bool up = (side != 0) == (d != 0);
        Macro<M> qm = mac;
        if (kind == BC_OUTFLOW || d == 1) {
            if (up)
                qm = moments<M, C>(zp1, mm);
            else
                qm = moments<M, C>(zm1, mm);
        }
        const Macro<M> q0 = pick_macro(d == 0, mac, qm);
        const Macro<M> q1 = pick_macro(kind == BC_REFLECT, q0, pick_macro(d == 0, qm, mac));
        // layer 1: the first neighbour of the nodes next to the face, the
        // second one of those one further in; layer 2: the second neighbour
        // of the nodes next to the face
#pragma unroll 1
        for (int j = 1; j + d <= 2; j++) {
            C lf[NV];
            M c, m;
            layer_coefs(kind, j, c, m);
            equilibrium<C, M>(layer_state(q0, q1, c, m, 2), mm, mc, lf);
            const bool lo1 = side == 0 && j + d == 1, hi1 = side == 1 && j + d == 1;
            const bool lo2 = side == 0 && j + d == 2, hi2 = side == 1 && j + d == 2;
            static_for<NV>([&](auto ic) {
                constexpr int I = decltype(ic)::value;
                constexpr int SG = vsign(I, 2);
                const C n = lf[I], m1 = zm1[I], p1 = zp1[I], m2 = zm2[I], p2 = zp2[I];
                zm1[I] = lo1 ? n : m1;
                zp1[I] = hi1 ? n : p1;
                if constexpr (SG > 0) zm2[I] = lo2 ? n : m2;
                if constexpr (SG < 0) zp2[I] = hi2 ? n : p2;
            });
        }
    }
}

// Block t of a solve: one step of its nodes from f to fn.  PM: the level is
// in plane-major order.  U2: the second-order upwind variant in place of NND.
template <int MODE, bool U2, bool PM, typename D>
__device__ __forceinline__ void step_block(uint64_t args, const BlockGrid& bg, uint32_t t,
                                           const typename Types<MODE>::S* __restrict__ f, typename Types<MODE>::S* fout,
                                           BlockPlane<typename Types<MODE>::S>& P,
                                           FaceNodes<typename Types<MODE>::M>& Q)
{
    using S = typename Types<MODE>::S;
    using C = typename Types<MODE>::C;
    using M = typename Types<MODE>::M;
    using Plane = BlockPlane<S>;
    constexpr int BX = Plane::BX, BY = Plane::BY;
    constexpr uint32_t ES = sizeof(S);
    const D& A = again<D>(args);
    const Grid& g = A.g;

    uint32_t sb, pb, bxi;
    const uint32_t si = div_rem(t, bg.strip, bg.smagic, sb);
    const bool tail = si >= bg.full;
    int z = (int)div_rem(sb, bg.ntx * (tail ? bg.last : bg.ys), tail ? bg.lmagic : bg.pmagic, pb);
    const uint32_t row = div_rem(pb, bg.ntx, bg.xmagic, bxi);
    const int y0 = (int)(si * bg.ys + row) * BY;
    // Consecutive workgroups of an XCD go to its shader engines in turn, and
    // the blocks at an x face take longer than the others: with as many
    // blocks per row as engines (or half) they would all go to the same
    // ones.  So each row starts one block further along x (for two blocks
    // per row every other row): 128^3 with an extrapolating x face, 54.8 us
    // a step without, 53.0 with (50.0 periodic, where the order stays).
    if (formed(A.bc.kind[0]) || formed(A.bc.kind[1])) {
        uint32_t rot;
        (void)div_rem(bg.ntx == 2 ? row >> 1 : row, bg.ntx, bg.xmagic, rot);
        bxi += rot;
        bxi -= bxi >= bg.ntx ? bg.ntx : 0;
    }
    const int x0 = (int)bxi * BX;
    const int tid = (int)threadIdx.x;
    const int tx = tid % BX, ty = tid / BX;
    const bool act = x0 + tx < g.nx && y0 + ty < g.ny;
    const int kx0 = A.bc.kind[0], kx1 = A.bc.kind[1], ky0 = A.bc.kind[2];
    const int kz0 = A.bc.kind[4], kz1 = A.bc.kind[5];
    // planes next to a formed z face first: their blocks take longer, and
    // the launch would end on them
    if (formed(kz1)) z = z < 2 ? z + g.nz - 2 : z - 2;

    // Byte offset of node (xx, yy) from row -2 of its plane: wrapped on
    // periodic axes, in the boundary layers of fixed-state faces (and of
    // every y face, where the rows are), else clamped.
    const uint32_t sy = (uint32_t)g.sy;
    const int xw = kx0 == BC_PERIODIC ? g.nx : 0, yw = ky0 == BC_PERIODIC ? g.ny : 0;
    const int ylo = yw ? 0 : -NG, yhi = yw ? g.ny - 1 : g.ny + 1;
    // fixed x layers in memory: in the row padding, or in the x-layer block
    // that follows the plane (xlb: its third element from row -2); levels
    // in velocity-major order keep that block elsewhere
    const bool dense = g.xg != 0, xmem = PM || !dense;
    const int xlo = kx0 == BC_INFLOW && xmem ? -NG : 0, xhi = kx1 == BC_INFLOW && xmem ? g.nx + 1 : g.nx - 1;
    const uint32_t xlb = (uint32_t)(g.xg - (g.org - NG * g.sz - NG * g.sy)) + NG;
    auto off = [&](int xx, int yy) {
        yy = min(yy, g.ny + 1);
        yy += yy < 0 ? yw : yy >= g.ny ? -yw : 0;
        yy = min(max(yy, ylo), yhi);
        xx = min(xx, g.nx + 1);
        xx += xx < 0 ? xw : xx >= g.nx ? -xw : 0;
        xx = min(max(xx, xlo), xhi);
        const uint32_t row = (uint32_t)(yy + NG);
        uint32_t o = row * sy + (uint32_t)xx;
        if (dense) {
            const uint32_t l = xlb + row * 4u + (uint32_t)(xx < 0 ? xx : xx - g.nx);
            o = (unsigned)xx >= (unsigned)g.nx ? l : o;
        }
        return o * ES;
    };
    const uint32_t o0 = off(x0 + tx, y0 + ty);

    // Uniform bases of row -2 of the planes read.  In plane-major order the
    // 15 velocities of a plane lie within a 32-bit offset of its base, so
    // the velocity goes into the lane offset, shared by all five planes;
    // otherwise each velocity has bases of its own.
    const int64_t org = g.org - NG * g.sy;
    auto zi = [&](int v) {
        const int w = v < 0 ? v + g.nz : v >= g.nz ? v - g.nz : v;
        return kz0 != BC_PERIODIC ? v : g.nz == 1 ? 0 : w;
    };
    auto plane = [&](int zz) { return f + (org + (int64_t)zz * g.sz); };
    const int64_t sv = g.sv;
    auto load = [&](auto ic, const S* base, uint32_t o) {
        constexpr int I = decltype(ic)::value;
        if constexpr (PM)
            return ld_lane(base, o + (uint32_t)I * ((uint32_t)sv * ES));
        else
            return ld_lane(sreg(base + I * sv), o);
    };
    const S* b0 = plane(z);

    C f0[NV];
    static_for<NV>([&](auto ic) { f0[decltype(ic)::value] = static_cast<C>(load(ic, b0, o0)); });

    // halo: thread k < HALO reads the k-th halo node of every velocity
    static_assert(Plane::HALO <= BLOCK_T, "one halo node per thread");
    const bool on = tid < Plane::HALO;
    S hv[NV];
    int hp = 0;  // its place in the plane
    if (on) {
        const bool hrow = tid < 4 * BX;
        const int hk = hrow ? tid / BX : (tid - 4 * BX) / BY, hl = hrow ? tid % BX : tid % BY;
        const int hc = hk < 2 ? hk - 2 : (hrow ? BY : BX) + hk - 2;
        hp = hrow ? (hc + 2) * BX + hl : Plane::COLS - 4 * BX + tid;
        const uint32_t oh = off(x0 + (hrow ? hl : hc), y0 + (hrow ? hc : hl));
        static_for<NV>([&](auto ic) { hv[decltype(ic)::value] = load(ic, b0, oh); });
    }

    // z neighbours (the offset made opaque: lane offsets formed here anew
    // keep the scalar-base form of the loads, those formed above would be
    // widened to 64-bit addresses)
    C zm2[NV], zm1[NV], zp1[NV], zp2[NV];
    {
        uint32_t oz = o0;
        asm("" : "+v"(oz));
        const S *bm2 = plane(zi(z - 2)), *bm1 = plane(zi(z - 1)), *bp1 = plane(zi(z + 1)), *bp2 = plane(zi(z + 2));
        static_for<NV>([&](auto ic) {
            constexpr int I = decltype(ic)::value;
            constexpr int SG = vsign(I, 2);
            zm2[I] = zp2[I] = C(0);
            if constexpr (SG > 0) zm2[I] = static_cast<C>(load(ic, bm2, oz));
            zm1[I] = static_cast<C>(load(ic, bm1, oz));
            zp1[I] = static_cast<C>(load(ic, bp1, oz));
            if constexpr (SG < 0) zp2[I] = static_cast<C>(load(ic, bp2, oz));
        });
    }

#pragma unroll
    for (int i = 0; i < NV; i++) P.v[i][2 * BX + tid] = static_cast<S>(f0[i]);
    if (on) {
#pragma unroll
        for (int i = 0; i < NV; i++) P.v[i][hp] = hv[i];
    }
    lds_barrier();

    if ((formed(kz0) && z < 2) || (formed(kz1) && z >= g.nz - 2)) block_z_layers<MODE, D>(args, z, f0, zm2, zm1, zp1, zp2);
    // (the values converted for the moments there are not kept for those below)
#pragma unroll
    for (int i = 0; i < NV; i++) asm("" : "+v"(f0[i]));
    C Dz[NV], lz[NV];
    static_for<NV>([&](auto ic) {
        constexpr int I = decltype(ic)::value;
        Dz[I] = lz[I] = C(0);
        axis_diff<I, 2, U2>(f0[I], zm2[I], zm1[I], zp1[I], zp2[I], Dz[I], lz[I]);
    });

    const D& K = again<D>(args);
    const Model<C>& mc = pick<C>(K.md, K.mf);
    const Model<M>& mm = pick<M>(K.md, K.mf);
    const Macro<M> mac = moments<M, C>(f0, mm);
    report_health(K.health, act ? health_bits(mac) : 0u);

    auto here = [&](int kind) { return formed(kind) || (kind == BC_INFLOW && !xmem); };
    const bool nearx = (x0 == 0 && here(kx0)) || (K.g.nx - x0 <= BX + 1 && here(kx1));
    const bool neary = (y0 == 0 && formed(ky0)) || (K.g.ny - y0 <= BY + 1 && formed(K.bc.kind[3]));
    if (nearx || neary) block_layers<MODE, D>(K, P, Q, x0, y0, xmem, mac);

    C feq[NV];
    equilibrium<C, M>(mac, mm, mc, feq);
    if (nearx || neary) lds_barrier();
    if (!act) return;
    S* fn = fout + (K.g.org - NG * K.g.sy + (int64_t)z * K.g.sz);
    const int64_t svn = K.g.sv;
    uint32_t os = o0;
    asm("" : "+v"(os));
    // places of this thread's neighbours: row -2 of its column (a y step is
    // BX), and along x
    const int la = tid, xo = 2 * BX + tid;
    const int xm1 = tx > 0 ? xo - 1 : Plane::COLS + BY + ty;
    const int xm2 = tx > 1 ? xo - 2 : Plane::COLS + tx * BY + ty;
    const int xp1 = tx < BX - 1 ? xo + 1 : Plane::COLS + 2 * BY + ty;
    const int xp2 = tx < BX - 2 ? xo + 2 : Plane::COLS + (tx - BX + 4) * BY + ty;
    static_for<NV>([&](auto ic) {
        constexpr int I = decltype(ic)::value;
        constexpr int SX = vsign(I, 0), SY = vsign(I, 1), G = vgroup(I);
        auto nb = [&](int p) { return static_cast<C>(P.v[I][p]); };
        const C v = f0[I];
        C Dx = C(0), Dy = C(0), lx = C(0), ly = C(0);
        if constexpr (SX != 0 || G <= 1)
            axis_diff<I, 0, U2>(v, SX > 0 ? nb(xm2) : C(0), nb(xm1), nb(xp1), SX < 0 ? nb(xp2) : C(0), Dx, lx);
        if constexpr (SY != 0 || G <= 1)
            axis_diff<I, 1, U2>(v, SY > 0 ? nb(la) : C(0), nb(la + BX), nb(la + 3 * BX),
                                SY < 0 ? nb(la + 4 * BX) : C(0), Dy, ly);
        const C out = node_update<I, C>(v, feq[I], Dx, Dy, Dz[I], lx, ly, lz[I], mc);
        if constexpr (PM)
            st_lane(fn, os + (uint32_t)I * ((uint32_t)svn * ES), static_cast<S>(out));
        else
            st_lane(sreg(fn + I * svn), os, static_cast<S>(out));
    });
}

template <int MODE, bool U2, bool PM>
__global__ void __launch_bounds__(BLOCK_T, MODE == MODE_FP64 ? 2 : 4)
k_step_block(BlockArgs args)
{
    using S = typename Types<MODE>::S;
    __shared__ BlockPlane<S> P;
    __shared__ FaceNodes<typename Types<MODE>::M> Q;
    const uint32_t t = (uint32_t)xcd_tile((int)blockIdx.x, (int)gridDim.x);
    step_block<MODE, U2, PM, BlockArgs>(reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr()), args.bg, t,
                                        (const S*)args.f, (S*)args.fn, P, Q);
}

// The untiled members of a batch: entry e names the solve of blocks
// [BATCH_BLOCKS e, BATCH_BLOCKS (e + 1)).
template <int MODE>
__global__ void __launch_bounds__(BLOCK_T, MODE == MODE_FP64 ? 2 : 4)
k_batch_block(const BatchSolve* __restrict__ solves, const BatchTile* __restrict__ entries,
              const BatchQueue* __restrict__ queue, int parity, const BatchCount* __restrict__ counts)
{
    using S = typename Types<MODE>::S;
    __shared__ BlockPlane<S> P;
    __shared__ FaceNodes<typename Types<MODE>::M> Q;
    if (parity < 0 && blockIdx.x == 0) advance_counts(*queue, parity);
    const uint32_t b = (uint32_t)xcd_tile((int)blockIdx.x, (int)gridDim.x);
    // (the tables through the constant address space: scalar loads)
    const BatchTile& entry = again<BatchTile>(reinterpret_cast<uint64_t>(entries + b / BATCH_BLOCKS));
    const int m = entry.solve;
    const uint32_t t = b - (uint32_t)entry.z0;
    const BlockGrid& bg = again<BlockGrid>(reinterpret_cast<uint64_t>(
        again<BatchQueue>(reinterpret_cast<uint64_t>(queue)).blocks + m));
    if (t >= bg.count) return;
    int par = parity;
    if (parity < 0) {
        const BatchCount& c = again<BatchCount>(reinterpret_cast<uint64_t>(counts + m));
        if (c.done >= c.target) return;
        par = c.done & 1;
    }
    const uint64_t at = reinterpret_cast<uint64_t>(solves + m);
    const BatchSolve& d = again<BatchSolve>(at);
    const bool flip = ((d.cur0 ^ par) & 1) != 0;
    const S* f = (const S*)(flip ? d.f[1] : d.f[0]);
    S* fn = (S*)(flip ? d.f[0] : d.f[1]);
    if (d.g.plane_major)
        step_block<MODE, false, true, BatchSolve>(at, bg, t, f, fn, P, Q);
    else
        step_block<MODE, false, false, BatchSolve>(at, bg, t, f, fn, P, Q);
}

}  // namespace lbm3d
