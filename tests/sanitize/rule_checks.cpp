// Host-side checks of rules that choose between paths, built like the other
// host checks with sanitizers and without kernels: how a transfer between
// caller memory and the device goes (copy_plan), and what the batched step
// does where the tables of its groups do not fit the room it is given, and
// where the host has no memory for its plan.
#include "../../include/lbm3d.h"
#include "../../paper_1010_4135_amd/csrc/lbm3d_api_impl.h"
#include "../../paper_1010_4135_amd/csrc/lbm3d_batch.h"
#include "../../paper_1010_4135_amd/csrc/lbm3d_internal.h"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <random>

// The allocation that fails, counted down (negative: none).
static long fail_at = -1;
void* operator new(size_t n)
{
    if (fail_at >= 0 && fail_at-- == 0) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return std::malloc(n ? n : 1); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

namespace lbm3d {
hipError_t launch_init(int, const Grid&, const Model<double>&, const double*, void*, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_step(int, const Grid&, const FaceBC&, const TileCfg&, const Model<double>&, const Model<float>&,
                       const double (*)[5], const void*, void*, uint32_t*, hipStream_t, bool, hipEvent_t,
                       hipEvent_t) { return hipErrorNoDevice; }
hipError_t launch_ghosts(int, const Grid&, const FaceBC&, const Model<double>&, const double (*)[5], bool, void*,
                         hipStream_t, uint32_t) { return hipErrorNoDevice; }
hipError_t launch_moments(int, const Grid&, const Model<double>&, const void*, double*, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_conserved(int, const Grid&, const Model<double>&, const void*, double*, int, double*, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_pack(int, const Grid&, const void*, void*, bool, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_batch_layers(int, const BatchSolve*, const BatchLayerJob*, const int32_t*, int, int, const BatchCount*,
                               hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_gather_health(const BatchSolve*, int, uint32_t*, hipStream_t) { return hipErrorNoDevice; }
hipError_t launch_batch_step(int, int, bool, const BatchSolve*, const BatchTile*, BatchQueue*, int, int, int,
                             const BatchCount*, hipStream_t) { return hipErrorNoDevice; }
}  // namespace lbm3d

static int failures = 0;
#define EXPECT(c)                                                            \
    do {                                                                     \
        if (!(c)) {                                                          \
            std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
            failures++;                                                      \
        }                                                                    \
    } while (0)

static constexpr size_t MIB = (size_t)1 << 20;

// The buffer as the transfers of a process leave it.
struct Process {
    size_t buffer = 0, passed = 0;
    int made = 0;
    lbm3d::CopyPlan move(size_t bytes, bool down, bool now = false)
    {
        const lbm3d::CopyPlan p = lbm3d::copy_plan(bytes, down, buffer, passed, now);
        if (p.make) {
            buffer = p.make;
            made++;
        }
        if (!p.threads && p.wants) passed += bytes;
        return p;
    }
};

static void check_copies(std::mt19937& rng)
{
    // a solve that is initialised, read back a few times, saved and destroyed
    // makes no buffer unless one of its transfers repays it
    for (size_t mib : {1, 3, 5, 10, 12, 31}) {
        Process p;
        p.move(mib * MIB, false);
        p.move(mib * MIB, true);
        p.move(mib * MIB * 3 / 2, true);
        EXPECT(p.made == (mib * 3 / 2 >= 32 ? 1 : 0));
    }
    // read back again and again, it is made once and then used
    for (size_t mib : {4, 10, 31}) {
        Process p;
        int first = -1;
        for (int k = 0; k < 60; k++) {
            const lbm3d::CopyPlan c = p.move(mib * MIB, true);
            if (c.threads && first < 0) first = k;
            EXPECT((c.threads != 0) == (first >= 0));
        }
        EXPECT(p.made == 1 && first >= 0 && (size_t)(first + 1) * mib >= 32 && (size_t)first * mib < 32);
        // a larger transfer needs a larger one, a smaller none
        EXPECT(p.move(200 * MIB, false).make != 0 && p.move(mib * MIB, true).make == 0 && p.made == 2);
    }
    // beside long work on the device, or for several users, the first read-back makes it
    for (size_t mib : {4, 10, 31}) {
        Process p;
        EXPECT(p.move(mib * MIB, true, true).make != 0 && p.move(mib * MIB, true).make == 0 && p.made == 1);
    }
    // below these sizes the runtime has no disadvantage to make good
    EXPECT(!lbm3d::copy_plan(4 * MIB - 1, true, 32 * MIB, 0, true).threads && !lbm3d::copy_plan(4 * MIB - 1, true, 0, 1 << 30, true).wants);
    EXPECT(!lbm3d::copy_plan(32 * MIB - 1, false, 32 * MIB, 0, false).threads);
    // every worker has a slot of its own within the buffer, and the chunks are
    // no smaller than they need be
    for (int k = 0; k < 20000; k++) {
        const size_t bytes = 1 + (size_t)(rng() % 300000) * 1021, buffers[3] = {0, 16 * MIB, 32 * MIB};
        const size_t buffer = buffers[rng() % 3], passed = (size_t)(rng() % 200) * MIB;
        const lbm3d::CopyPlan c = lbm3d::copy_plan(bytes, rng() % 2, buffer, passed, rng() % 2);
        if (!c.threads) {
            EXPECT(c.make == 0);
            continue;
        }
        EXPECT(c.wants && c.threads <= 8 && c.chunk > 0 && c.chunk % 65536 == 0);
        EXPECT(c.threads * c.chunk <= (c.make ? c.make : buffer));
        EXPECT(c.make == 0 || c.make > buffer);
        EXPECT(c.chunk >= 2 * MIB || c.threads * c.chunk >= bytes);
    }
}

// A solve as far as a plan looks at it (nothing of it is on a device).
static void shape(lbm3d_solver& h, int nx, int ny, int nz, int precision)
{
    std::memset(&h.p, 0, sizeof h.p);
    h.p.nx = nx;
    h.p.ny = ny;
    h.p.nz = nz;
    h.p.precision = precision;
    h.mode = precision;
    h.g = lbm3d::make_grid(&h.p);
}

// Bytes build asks for: the least room it does not refuse (with room, it fails
// where it would copy the tables to the device that is not there).
static size_t room(const std::vector<lbm3d_solver*>& members, int tz)
{
    static char somewhere[256];
    size_t lo = 0, hi = (size_t)1 << 26;  // refused, enough
    while (hi - lo > 1) {
        lbm3d::BatchPlan plan;
        const size_t mid = (lo + hi) / 2;
        const int32_t rc = plan.build(members, nullptr, tz, somewhere, mid);
        EXPECT(rc == LBM3D_E_NOMEM || rc == LBM3D_E_DEVICE);
        (rc == LBM3D_E_NOMEM ? lo : hi) = mid;
    }
    return hi;
}

static void check_tables()
{
    EXPECT(lbm3d::noalloc_scratch_bytes() <= 4 * MIB + MIB / 16);
    // thin and long: by blocks an entry per 64 planes, in few tiles if tiled
    for (int precision : {LBM3D_FP64, LBM3D_FP32}) {
        lbm3d_solver a, b;
        shape(a, 3, 2, 60000, precision);
        shape(b, 9, 4, 30000, precision);
        const std::vector<lbm3d_solver*> members{&a, &b};
        std::vector<lbm3d::BatchMember> shapes;
        for (lbm3d_solver* h : members) shapes.push_back(lbm3d::BatchMember{h->g, h->bc});
        EXPECT(!lbm3d::plan_groups(precision, shapes, 0, lbm3d::device_cus())[0].tiled);
        const int depth = lbm3d::batch_model_depth(precision, shapes, lbm3d::device_cus());
        const size_t tiled = room(members, depth);
        EXPECT(room(members, 0) == tiled && tiled <= lbm3d::BatchPlan::table_bytes(members) + 1024);
    }
}

static void check_no_memory()
{
    lbm3d_params ps[3];
    const int grids[3][3] = {{192, 128, 128}, {40, 33, 20}, {128, 64, 64}};
    for (int k = 0; k < 3; k++) {
        lbm3d_solver h;
        shape(h, grids[k][0], grids[k][1], grids[k][2], LBM3D_FP32);
        ps[k] = h.p;
        ps[k].c1 = ps[k].eta0 = 8;
        ps[k].c2 = 24;
        ps[k].gamma = 1.4;
        ps[k].tau = ps[k].dt = 1e-5;
        ps[k].dx = 1.0 / 256;
    }
    int32_t n = 0, group[3], tiled[3];
    for (int which = 0; which < 2; which++) {
        int32_t rc = LBM3D_E_NOMEM;
        long allocations = 0;
        for (; rc == LBM3D_E_NOMEM && allocations < 100000; allocations++) {
            fail_at = allocations;
            rc = which ? lbm3d_batch_groups(ps, 3, 0, 256, group, tiled)
                       : lbm3d_batch_plan(ps, 3, -1, 256, &n, nullptr, nullptr, nullptr, 0, nullptr);
        }
        EXPECT(rc == LBM3D_OK && fail_at >= 0 && allocations > 3);
        fail_at = -1;
    }
}

int main()
{
    std::mt19937 rng(4711);
    check_no_memory();
    check_copies(rng);
    check_tables();
    if (failures) {
        std::fprintf(stderr, "%d rule checks failed\n", failures);
        return 1;
    }
    std::printf("rule checks passed\n");
    return 0;
}
