// Host-side solver object shared by the C ABI, the batched step and the
// server (internal).
#pragma once

#include "../../include/lbm3d.h"
#include "lbm3d_internal.h"

struct lbm3d_solver {
    lbm3d_params p{};
    int mode = 0;
    lbm3d::Grid g{};
    lbm3d::FaceBC bc{};
    lbm3d::TileCfg tile{};
    lbm3d::Model<double> md{};
    lbm3d::Model<float> mf{};
    int64_t n = 0;             // interior nodes
    size_t bytes = 0;          // device bytes held
    void* mem = nullptr;       // one allocation for everything below
    void* f[2] = {nullptr, nullptr};
    double* q5 = nullptr;      // 5 x n staging for init / moments
    double* partial = nullptr; // per-block totals
    double* out5 = nullptr;
    uint32_t* health = nullptr;
    int nred = 0;
    bool layers_stale = false; // the current level's boundary layers in memory are an older level's: the
                               // untiled kernel forms layers itself, the tiled ones read some from memory
    bool upwind2 = false;      // the second-order upwind variant (steps untiled)
    int cur = 0;               // buffer holding the current level
    int64_t steps = 0;
    int64_t read_steps = 0;    // the step count when the fields or the state were last read back
    bool initialised = false;
    hipStream_t own_stream = nullptr;
    hipStream_t stream = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    hipGraphExec_t graph_exec[2] = {nullptr, nullptr};
    lbm3d_solver();
    ~lbm3d_solver();
};

namespace lbm3d {

constexpr int GRAPH_STEPS = 32;  // steps per captured graph (even)

int32_t validate(const lbm3d_params* p);
Model<double> make_model(const lbm3d_params* p);
Model<float> model_to_float(const Model<double>& d);
Grid make_grid(const lbm3d_params* p);
size_t elem_size(int precision);
size_t f_bytes(const Grid& g, int precision);
size_t footprint_of(const lbm3d_params* p);
int32_t solver_create(const lbm3d_params* p, lbm3d_solver** out);
int32_t solver_enqueue_steps(lbm3d_solver* h, int64_t nsteps);
// What f returns, or E_NOMEM if it throws: plans and their tables are host
// allocations, and nothing may leave a C entry point, or end a server's worker.
template <typename F>
int32_t no_throw(F&& f) noexcept
{
    try {
        return f();
    } catch (...) {
        return LBM3D_E_NOMEM;
    }
}
// ---- host copies (lbm3d_api.cpp) ----
// dst[0 .. n) = src[0 .. n), by several threads where that pays.
void copy_host(double* dst, const double* src, size_t n);
struct HostCopy {
    void* host;
    void* dev;
    size_t bytes;
};
// How a transfer of `total` bytes goes when the pinned buffer has `buffer`
// bytes (0: there is none) and `passed` bytes have gone through the runtime
// for want of it, making it worth while now or not yet (`now`): by `threads`
// threads in chunks of `chunk` bytes, after making a buffer of `make` bytes if
// that is not 0, or, with no threads, through the runtime, `wants` saying that
// the buffer would have served.
struct CopyPlan {
    unsigned threads = 0;
    size_t chunk = 0, make = 0;
    bool wants = false;
};
CopyPlan copy_plan(size_t total, bool down, size_t buffer, size_t passed, bool now);
// Copies between caller memory and the device, after the work on s, complete
// when s has been waited for; until then the host memory must stay as it is,
// in both directions (pinned memory is read by the device itself).  `beside`:
// the device has 2 ms of work and more to do before it.
hipError_t copy_to_host(const HostCopy* items, int n, bool beside, hipStream_t s);
hipError_t copy_to_device(const HostCopy* items, int n, hipStream_t s);
// The pinned buffer those copies go through exists while a user of it does
// (every solver and server is one).
void staging_ref();
void staging_unref();

// Stability admission of an initial state (lbm3d_admit): E_UNSTABLE if the
// von Neumann analysis at the state's extremes exceeds 1 + STABILITY_TOL.
constexpr double STABILITY_TOL = 1e-3;
int32_t admission(const lbm3d_params* p, const double* rho, const double* ux, const double* uy, const double* uz,
                  const double* pr, double* worst);
// autotuner results (lbm3d_tune.cpp): the tuned tile of a solve shape, and
// the set or tuned batch tile depth of a precision (0 if there is none), and
// whether it was set (lbm3d_batch_set_depth)
bool cached_tile(int mode, const Grid& g, const FaceBC& bc, TileCfg* out);
int batch_tile_depth(int mode);
bool batch_depth_set(int mode);

}  // namespace lbm3d
