// Host runtime and C ABI of the lbm3d library: parameter validation, device
// state, step loops replayed from captured HIP graphs, moments, totals,
// checkpoints.  The batched step and the server live in their own files.
#include "lbm3d_api_impl.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

using namespace lbm3d;

namespace lbm3d {

static bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

int32_t validate(const lbm3d_params* p)
{
    if (!p) return LBM3D_E_INVAL;
    const int32_t n[3] = {p->nx, p->ny, p->nz};
    for (int a = 0; a < 3; a++) {
        if (n[a] < 1 || n[a] > (1 << 20)) return LBM3D_E_INVAL;
        const int lo = p->bc[2 * a], hi = p->bc[2 * a + 1];
        if (lo < LBM3D_PERIODIC || lo > LBM3D_REFLECT || hi < LBM3D_PERIODIC || hi > LBM3D_REFLECT)
            return LBM3D_E_INVAL;
        if ((lo == LBM3D_PERIODIC) != (hi == LBM3D_PERIODIC)) return LBM3D_E_INVAL;
        if (lo != LBM3D_PERIODIC && n[a] < 2) return LBM3D_E_INVAL;
    }
    if (p->nz > 65535) return LBM3D_E_INVAL;
    {
        // one velocity plane (with boundary layers and padding) must be
        // addressable with 32-bit element offsets
        const double plane = (double)(p->nx + 64 + NG) * (p->ny + 2 * NG) * (p->nz + 2 * NG);
        if (plane > 2.0e9) return LBM3D_E_INVAL;
    }
    if (!finite_pos(p->c1) || !finite_pos(p->c2) || !finite_pos(p->eta0)) return LBM3D_E_INVAL;
    if (p->c1 == p->c2) return LBM3D_E_INVAL;  // A_i and B_i divide by c1^2 - c2^2
    if (!std::isfinite(p->gamma) || !(p->gamma > 1.0)) return LBM3D_E_INVAL;
    if (!finite_pos(p->tau) || !finite_pos(p->dt) || !finite_pos(p->dx)) return LBM3D_E_INVAL;
    if (p->precision < LBM3D_FP64 || p->precision > LBM3D_FP32_T64) return LBM3D_E_INVAL;
    if (p->flags & ~(uint32_t)(LBM3D_NO_DISSIPATION | LBM3D_UPWIND2 | LBM3D_CHECK_STABILITY | LBM3D_VELOCITY_MAJOR))
        return LBM3D_E_INVAL;
    for (int face = 0; face < 6; face++) {
        if (p->bc[face] != LBM3D_INFLOW) continue;
        const double* s = p->inflow[face];
        if (!finite_pos(s[0]) || !finite_pos(s[4])) return LBM3D_E_INVAL;
        if (!std::isfinite(s[1]) || !std::isfinite(s[2]) || !std::isfinite(s[3])) return LBM3D_E_INVAL;
    }
    // explicit-step admission: Courant number of the diagonal velocities,
    // diffusion number of the rest particle, relaxation factor dt/tau
    const double cfl = std::sqrt(3.0) * p->c2 * p->dt / p->dx;
    const double dif = (p->flags & LBM3D_NO_DISSIPATION) ? 0.0 : 6.0 * p->c1 * p->dt / p->dx;
    if (cfl > 1.0 || dif > 1.0 || p->dt / p->tau > 2.0) return LBM3D_E_UNSTABLE;
    return LBM3D_OK;
}

Model<double> make_model(const lbm3d_params* p)
{
    Model<double> m;
    const double c1 = p->c1, c2 = p->c2, e0 = p->eta0;
    const double b = 2.0 / (p->gamma - 1.0);
    const double c1s = c1 * c1, c2s = c2 * c2, e0s = e0 * e0;
    m.c1 = c1;
    m.k = c2 / std::sqrt(3.0);
    m.c1sq = c1s;
    m.c2sq = c2s;
    m.e0sq = e0s;
    m.inv_b = 1.0 / b;
    // Eq. (e18): rest A_1 = (b-3) T / eta0^2
    m.r_aT = (b - 3.0) / e0s;
    // axis group i = 2..7
    const double ia = 1.0 / (6.0 * (c1s - c2s));
    m.x_a0 = -c2s * ia;
    m.x_aT = ((b - 3.0) * c2s / e0s + 3.0) * ia;
    m.x_au = c2s / c1s * ia;
    const double ib = 1.0 / (2.0 * c1s * (c1s - c2s));
    m.x_b0 = -c2s * ib;
    m.x_bT = (b + 2.0) * ib;
    m.x_bu = ib;
    m.x_d = 1.0 / (2.0 * c1s * c1s);
    // diagonal group i = 8..15
    const double da = 1.0 / (8.0 * (c2s - c1s));
    m.d_a0 = -c1s * da;
    m.d_aT = ((b - 3.0) * c1s / e0s + 3.0) * da;
    m.d_au = (3.0 * c1s - c2s) / (2.0 * c2s) * da;
    const double db = 3.0 / (8.0 * c2s * (c2s - c1s));
    m.d_b0 = -c1s * db;
    m.d_bT = (b + 2.0) * db;
    m.d_bu = db;
    m.d_d = 9.0 / (16.0 * c2s * c2s);
    // time-step factors; lambda_i of Eq. (lp): c1 dx (rest), c1 dx / 10 (axis), 0 (diagonal)
    m.k_adv = p->dt / p->dx;
    m.k_bgk = p->dt / p->tau;
    const bool diss = !(p->flags & LBM3D_NO_DISSIPATION);
    m.k_lap0 = diss ? c1 * p->dx * p->dt / (p->dx * p->dx) : 0.0;
    m.k_lap1 = diss ? c1 * p->dx / 10.0 * p->dt / (p->dx * p->dx) : 0.0;
    m.a1 = m.k_adv * m.c1;
    m.ad = m.k_adv * m.k;
    return m;
}

Model<float> model_to_float(const Model<double>& d)
{
    Model<float> f;
    const double* src = reinterpret_cast<const double*>(&d);
    float* dst = reinterpret_cast<float*>(&f);
    static_assert(sizeof(Model<double>) == 2 * sizeof(Model<float>), "model layout");
    for (size_t i = 0; i < sizeof(Model<float>) / sizeof(float); i++) dst[i] = (float)src[i];
    return f;
}


size_t footprint_of(const lbm3d_params* p)
{
    const Grid g = make_grid(p);
    const size_t n = (size_t)p->nx * p->ny * p->nz;
    return 2 * f_bytes(g, p->precision) + 5 * n * sizeof(double) + 1024 * 5 * sizeof(double) + 4096;
}

}  // namespace lbm3d

// ------------------------------------------------------------- host copies --
// Fields come from and go to pageable memory of the caller.  The runtime
// copies that through its own pinned buffer with one thread, whose memcpy and,
// in fresh memory, page faults hold the transfer to 8 - 18 GB/s; here several
// threads each move chunks through a slot of a pinned buffer of the library.
// Reading back the five fields of a 128^3 solve (84 MB) takes 2.1 ms instead
// of 4.7, an FP64 state of it (252 MB, fresh memory) 14 instead of 27.
namespace lbm3d {

constexpr unsigned COPY_THREADS = 8, COPY_FEW = 5;
constexpr size_t COPY_SLOT = (size_t)4 << 20, COPY_SMALL_SLOT = (size_t)2 << 20;  // bytes of a slot, the largest chunk
constexpr size_t COPY_HOST_CHUNK = (size_t)1 << 20, COPY_HOST_MIN = (size_t)2 << 20;  // copies within the host
// Below COPY_MIN (to the host) and COPY_MIN_UP, one thread and the runtime's
// own path: to the host, starting the threads costs some 0.1 ms (3 MiB 0.18 -
// 0.25 ms either way); from it, the runtime stages small copies at 30 GB/s (16
// MB 0.52 ms against 0.66, 24 MB 0.81 against 0.93) and large ones at 8 (126 MB
// 15.6 ms against 5.9).  To the host, in memory touched before and in memory
// fresh from the system, whose page faults are shared out: 4 MiB by the runtime
// 0.22 and 0.85 ms, by five threads 0.23 and 0.45, by eight 0.30 and 0.45; 10
// MiB 0.60 and 2.5, 0.40 and 1.0, 0.44 and 0.86; 24 MiB 1.4 and 5.8, 0.76 and
// 2.1, 0.79 and 1.7.  Hence five threads below COPY_FEW_BELOW and eight above.
// Slots of 2 MiB (1 MiB: 24 MiB 0.93 ms instead of 0.79), and of 4 MiB where
// the buffer is worth it (84 MiB 2.06 ms instead of 2.25).
constexpr size_t COPY_MIN = (size_t)4 << 20, COPY_FEW_BELOW = (size_t)10 << 20;
constexpr size_t COPY_MIN_UP = (size_t)32 << 20, COPY_MANY = (size_t)32 << 20;

// Making the buffer costs 1.5 - 2.5 ms (its pages are faulted in) where a
// transfer of 10 MiB gains 0.2 ms in touched and 1.6 ms in fresh memory.  So it
// is made by a transfer that gains more than that by itself (COPY_MANY), beside
// that much work still queued on the device, where another solve or a server
// will keep it (`now`), or once as much has gone through the runtime for want
// of it (COPY_EARN).  A 64^3 solve created, stepped 5 times, read back and
// destroyed: 1.6 ms, and 5.3 - 6.5 with a buffer each time; 96x64x64 stepped
// 250 times and read back: 4.5 ms with a buffer each time, 5.0 without.
constexpr size_t COPY_EARN = (size_t)32 << 20;
CopyPlan copy_plan(size_t total, bool down, size_t buffer, size_t passed, bool now)
{
    CopyPlan p;
    if (total < (down ? COPY_MIN : COPY_MIN_UP)) return p;
    const bool many = total >= COPY_MANY;
    const unsigned threads = total < COPY_FEW_BELOW ? COPY_FEW : COPY_THREADS;
    const size_t slot = many ? COPY_SLOT : COPY_SMALL_SLOT;
    p.wants = true;
    if (buffer < COPY_THREADS * slot) {
        if (!many && !now && passed + total < COPY_EARN) return p;
        p.make = COPY_THREADS * slot;
    }
    p.threads = threads;
    p.chunk = std::min(((total + threads - 1) / threads + 65535) & ~(size_t)65535, slot);
    return p;
}

// Runs work(k) for k = 0 .. chunks - 1 (none may throw) on up to COPY_THREADS
// threads, the calling one among them: it does all that is left if no other
// can be started.
template <typename Work>
static void for_chunks(size_t chunks, const Work& work)
{
    std::atomic<size_t> next{0};
    auto loop = [&] {
        for (size_t k; (k = next.fetch_add(1)) < chunks;) work(k);
    };
    const size_t want = std::min<size_t>({chunks, COPY_THREADS, std::max(1u, std::thread::hardware_concurrency())});
    std::vector<std::thread> more;
    try {
        more.reserve(want);
        for (size_t t = 1; t < want; t++) more.emplace_back(loop);
    } catch (...) {
        // (the threads there are, or this one alone, do the rest)
    }
    loop();
    for (std::thread& t : more) t.join();
}

void copy_host(double* dst, const double* src, size_t n)
{
    constexpr size_t per = COPY_HOST_CHUNK / sizeof(double);
    if (n * sizeof(double) < COPY_HOST_MIN) {
        std::memcpy(dst, src, n * sizeof(double));
        return;
    }
    for_chunks((n + per - 1) / per, [&](size_t k) {
        const size_t a = k * per, m = std::min(per, n - a);
        std::memcpy(dst + a, src + a, m * sizeof(double));
    });
}

// Any rho <= 0 or p <= 0 or value that is not finite in n nodes?
static bool bad_state(size_t n, const double* rho, const double* ux, const double* uy, const double* uz, const double* p)
{
    constexpr size_t per = (size_t)1 << 17;
    std::atomic<bool> bad{false};
    auto check = [&](size_t c) {
        if (bad.load(std::memory_order_relaxed)) return;
        for (size_t k = c * per, e = std::min(n, k + per); k < e; k++)
            if (!finite_pos(rho[k]) || !finite_pos(p[k]) || !std::isfinite(ux[k]) || !std::isfinite(uy[k]) ||
                !std::isfinite(uz[k])) {
                bad = true;
                return;
            }
    };
    const size_t chunks = (n + per - 1) / per;
    if (chunks < 2)
        check(0);
    else
        for_chunks(chunks, check);
    return bad;
}

// The pinned buffer (16 or 32 MiB, see copy_plan), for one transfer at a time
// (another one meanwhile takes the runtime's own path), given back with the
// last user.
static std::mutex g_staging_mu;       // held by the transfer that uses the buffer
static char* g_staging = nullptr;
static size_t g_staging_bytes = 0;
static size_t g_passed = 0;           // bytes that went through the runtime for want of the buffer
static std::atomic<long> g_staging_users{0};

void staging_ref() { g_staging_users++; }
void staging_unref()
{
    if (--g_staging_users > 0) return;
    std::lock_guard<std::mutex> lk(g_staging_mu);
    if (g_staging_users != 0) return;
    if (g_staging) (void)hipHostFree(g_staging);
    g_staging = nullptr;
    g_staging_bytes = 0;
    g_passed = 0;
}

// Moves every chunk of the items through a slot; false (and nothing done) if
// the buffer is in use or there is none.
static bool staged(const HostCopy* items, int n, bool down, bool beside, hipStream_t s, hipError_t* result)
{
    struct Chunk {
        char* host;
        char* dev;
        size_t bytes;
    };
    size_t total = 0;
    for (int i = 0; i < n; i++) total += items[i].bytes;
    std::unique_lock<std::mutex> lk(g_staging_mu, std::try_to_lock);
    if (!lk.owns_lock()) return false;
    const CopyPlan plan = copy_plan(total, down, g_staging_bytes, g_passed, beside || g_staging_users > 1);
    if (!plan.threads) {
        if (plan.wants) g_passed += total;
        return false;
    }
    std::vector<Chunk> chunks;
    for (int i = 0; i < n; i++)
        for (size_t a = 0; a < items[i].bytes; a += plan.chunk)
            chunks.push_back(
                Chunk{(char*)items[i].host + a, (char*)items[i].dev + a, std::min(plan.chunk, items[i].bytes - a)});
    if (plan.make) {
        if (g_staging) (void)hipHostFree(g_staging);
        g_staging_bytes = 0;
        if (hipHostMalloc((void**)&g_staging, plan.make, hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();
            g_staging = nullptr;
            return false;
        }
        g_staging_bytes = plan.make;
    }
    // events belong to the device current when they are made and are recorded
    // on streams of it only: that of s, which the caller may have left
    int device = 0, mine = 0;
    if (hipStreamGetDevice(s, &device) != hipSuccess || hipGetDevice(&mine) != hipSuccess ||
        hipSetDevice(device) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    struct Back {
        int device;
        ~Back() { (void)hipSetDevice(device); }
    } back{mine};
    hipEvent_t done[COPY_THREADS] = {};
    for (unsigned t = 0; t < plan.threads; t++)
        if (hipEventCreateWithFlags(&done[t], hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            for (unsigned u = 0; u < t; u++) (void)hipEventDestroy(done[u]);
            return false;
        }
    std::atomic<size_t> next{0};
    std::atomic<int> error{hipSuccess};
    // one slot per worker, each chunk through it and out before the next
    for_chunks(std::min<size_t>(plan.threads, chunks.size()), [&](size_t w) {
        char* slot = g_staging + w * plan.chunk;
        hipError_t e = hipSetDevice(device);
        for (size_t k; e == hipSuccess && error == hipSuccess && (k = next.fetch_add(1)) < chunks.size();) {
            const Chunk& c = chunks[k];
            if (!down) std::memcpy(slot, c.host, c.bytes);
            e = down ? hipMemcpyAsync(slot, c.dev, c.bytes, hipMemcpyDeviceToHost, s)
                     : hipMemcpyAsync(c.dev, slot, c.bytes, hipMemcpyHostToDevice, s);
            if (e == hipSuccess) e = hipEventRecord(done[w], s);
            if (e == hipSuccess) e = hipEventSynchronize(done[w]);
            if (e == hipSuccess && down) std::memcpy(c.host, slot, c.bytes);
        }
        if (e != hipSuccess) error = e;
    });
    // (an error may leave a copy into a slot queued)
    if (error != hipSuccess) (void)hipStreamSynchronize(s);
    for (unsigned t = 0; t < plan.threads; t++) (void)hipEventDestroy(done[t]);
    *result = (hipError_t)error.load();
    return true;
}

// Memory that the runtime does not know?  (Pinned memory it reaches itself at
// the link's rate; device memory is not for the host to touch.)
static bool pageable(const void* p)
{
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return a.type == hipMemoryTypeUnregistered;
}

static hipError_t copy_items(const HostCopy* items, int n, bool down, bool beside, hipStream_t s)
{
    size_t total = 0;
    bool plain = true;
    for (int i = 0; i < n; i++) total += items[i].bytes;
    const bool large = total >= (down ? COPY_MIN : COPY_MIN_UP);
    if (large)
        for (int i = 0; i < n; i++) plain = plain && pageable(items[i].host);
    hipError_t e = hipSuccess;
    if (large && plain) try {
            if (staged(items, n, down, beside, s, &e)) return e;
        } catch (...) {
            // (no memory for the chunk list, before anything was copied)
        }
    e = hipSuccess;
    for (int i = 0; i < n && e == hipSuccess; i++)
        e = down ? hipMemcpyAsync(items[i].host, items[i].dev, items[i].bytes, hipMemcpyDeviceToHost, s)
                 : hipMemcpyAsync(items[i].dev, items[i].host, items[i].bytes, hipMemcpyHostToDevice, s);
    return e;
}
hipError_t copy_to_host(const HostCopy* items, int n, bool beside, hipStream_t s)
{
    return copy_items(items, n, true, beside, s);
}
hipError_t copy_to_device(const HostCopy* items, int n, hipStream_t s) { return copy_items(items, n, false, false, s); }

}  // namespace lbm3d

// ------------------------------------------------------------------ solver --
static int32_t dev_err(hipError_t e) { return e == hipSuccess ? LBM3D_OK : (e == hipErrorOutOfMemory ? LBM3D_E_NOMEM : LBM3D_E_DEVICE); }

#define HIPCHK(x)                                  \
    do {                                           \
        hipError_t _e = (x);                       \
        if (_e != hipSuccess) return dev_err(_e);  \
    } while (0)

lbm3d_solver::lbm3d_solver() { staging_ref(); }

lbm3d_solver::~lbm3d_solver()
{
    for (int k = 0; k < 2; k++)
        if (graph_exec[k]) (void)hipGraphExecDestroy(graph_exec[k]);
    if (ev0) (void)hipEventDestroy(ev0);
    if (ev1) (void)hipEventDestroy(ev1);
    if (own_stream) (void)hipStreamDestroy(own_stream);
    if (mem) (void)hipFree(mem);
    staging_unref();
}

namespace lbm3d {

int32_t solver_create(const lbm3d_params* p, lbm3d_solver** out)
{
    if (!out) return LBM3D_E_INVAL;
    *out = nullptr;
    int32_t rc = validate(p);
    if (rc) return rc;
    lbm3d_solver* h = new (std::nothrow) lbm3d_solver();
    if (!h) return LBM3D_E_NOMEM;
    h->p = *p;
    h->mode = p->precision;
    h->g = make_grid(p);
    h->md = make_model(p);
    h->mf = model_to_float(h->md);
    for (int f = 0; f < 6; f++) h->bc.kind[f] = p->bc[f];
    h->upwind2 = (p->flags & LBM3D_UPWIND2) != 0;
    h->tile = default_tile(h->mode, h->g);
    TileCfg tuned;
    if (cached_tile(h->mode, h->g, h->bc, &tuned) && tile_supported(h->mode, h->g, tuned)) h->tile = tuned;
    if (h->upwind2) {
        // the variant runs in the untiled kernel
        h->tile.by = 0;
        h->tile.tz = 1;
    }
    h->n = (int64_t)p->nx * p->ny * p->nz;
    const size_t fb = f_bytes(h->g, h->mode);
    h->nred = conserved_blocks(h->g);
    const size_t q5b = (size_t)5 * h->n * sizeof(double);
    const size_t redb = (size_t)h->nred * 5 * sizeof(double) + 8 * sizeof(double);
    h->bytes = 2 * fb + q5b + redb + 256;
    hipError_t e = hipMalloc(&h->mem, h->bytes);
    if (e != hipSuccess) {
        delete h;
        return dev_err(e);
    }
    char* base = (char*)h->mem;
    h->f[0] = base;
    h->f[1] = base + fb;
    h->q5 = (double*)(base + 2 * fb);
    h->partial = (double*)(base + 2 * fb + q5b);
    h->out5 = h->partial + (size_t)h->nred * 5;
    h->health = (uint32_t*)(h->out5 + 5);
    e = hipStreamCreateWithFlags(&h->own_stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreate(&h->ev0);
    if (e == hipSuccess) e = hipEventCreate(&h->ev1);
    // zero both buffers once so the unused padding never holds garbage
    if (e == hipSuccess) e = hipMemsetAsync(h->mem, 0, h->bytes, h->own_stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->own_stream);
    if (e != hipSuccess) {
        delete h;
        return dev_err(e);
    }
    h->stream = h->own_stream;
    *out = h;
    return LBM3D_OK;
}

// One time step of a solve: fused update f[cur] -> f[cur^1], then the
// boundary layers of the new level that the next step reads from memory.
static hipError_t enqueue_one(lbm3d_solver* h, int cur, hipStream_t s)
{
    hipError_t e = launch_step(h->mode, h->g, h->bc, h->tile, h->md, h->mf, h->p.inflow, h->f[cur], h->f[cur ^ 1],
                               h->health, s, h->upwind2);
    if (e != hipSuccess) return e;
    const uint32_t rest = ghost_faces(h->g, h->bc, h->tile.by != 0);
    if (!rest) return hipSuccess;
    return launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, false, h->f[cur ^ 1], s, rest);
}

// Before steps of the tiled kernel: the layers it reads from memory, if the
// solve last stepped untiled (as a member of a batch; lbm3d_set_tile
// refreshes them itself).
static hipError_t refresh_layers(lbm3d_solver* h)
{
    if (!h->layers_stale || h->tile.by == 0) return hipSuccess;
    const hipError_t e = launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, false, h->f[h->cur], h->stream,
                                       ghost_faces(h->g, h->bc, true));
    if (e == hipSuccess) h->layers_stale = false;
    return e;
}

// Does the device still have some 2 ms of a solve's steps to do (64 M node
// updates at 18 - 40 G/s, unless they have run since they were queued)?
static bool stepping(lbm3d_solver* h)
{
    if ((double)(h->steps - h->read_steps) * (double)h->n < 64.0 * 1048576.0) return false;
    const bool busy = hipStreamQuery(h->stream) == hipErrorNotReady;
    (void)hipGetLastError();
    return busy;
}

int32_t solver_enqueue_steps(lbm3d_solver* h, int64_t nsteps)
{
    hipStream_t s = h->stream;
    if (nsteps > 0) HIPCHK(refresh_layers(h));
    int64_t left = nsteps;
    // runs of GRAPH_STEPS steps are replayed from a graph captured once per
    // starting buffer (the step count is even, so the run ends where it began)
    while (left >= GRAPH_STEPS) {
        hipGraphExec_t& ge = h->graph_exec[h->cur];
        if (!ge) {
            hipGraph_t graph = nullptr;
            hipStream_t cs = h->own_stream;
            HIPCHK(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
            hipError_t e = hipSuccess;
            int c = h->cur;
            for (int k = 0; k < GRAPH_STEPS && e == hipSuccess; k++) {
                e = enqueue_one(h, c, cs);
                c ^= 1;
            }
            hipError_t e2 = hipStreamEndCapture(cs, &graph);
            if (e != hipSuccess) {
                if (graph) (void)hipGraphDestroy(graph);
                return dev_err(e);
            }
            HIPCHK(e2);
            e = hipGraphInstantiate(&ge, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            HIPCHK(e);
        }
        HIPCHK(hipGraphLaunch(ge, s));
        left -= GRAPH_STEPS;
        h->steps += GRAPH_STEPS;
        if (h->tile.by == 0) h->layers_stale = true;
    }
    for (; left > 0; left--) {
        HIPCHK(enqueue_one(h, h->cur, s));
        h->cur ^= 1;
        h->steps++;
        if (h->tile.by == 0) h->layers_stale = true;
    }
    return LBM3D_OK;
}

}  // namespace lbm3d

// ------------------------------------------------------------------- C ABI --
extern "C" {

const char* lbm3d_version(void) { return "lbm3d 0.1 (gfx950)"; }

const char* lbm3d_strerror(int32_t code)
{
    switch (code) {
    case LBM3D_OK: return "ok";
    case LBM3D_E_INVAL: return "invalid argument";
    case LBM3D_E_UNSTABLE: return "explicit step not admitted (Courant, diffusion or relaxation number too large)";
    case LBM3D_E_NOMEM: return "out of memory or over budget";
    case LBM3D_E_DEVICE: return "HIP runtime error";
    case LBM3D_E_STATE: return "call out of order";
    case LBM3D_E_NONFINITE: return "solution is not finite";
    case LBM3D_E_NOTFOUND: return "unknown ticket";
    case LBM3D_E_CANCELLED: return "cancelled";
    default: return "unknown status";
    }
}

int32_t lbm3d_device_count(int32_t* count)
{
    if (!count) return LBM3D_E_INVAL;
    int c = 0;
    hipError_t e = hipGetDeviceCount(&c);
    *count = (e == hipSuccess) ? c : 0;
    return LBM3D_OK;
}

int32_t lbm3d_footprint(const lbm3d_params* p, size_t* bytes)
{
    if (!bytes) return LBM3D_E_INVAL;
    int32_t rc = validate(p);
    if (rc) return rc;
    *bytes = footprint_of(p);
    return LBM3D_OK;
}

int32_t lbm3d_create(const lbm3d_params* p, lbm3d_t* out)
{
    return no_throw([&] { return solver_create(p, out); });
}

int32_t lbm3d_destroy(lbm3d_t h)
{
    if (!h) return LBM3D_OK;
    (void)hipStreamSynchronize(h->stream);
    delete h;
    return LBM3D_OK;
}

int32_t lbm3d_set_stream(lbm3d_t h, void* hip_stream)
{
    if (!h) return LBM3D_E_INVAL;
    HIPCHK(hipStreamSynchronize(h->stream));
    h->stream = hip_stream ? (hipStream_t)hip_stream : h->own_stream;
    return LBM3D_OK;
}

int32_t lbm3d_init(lbm3d_t h, const double* rho, const double* ux, const double* uy, const double* uz,
                   const double* p)
{
    if (!h || !rho || !ux || !uy || !uz || !p) return LBM3D_E_INVAL;
    if (bad_state((size_t)h->n, rho, ux, uy, uz, p)) return LBM3D_E_INVAL;
    if (h->p.flags & LBM3D_CHECK_STABILITY) {
        const int32_t rc = no_throw([&] { return admission(&h->p, rho, ux, uy, uz, p, nullptr); });
        if (rc) return rc;
    }
    hipStream_t s = h->stream;
    const double* src[5] = {rho, ux, uy, uz, p};
    HostCopy up[5];
    for (int c = 0; c < 5; c++)
        up[c] = HostCopy{const_cast<double*>(src[c]), h->q5 + (size_t)c * h->n, (size_t)h->n * sizeof(double)};
    HIPCHK(copy_to_device(up, 5, s));
    HIPCHK(launch_init(h->mode, h->g, h->md, h->q5, h->f[0], s));
    HIPCHK(launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, true, h->f[0], s));
    // the fixed-state layers never change: write them into the other buffer too
    HIPCHK(launch_init(h->mode, h->g, h->md, h->q5, h->f[1], s));
    HIPCHK(launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, true, h->f[1], s));
    HIPCHK(hipMemsetAsync(h->health, 0, sizeof(uint32_t), s));
    HIPCHK(hipStreamSynchronize(s));
    h->cur = 0;
    h->steps = h->read_steps = 0;
    h->layers_stale = false;
    h->initialised = true;
    return LBM3D_OK;
}

int32_t lbm3d_step(lbm3d_t h, int64_t nsteps)
{
    if (!h || nsteps < 0) return LBM3D_E_INVAL;
    if (!h->initialised) return LBM3D_E_STATE;
    return solver_enqueue_steps(h, nsteps);
}

int32_t lbm3d_step_timed(lbm3d_t h, int64_t nsteps, double* ms)
{
    if (!h || nsteps < 0) return LBM3D_E_INVAL;
    if (!h->initialised) return LBM3D_E_STATE;
    HIPCHK(hipEventRecord(h->ev0, h->stream));
    int32_t rc = solver_enqueue_steps(h, nsteps);
    if (rc) return rc;
    HIPCHK(hipEventRecord(h->ev1, h->stream));
    HIPCHK(hipEventSynchronize(h->ev1));
    float t = 0.0f;
    HIPCHK(hipEventElapsedTime(&t, h->ev0, h->ev1));
    if (ms) *ms = (double)t;
    return LBM3D_OK;
}

int32_t lbm3d_step_profiled(lbm3d_t h, int64_t nsteps, double* total_ms, double* step_kernel_ms)
{
    if (!h || nsteps < 1) return LBM3D_E_INVAL;
    if (!h->initialised) return LBM3D_E_STATE;
    std::vector<hipEvent_t> ev;
    const int32_t room = no_throw([&]() -> int32_t {
        ev.assign((size_t)2 * nsteps, nullptr);
        return LBM3D_OK;
    });
    if (room != LBM3D_OK) return room;
    hipError_t e = hipSuccess;
    for (auto& x : ev)
        if (e == hipSuccess) e = hipEventCreate(&x);
    hipStream_t s = h->stream;
    if (e == hipSuccess) e = refresh_layers(h);
    if (e == hipSuccess) e = hipEventRecord(h->ev0, s);
    for (int64_t k = 0; k < nsteps && e == hipSuccess; k++) {
        const int c = h->cur;
        // the step kernel's own dispatch records its start and end (no
        // markers of their own around it, whose overhead would count)
        e = launch_step(h->mode, h->g, h->bc, h->tile, h->md, h->mf, h->p.inflow, h->f[c], h->f[c ^ 1],
                        h->health, s, h->upwind2, ev[2 * k], ev[2 * k + 1]);
        const uint32_t rest = ghost_faces(h->g, h->bc, h->tile.by != 0);
        if (e == hipSuccess && rest)
            e = launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, false, h->f[c ^ 1], s, rest);
        if (e == hipSuccess) {
            h->cur ^= 1;
            h->steps++;
            if (h->tile.by == 0) h->layers_stale = true;
        }
    }
    if (e == hipSuccess) e = hipEventRecord(h->ev1, s);
    if (e == hipSuccess) e = hipEventSynchronize(h->ev1);
    double ksum = 0.0;
    float t = 0.0f;
    for (int64_t k = 0; k < nsteps && e == hipSuccess; k++) {
        e = hipEventElapsedTime(&t, ev[2 * k], ev[2 * k + 1]);
        ksum += t;
    }
    if (e == hipSuccess) e = hipEventElapsedTime(&t, h->ev0, h->ev1);
    for (auto& x : ev)
        if (x) (void)hipEventDestroy(x);
    if (e != hipSuccess) return dev_err(e);
    if (total_ms) *total_ms = (double)t;
    if (step_kernel_ms) *step_kernel_ms = ksum / (double)nsteps;
    return LBM3D_OK;
}

// A new launch shape (or store kind) for the solve's next steps.
static int32_t set_launch(lbm3d_t h, const TileCfg& t)
{
    if (!tile_supported(h->mode, h->g, t) || (h->upwind2 && t.by != 0)) return LBM3D_E_INVAL;
    HIPCHK(hipStreamSynchronize(h->stream));
    for (int k = 0; k < 2; k++)
        if (h->graph_exec[k]) {
            (void)hipGraphExecDestroy(h->graph_exec[k]);
            h->graph_exec[k] = nullptr;
        }
    h->tile = t;
    // the layers a step forms itself are not kept in memory: refresh them
    // all, so any launch shape can take over
    if (h->initialised) {
        HIPCHK(launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, true, h->f[h->cur], h->stream));
        h->layers_stale = false;
        HIPCHK(hipStreamSynchronize(h->stream));
    }
    return LBM3D_OK;
}

int32_t lbm3d_set_tile(lbm3d_t h, int32_t by, int32_t tz)
{
    if (!h) return LBM3D_E_INVAL;
    TileCfg t = h->tile;  // (the store kind is kept)
    t.by = by;
    t.tz = tz;
    return set_launch(h, t);
}

int32_t lbm3d_set_streaming(lbm3d_t h, int32_t streaming)
{
    if (!h || (streaming != 0 && streaming != 1)) return LBM3D_E_INVAL;
    TileCfg t = h->tile;
    t.stream = streaming == 1;
    return set_launch(h, t);
}

int32_t lbm3d_get_streaming(lbm3d_t h, int32_t* streaming)
{
    if (!h || !streaming) return LBM3D_E_INVAL;
    *streaming = h->tile.stream ? 1 : 0;
    return LBM3D_OK;
}

int32_t lbm3d_get_tile(lbm3d_t h, int32_t* by, int32_t* tz)
{
    if (!h) return LBM3D_E_INVAL;
    if (by) *by = h->tile.by;
    if (tz) *tz = h->tile.tz;
    return LBM3D_OK;
}

int32_t lbm3d_sync(lbm3d_t h)
{
    if (!h) return LBM3D_E_INVAL;
    HIPCHK(hipStreamSynchronize(h->stream));
    return LBM3D_OK;
}

int32_t lbm3d_moments(lbm3d_t h, double* rho, double* ux, double* uy, double* uz, double* p)
{
    if (!h) return LBM3D_E_INVAL;
    if (!h->initialised) return LBM3D_E_STATE;
    hipStream_t s = h->stream;
    const bool beside = stepping(h);
    h->read_steps = h->steps;
    HIPCHK(launch_moments(h->mode, h->g, h->md, h->f[h->cur], h->q5, s));
    double* dst[5] = {rho, ux, uy, uz, p};
    HostCopy down[5];
    int n = 0;
    for (int c = 0; c < 5; c++)
        if (dst[c]) down[n++] = HostCopy{dst[c], h->q5 + (size_t)c * h->n, (size_t)h->n * sizeof(double)};
    HIPCHK(copy_to_host(down, n, beside, s));
    uint32_t hw = 0;
    HIPCHK(hipMemcpyAsync(&hw, h->health, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    return (hw & LBM3D_HEALTH_NONFINITE) ? LBM3D_E_NONFINITE : LBM3D_OK;
}

int32_t lbm3d_conserved(lbm3d_t h, double out[5])
{
    if (!h || !out) return LBM3D_E_INVAL;
    if (!h->initialised) return LBM3D_E_STATE;
    hipStream_t s = h->stream;
    HIPCHK(launch_conserved(h->mode, h->g, h->md, h->f[h->cur], h->partial, h->nred, h->out5, s));
    HIPCHK(hipMemcpyAsync(out, h->out5, 5 * sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    return LBM3D_OK;
}

int32_t lbm3d_status(lbm3d_t h, uint32_t* health, int64_t* steps_done)
{
    if (!h) return LBM3D_E_INVAL;
    uint32_t hw = 0;
    HIPCHK(hipMemcpyAsync(&hw, h->health, sizeof(uint32_t), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    if (health) *health = hw;
    if (steps_done) *steps_done = h->steps;
    return LBM3D_OK;
}

int32_t lbm3d_poison_next(lbm3d_t h)
{
    if (!h) return LBM3D_E_INVAL;
    if (!h->initialised) return LBM3D_E_STATE;
    hipStream_t s = h->stream;
    // all ones is a quiet NaN in both float and double
    HIPCHK(hipMemsetAsync(h->f[h->cur ^ 1], 0xff, f_bytes(h->g, h->mode), s));
    // the fixed-state layers are written once per buffer (at init), not by
    // the steps: restore them
    HIPCHK(launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, true, h->f[h->cur ^ 1], s, 0u));
    HIPCHK(hipStreamSynchronize(s));
    return LBM3D_OK;
}

int32_t lbm3d_get_f(lbm3d_t h, void* host, size_t bytes)
{
    if (!h || !host) return LBM3D_E_INVAL;
    if (!h->initialised) return LBM3D_E_STATE;
    const size_t need = (size_t)NV * h->n * elem_size(h->mode);
    if (bytes != need) return LBM3D_E_INVAL;
    const bool beside = stepping(h);
    h->read_steps = h->steps;
    void* dense = nullptr;
    HIPCHK(hipMalloc(&dense, need));
    hipStream_t s = h->stream;
    hipError_t e = launch_pack(h->mode, h->g, h->f[h->cur], dense, true, s);
    const HostCopy down{host, dense, need};
    if (e == hipSuccess) e = copy_to_host(&down, 1, beside, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(dense);
    return dev_err(e);
}

int32_t lbm3d_set_f(lbm3d_t h, const void* host, size_t bytes)
{
    if (!h || !host) return LBM3D_E_INVAL;
    if (!h->initialised) return LBM3D_E_STATE;
    const size_t need = (size_t)NV * h->n * elem_size(h->mode);
    if (bytes != need) return LBM3D_E_INVAL;
    void* dense = nullptr;
    HIPCHK(hipMalloc(&dense, need));
    hipStream_t s = h->stream;
    const HostCopy up{const_cast<void*>(host), dense, need};
    hipError_t e = copy_to_device(&up, 1, s);
    if (e == hipSuccess) e = launch_pack(h->mode, h->g, h->f[h->cur], dense, false, s);
    if (e == hipSuccess)
        e = launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, true, h->f[h->cur], s);
    if (e == hipSuccess) h->layers_stale = false;
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(dense);
    return dev_err(e);
}

}  // extern "C"
