// Batched stepping of many solves with one launch per step (internal).
#pragma once

#include <vector>

#include "lbm3d_api_impl.h"

namespace lbm3d {

// Work plan of a batched step, computed on the host: the tiles of every
// member split into per-XCD lists (see plan_tiles).
struct TilePlan {
    std::vector<BatchTile> tiles;  // list 0's tiles, then list 1's, ...
    BatchQueue queue{};            // list boundaries; counters zero
    int nlists = 0;                // lists (one per XCD, fewer for tiny batches)
    int nblocks = 0;               // persistent workgroups, a multiple of nlists
    double cost[BATCH_MAX_LISTS] = {};  // planes marched per list (balance)
};

// Tiles of 64 x `by` x `tz` nodes (tz >= nz: whole columns) over the grids,
// for `cus` compute units.  Each member's tiles are cut into contiguous
// pieces (row slabs, which share their halo rows through one L2), the pieces
// are dealt to the lists largest first onto the least-loaded list, and each
// list runs its deepest tiles first.  Host only.
int32_t plan_tiles(const std::vector<Grid>& grids, int by, int tz, int cus, TilePlan& out);

// What the plan of a batch depends on of a member.
struct BatchMember {
    Grid g;
    FaceBC bc;
};
// Members stepped by one launch (their places in the membership), by the
// tiled kernel or by untiled blocks.
struct GroupMembers {
    std::vector<int32_t> who;
    int64_t bytes = 0;
    bool tiled = false;
    int depth = 0;  // of a tiled group, where the grouping has found it
};
// The groups of a plan at tile depth tz (as for BatchPlan::build): all members
// tiled in one group where the caller asks for a depth (tz > 0, or the
// precision's was set by lbm3d_batch_set_depth), or where a model of both
// kernels finds that the faster; else cache-sized groups of untiled blocks and
// one of the larger members, tiled.  Host only.
std::vector<GroupMembers> plan_groups(int mode, const std::vector<BatchMember>& members, int tz, int cus);
// The launch model's depth for these members, were they all tiled.
int batch_model_depth(int mode, const std::vector<BatchMember>& members, int cus);

// A fixed set of solves (one precision) advanced together, group by group
// (see plan_groups): a device table of the solves, the work items of each
// group and one launch per step and group (and one for the boundary layers
// tiles leave to memory); runs of steps are replayed from captured graphs.
class BatchPlan {
public:
    BatchPlan() = default;
    ~BatchPlan();
    BatchPlan(const BatchPlan&) = delete;
    BatchPlan& operator=(const BatchPlan&) = delete;

    // (Re)build for `members` (all initialised, same precision); each
    // member's current buffer is taken as parity 0.  Enqueued on `s`.
    // `tz` > 0 sets the tile depth of every member; 0 takes the set or tuned
    // depth of the precision, else the launch model's; < 0 the launch model's.
    // The device tables go into a buffer the plan allocates, or, with
    // `dev` != nullptr, into the caller's `cap` bytes at `dev` (then nothing
    // is allocated; the members go tiled in one group if the tables of more
    // groups do not fit, and E_NOMEM is returned if those do not either).
    int32_t build(const std::vector<lbm3d_solver*>& members, hipStream_t s, int tz = 0,
                  void* dev = nullptr, size_t cap = 0);
    // Device bytes the tables of `members` need at tile depth tz (0: the
    // depth as for build).
    static size_t table_bytes(const std::vector<lbm3d_solver*>& members, int tz = 0);
    // One step of every member from its buffer of the given parity
    // (relative to build) into the other one, boundary layers included,
    // without advancing the members' step counters or parity (for timing).
    hipError_t launch_at(int parity, hipStream_t s);
    // Enqueue k launches of the step on `s`, in which member m takes
    // min(k, limit[m]) steps (k each without `limit`; a member that is done
    // sits out the remaining launches), and update the members' buffer
    // parity and step counters; `graphs` = false launches every step
    // directly (no graph is instantiated).
    int32_t run(int64_t k, hipStream_t s, bool graphs = true, const std::vector<int64_t>* limit = nullptr);
    // Health words of the members (in build order) after the work queued
    // on `s`; waits for `s`.
    int32_t health(std::vector<uint32_t>& out, hipStream_t s);
    bool empty() const { return members_.empty(); }

private:
    struct Group {
        int first = 0, n = 0;  // its members in members_
        bool tiled = false;    // stepped by the tiled kernel, else by the untiled one
        bool stream = false;   // non-temporal stores (tiled, levels beyond STREAM_MIN_BYTES)
        int nlists = 0, nblocks = 0, nlblocks = 0;
        BatchQueue* queue = nullptr;      // (device)
        BatchCount* counts = nullptr;     // step counts in the current run, two copies
        BatchTile* items = nullptr;       // tiles, or entries of blocks
        BatchLayerJob* layers = nullptr;  // boundary-layer jobs (sorted by first workgroup)
        int32_t* blockjob = nullptr;      // job of each boundary-layer workgroup
        hipGraphExec_t graph = nullptr;
    };
    // A plan's tables as they go to the device, and where they lie there.
    struct Layout {
        struct Offsets {
            size_t queue, counts, items, grids, layers, blockjob;
        };
        std::vector<char> image;
        size_t solves = 0, health = 0;
        std::vector<Offsets> groups;
    };
    int32_t lay_out(const std::vector<BatchMember>& shapes, const std::vector<GroupMembers>& parts, int tz, int cus,
                    Layout& t);  // fills groups_ and order_ too
    hipError_t enqueue(const Group& q, int parity, hipStream_t s);  // parity < 0: by the counts (-1, -2: which copy)
    void release_graphs();

    std::vector<lbm3d_solver*> members_;  // group by group
    std::vector<int32_t> order_;          // their places in the caller's list
    std::vector<Group> groups_;
    int mode_ = 0, by_ = 8;
    void* dmem_ = nullptr;  // tables allocated by the plan (nullptr with a caller's buffer)
    size_t dbytes_ = 0;
    BatchSolve* dsolves_ = nullptr;
    uint32_t* dhealth_ = nullptr;     // gathered health words, one per member
    std::vector<BatchCount> hcount_;  // host copy of the counts (source of the upload; done = parity since build)
    bool count_pending_ = false;      // hcount_ was uploaded and the stream not waited for since
    hipStream_t capture_stream_ = nullptr;
    hipStream_t last_stream_ = nullptr;  // stream of the last enqueued work (drained before teardown)
};

// Bytes of the static device array of the step that allocates nothing.
size_t noalloc_scratch_bytes();

// Checks shared by the batched entry points (E_INVAL / E_STATE).
int32_t check_batch(lbm3d_t* hs, int32_t count);
// Advance members by their own step counts (one run of the largest count,
// the others sitting out its last launches), then wait for `s`.  Tables go
// into `dev` (cap bytes) when given; `graphs` = false launches every step
// directly.
int32_t batch_advance(lbm3d_t* hs, int32_t count, const int64_t* nsteps, hipStream_t s, BatchPlan& plan,
                      void* dev, size_t cap, bool graphs);

}  // namespace lbm3d
