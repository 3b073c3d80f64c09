// Batched stepping: many solves of uneven size advanced group by group, a
// step of a group one launch (persistent, over per-XCD tile lists, or of
// untiled blocks), with step runs replayed from captured HIP graphs.
#include "lbm3d_batch.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <new>
#include <set>

namespace lbm3d {

static int32_t herr(hipError_t e)
{
    return e == hipSuccess ? LBM3D_OK : (e == hipErrorOutOfMemory ? LBM3D_E_NOMEM : LBM3D_E_DEVICE);
}

// Steps per captured graph of the batched step (even: parities 0,1,...).
constexpr int BATCH_GRAPH_STEPS = 16;
// Planes a tile marches before its first update (the z prologue), counted
// in the cost that balances the lists.
constexpr double TILE_PROLOGUE_PLANES = 3.0;

static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

int32_t plan_tiles(const std::vector<Grid>& grids, int by, int tz, int cus, TilePlan& out)
{
    out = TilePlan();
    if (by < 1 || tz < 1 || cus < 1) return LBM3D_E_INVAL;
    // every member's tiles in natural order: z chunk, then row, then column
    std::vector<BatchTile> all;
    std::vector<double> tcost;
    std::vector<size_t> mbegin(grids.size() + 1, 0);
    for (size_t k = 0; k < grids.size(); k++) {
        const Grid& g = grids[k];
        mbegin[k] = all.size();
        const int64_t ntx = (g.nx + TILE_X - 1) / TILE_X;
        const int64_t nty = (g.ny + by - 1) / by;
        const int64_t ntz = (g.nz + (int64_t)tz - 1) / tz;
        if ((int64_t)all.size() + ntx * nty * ntz > (int64_t)INT32_MAX) return LBM3D_E_INVAL;
        for (int64_t cz = 0; cz < ntz; cz++) {
            const int z0 = (int)(cz * tz);
            const int z1 = (int)std::min<int64_t>((int64_t)z0 + tz, g.nz);
            for (int64_t ty = 0; ty < nty; ty++)
                for (int64_t tx = 0; tx < ntx; tx++) {
                    BatchTile t;
                    t.solve = (int32_t)k;
                    t.txi = (int32_t)tx;
                    t.tyi = (int32_t)ty;
                    t.z0 = z0;
                    t.z1 = z1;
                    all.push_back(t);
                    tcost.push_back((z1 - z0) + TILE_PROLOGUE_PLANES);
                }
        }
    }
    mbegin[grids.size()] = all.size();
    const int n = (int)all.size();
    if (n == 0) return LBM3D_OK;
    int nblocks = std::min(n, cus);
    if (nblocks >= BATCH_MAX_LISTS) nblocks -= nblocks % BATCH_MAX_LISTS;
    const int nlists = std::min(BATCH_MAX_LISTS, nblocks);
    out.nblocks = nblocks;
    out.nlists = nlists;

    // contiguous pieces of each member, at most a quarter of a list's share each
    struct Piece {
        size_t begin, end;
        double cost;
    };
    double total = 0.0;
    for (double c : tcost) total += c;
    const double piece_max = nlists > 1 ? 0.25 * total / nlists : total;
    std::vector<Piece> pieces;
    for (size_t k = 0; k < grids.size(); k++) {
        double ck = 0.0;
        for (size_t j = mbegin[k]; j < mbegin[k + 1]; j++) ck += tcost[j];
        const int np = std::max(1, (int)std::ceil(ck / piece_max - 1e-9));
        size_t b = mbegin[k];
        double acc = 0.0;
        for (int p = 0; p < np; p++) {
            const double upto = ck * (p + 1) / np;
            size_t e = b;
            double pc = 0.0;
            while (e < mbegin[k + 1] && (p == np - 1 || acc + tcost[e] <= upto + 1e-9 || e == b)) {
                acc += tcost[e];
                pc += tcost[e];
                e++;
            }
            if (e > b) pieces.push_back(Piece{b, e, pc});
            b = e;
        }
    }
    // largest piece first onto the least-loaded list
    std::stable_sort(pieces.begin(), pieces.end(), [](const Piece& a, const Piece& b) { return a.cost > b.cost; });
    std::vector<std::vector<const Piece*>> lists((size_t)nlists);
    for (const Piece& p : pieces) {
        int best = 0;
        for (int l = 1; l < nlists; l++)
            if (out.cost[l] < out.cost[best]) best = l;
        lists[(size_t)best].push_back(&p);
        out.cost[best] += p.cost;
    }
    // each list: its pieces' tiles, deepest first (the order within a depth
    // is kept, so neighbouring tiles run together)
    out.tiles.reserve((size_t)n);
    for (int l = 0; l < nlists; l++) {
        out.queue.first[l] = (int32_t)out.tiles.size();
        std::vector<BatchTile> lt;
        for (const Piece* p : lists[(size_t)l])
            for (size_t j = p->begin; j < p->end; j++) lt.push_back(all[j]);
        std::stable_sort(lt.begin(), lt.end(),
                         [](const BatchTile& a, const BatchTile& b) { return (a.z1 - a.z0) > (b.z1 - b.z0); });
        out.tiles.insert(out.tiles.end(), lt.begin(), lt.end());
    }
    for (int l = nlists; l <= BATCH_MAX_LISTS; l++) out.queue.first[l] = (int32_t)out.tiles.size();
    for (int l = 0; l < BATCH_MAX_LISTS; l++) out.queue.next[l] = 0;
    return LBM3D_OK;
}

BatchPlan::~BatchPlan()
{
    if (last_stream_) (void)hipStreamSynchronize(last_stream_);
    release_graphs();
    if (capture_stream_) (void)hipStreamDestroy(capture_stream_);
    if (dmem_) (void)hipFree(dmem_);
}

void BatchPlan::release_graphs()
{
    // (callers have drained the stream the graphs were launched on)
    for (Group& q : groups_)
        if (q.graph) (void)hipGraphExecDestroy(q.graph);
    groups_.clear();
}

// The least planes the busiest compute unit can march when the tiles of a
// membership at depth d are dealt out longest first, each to the unit that is
// free first: each tile its planes plus the ones its z ring loads first.
static double tile_makespan(const std::vector<Grid>& grids, int by, int d, int cus)
{
    std::map<int, int64_t, std::greater<int>> tiles;  // by depth
    for (const Grid& g : grids) {
        const int64_t cols = (int64_t)((g.nx + TILE_X - 1) / TILE_X) * ((g.ny + by - 1) / by);
        if (g.nz / d) tiles[d] += cols * (g.nz / d);
        if (g.nz % d) tiles[g.nz % d] += cols;
    }
    std::map<double, int64_t> units{{0.0, (int64_t)cus}};  // compute units by the planes they have
    double last = 0.0;
    for (const auto& t : tiles) {
        const double cost = t.first + TILE_PROLOGUE_PLANES;
        int64_t left = t.second;
        // (whole rounds over all units at once)
        const int64_t rounds = left / cus - 1;
        if (rounds > 0) {
            std::map<double, int64_t> moved;
            for (const auto& u : units) moved[u.first + (double)rounds * cost] = u.second;
            units.swap(moved);
            left -= rounds * cus;
        }
        while (left > 0) {
            const auto u = units.begin();
            const double load = u->first;
            const int64_t n = std::min(left, u->second);
            if ((u->second -= n) == 0) units.erase(u);
            units[load + cost] += n;
            left -= n;
        }
    }
    for (const auto& u : units) last = std::max(last, u.first);
    return last;
}

// Planes the busiest workgroup of a plan marches: the workgroups of a list
// take its tiles in order, each when it is free.  A list that holds one more
// deep tile than it has workgroups takes a whole tile longer than tile_makespan
// has it (a 192x128x128 solve and three of 40^3, FP32 with FP64 moments: tiles
// of 32 planes are 222 in all, but one list gets 32 of them for its 27
// workgroups; 210 us a step, and 135 with the 16 planes this picks).
static double plan_makespan(const TilePlan& p)
{
    double last = 0.0;
    std::vector<double> load;  // a heap, the workgroup that is free first on top
    for (int l = 0; l < p.nlists; l++) {
        load.assign((size_t)(p.nblocks / p.nlists), 0.0);
        for (int32_t j = p.queue.first[l]; j < p.queue.first[l + 1]; j++) {
            std::pop_heap(load.begin(), load.end(), std::greater<double>());
            load.back() += p.tiles[(size_t)j].z1 - p.tiles[(size_t)j].z0 + TILE_PROLOGUE_PLANES;
            last = std::max(last, load.back());
            std::push_heap(load.begin(), load.end(), std::greater<double>());
        }
    }
    return last;
}
static double plan_makespan(const std::vector<Grid>& grids, int by, int d, int cus)
{
    TilePlan p;
    // (a plan of more tiles than can be counted is refused when it is built)
    return plan_tiles(grids, by, d, cus, p) == LBM3D_OK ? plan_makespan(p) : tile_makespan(grids, by, d, cus);
}

// Tile depth of a membership, of 16, 32, ... up to whole columns: in the FP32
// modes the deepest whose plan's makespan is within 5% of the shortest (whole
// columns for a batch as large as the 64-solve mix, as the tuner finds, short
// chunks for a few solves, whose whole columns would leave most compute units
// idle); in FP64, which leans less on the caches, the shortest (the shallower
// of two: 100x164x238 and 173x85x266 752 us a step with 32 planes, 761 with 64;
// six solves of about 90^3 607 and 645).  Plans are made for the depths that
// can be among those only.  Over 12 memberships of 1 - 20 solves, depths in
// between tried too, this takes the fastest depth or one 1% behind in the FP32
// modes, and one a few percent behind in FP64.
static std::vector<std::pair<double, int>> least_makespans(const std::vector<Grid>& grids, int by, int cus)
{
    int maxnz = 1;
    for (const Grid& g : grids) maxnz = std::max(maxnz, g.nz);
    std::vector<std::pair<double, int>> least;  // makespan at best, depth
    for (int d = 16;; d *= 2) {
        const int dd = std::min(d, maxnz);
        least.emplace_back(tile_makespan(grids, by, dd, cus), dd);
        if (dd >= maxnz) break;
    }
    std::sort(least.begin(), least.end());
    return least;
}
static int model_depth(int mode, const std::vector<Grid>& grids, int by, int cus, double* planes = nullptr)
{
    const double slack = mode == LBM3D_FP64 ? 1.0 : 1.05;
    std::vector<std::pair<double, int>> tried;
    double best = 0.0;
    for (const auto& c : least_makespans(grids, by, cus)) {
        if (!tried.empty() && c.first > slack * best) break;
        tried.emplace_back(plan_makespan(grids, by, c.second, cus), c.second);
        best = tried.size() == 1 ? tried[0].first : std::min(best, tried.back().first);
    }
    std::pair<double, int> pick{0.0, 0};
    for (const auto& t : tried)
        if (t.first <= slack * best && (pick.second == 0 || (mode != LBM3D_FP64) == (t.second > pick.second))) pick = t;
    if (planes) *planes = pick.first;
    return pick.second;
}

// Tile depth of a plan: tz > 0 as given; 0: the precision's tuned depth,
// else the model's; < 0: the model's (memberships that change from tick to
// tick, whose best depth no earlier tuning knows).
static int fixed_depth(int mode, int tz) { return tz == 0 ? batch_tile_depth(mode) : std::max(tz, 0); }
static int plan_depth(int mode, int tz, const std::vector<Grid>& grids, int by, int cus)
{
    const int t = fixed_depth(mode, tz);
    return t > 0 ? t : model_depth(mode, grids, by, cus);
}

// Members are independent, so a run steps them group by group, all its steps
// for one group before the next: a group whose two levels fit the 256 MB
// memory-side cache steps from there instead of from HBM.  The bytes a step
// touches are 30 values per node; GROUP_BYTES leaves room for the uneven
// spread of several members' pages over the cache (six 64^3 solves in FP32
// with FP64 moments, 189 MB, run at 39.5 G node updates/s, seven at 32.7,
// eight at 28.4), a member alone may fill it (128^3, 252 MB: 40).  Such
// groups are stepped by the untiled kernel, whose blocks fill the device at
// once and form their own boundary layers: a small solve has few tiles, each
// a long serial march (one 64^3 solve 53.9 us a step tiled, 11.6 untiled;
// 128^3 bubble 65.3 and 55).  Larger members form one group of their own,
// stepped by the tiled kernel: from HBM it streams faster than the blocks,
// which read their z neighbours several times (256x128x128: 114 us against
// 150).
constexpr int64_t GROUP_BYTES = (int64_t)192 << 20, ALONE_BYTES = (int64_t)256 << 20;

static std::vector<GroupMembers> group_members(int mode, const std::vector<BatchMember>& members)
{
    std::vector<GroupMembers> out;
    GroupMembers large;
    large.tiled = true;
    std::vector<std::pair<int64_t, int32_t>> fits;
    for (size_t k = 0; k < members.size(); k++) {
        const Grid& g = members[k].g;
        const int64_t b = (int64_t)g.nx * g.ny * g.nz * 2 * NV * (int64_t)elem_size(mode);
        if (b > ALONE_BYTES)
            large.who.push_back((int32_t)k);
        else
            fits.emplace_back(-b, (int32_t)k);
    }
    // largest first, each into the fullest group it fits
    std::stable_sort(fits.begin(), fits.end(),
                     [](const auto& a, const auto& b) { return a.first < b.first; });
    for (const auto& m : fits) {
        GroupMembers* best = nullptr;
        for (GroupMembers& q : out)
            if (q.bytes - m.first <= GROUP_BYTES && (!best || q.bytes > best->bytes)) best = &q;
        if (!best) {
            out.emplace_back();
            best = &out.back();
        }
        best->who.push_back(m.second);
        best->bytes -= m.first;
    }
    if (!large.who.empty()) out.push_back(large);
    return out;
}

// Time of a step of tiled members or of one untiled group, from what their
// kernels take per plane of a tile (over the memberships above 3.1 - 3.8 us in
// FP64, 2.5 - 3.6 in the FP32 modes) and per block (14 - 19 ns in FP64, 7 - 9 in
// the FP32 modes, at 256 compute units), with their launches.
static double tiled_us(int mode, double planes, const std::vector<BatchMember>& members)
{
    bool layers = false;
    for (const BatchMember& m : members) layers = layers || ghost_faces(m.g, m.bc, true) != 0;
    return planes * (mode == LBM3D_FP64 ? 3.5 : 3.1) + (layers ? 9.0 : 3.0);
}
static double blocks_us(int mode, const std::vector<BatchMember>& members, int cus)
{
    double blocks = 0.0;
    for (const BatchMember& m : members) blocks += block_grid(m.g).count;
    return 2.5 + blocks * (mode == LBM3D_FP64 ? 0.017 : 0.007) * 256.0 / cus;
}

static std::vector<GroupMembers> all_tiled(size_t members)
{
    GroupMembers all;
    all.tiled = true;
    for (size_t k = 0; k < members; k++) all.who.push_back((int32_t)k);
    return {all};
}

std::vector<GroupMembers> plan_groups(int mode, const std::vector<BatchMember>& members, int tz, int cus)
{
    const int by = mode == LBM3D_FP64 ? 4 : 8, fixed = fixed_depth(mode, tz);
    if (tz > 0 || (tz == 0 && batch_depth_set(mode))) return all_tiled(members.size());
    std::vector<GroupMembers> parts = group_members(mode, members);
    if (parts.size() == 1 && parts[0].tiled) return parts;
    auto grids_of = [](const std::vector<BatchMember>& who) {
        std::vector<Grid> grids;
        for (const BatchMember& m : who) grids.push_back(m.g);
        return grids;
    };
    // a tiled group's time, and the depth that it takes
    auto tiled = [&](const std::vector<BatchMember>& who, int* depth) {
        const std::vector<Grid> grids = grids_of(who);
        double planes = 0.0;
        *depth = fixed > 0 ? fixed : model_depth(mode, grids, by, cus, &planes);
        if (fixed > 0) planes = plan_makespan(grids, by, fixed, cus);
        return tiled_us(mode, planes, who);
    };
    double apart = 0.0;
    for (GroupMembers& part : parts) {
        std::vector<BatchMember> mine;
        for (int32_t k : part.who) mine.push_back(members[(size_t)k]);
        apart += part.tiled ? tiled(mine, &part.depth) : blocks_us(mode, mine, cus);
    }
    // (no plan of all members is made where it could not win at best)
    const std::vector<Grid> grids = grids_of(members);
    const double least = fixed > 0 ? tile_makespan(grids, by, fixed, cus) : least_makespans(grids, by, cus)[0].first;
    if (apart <= tiled_us(mode, least, members)) return parts;
    std::vector<GroupMembers> all = all_tiled(members.size());
    return apart <= tiled(members, &all[0].depth) ? parts : all;
}

int batch_model_depth(int mode, const std::vector<BatchMember>& members, int cus)
{
    std::vector<Grid> grids;
    for (const BatchMember& m : members) grids.push_back(m.g);
    return model_depth(mode, grids, mode == LBM3D_FP64 ? 4 : 8, cus);
}

// layer jobs of tiled members (faces the tiles leave to memory)
static void layer_jobs(const std::vector<BatchMember>& members, std::vector<BatchLayerJob>& ljobs,
                       std::vector<int32_t>& block_job, int& nlblocks)
{
    ljobs.clear();
    nlblocks = 0;
    for (size_t k = 0; k < members.size(); k++) {
        const Grid& g = members[k].g;
        const uint32_t faces = ghost_faces(g, members[k].bc, true);
        if (!faces) continue;
        int64_t lines = 0;
        for (int face = 0; face < 6; face++) {
            if (!((faces >> face) & 1)) continue;
            const int axis = face >> 1;
            lines += axis == 0 ? (int64_t)g.ny * g.nz : axis == 1 ? (int64_t)g.nx * g.nz : (int64_t)g.nx * g.ny;
        }
        BatchLayerJob jb;
        jb.solve = (int32_t)k;
        jb.faces = faces;
        jb.first = nlblocks;
        ljobs.push_back(jb);
        nlblocks += (int)((lines + 63) / 64);
    }
    block_job.assign((size_t)nlblocks, 0);
    for (size_t j = 0; j < ljobs.size(); j++) {
        const int end = j + 1 < ljobs.size() ? ljobs[j + 1].first : nlblocks;
        for (int b = ljobs[j].first; b < end; b++) block_job[(size_t)b] = (int32_t)j;
    }
}

static size_t tables_need(size_t nmembers, size_t ntiles, size_t nljobs, size_t nlblocks)
{
    return align256(nmembers * sizeof(BatchSolve)) + align256(ntiles * sizeof(BatchTile)) +
           align256(9 * sizeof(int32_t) + BATCH_MAX_LISTS * sizeof(uint32_t)) +
           align256(nljobs * sizeof(BatchLayerJob)) + align256(nlblocks * sizeof(int32_t)) +
           align256(nmembers * sizeof(BatchCount)) + nmembers * sizeof(uint32_t) + 256;
}

size_t BatchPlan::table_bytes(const std::vector<lbm3d_solver*>& members, int tz)
{
    if (members.empty()) return 0;
    const int mode = members[0]->mode;
    const int by = mode == LBM3D_FP64 ? 4 : 8;
    std::vector<Grid> grids;
    std::vector<BatchMember> all;
    for (lbm3d_solver* h : members) {
        grids.push_back(h->g);
        all.push_back(BatchMember{h->g, h->bc});
    }
    TilePlan p;
    const int cus = device_cus();
    if (plan_tiles(grids, by, plan_depth(mode, tz, grids, by, cus), cus, p) != LBM3D_OK) return (size_t)-1;
    std::vector<BatchLayerJob> lj;
    std::vector<int32_t> bj;
    int nlb = 0;
    layer_jobs(all, lj, bj, nlb);
    return tables_need(members.size(), p.tiles.size(), lj.size(), (size_t)nlb);
}

// The tables, laid out in a host image of the device memory: the solves in
// group order and the members' health words, then per group its queue, counts
// and work items (with the solves' indices in the group).
int32_t BatchPlan::lay_out(const std::vector<BatchMember>& shapes, const std::vector<GroupMembers>& parts, int tz,
                           int cus, Layout& t)
{
    groups_.clear();
    order_.clear();
    t = Layout();
    std::vector<char>& image = t.image;
    auto place = [&](size_t bytes) {
        const size_t at = align256(image.size());
        image.resize(at + bytes, 0);
        return at;
    };
    t.solves = place(shapes.size() * sizeof(BatchSolve));
    t.health = place(shapes.size() * sizeof(uint32_t));
    for (const GroupMembers& part : parts) {
        Group q;
        q.first = (int)order_.size();
        q.n = (int)part.who.size();
        q.tiled = part.tiled;
        std::vector<BatchMember> mine;
        for (int32_t k : part.who) {
            order_.push_back(k);
            mine.push_back(shapes[(size_t)k]);
        }
        Layout::Offsets o{};
        o.queue = place(sizeof(BatchQueue));
        o.counts = place(2 * mine.size() * sizeof(BatchCount));
        std::vector<BatchTile> items;
        if (part.tiled) {
            std::vector<Grid> grids;
            int64_t level_bytes = 0, dense_bytes = 0;
            for (const BatchMember& m : mine) {
                grids.push_back(m.g);
                const int64_t bytes = 2 * (int64_t)f_bytes(m.g, mode_);
                level_bytes += bytes;
                if (dense_rows(m.g.nx) || mode_ == LBM3D_FP64) dense_bytes += bytes;
            }
            // plain stores when the levels together fit the memory-side
            // cache, or most of them have rows that end inside a cache
            // line (in the FP32 modes), as for a single solve
            q.stream = level_bytes > STREAM_MIN_BYTES && 2 * dense_bytes > level_bytes;
            TilePlan plan;
            const int depth = part.depth > 0 ? part.depth : plan_depth(mode_, tz, grids, by_, cus);
            int32_t rc = plan_tiles(grids, by_, depth, cus, plan);
            if (rc) return rc;
            items.swap(plan.tiles);
            q.nlists = plan.nlists;
            q.nblocks = plan.nblocks;
            std::memcpy(image.data() + o.queue, &plan.queue, sizeof(BatchQueue));
            std::vector<BatchLayerJob> ljobs;
            std::vector<int32_t> block_job;
            layer_jobs(mine, ljobs, block_job, q.nlblocks);
            if (q.nlblocks) {
                o.layers = place(ljobs.size() * sizeof(BatchLayerJob));
                std::memcpy(image.data() + o.layers, ljobs.data(), ljobs.size() * sizeof(BatchLayerJob));
                o.blockjob = place(block_job.size() * sizeof(int32_t));
                std::memcpy(image.data() + o.blockjob, block_job.data(), block_job.size() * sizeof(int32_t));
            }
        } else {
            o.grids = place(mine.size() * sizeof(BlockGrid));
            for (size_t k = 0; k < mine.size(); k++) {
                const BlockGrid bg = block_grid(mine[k].g);
                std::memcpy(image.data() + o.grids + k * sizeof(BlockGrid), &bg, sizeof(BlockGrid));
                const int first = q.nblocks;
                for (uint32_t b = 0; b < bg.count; b += BATCH_BLOCKS) {
                    items.push_back(BatchTile{(int32_t)k, 0, 0, first, 0});
                    q.nblocks += BATCH_BLOCKS;
                }
            }
        }
        o.items = place(items.size() * sizeof(BatchTile));
        std::memcpy(image.data() + o.items, items.data(), items.size() * sizeof(BatchTile));
        groups_.push_back(q);
        t.groups.push_back(o);
    }
    return LBM3D_OK;
}

int32_t BatchPlan::build(const std::vector<lbm3d_solver*>& members, hipStream_t s, int tz, void* dev, size_t cap)
{
    // work still queued may read the old tables or replay the old graphs
    if (last_stream_ && hipStreamSynchronize(last_stream_) != hipSuccess) return LBM3D_E_DEVICE;
    last_stream_ = nullptr;
    release_graphs();
    members_.clear();
    count_pending_ = false;
    if (members.empty()) return LBM3D_OK;
    mode_ = members[0]->mode;
    by_ = mode_ == LBM3D_FP64 ? 4 : 8;
    const int cus = device_cus();
    std::vector<BatchMember> shapes;
    for (lbm3d_solver* h : members) shapes.push_back(BatchMember{h->g, h->bc});
    Layout t;
    int32_t rc = lay_out(shapes, plan_groups(mode_, shapes, tz, cus), tz, cus, t);
    // tables of groups may need more room than those of one tiled plan (an
    // entry per 64 blocks of a member, where a deep tile takes as many bytes
    // for more nodes)
    if (rc == LBM3D_OK && dev && t.image.size() > cap) rc = lay_out(shapes, all_tiled(shapes.size()), tz, cus, t);
    const size_t need = t.image.size();
    char* base = (char*)dev;
    if (rc == LBM3D_OK && dev && need > cap) rc = LBM3D_E_NOMEM;
    if (rc == LBM3D_OK && (dev || need > dbytes_)) {
        if (dmem_) (void)hipFree(dmem_);
        dmem_ = nullptr;
        dbytes_ = 0;
        if (!dev) {
            rc = herr(hipMalloc(&dmem_, need));
            if (rc == LBM3D_OK) dbytes_ = need;
        }
    }
    if (rc) {
        groups_.clear();
        return rc;
    }
    if (!dev) base = (char*)dmem_;
    for (int32_t k : order_) members_.push_back(members[(size_t)k]);
    std::vector<char>& image = t.image;
    dsolves_ = (BatchSolve*)(base + t.solves);
    dhealth_ = (uint32_t*)(base + t.health);
    for (size_t j = 0; j < groups_.size(); j++) {
        Group& q = groups_[j];
        const Layout::Offsets& o = t.groups[j];
        q.queue = (BatchQueue*)(base + o.queue);
        q.counts = (BatchCount*)(base + o.counts);
        q.items = (BatchTile*)(base + o.items);
        q.layers = (BatchLayerJob*)(base + o.layers);
        q.blockjob = (int32_t*)(base + o.blockjob);
        BatchQueue hq;
        std::memcpy(&hq, image.data() + o.queue, sizeof(hq));
        hq.blocks = (const BlockGrid*)(base + o.grids);
        hq.counts = q.counts;
        hq.members = q.n;
        std::memcpy(image.data() + o.queue, &hq, sizeof(hq));
    }
    for (size_t k = 0; k < members_.size(); k++) {
        const lbm3d_solver* h = members_[k];
        BatchSolve d;
        std::memset(&d, 0, sizeof(d));
        d.g = h->g;
        d.bc = h->bc;
        d.cur0 = h->cur;
        x_fixed_states(h->p.inflow, d.xin);
        d.f[0] = h->f[0];
        d.f[1] = h->f[1];
        d.health = h->health;
        d.md = h->md;
        d.mf = h->mf;
        std::memcpy(image.data() + t.solves + k * sizeof(BatchSolve), &d, sizeof(d));
    }
    hcount_.assign(members_.size(), BatchCount{0, 0});
    // the tiles read some layers from memory, which members that last
    // stepped untiled have left behind
    hipError_t e = hipSuccess;
    for (const Group& q : groups_)
        for (int k = q.first; q.tiled && k < q.first + q.n && e == hipSuccess; k++) {
            lbm3d_solver* h = members_[(size_t)k];
            if (!h->layers_stale) continue;
            e = launch_ghosts(h->mode, h->g, h->bc, h->md, h->p.inflow, false, h->f[h->cur], s,
                              ghost_faces(h->g, h->bc, true));
            if (e == hipSuccess) h->layers_stale = false;
        }
    if (e == hipSuccess) e = hipMemcpyAsync(base, image.data(), need, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);  // the host image dies at return
    last_stream_ = nullptr;
    return herr(e);
}

int32_t BatchPlan::health(std::vector<uint32_t>& out, hipStream_t s)
{
    out.assign(members_.size(), 0u);
    if (members_.empty()) return LBM3D_OK;
    std::vector<uint32_t> got(members_.size(), 0u);
    hipError_t e = launch_gather_health(dsolves_, (int)members_.size(), dhealth_, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(got.data(), dhealth_, got.size() * sizeof(uint32_t), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess && s == last_stream_) count_pending_ = false;
    for (size_t k = 0; k < got.size(); k++) out[(size_t)order_[k]] = got[k];
    return herr(e);
}

hipError_t BatchPlan::launch_at(int parity, hipStream_t s)
{
    last_stream_ = s;
    hipError_t e = hipSuccess;
    for (const Group& q : groups_)
        if (e == hipSuccess) e = enqueue(q, parity & 1, s);
    return e;
}

hipError_t BatchPlan::enqueue(const Group& q, int parity, hipStream_t s)
{
    const BatchCount* counts = q.counts + (parity == -2 ? q.n : 0);
    const BatchSolve* solves = dsolves_ + q.first;
    hipError_t e = launch_batch_step(mode_, q.tiled ? by_ : 0, q.stream, solves, q.items, q.queue, q.nlists, q.nblocks,
                                     parity, counts, s);
    // boundary layers the tiles do not form themselves, all members at once
    if (e == hipSuccess && q.nlblocks)
        e = launch_batch_layers(mode_, solves, q.layers, q.blockjob, q.nlblocks, parity, counts, s);
    return e;
}

int32_t BatchPlan::run(int64_t k, hipStream_t s, bool graphs, const std::vector<int64_t>* limit)
{
    if (members_.empty() || k <= 0) return LBM3D_OK;
    if (limit && limit->size() != members_.size()) return LBM3D_E_INVAL;
    // the counts are 32-bit: very long runs go in pieces
    constexpr int64_t PIECE = (int64_t)1 << 30;
    if (k > PIECE) {
        std::vector<int64_t> rest = limit ? *limit : std::vector<int64_t>(members_.size(), k);
        for (int64_t left = k; left > 0;) {
            const int64_t c = std::min(left, PIECE);
            int32_t rc = run(c, s, graphs, &rest);
            if (rc) return rc;
            for (int64_t& r : rest) r = std::max<int64_t>(0, r - c);
            left -= c;
        }
        return LBM3D_OK;
    }
    // the counts of the last run may still be on their way from hcount_
    if (count_pending_ && last_stream_ && hipStreamSynchronize(last_stream_) != hipSuccess) return LBM3D_E_DEVICE;
    count_pending_ = false;
    last_stream_ = s;
    // this run's counts: done restarts at each member's parity since build
    // (so it never grows), target = done + the member's steps
    std::vector<int64_t> steps(members_.size(), k);
    for (size_t m = 0; m < members_.size(); m++) {
        if (limit) steps[m] = std::max<int64_t>(0, std::min<int64_t>(k, (*limit)[(size_t)order_[m]]));
        hcount_[m].done &= 1;
        hcount_[m].target = hcount_[m].done + (int32_t)steps[m];
    }
    for (Group& q : groups_) {
        int64_t left = 0;
        for (int m = q.first; m < q.first + q.n; m++) left = std::max(left, steps[(size_t)m]);
        if (left == 0) continue;
        hipError_t e = hipMemcpyAsync(q.counts, hcount_.data() + q.first, (size_t)q.n * sizeof(BatchCount),
                                      hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return herr(e);
        count_pending_ = true;
        // the launches carry nothing step-specific but which copy of the
        // counts they read (each member's parity comes from its count), so
        // one captured run of BATCH_GRAPH_STEPS, an even number, serves all
        while (graphs && left >= BATCH_GRAPH_STEPS) {
            if (!q.graph) {
                if (!capture_stream_) {
                    e = hipStreamCreateWithFlags(&capture_stream_, hipStreamNonBlocking);
                    if (e != hipSuccess) return herr(e);
                }
                hipGraph_t graph = nullptr;
                e = hipStreamBeginCapture(capture_stream_, hipStreamCaptureModeThreadLocal);
                if (e != hipSuccess) return herr(e);
                for (int j = 0; j < BATCH_GRAPH_STEPS && e == hipSuccess; j++)
                    e = enqueue(q, -1 - (j & 1), capture_stream_);
                hipError_t e2 = hipStreamEndCapture(capture_stream_, &graph);
                if (e != hipSuccess || e2 != hipSuccess) {
                    if (graph) (void)hipGraphDestroy(graph);
                    return herr(e != hipSuccess ? e : e2);
                }
                e = hipGraphInstantiate(&q.graph, graph, nullptr, nullptr, 0);
                (void)hipGraphDestroy(graph);
                if (e != hipSuccess) return herr(e);
            }
            e = hipGraphLaunch(q.graph, s);
            if (e != hipSuccess) return herr(e);
            left -= BATCH_GRAPH_STEPS;
        }
        for (int j = 0; j < left; j++) {
            e = enqueue(q, -1 - (j & 1), s);
            if (e != hipSuccess) return herr(e);
        }
        // members advance by their steps; their current buffer flips with
        // an odd count (the device table keeps the build-time buffers, and
        // each count's done its parity since build)
        for (int m = q.first; m < q.first + q.n; m++) {
            lbm3d_solver* h = members_[(size_t)m];
            const int64_t n = steps[(size_t)m];
            hcount_[(size_t)m].done = (hcount_[(size_t)m].done + (int32_t)(n & 1)) & 1;
            if (n == 0) continue;
            h->steps += n;
            if (n & 1) h->cur ^= 1;
            if (!q.tiled) h->layers_stale = true;
        }
    }
    return LBM3D_OK;
}

// Checks shared by the batched entry points: non-null distinct handles,
// initialised, one precision, within the tiled kernels' addressing.
int32_t check_batch(lbm3d_t* hs, int32_t count)
{
    if (!hs || count < 1) return LBM3D_E_INVAL;
    std::set<lbm3d_t> seen;
    for (int32_t k = 0; k < count; k++) {
        if (!hs[k] || !seen.insert(hs[k]).second) return LBM3D_E_INVAL;
        if (!hs[k]->initialised) return LBM3D_E_STATE;
        if (hs[k]->mode != hs[0]->mode) return LBM3D_E_INVAL;
        if (!tiled_fits(hs[k]->mode, hs[k]->g)) return LBM3D_E_INVAL;
        if (hs[k]->upwind2) return LBM3D_E_INVAL;  // the batched kernel is NND only
    }
    return LBM3D_OK;
}

// Steps of a batch whose members need different step counts: runs of the
// common count with the members that still have steps to do.
int32_t batch_advance(lbm3d_t* hs, int32_t count, const int64_t* nsteps, hipStream_t s, BatchPlan& plan,
                      void* dev, size_t cap, bool graphs)
{
    std::vector<lbm3d_solver*> active;
    std::vector<int64_t> limit;
    int64_t k = 0;
    for (int32_t j = 0; j < count; j++)
        if (nsteps[j] > 0) {
            active.push_back(hs[j]);
            limit.push_back(nsteps[j]);
            k = std::max(k, nsteps[j]);
        }
    if (!active.empty()) {
        int32_t rc = plan.build(active, s, 0, dev, cap);
        if (rc) return rc;
        rc = plan.run(k, s, graphs, &limit);
        if (rc) return rc;
    }
    return hipStreamSynchronize(s) == hipSuccess ? LBM3D_OK : LBM3D_E_DEVICE;
}

}  // namespace lbm3d

// ------------------------------------------------------------------- C ABI --
using namespace lbm3d;

static int32_t batch_step(lbm3d_t* hs, int32_t count, const int64_t* nsteps)
{
    int32_t rc = check_batch(hs, count);
    if (rc) return rc;
    if (!nsteps) return LBM3D_E_INVAL;
    for (int32_t k = 0; k < count; k++)
        if (nsteps[k] < 0) return LBM3D_E_INVAL;
    hipStream_t s = hs[0]->stream;
    // work already queued on the other solves' streams precedes the batch
    for (int32_t k = 1; k < count; k++)
        if (hs[k]->stream != s && hipStreamSynchronize(hs[k]->stream) != hipSuccess) return LBM3D_E_DEVICE;
    BatchPlan plan;
    return batch_advance(hs, count, nsteps, s, plan, nullptr, 0, true);
}

extern "C" int32_t lbm3d_batch_step(lbm3d_t* hs, int32_t count, const int64_t* nsteps)
{
    return no_throw([&] { return batch_step(hs, count, nsteps); });
}

// ------------------------------------------------ the allocation-free step --
// The tables of lbm3d_batch_step_noalloc (solve table, tile lists and their
// counters, boundary-layer jobs, health words) live in this array, one copy
// per device, held until the process ends.  In host code its name is only a
// stand-in: the device address of each device's copy comes from
// hipGetSymbolAddress and is kept per device.
// A batch is taken if its tables with every member tiled in one group fit
// NOALLOC_SCRATCH_BYTES, and goes that way where those of its groups do not
// fit; the slack is for what build adds to the former (a second copy of the
// counts, a longer queue).
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)4 << 20, NOALLOC_SLACK = (size_t)64 << 10;
static_assert(NOALLOC_SCRATCH_BYTES / sizeof(BatchSolve) * sizeof(BatchCount) + 4096 <= NOALLOC_SLACK,
              "as many members as there is room for");
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES + NOALLOC_SLACK];

size_t lbm3d::noalloc_scratch_bytes() { return sizeof(scratch); }

namespace {
std::mutex g_scratch_mu;
std::vector<void*> g_scratch;  // device address of `scratch` per device (nullptr: not looked up yet)
}  // namespace

// The device address of the current device's scratch array (looked up once
// per device, with that device current).
static int32_t scratch_address(void** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return LBM3D_E_DEVICE;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((size_t)dev >= g_scratch.size()) g_scratch.resize((size_t)dev + 1, nullptr);
    if (!g_scratch[(size_t)dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LBM3D_E_DEVICE;
        g_scratch[(size_t)dev] = ptr;
    }
    *out = g_scratch[(size_t)dev];
    return LBM3D_OK;
}

static int32_t batch_step_noalloc(lbm3d_t* hs, int32_t count, const int64_t* nsteps)
{
    int32_t rc = check_batch(hs, count);
    if (rc) return rc;
    if (!nsteps) return LBM3D_E_INVAL;
    for (int32_t k = 0; k < count; k++)
        if (nsteps[k] < 0) return LBM3D_E_INVAL;
    std::vector<lbm3d_solver*> members(hs, hs + count);
    // the full membership needs the largest tables of the call
    if (BatchPlan::table_bytes(members) > NOALLOC_SCRATCH_BYTES) return LBM3D_E_NOMEM;
    void* ptr = nullptr;
    rc = scratch_address(&ptr);
    if (rc) return rc;
    hipStream_t s = hs[0]->stream;
    for (int32_t k = 1; k < count; k++)
        if (hs[k]->stream != s && hipStreamSynchronize(hs[k]->stream) != hipSuccess) return LBM3D_E_DEVICE;
    BatchPlan plan;  // tables in the scratch array, steps launched directly (no graph)
    return batch_advance(hs, count, nsteps, s, plan, ptr, NOALLOC_SCRATCH_BYTES + NOALLOC_SLACK, false);
}

extern "C" int32_t lbm3d_batch_step_noalloc(lbm3d_t* hs, int32_t count, const int64_t* nsteps)
{
    return no_throw([&] { return batch_step_noalloc(hs, count, nsteps); });
}

static int32_t batch_plan(const lbm3d_params* ps, int32_t count, int32_t tz, int32_t cus,
                          int32_t* ntiles, int32_t* nlists, int32_t* nblocks, int32_t* tiles,
                          int64_t cap, int32_t* list_first)
{
    if (!ps || count < 1 || cus < 1) return LBM3D_E_INVAL;
    std::vector<Grid> grids;
    for (int32_t k = 0; k < count; k++) {
        int32_t rc = validate(&ps[k]);
        if (rc) return rc;
        if (ps[k].precision != ps[0].precision || (ps[k].flags & LBM3D_UPWIND2)) return LBM3D_E_INVAL;
        const Grid g = make_grid(&ps[k]);
        if (!tiled_fits(ps[k].precision, g)) return LBM3D_E_INVAL;
        grids.push_back(g);
    }
    const int mode = ps[0].precision;
    const int by = mode == LBM3D_FP64 ? 4 : 8;
    TilePlan p;
    int32_t rc = plan_tiles(grids, by, plan_depth(mode, tz, grids, by, cus), cus, p);
    if (rc) return rc;
    const int64_t n = (int64_t)p.tiles.size();
    if (ntiles) *ntiles = (int32_t)n;
    if (nlists) *nlists = p.nlists;
    if (nblocks) *nblocks = p.nblocks;
    if (list_first)
        for (int l = 0; l <= BATCH_MAX_LISTS; l++) list_first[l] = p.queue.first[l];
    if (tiles) {
        if (cap < n) return LBM3D_E_NOMEM;
        for (int64_t j = 0; j < n; j++) {
            const BatchTile& t = p.tiles[(size_t)j];
            const Grid& g = grids[(size_t)t.solve];
            int32_t* o = tiles + 7 * j;
            o[0] = t.solve;
            o[1] = t.txi * TILE_X;
            o[2] = std::min(o[1] + TILE_X, g.nx);
            o[3] = t.tyi * by;
            o[4] = std::min(o[3] + by, g.ny);
            o[5] = t.z0;
            o[6] = t.z1;
        }
    }
    return LBM3D_OK;
}

extern "C" int32_t lbm3d_batch_plan(const lbm3d_params* ps, int32_t count, int32_t tz, int32_t cus,
                                    int32_t* ntiles, int32_t* nlists, int32_t* nblocks, int32_t* tiles,
                                    int64_t cap, int32_t* list_first)
{
    return no_throw([&] { return batch_plan(ps, count, tz, cus, ntiles, nlists, nblocks, tiles, cap, list_first); });
}

static int32_t batch_groups(const lbm3d_params* ps, int32_t count, int32_t tz, int32_t cus, int32_t* group,
                            int32_t* tiled)
{
    if (!ps || count < 1 || cus < 1 || !group || !tiled) return LBM3D_E_INVAL;
    std::vector<BatchMember> members;
    for (int32_t k = 0; k < count; k++) {
        int32_t rc = validate(&ps[k]);
        if (rc) return rc;
        if (ps[k].precision != ps[0].precision || (ps[k].flags & LBM3D_UPWIND2)) return LBM3D_E_INVAL;
        BatchMember m;
        m.g = make_grid(&ps[k]);
        if (!tiled_fits(ps[k].precision, m.g)) return LBM3D_E_INVAL;
        for (int f = 0; f < 6; f++) m.bc.kind[f] = ps[k].bc[f];
        members.push_back(m);
    }
    const std::vector<GroupMembers> parts = plan_groups(ps[0].precision, members, tz, cus);
    for (size_t j = 0; j < parts.size(); j++)
        for (int32_t k : parts[j].who) {
            group[k] = (int32_t)j;
            tiled[k] = parts[j].tiled ? 1 : 0;
        }
    return LBM3D_OK;
}

extern "C" int32_t lbm3d_batch_groups(const lbm3d_params* ps, int32_t count, int32_t tz, int32_t cus, int32_t* group,
                                      int32_t* tiled)
{
    return no_throw([&] { return batch_groups(ps, count, tz, cus, group, tiled); });
}
