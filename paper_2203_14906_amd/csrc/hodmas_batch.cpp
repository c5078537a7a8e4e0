// Batched form: a work list of (frame, tile) units over many frames, grouped by
// kind (order x storage type x mirror pairing x coherence weighting, or several
// orders and pairings of one storage type as one mixed kind) and walked by one
// kernel per kind; a HIP graph holds the kernels so one graph launch
// runs the batch.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <numeric>
#include <vector>

#include "hodmas_internal.h"

using hodmas::BatchFrame;
using hodmas::BatchHeader;
using hodmas::BatchUnit;
using hodmas::DrawCount;

namespace {

constexpr uint32_t kBatchMagic = 0x48424154u;  // "HBAT"
constexpr size_t kAlign = 256;
// Estimated VALU slots per pixel-element by order (delay, gather, root, sums):
// only used to order the work list, heaviest units first.
constexpr int64_t kSlots[7] = {0, 19, 25, 32, 32, 36, 38};
constexpr int64_t kCfSlots = 4;   // coherence weighting: two more compensated sums
constexpr int kLaunches = 4;      // direct launches of one list with draw counts of their own

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// How a kind of one order runs: not at all, in the mixed kind or by itself.
enum class RunsAs : char { none, mixed, apart };

}  // namespace

struct hodmas_batch_s {
    uint32_t magic = kBatchMagic;
    int device = -1;
    int32_t max_frames = 0;
    int64_t max_units = 0;
    int64_t lds_bytes = 0;
    uint32_t flags = 0;
    int cus = 0;                          // compute units of the device
    int grid[hodmas::kBatchKinds] = {};   // workgroups the device holds per kind at lds_bytes
    // the current work list's kinds: LDS of their largest member plan and the
    // workgroups the device holds at that LDS
    int64_t kind_lds[hodmas::kBatchKinds] = {};
    int kind_grid[hodmas::kBatchKinds] = {};
    int32_t longest[hodmas::kBatchKinds] = {};   // units of the longest XCD run
    // the last occupancy answer per kind (a serving loop sets a list per launch)
    int64_t occ_lds[hodmas::kBatchKinds] = {};
    int occ_per_cu[hodmas::kBatchKinds] = {};
    bool draws[3] = {};                   // by storage type: the list's mixed kind draws its units
    // how the list runs the kinds it has, and how captured launches have run them
    RunsAs runs_as[hodmas::kOrderKinds] = {}, captured[hodmas::kOrderKinds] = {};
    size_t off_frames = 0, off_units = 0, off_counts = 0, bytes = 0;
    char* d_buf = nullptr;
    char* h_buf = nullptr;           // pinned staging of the work list
    hipEvent_t copied = nullptr;     // last host->device copy of h_buf
    bool copy_pending = false;
    bool has_list = false;
    int32_t begin[hodmas::kBatchKinds] = {}, end[hodmas::kBatchKinds] = {};   // host copy of the ranges
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipGraphNode_t node[hodmas::kBatchKinds] = {};   // one kernel node per kind
    int node_grid[hodmas::kBatchKinds] = {};         // its current grid in `exec`
    int64_t node_lds[hodmas::kBatchKinds] = {};      // and its dynamic LDS
    bool node_on[hodmas::kBatchKinds] = {};          // enabled in `exec`
    bool node_draws[hodmas::kBatchKinds] = {};       // with the graph's draw counts
    // Draw counts belong to one launch at a time: set 0 to the graph, set 1 + i
    // to the direct launches that take runs[i] in turn.  A launch on another
    // stream than the one before it with the same set waits for that one's end.
    struct Run {
        hipEvent_t done = nullptr;   // destroy waits for it
        hipStream_t stream = nullptr;
        bool pending = false;
    };
    Run replayed, runs[kLaunches];
    bool list_replayed = false;      // the current list, by the graph or in its place
    int next_run = 0;
    hodmas_batch_info info{};
};

namespace {

void release(hodmas_batch_s* b)
{
    for (hodmas_batch_s::Run* r : {&b->replayed, &b->runs[0], &b->runs[1], &b->runs[2], &b->runs[3]}) {
        static_assert(kLaunches == 4, "every run");
        if (r->done) {
            (void)hipEventSynchronize(r->done);
            (void)hipEventDestroy(r->done);
            r->done = nullptr;
        }
    }
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    if (b->copied) {
        (void)hipEventSynchronize(b->copied);
        (void)hipEventDestroy(b->copied);
    }
    if (b->d_buf) (void)hipFree(b->d_buf);
    if (b->h_buf) (void)hipHostFree(b->h_buf);
    b->exec = nullptr;
    b->graph = nullptr;
    b->copied = nullptr;
    b->d_buf = nullptr;
    b->h_buf = nullptr;
}

bool valid_batch(const hodmas_batch_s* b) { return b && b->magic == kBatchMagic; }

struct Unit {
    int64_t cost;
    int32_t kind, frame, tile;
};

// A mixed kind's n units, in frame and tile order, dealt to `used` XCDs: every
// frame is cut into that many bands of tile rows of about equal estimated cost,
// and each XCD takes one of each frame -- another one of the next, as costs
// that the estimate misses go with depth -- so all have the same mix of orders
// and record ends whatever those cost.  (Contiguous runs, an XCD all of a few
// frames, as the kinds of one order are cut, rest on the estimate across orders:
// 753 us where this took 685, 24 frames of 17 shapes.)  cut[x] .. cut[x + 1]
// becomes XCD x's run: its bands, those of the heaviest units first.
void deal_frames(Unit* run, int n, int used, int32_t* cut, std::vector<Unit>& dealt)
{
    struct Band {
        int64_t unit_cost;
        int first, end;
    };
    std::vector<Band> mine[hodmas::kXcds];
    for (int f0 = 0, frame = 0; f0 < n; ++frame) {
        int f1 = f0;
        int64_t total = 0;
        for (; f1 < n && run[f1].frame == run[f0].frame; ++f1)
            total += run[f1].cost;
        int u = f0;
        int64_t before = 0;
        for (int band = 0; band < used; ++band) {
            const int first = u;
            const int64_t start = before;
            // a unit belongs to the band its middle falls in
            for (; u < f1 && (2 * before + run[u].cost) * used < 2 * total * (band + 1); ++u)
                before += run[u].cost;
            if (u > first)
                mine[(band + frame) % used].push_back({(before - start) / (u - first), first, u});
        }
        f0 = f1;
    }
    dealt.clear();
    for (int x = 0; x <= hodmas::kXcds; ++x) {
        cut[x] = (int32_t)dealt.size();
        if (x < used) {
            std::stable_sort(mine[x].begin(), mine[x].end(),
                             [](const Band& a, const Band& c) { return a.unit_cost > c.unit_cost; });
            for (const Band& m : mine[x])
                dealt.insert(dealt.end(), run + m.first, run + m.end);
        }
    }
    std::copy(dealt.begin(), dealt.end(), run);
}

// Joins the unweighted kinds of a storage type, where there are two or more, to
// its mixed kind: one kernel and one tail instead of each kind's.  In us, mixed and
// apart (launched; replayed as a graph, whose nodes cost more): two frames of 256 x
// 256 from 64 elements at orders 2 and 3 13.8 and 17.0 (20.6 and 42.3); 18 paired
// of 128 x 128 at six orders 33 and 50 (40 and 88); 24 paired of 512 x 512 from 128
// elements 350 and 396 (357 and 389); 24 unpaired of 768 x 768 924 and 1063 (931
// and 1069).  Left apart are
// - kinds whose LDS would hold the workgroups of half of the work (by cost) or more
//   to fewer per CU, in lists that fill the device more than kLong times, where
//   that decides: 48 frames of 512 x 512 with 7 KB tiles and one of 256 x 256 with
//   36 KB, all mixed 567 (575), its kind apart 532 (527); 24 of 512 x 512 with 14
//   KB, which fill it 8 times, 212 (218) and 220 (245).
// - two kinds of short units that fill it once: the kinds' own kernels hold seven
//   workgroups instead of six and switch nothing between units (24 frames of 256 x
//   256 at orders 2 and 3 85 mixed and 78; replayed 91 and 95).
// - any number of short unpaired kinds each of which fills it kManyFills times: the
//   tails are small by then (192 of 128 x 128 at six orders, and one with 36 KB
//   whose kind is apart, 252 mixed and 250; replayed 261 and 250).
// A kind that a captured launch has run mixed, or apart, stays so in every later
// list: the capture holds that kernel and no other.
void mix_kinds(std::vector<Unit>& units, int64_t (&lds)[hodmas::kBatchKinds], int cus,
               const RunsAs (&captured)[hodmas::kOrderKinds])
{
    constexpr int kMixedPerCu = 6;                   // workgroups of the mixed kernel its registers allow
    constexpr int64_t kLong = 12, kManyFills = 5;    // times what the device holds at once
    constexpr int64_t kShortUnit = 500000;           // slots
    int64_t count[hodmas::kOrderKinds] = {}, cost[hodmas::kOrderKinds] = {};
    for (const Unit& u : units) {
        ++count[u.kind];
        cost[u.kind] += u.cost;
    }
    bool joins[hodmas::kOrderKinds] = {};
    for (int dt = 0; dt < 3; ++dt) {
        // the mixed kernel's workgroups per CU at each kind's LDS (0: not of this type)
        int per_cu[hodmas::kOrderKinds] = {};
        int64_t n = 0, total = 0, no_more[kMixedPerCu + 1] = {};
        for (int kind = 0; kind < hodmas::kOrderKinds; ++kind) {
            if (!count[kind] || hodmas::kind_dtype(kind) != dt || hodmas::kind_cf(kind))
                continue;
            per_cu[kind] = (int)std::min<int64_t>(kMixedPerCu, std::max<int64_t>(1, hodmas::kMaxLdsBytes / lds[kind]));
            n += count[kind];
            total += cost[kind];
            for (int w = per_cu[kind]; w <= kMixedPerCu; ++w)
                no_more[w] += cost[kind];
        }
        // half of the work or more is in kinds that leave room for `least`
        int least = 1;
        while (least < kMixedPerCu && 2 * no_more[least] <= total)
            ++least;
        const int64_t fill = (int64_t)least * cus;
        if (n <= kLong * fill)
            least = 1;
        int members = 0, pairing = 1;
        int64_t fewest = 0, member_cost = 0, member_units = 0;
        for (int kind = 0; kind < hodmas::kOrderKinds; ++kind) {
            if (per_cu[kind] < least)
                continue;
            fewest = members++ ? std::min(fewest, count[kind]) : count[kind];
            pairing = std::max(pairing, hodmas::kind_pairing(kind));
            member_cost += cost[kind];
            member_units += count[kind];
        }
        const bool fills = members == 2 ? member_units > 4 * cus : pairing == 1 && fewest >= kManyFills * fill;
        const bool mixes = members >= 2 && !(member_cost < kShortUnit * member_units && fills);
        const int mixed = hodmas::mixed_kind(dt);
        for (int kind = 0; kind < hodmas::kOrderKinds; ++kind) {
            if (!per_cu[kind])
                continue;
            joins[kind] = captured[kind] == RunsAs::none ? mixes && per_cu[kind] >= least
                                                         : captured[kind] == RunsAs::mixed;
            if (joins[kind]) {
                lds[mixed] = std::max(lds[mixed], lds[kind]);
                lds[kind] = 0;
            }
        }
    }
    for (Unit& u : units)
        if (joins[u.kind])
            u.kind = hodmas::mixed_kind(hodmas::kind_dtype(u.kind));
}

// Workgroups a kind's kernel launches with: one per unit.  The device hands a
// workgroup out as another ends, which evens out better than fixed shares of a
// grid that just fills the device.  Measured so, and with fixed shares: one
// unpaired 2048 x 2048 frame from 256 elements at order 1 501 and 659 us, at
// order 6 789 and 917; one of 512 x 512 from 128 at order 2 28.8 and 39.5; eight
// of them at order 6, paired, 187 and 191; at order 1 90 and 89; 256 of 128 x 128
// at order 1 264 and 309.  From kMostWorkgroups on each takes several (1100 of 128 x
// 128, 70400 units: 1031 and 1254 us).  A mixed kind that fills the device twice
// draws its units instead, with as many workgroups as the device holds, which
// saves the start of a workgroup for each (24 FP16 frames of 17 shapes at all
// orders 862 us with fixed shares, 697 one per unit, 679 drawn).
int launch_grid(const hodmas_batch_s* b, int kind, bool draws)
{
    constexpr int kMostWorkgroups = 1 << 16;
    if (draws)
        return b->kind_grid[kind];
    return (int)std::min<int64_t>((int64_t)b->longest[kind] * hodmas::kXcds, kMostWorkgroups);
}

bool kind_draws(const hodmas_batch_s* b, int kind)
{
    return kind >= hodmas::kOrderKinds && b->draws[kind - hodmas::kOrderKinds];
}

// What the batch kernels take.
struct KernelArgs {
    const BatchHeader* hdr;
    const BatchFrame* frames;
    const BatchUnit* units;
    DrawCount* counts;
    void* ptr[4] = {&hdr, &frames, &units, &counts};
    // counts: the set the launch draws with, or -1
    KernelArgs(const hodmas_batch_s* b, int set)
        : hdr(reinterpret_cast<const BatchHeader*>(b->d_buf)),
          frames(reinterpret_cast<const BatchFrame*>(b->d_buf + b->off_frames)),
          units(reinterpret_cast<const BatchUnit*>(b->d_buf + b->off_units)),
          counts(set < 0 ? nullptr
                         : reinterpret_cast<DrawCount*>(b->d_buf + b->off_counts) + set * hodmas::kDrawCounts)
    {
    }
    KernelArgs(const KernelArgs&) = delete;
};

// Puts work on `st` behind the run's last, if that was on another stream.
bool follow(const hodmas_batch_s::Run& run, hipStream_t st)
{
    return !run.pending || run.stream == st || hipStreamWaitEvent(st, run.done, 0) == hipSuccess;
}
bool finish(hodmas_batch_s::Run& run, hipStream_t st)
{
    run.stream = st;
    run.pending = hipEventRecord(run.done, st) == hipSuccess;
    return run.pending;
}

}  // namespace

extern "C" {

hodmas_status hodmas_batch_create(int32_t max_frames, int64_t max_units, int64_t max_lds_bytes,
                                  uint32_t flags, hodmas_batch_t* out)
{
    if (!out)
        return HODMAS_EINVAL;
    *out = nullptr;
    if (max_frames < 1 || max_units < 1 || max_units > (int64_t(1) << 31) || max_lds_bytes < 0 ||
        max_lds_bytes > hodmas::kMaxLdsBytes || (flags & ~HODMAS_FLAG_ACC_PLAIN))
        return HODMAS_EINVAL;
    hodmas_batch_s* b = new (std::nothrow) hodmas_batch_s;
    if (!b)
        return HODMAS_ENOMEM;
    b->max_frames = max_frames;
    b->max_units = max_units;
    b->lds_bytes = max_lds_bytes > 0 ? max_lds_bytes : 64 * 1024;
    b->flags = flags;
    const bool comp = !(flags & HODMAS_FLAG_ACC_PLAIN);
    hipDeviceProp_t prop;
    if (hipGetDevice(&b->device) != hipSuccess || hipGetDeviceProperties(&prop, b->device) != hipSuccess) {
        delete b;
        return HODMAS_EDEVICE;
    }
    int max_grid = 0;
    for (int kind = 0; kind < hodmas::kBatchKinds; ++kind) {
        const void* fn = hodmas::batch_kernel(kind, comp);
        if (!fn)
            continue;   // no such kind under this accumulation mode
        if (b->lds_bytes > 64 * 1024 &&
            hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)b->lds_bytes) != hipSuccess) {
            (void)hipGetLastError();
            delete b;
            return HODMAS_EUNSUPPORTED;
        }
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, hodmas::kBlock, (size_t)b->lds_bytes) !=
                hipSuccess || per_cu < 1) {
            (void)hipGetLastError();
            delete b;
            return HODMAS_EUNSUPPORTED;
        }
        b->grid[kind] = per_cu * prop.multiProcessorCount;
        max_grid = std::max(max_grid, per_cu * prop.multiProcessorCount);
    }
    b->cus = prop.multiProcessorCount;
    b->off_frames = align_up(sizeof(BatchHeader));
    b->off_units = b->off_frames + align_up(sizeof(BatchFrame) * (size_t)max_frames);
    b->off_counts = b->off_units + align_up(sizeof(BatchUnit) * (size_t)max_units);
    b->bytes = b->off_counts + sizeof(DrawCount) * hodmas::kDrawCounts * (1 + kLaunches);
    bool ok = hipMalloc((void**)&b->d_buf, b->bytes) == hipSuccess &&
              hipHostMalloc((void**)&b->h_buf, b->bytes, hipHostMallocDefault) == hipSuccess &&
              hipEventCreateWithFlags(&b->copied, hipEventDisableTiming) == hipSuccess;
    for (hodmas_batch_s::Run& r : b->runs)
        ok = ok && hipEventCreateWithFlags(&r.done, hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        release(b);
        delete b;
        return HODMAS_ENOMEM;
    }
    std::memset(b->h_buf, 0, b->bytes);
    if (hipMemcpy(b->d_buf, b->h_buf, b->bytes, hipMemcpyHostToDevice) != hipSuccess) {
        release(b);
        delete b;
        return HODMAS_EDEVICE;
    }
    b->info.grid = max_grid;
    b->info.lds_bytes = b->lds_bytes;
    *out = b;
    return HODMAS_OK;
}

hodmas_status hodmas_batch_set(hodmas_batch_t b, const hodmas_plan_t* plans, const void* const* rf,
                               const int32_t* orders, float* const* images, int32_t n_frames,
                               void* stream)
{
    if (!valid_batch(b) || !plans || !rf || !orders || !images || n_frames < 1 ||
        n_frames > b->max_frames)
        return HODMAS_EINVAL;
    std::vector<Unit> units;
    int64_t pixch = 0;
    const bool comp = !(b->flags & HODMAS_FLAG_ACC_PLAIN);
    int64_t kl[hodmas::kBatchKinds] = {};   // LDS each kind's largest plan needs
    try {
        for (int32_t f = 0; f < n_frames; ++f) {
            const hodmas_plan_s* p = plans[f];
            if (!p || p->magic != hodmas::kPlanMagic || !rf[f] || !images[f])
                return HODMAS_EINVAL;
            if ((p->flags & HODMAS_FLAG_HOST_ONLY) || p->device != b->device)
                return HODMAS_EINVAL;
            if ((p->flags & HODMAS_FLAG_ACC_PLAIN) != (b->flags & HODMAS_FLAG_ACC_PLAIN))
                return HODMAS_EINVAL;
            const int cf = (p->flags & HODMAS_FLAG_CF) ? 1 : 0;
            if (cf && (b->flags & HODMAS_FLAG_ACC_PLAIN))
                return HODMAS_EUNSUPPORTED;   // coherence-weighted kinds accumulate compensated
            if (orders[f] < 1 || orders[f] > p->max_order)
                return HODMAS_EUNSUPPORTED;
            if (p->lds_bytes > b->lds_bytes)
                return HODMAS_EINVAL;
            if (p->tiling.tile_x * p->tiling.tile_z * p->tiling.split != hodmas::kBlock)
                return HODMAS_EINVAL;   // the batched kernels run 256-thread tiles
            // a mirror plan's units are the pairs: each left-half tile with its mirror
            const int pairing = (p->flags & HODMAS_FLAG_MIRROR) ? 2 : 1;
            const int n_units = (int)p->tiles.size() / pairing;
            const int half = p->grid.nx / p->tiling.tile_x / 2;   // tile columns left of the centre
            if ((int64_t)units.size() + n_units > b->max_units)
                return HODMAS_EINVAL;
            pixch += int64_t(p->grid.nx) * p->grid.nz * p->geom.n_elements;
            const int kind = hodmas::batch_kind(orders[f], p->rf.dtype, pairing, cf);
            kl[kind] = std::max(kl[kind], hodmas::launch_lds(p, orders[f]));
            for (int i = 0; i < n_units; ++i) {
                const int t = pairing == 1 ? i : i / half * 2 * half + i % half;
                const hodmas_tile_desc& td = p->tiles[t];
                const int64_t pix = int64_t(td.nx) * td.nz;
                int64_t cost = pix;  // zero-fill only
                if (td.n_active >= orders[f])
                    cost = td.n_active * (pix * (kSlots[orders[f]] + kCfSlots * cf) + int64_t(td.window) * 2);
                units.push_back(Unit{cost, kind, f, (int32_t)t});
            }
        }
    } catch (const std::bad_alloc&) {
        return HODMAS_ENOMEM;
    }
    RunsAs runs_as[hodmas::kOrderKinds];
    for (int kind = 0; kind < hodmas::kOrderKinds; ++kind)
        runs_as[kind] = kl[kind] ? RunsAs::apart : RunsAs::none;
    if (comp)
        mix_kinds(units, kl, b->cus, b->captured);
    for (int kind = 0; kind < hodmas::kOrderKinds; ++kind)
        if (runs_as[kind] != RunsAs::none && !kl[kind])
            runs_as[kind] = RunsAs::mixed;
    // Each kind runs with the LDS its own plans need, and with as many
    // workgroups at once as that LDS lets a CU hold.
    int kg[hodmas::kBatchKinds] = {};
    for (int kind = 0; kind < hodmas::kBatchKinds; ++kind) {
        if (kl[kind] == 0)
            continue;
        if (b->occ_lds[kind] != kl[kind]) {
            const void* fn = hodmas::batch_kernel(kind, comp);
            int per_cu = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, hodmas::kBlock, (size_t)kl[kind]) !=
                    hipSuccess || per_cu < 1) {
                (void)hipGetLastError();
                return HODMAS_EDEVICE;
            }
            b->occ_lds[kind] = kl[kind];
            b->occ_per_cu[kind] = per_cu;
        }
        kg[kind] = b->occ_per_cu[kind] * b->cus;
    }
    // grouped by kind (one kernel each), in frame and tile order
    auto by_kind = [](const Unit& x, const Unit& y) { return x.kind < y.kind; };
    if (!std::is_sorted(units.begin(), units.end(), by_kind))
        std::stable_sort(units.begin(), units.end(), by_kind);
    int32_t kb[hodmas::kBatchKinds] = {}, ke[hodmas::kBatchKinds] = {};
    for (size_t u = 0; u < units.size(); ++u) {
        const int k = units[u].kind;
        if (u == 0 || units[u - 1].kind != k)
            kb[k] = (int32_t)u;
        ke[k] = (int32_t)u + 1;
    }
    // Each kind's units, in frame and tile order (tile rows are depth bands),
    // are cut into one contiguous run per XCD that has workgroups, of about
    // equal estimated cost: an XCD then stages the RF of one frame, or of a
    // band of depths, and reads that frame's tables, instead of every XCD
    // fetching every frame.  Within a run the heaviest units go first.
    int32_t cuts[hodmas::kBatchKinds][hodmas::kXcds + 1] = {};
    try {
        std::vector<int64_t> pre;
        std::vector<Unit> dealt;
        for (int k = 0; k < hodmas::kBatchKinds; ++k) {
            const int n = ke[k] - kb[k];
            if (n <= 0)
                continue;
            const int used = std::min<int>(hodmas::kXcds, (int)std::min<int64_t>(kg[k], n));
            Unit* run = units.data() + kb[k];
            int32_t* cut = cuts[k];
            if (k >= hodmas::kOrderKinds) {
                deal_frames(run, n, used, cut, dealt);
                continue;
            }
            pre.assign((size_t)n + 1, 0);
            for (int u = 0; u < n; ++u)
                pre[u + 1] = pre[u] + run[u].cost;
            for (int x = 1; x < used; ++x) {
                const int64_t target = pre[n] * x / used;
                int i = (int)(std::lower_bound(pre.begin(), pre.end(), target) - pre.begin());
                i = std::max(i, cut[x - 1] + 1);     // every XCD in use gets a unit
                i = std::min(i, n - (used - x));
                cut[x] = i;
            }
            for (int x = used; x <= hodmas::kXcds; ++x)
                cut[x] = n;
            for (int x = 0; x < used; ++x)
                std::stable_sort(run + cut[x], run + cut[x + 1],
                                 [](const Unit& a, const Unit& c) { return a.cost > c.cost; });
        }
    } catch (const std::bad_alloc&) {
        return HODMAS_ENOMEM;
    }
    // the pinned staging buffer may still feed the previous asynchronous copy
    if (b->copy_pending && hipEventSynchronize(b->copied) != hipSuccess)
        return HODMAS_EDEVICE;
    b->copy_pending = false;
    BatchHeader* hdr = reinterpret_cast<BatchHeader*>(b->h_buf);
    BatchFrame* frames = reinterpret_cast<BatchFrame*>(b->h_buf + b->off_frames);
    BatchUnit* list = reinterpret_cast<BatchUnit*>(b->h_buf + b->off_units);
    std::memset(hdr, 0, sizeof(BatchHeader));
    hdr->n_units = (int32_t)units.size();
    hdr->n_frames = n_frames;
    std::memcpy(hdr->begin, kb, sizeof(kb));
    std::memcpy(hdr->end, ke, sizeof(ke));
    std::memcpy(hdr->xcd, cuts, sizeof(cuts));
    for (int k = 0; k < hodmas::kBatchKinds; ++k) {
        b->longest[k] = 0;
        for (int x = 0; x < hodmas::kXcds; ++x)
            b->longest[k] = std::max(b->longest[k], cuts[k][x + 1] - cuts[k][x]);
    }
    for (int dt = 0; dt < 3; ++dt) {
        const int k = hodmas::mixed_kind(dt);
        b->draws[dt] = ke[k] - kb[k] > 2 * kg[k];   // two units without drawing
    }
    std::memcpy(b->begin, hdr->begin, sizeof(b->begin));
    std::memcpy(b->end, hdr->end, sizeof(b->end));
    std::memcpy(b->runs_as, runs_as, sizeof(runs_as));
    std::memcpy(b->kind_lds, kl, sizeof(kl));
    std::memcpy(b->kind_grid, kg, sizeof(kg));
    for (int32_t f = 0; f < n_frames; ++f) {
        std::memset(&frames[f], 0, sizeof(BatchFrame));
        frames[f].args = hodmas::frame_args(plans[f], rf[f], images[f]);
        frames[f].order = orders[f];
        frames[f].dtype = plans[f]->rf.dtype;
        frames[f].pairing = (plans[f]->flags & HODMAS_FLAG_MIRROR) ? 2 : 1;
    }
    for (size_t u = 0; u < units.size(); ++u)
        list[u] = BatchUnit{units[u].frame, units[u].tile};
    const size_t used = b->off_units + sizeof(BatchUnit) * units.size();
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (hipMemcpyAsync(b->d_buf, b->h_buf, used, hipMemcpyHostToDevice, st) != hipSuccess ||
        hipEventRecord(b->copied, st) != hipSuccess) {
        (void)hipGetLastError();
        return HODMAS_EDEVICE;
    }
    b->copy_pending = true;
    b->has_list = true;
    b->list_replayed = false;
    b->info.n_frames = n_frames;
    b->info.n_units = (int64_t)units.size();
    b->info.pixel_channels = pixch;
    b->info.grid = *std::max_element(kg, kg + hodmas::kBatchKinds);
    b->info.lds_bytes = *std::max_element(kl, kl + hodmas::kBatchKinds);
    return HODMAS_OK;
}

hodmas_status hodmas_batch_launch(hodmas_batch_t b, void* stream)
{
    if (!valid_batch(b) || !b->has_list)
        return HODMAS_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // A captured launch may run again at any time beside others, so it gets no
    // draw counts (and the event would be the capture's, not this launch's).
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const bool captured = hipStreamIsCapturing(st, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
    const int turn = b->next_run;
    hodmas_batch_s::Run& run = b->runs[turn];
    KernelArgs drawing(b, 1 + turn), fixed(b, -1);
    bool ok = true;
    for (int kind = 0; kind < hodmas::kBatchKinds && ok; ++kind) {
        if (b->end[kind] <= b->begin[kind])
            continue;
        const bool draws = !captured && kind_draws(b, kind);
        const int grid = launch_grid(b, kind, draws);
        if (kind < hodmas::kOrderKinds)
            ok = hodmas::launch_batch(kind, fixed.hdr, fixed.frames, fixed.units, grid,
                                      !(b->flags & HODMAS_FLAG_ACC_PLAIN), b->kind_lds[kind], stream) == 0;
        else
            ok = (!draws || follow(run, st)) &&
                 hipLaunchKernel(hodmas::batch_kernel(kind, true), dim3(grid), dim3(hodmas::kBlock),
                                 (draws ? drawing : fixed).ptr, (size_t)b->kind_lds[kind], st) == hipSuccess;
    }
    if (!captured) {
        ok = finish(run, st) && ok;
        b->next_run = (turn + 1) % kLaunches;
    } else if (ok) {
        for (int kind = 0; kind < hodmas::kOrderKinds; ++kind)
            if (b->runs_as[kind] != RunsAs::none)
                b->captured[kind] = b->runs_as[kind];
    }
    if (!ok) {
        (void)hipGetLastError();
        return HODMAS_EDEVICE;
    }
    return HODMAS_OK;
}

}  // extern "C"

// The graph holds one node per kind of the work list it was captured for and
// no edges between them: kinds write disjoint images, so one kind's last
// units overlap the next kind's start instead of the GPU draining between
// kinds.  Each node reads its unit range from the device header, so a later
// hodmas_batch_set with the same kinds (or fewer) needs no re-capture; a set
// that brings a kind the graph lacks has the graph rebuilt at the next
// replay, with a node for every kind seen so far.  Nodes are not made for
// absent kinds: every node of a graph launch costs time even when switched
// off.  Before each replay the nodes are fitted to the current work list in
// the instantiated graph itself: a kind that is absent is switched off, and a
// present kind runs with the LDS its own plans need and the grid of its units
// (launch_grid), which differs from list to list.
namespace {

hipKernelNodeParams node_params(const hodmas_batch_s* b, int kind, int grid, int64_t lds, KernelArgs& args)
{
    hipKernelNodeParams kp;
    std::memset(&kp, 0, sizeof(kp));
    kp.func = const_cast<void*>(hodmas::batch_kernel(kind, !(b->flags & HODMAS_FLAG_ACC_PLAIN)));
    kp.gridDim = dim3(grid);
    kp.blockDim = dim3(hodmas::kBlock);
    kp.sharedMemBytes = (unsigned)lds;
    kp.kernelParams = args.ptr;
    kp.extra = nullptr;
    return kp;
}

// (Re)build the graph with a node for every kind in `want`.
bool build_graph(hodmas_batch_s* b, const bool* want)
{
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->exec = nullptr;
    b->graph = nullptr;
    KernelArgs args(b, -1);
    bool ok = hipGraphCreate(&b->graph, 0) == hipSuccess;
    for (int kind = 0; kind < hodmas::kBatchKinds && ok; ++kind) {
        b->node[kind] = nullptr;
        b->node_on[kind] = false;
        if (!want[kind] || !hodmas::batch_kernel(kind, !(b->flags & HODMAS_FLAG_ACC_PLAIN)))
            continue;   // not wanted, or no such kind under this accumulation mode
        const hipKernelNodeParams kp = node_params(b, kind, b->grid[kind], b->lds_bytes, args);
        hipGraphNode_t node = nullptr;
        ok = hipGraphAddKernelNode(&node, b->graph, nullptr, 0, &kp) == hipSuccess;
        b->node[kind] = node;
        b->node_grid[kind] = b->grid[kind];
        b->node_lds[kind] = b->lds_bytes;
        b->node_on[kind] = true;
        b->node_draws[kind] = false;
    }
    if (ok)
        ok = hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0) == hipSuccess;
    if (ok && !b->replayed.done)
        ok = hipEventCreateWithFlags(&b->replayed.done, hipEventDisableTiming) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        if (b->exec) (void)hipGraphExecDestroy(b->exec);
        if (b->graph) (void)hipGraphDestroy(b->graph);
        b->graph = nullptr;
        b->exec = nullptr;
        for (int kind = 0; kind < hodmas::kBatchKinds; ++kind)
            b->node[kind] = nullptr;
    }
    return ok;
}

}  // namespace

extern "C" {

hodmas_status hodmas_batch_capture(hodmas_batch_t b)
{
    if (!valid_batch(b))
        return HODMAS_EINVAL;
    if (b->exec)
        return HODMAS_OK;
    // the kinds of the current work list, or every kind before any list is set
    bool want[hodmas::kBatchKinds];
    for (int kind = 0; kind < hodmas::kBatchKinds; ++kind)
        want[kind] = !b->has_list || b->end[kind] > b->begin[kind];
    return build_graph(b, want) ? HODMAS_OK : HODMAS_EDEVICE;
}

hodmas_status hodmas_batch_replay(hodmas_batch_t b, void* stream)
{
    if (!valid_batch(b) || !b->exec || !b->has_list)
        return HODMAS_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // a launch of `exec` still in flight must not see its nodes change
    bool change = false, missing = false;
    for (int kind = 0; kind < hodmas::kBatchKinds; ++kind) {
        const int n = b->end[kind] - b->begin[kind];
        missing = missing || (n > 0 && !b->node[kind]);
        change = change || (n > 0) != b->node_on[kind] ||
                 (n > 0 && (launch_grid(b, kind, kind_draws(b, kind)) != b->node_grid[kind] ||
                            kind_draws(b, kind) != b->node_draws[kind] || b->kind_lds[kind] != b->node_lds[kind]));
    }
    const bool first = !b->list_replayed;
    b->list_replayed = true;
    if ((change || missing) && b->replayed.pending) {
        // ... so a list's first replay runs its kernels directly while one is:
        // a loop of sets and replays then never waits for the GPU.  (Fitting a
        // graph pays from the list's second replay on.)
        if (first && hipEventQuery(b->replayed.done) == hipErrorNotReady) {
            (void)hipGetLastError();
            return hodmas_batch_launch(b, stream);
        }
        if (hipEventSynchronize(b->replayed.done) != hipSuccess) {
            (void)hipGetLastError();
            return HODMAS_EDEVICE;
        }
        b->replayed.pending = false;
    }
    if (missing) {
        // a kind the graph has no node for: rebuild with every kind seen so far
        bool want[hodmas::kBatchKinds];
        for (int kind = 0; kind < hodmas::kBatchKinds; ++kind)
            want[kind] = b->node[kind] != nullptr || b->end[kind] > b->begin[kind];
        if (!build_graph(b, want))
            return HODMAS_EDEVICE;
        change = true;
    }
    for (int kind = 0; kind < hodmas::kBatchKinds && change; ++kind) {
        if (!b->node[kind])
            continue;
        const int n = b->end[kind] - b->begin[kind];
        const bool on = n > 0;
        if (on) {
            const bool draws = kind_draws(b, kind);
            const int grid = launch_grid(b, kind, draws);
            if (grid != b->node_grid[kind] || draws != b->node_draws[kind] ||
                b->kind_lds[kind] != b->node_lds[kind]) {
                KernelArgs args(b, draws ? 0 : -1);
                const hipKernelNodeParams kp = node_params(b, kind, grid, b->kind_lds[kind], args);
                if (hipGraphExecKernelNodeSetParams(b->exec, b->node[kind], &kp) != hipSuccess) {
                    (void)hipGetLastError();
                    return HODMAS_EDEVICE;
                }
                b->node_grid[kind] = grid;
                b->node_draws[kind] = draws;
                b->node_lds[kind] = b->kind_lds[kind];
            }
        }
        if (on != b->node_on[kind]) {
            if (hipGraphNodeSetEnabled(b->exec, b->node[kind], on ? 1 : 0) != hipSuccess) {
                (void)hipGetLastError();
                return HODMAS_EDEVICE;
            }
            b->node_on[kind] = on;
        }
    }
    const bool ok = follow(b->replayed, st) && hipGraphLaunch(b->exec, st) == hipSuccess;
    if (!(finish(b->replayed, st) && ok)) {
        (void)hipGetLastError();
        return HODMAS_EDEVICE;
    }
    return HODMAS_OK;
}

hodmas_status hodmas_batch_get_info(hodmas_batch_t b, hodmas_batch_info* info)
{
    if (!valid_batch(b) || !info)
        return HODMAS_EINVAL;
    *info = b->info;
    return HODMAS_OK;
}

hodmas_status hodmas_batch_destroy(hodmas_batch_t b)
{
    if (!b)
        return HODMAS_OK;
    if (b->magic != kBatchMagic)
        return HODMAS_EINVAL;
    release(b);
    b->magic = 0;
    delete b;
    return HODMAS_OK;
}

}  // extern "C"
