// batch.cpp -- batched ECB: validation, tile planning, graph capture, tuning.
//
// A batch is many messages, each with its own key triple (an index into a
// device table of schedules) and direction.  The paper runs one message and
// launches one kernel per 1 MiB chunk (Listing 1.1, Section II.B); with
// thousands of short messages, per-launch cost would dominate, so the whole
// batch becomes one launch: of the persistent kernel in k_batch.hip, or of
// k_batch_team.hip's for few tiles.
//
// Planning.  Each message is cut into wave tiles of 2048 blocks (one key per
// wave, scalar key masks).  Its remainder, if shorter than the context's
// wave_remainder (1800 unless tuned), is cut into lane slots of 32 blocks
// instead; lane slots from all messages are packed 64 to a lane tile, where
// each lane has its own key.  A 2048-block
// tile then never runs mostly empty for short messages.  Lane tiles go first
// so that the cheaper wave tiles fill the tail of the launch.  The host only
// counts: it leaves one record per message in pinned memory, and a kernel
// (k_plan.hip) writes the slots on the device.
//
// Graphs.  The kernels read the tile count from the plan's header, so one
// captured graph (a single kernel node) serves every batch with the same
// base pointer, schedule table and launch shape; it is captured on a private
// stream, behind a context's first batch or by the first replay that needs it,
// and replayed on the caller's by tdes_ecb_batch_replay.  Batches of few tiles have a kernel,
// and a graph, of their own.
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "batch_plan.h"
#include "internal.h"

namespace {

constexpr uint32_t kWaveBlocks = 2048;
constexpr uint32_t kLaneBlocks = 32;
constexpr uint32_t kLanesPerTile = 64;
// Default cut-over: a remainder this long still takes a wave tile.  A lane tile
// costs more per block (a key per lane); the autotuner may choose another value,
// and for 4096 messages does: 1536, 1.4% faster (360.0 -> 355.1 us).  The default
// is what the interface states.
constexpr uint32_t kDefaultWaveRemainder = 1800;
constexpr uint32_t kMaxTilesPerDraw = 16;
constexpr uint64_t kMaxJobBlocks = 1ull << 40;

}  // namespace

struct tdes_ctx {
    int device = 0;
    int cu_count = 0;
    hipStream_t capture_stream = nullptr;
    uint32_t *d_counter = nullptr;
    // The plan: the messages' records in pinned host memory, in two buffers in turn so that the host writes one
    // batch's while the GPU works on the last; the header and slots on the device.
    uint8_t *d_plan = nullptr;
    size_t cap_slots = 0;
    struct Records {
        tdes::PlanMessage *host = nullptr;
        size_t cap = 0;
        hipEvent_t done = nullptr;  // the batch with these records, and its last replay, have finished
    } records[2];
    int last = 0;  // the last batch's records
    bool have_plan = false;
    // Last planned batch (for replay).
    const void *last_sched = nullptr;
    uint8_t *last_base = nullptr;
    uint32_t last_tiles = 0;
    // Launch shape and tiling.
    uint32_t threads = 256;
    uint32_t groups_per_cu = 4;
    uint32_t wave_remainder = kDefaultWaveRemainder;  // remainders this long take a wave tile
    uint32_t tiles_per_draw = 1;                      // tiles a wave takes per counter draw
    bool capped = false;                              // launch the 120-VGPR kernel variant
    // Captured graphs (one wave per tile; a workgroup per tile) and everything their kernel nodes were captured with.
    struct Graph {
        hipGraphExec_t exec = nullptr;
        const void *sched = nullptr, *base = nullptr, *plan = nullptr;
        uint32_t grid = 0, threads = 0, draw = 0;
        bool capped = false;

        void drop() {
            if (exec) (void)hipGraphExecDestroy(exec);
            exec = nullptr;
        }
    } graphs[2];
    tdes_batch_info info{};
};

namespace {

// Room for n_messages records, no longer read by an earlier batch's plan kernel.
int ensure_records(tdes_ctx::Records *r, size_t n_messages) {
    if (hipEventSynchronize(r->done) != hipSuccess) return TDES_ERR_HIP;
    if (n_messages <= r->cap) return TDES_OK;
    const size_t n = std::max<size_t>(n_messages, std::max<size_t>(1024, r->cap * 2));
    if (r->host) (void)hipHostFree(r->host);
    r->host = nullptr;
    r->cap = 0;
    if (hipHostMalloc(&r->host, n * sizeof(tdes::PlanMessage), hipHostMallocDefault) != hipSuccess) {
        r->host = nullptr;
        return TDES_ERR_NOMEM;
    }
    r->cap = n;
    return TDES_OK;
}

// Room for n_slots slots on the device.
int ensure_slots(tdes_ctx *c, size_t n_slots) {
    if (n_slots <= c->cap_slots && c->d_plan) return TDES_OK;
    const size_t n = std::max<size_t>(n_slots, std::max<size_t>(8192, c->cap_slots * 2));
    if (c->d_plan) {
        // The old buffer may still be in use by a kernel, and the captured graphs point into it.
        if (hipEventSynchronize(c->records[c->last].done) != hipSuccess) return TDES_ERR_HIP;
        for (auto &g : c->graphs) g.drop();
        (void)hipFree(c->d_plan);
        c->d_plan = nullptr;
        c->have_plan = false;
        c->cap_slots = 0;
    }
    if (hipMalloc(&c->d_plan, sizeof(tdes::PlanHeader) + n * sizeof(tdes::Slot)) != hipSuccess) {
        c->d_plan = nullptr;
        return TDES_ERR_NOMEM;
    }
    c->cap_slots = n;
    return TDES_OK;
}

struct Interval {
    uint64_t lo, hi;
    uint32_t job;
};

int validate_jobs(const tdes_job *jobs, uint32_t n_jobs, uint64_t n_scheds, uintptr_t base) {
    // Batches are usually laid out in order, inputs apart from outputs or every message in place: then the
    // outputs ascend without touching, no input reaches another message's output, and nothing is left to
    // sort or search (4096 messages: 0.3 ms).
    uint64_t in_lo = ~0ull, in_hi = 0, out_lo = ~0ull, out_hi = 0;
    bool ascending = true, in_place = true;
    for (uint32_t j = 0; j < n_jobs; j++) {
        const tdes_job &x = jobs[j];
        if (x.direction != TDES_ENCRYPT && x.direction != TDES_DECRYPT) return TDES_ERR_ARG;
        if (x.sched_idx >= n_scheds) return TDES_ERR_SIZE;
        if (x.n_blocks > kMaxJobBlocks) return TDES_ERR_SIZE;
        if (((base + x.in_off) | (base + x.out_off)) & 7) return TDES_ERR_ALIGN;
        if (x.n_blocks == 0) continue;
        const uint64_t bytes = x.n_blocks * 8;
        if (x.in_off + bytes < x.in_off || x.out_off + bytes < x.out_off) return TDES_ERR_SIZE;
        if (x.in_off != x.out_off && x.in_off < x.out_off + bytes && x.out_off < x.in_off + bytes)
            return TDES_ERR_OVERLAP;
        ascending = ascending && x.out_off >= out_hi;
        in_place = in_place && x.in_off == x.out_off;
        in_lo = std::min(in_lo, x.in_off);
        in_hi = std::max(in_hi, x.in_off + bytes);
        out_lo = std::min(out_lo, x.out_off);
        out_hi = std::max(out_hi, x.out_off + bytes);
    }
    if (ascending && (in_place || in_hi <= out_lo || out_hi <= in_lo)) return TDES_OK;
    std::vector<Interval> outs;
    outs.reserve(n_jobs);
    for (uint32_t j = 0; j < n_jobs; j++)
        if (jobs[j].n_blocks) outs.push_back({jobs[j].out_off, jobs[j].out_off + jobs[j].n_blocks * 8, j});
    std::sort(outs.begin(), outs.end(), [](const Interval &a, const Interval &b) { return a.lo < b.lo; });
    for (size_t i = 1; i < outs.size(); i++)
        if (outs[i].lo < outs[i - 1].hi) return TDES_ERR_OVERLAP;  // two outputs share bytes
    // No message may read bytes that another message writes.
    for (uint32_t j = 0; j < n_jobs; j++) {
        const tdes_job &x = jobs[j];
        if (x.n_blocks == 0) continue;
        const uint64_t lo = x.in_off, hi = x.in_off + x.n_blocks * 8;
        size_t k = std::upper_bound(outs.begin(), outs.end(), hi,
                                    [](uint64_t v, const Interval &iv) { return v <= iv.lo; }) -
                   outs.begin();
        while (k > 0) {
            const Interval &iv = outs[--k];
            if (iv.hi <= lo) break;
            if (iv.job != j) return TDES_ERR_OVERLAP;
        }
    }
    return TDES_OK;
}

struct Plan {
    uint32_t messages = 0;        // records written
    uint64_t wave = 0, lane = 0;  // slots
    uint64_t blocks = 0;
    uint32_t max_wave = 0;        // wave tiles of the longest message

    uint64_t lane_tiles() const { return (lane + kLanesPerTile - 1) / kLanesPerTile; }
    uint64_t tiles() const { return lane_tiles() + wave; }
    uint64_t slots() const { return lane_tiles() * kLanesPerTile + wave; }
};

// Writes the records of a batch (there is room for n_jobs).  TDES_ERR_SIZE if it has too many slots.
int plan_jobs(uint32_t wave_remainder, const tdes_job *jobs, uint32_t n_jobs, tdes::PlanMessage *records, Plan *plan) {
    Plan p;
    for (uint32_t j = 0; j < n_jobs; j++) {
        const tdes_job &x = jobs[j];
        if (x.n_blocks == 0) continue;
        const uint32_t rem = (uint32_t)(x.n_blocks % kWaveBlocks);
        const bool wave_rem = rem >= wave_remainder;
        const uint64_t wave = x.n_blocks / kWaveBlocks + wave_rem;
        tdes::PlanMessage &m = records[p.messages++];
        m.in_off = x.in_off;
        m.out_off = x.out_off;
        m.n_blocks = x.n_blocks;
        m.ks_off = x.sched_idx * (TDES_SCHED_BYTES / 4) + x.direction * tdes::kDirWords;
        m.wave_first = (uint32_t)p.wave;
        m.lane_first = (uint32_t)p.lane;
        m.wave_tiles = (uint32_t)wave;
        p.wave += wave;
        if (!wave_rem) p.lane += (rem + kLaneBlocks - 1) / kLaneBlocks;
        p.blocks += x.n_blocks;
        p.max_wave = std::max(p.max_wave, m.wave_tiles);
        if (p.slots() >= 1ull << 31) return TDES_ERR_SIZE;
    }
    *plan = p;
    return TDES_OK;
}

// The planned batch's kernel: a workgroup per tile for few tiles, one wave per tile for many.
// captured: the launch is replayed for other batches of its kind too.
hipError_t launch_kernel(tdes_ctx *c, const void *sched, uint8_t *base, bool captured, hipStream_t stream) {
    const tdes::PlanHeader *hdr = reinterpret_cast<const tdes::PlanHeader *>(c->d_plan);
    const tdes::Slot *slots = reinterpret_cast<const tdes::Slot *>(c->d_plan + sizeof(tdes::PlanHeader));
    const uint32_t *ks = static_cast<const uint32_t *>(sched);
    if (c->last_tiles <= tdes::kTeamTiles)
        return tdes::launch_batch_team(ks, hdr, slots, base, captured ? tdes::kTeamTiles : c->last_tiles, stream);
    return tdes::launch_batch(ks, hdr, slots, c->d_counter, base, (uint32_t)c->cu_count * c->groups_per_cu, c->threads,
                              c->tiles_per_draw, c->capped, stream);
}

// The graph of that launch, captured if the context has none for it; nullptr on failure (which leaves no error
// behind for the next launch's check to find).
hipGraphExec_t plan_graph(tdes_ctx *c, const void *sched, uint8_t *base) {
    const bool team = c->last_tiles <= tdes::kTeamTiles;
    const uint32_t grid = (uint32_t)c->cu_count * c->groups_per_cu;
    tdes_ctx::Graph &g = c->graphs[team];
    const bool same_shape = team || (g.grid == grid && g.threads == c->threads && g.draw == c->tiles_per_draw &&
                                     g.capped == c->capped);
    if (g.exec && g.sched == sched && g.base == base && g.plan == c->d_plan && same_shape) return g.exec;
    g.drop();
    hipGraph_t graph = nullptr;
    if (hipStreamBeginCapture(c->capture_stream, hipStreamCaptureModeThreadLocal) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    const hipError_t le = launch_kernel(c, sched, base, true, c->capture_stream);
    const hipError_t ce = hipStreamEndCapture(c->capture_stream, &graph);
    if (le != hipSuccess || ce != hipSuccess || !graph) {
        if (graph) (void)hipGraphDestroy(graph);
        (void)hipGetLastError();
        return nullptr;
    }
    const hipError_t ie = hipGraphInstantiate(&g.exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (ie != hipSuccess) {
        g.exec = nullptr;
        (void)hipGetLastError();
        return nullptr;
    }
    g.sched = sched;
    g.base = base;
    g.plan = c->d_plan;
    g.grid = grid;
    g.threads = c->threads;
    g.draw = c->tiles_per_draw;
    g.capped = c->capped;
    c->info.graph_captures++;
    return g.exec;
}

}  // namespace

extern "C" int tdes_ctx_create(tdes_ctx **out, int device) {
    if (!out) return TDES_ERR_NULL;
    *out = nullptr;
    int n_dev = 0;
    if (hipGetDeviceCount(&n_dev) != hipSuccess) return TDES_ERR_HIP;
    if (device >= n_dev) return TDES_ERR_ARG;
    if (device < 0 && hipGetDevice(&device) != hipSuccess) return TDES_ERR_HIP;
    tdes::DeviceGuard guard(device);
    if (!guard.ok()) return TDES_ERR_HIP;
    tdes::DeviceInfo dinfo;
    if (tdes::device_info(&dinfo) != TDES_OK) return TDES_ERR_HIP;
    tdes_ctx *c = new (std::nothrow) tdes_ctx;
    if (!c) return TDES_ERR_NOMEM;
    c->device = dinfo.device;
    c->cu_count = dinfo.cu_count;
    bool ok = hipStreamCreateWithFlags(&c->capture_stream, hipStreamNonBlocking) == hipSuccess &&
              hipEventCreateWithFlags(&c->records[0].done, hipEventDisableTiming) == hipSuccess &&
              hipEventCreateWithFlags(&c->records[1].done, hipEventDisableTiming) == hipSuccess &&
              hipMalloc(&c->d_counter, 256) == hipSuccess && hipMemset(c->d_counter, 0, 256) == hipSuccess &&
              hipDeviceSynchronize() == hipSuccess;
    if (!ok) {
        tdes_ctx_destroy(c);
        return TDES_ERR_HIP;
    }
    c->info.threads = c->threads;
    c->info.groups_per_cu = c->groups_per_cu;
    c->info.wave_remainder = c->wave_remainder;
    c->info.tiles_per_draw = c->tiles_per_draw;
    *out = c;
    return TDES_OK;
}

extern "C" int tdes_ctx_destroy(tdes_ctx *c) {
    if (!c) return TDES_OK;
    tdes::DeviceGuard guard(c->device);
    for (auto &r : c->records)
        if (r.done) (void)hipEventSynchronize(r.done);
    for (auto &g : c->graphs) g.drop();
    if (c->d_plan) (void)hipFree(c->d_plan);
    for (auto &r : c->records) {
        if (r.host) (void)hipHostFree(r.host);
        if (r.done) (void)hipEventDestroy(r.done);
    }
    if (c->d_counter) (void)hipFree(c->d_counter);
    if (c->capture_stream) (void)hipStreamDestroy(c->capture_stream);
    delete c;
    return TDES_OK;
}

extern "C" int tdes_ctx_set_tuning(tdes_ctx *c, uint32_t threads, uint32_t groups_per_cu, uint32_t wave_remainder,
                                   uint32_t tiles_per_draw) {
    if (!c) return TDES_ERR_NULL;
    if (threads == 0 || threads > 256 || threads % 64 != 0 || groups_per_cu == 0 || groups_per_cu > 64)
        return TDES_ERR_ARG;
    if (wave_remainder > kWaveBlocks || tiles_per_draw > kMaxTilesPerDraw) return TDES_ERR_ARG;
    c->threads = threads;
    c->groups_per_cu = groups_per_cu;
    c->wave_remainder = wave_remainder ? wave_remainder : kDefaultWaveRemainder;
    c->tiles_per_draw = tiles_per_draw ? tiles_per_draw : 1;
    c->info.threads = threads;
    c->info.groups_per_cu = groups_per_cu;
    c->info.wave_remainder = c->wave_remainder;
    c->info.tiles_per_draw = c->tiles_per_draw;
    return TDES_OK;
}

namespace tdes {
void ctx_set_capped(tdes_ctx *c, bool capped) { c->capped = capped; }
}  // namespace tdes

extern "C" int tdes_ctx_get_info(const tdes_ctx *c, tdes_batch_info *info) {
    if (!c || !info) return TDES_ERR_NULL;
    *info = c->info;
    return TDES_OK;
}

extern "C" int tdes_ecb_batch(tdes_ctx *c, const tdes_job *jobs, uint32_t n_jobs, const void *dev_sched_table,
                              uint64_t n_scheds, void *dev_base, uint32_t flags, void *stream) {
    if (!c) return TDES_ERR_NULL;
    if (n_jobs == 0) return TDES_OK;
    if (!jobs || !dev_sched_table || !dev_base) return TDES_ERR_NULL;
    if (flags & ~(TDES_BATCH_NO_GRAPH | TDES_BATCH_PER_MESSAGE)) return TDES_ERR_ARG;
    if ((reinterpret_cast<uintptr_t>(dev_sched_table) & 3) != 0) return TDES_ERR_ALIGN;
    if (n_scheds == 0 || n_scheds > (1ull << 32) / (TDES_SCHED_BYTES / 4)) return TDES_ERR_SIZE;
    int rc = validate_jobs(jobs, n_jobs, n_scheds, reinterpret_cast<uintptr_t>(dev_base));
    if (rc != TDES_OK) return rc;
    tdes::DeviceGuard guard(c->device);
    if (!guard.ok()) return TDES_ERR_HIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t *base = static_cast<uint8_t *>(dev_base);
    const uint32_t *table = static_cast<const uint32_t *>(dev_sched_table);

    if (flags & TDES_BATCH_PER_MESSAGE) {
        // The baseline: one plain launch per message, in order, on the stream.
        for (uint32_t j = 0; j < n_jobs; j++) {
            const tdes_job &x = jobs[j];
            if (x.n_blocks == 0) continue;
            const uint32_t *ks = table + x.sched_idx * (TDES_SCHED_BYTES / 4) + x.direction * tdes::kDirWords;
            if (tdes::launch_auto(ks, base + x.in_off, base + x.out_off, x.n_blocks, s) != hipSuccess)
                return TDES_ERR_HIP;
        }
        return TDES_OK;
    }

    tdes_ctx::Records &rec = c->records[c->last ^ 1];
    rc = ensure_records(&rec, n_jobs);
    if (rc != TDES_OK) return rc;
    Plan p;
    rc = plan_jobs(c->wave_remainder, jobs, n_jobs, rec.host, &p);
    if (rc != TDES_OK) return rc;
    rc = ensure_slots(c, p.slots());
    if (rc != TDES_OK) return rc;
    c->info.tiles = p.tiles();
    c->info.wave_tiles = p.wave;
    c->info.lane_tiles = p.lane_tiles();
    c->info.slots = p.slots();
    c->info.blocks = p.blocks;
    c->info.padded_blocks = p.tiles() * kWaveBlocks;
    c->have_plan = true;
    c->last_sched = dev_sched_table;
    c->last_base = base;
    c->last_tiles = (uint32_t)p.tiles();
    if (p.messages == 0) return TDES_OK;
    // A previous launch on another stream may still read the device plan.
    if (hipStreamWaitEvent(s, c->records[c->last].done, 0) != hipSuccess) {
        c->have_plan = false;
        return TDES_ERR_HIP;
    }
    // The batch's launch follows the plan kernel directly: as a graph it would start 7 us later, and with an event
    // recorded between the two kernels 3 us later.
    if (tdes::launch_plan(rec.host, p.messages, p.max_wave, reinterpret_cast<tdes::PlanHeader *>(c->d_plan),
                          reinterpret_cast<tdes::Slot *>(c->d_plan + sizeof(tdes::PlanHeader)), (uint32_t)p.tiles(),
                          (uint32_t)p.lane, s) != hipSuccess ||
        launch_kernel(c, dev_sched_table, base, false, s) != hipSuccess)
        rc = TDES_ERR_HIP;
    if (hipEventRecord(rec.done, s) != hipSuccess) rc = TDES_ERR_HIP;
    c->last ^= 1;
    if (rc != TDES_OK) {
        c->have_plan = false;
        return rc;
    }
    // The first graph of the batch's kind, for replays, captured while the GPU is at work.  This call does not need
    // it: if the capture fails, a replay tries again, and a graph for other buffers or another shape is left to the
    // replay that wants it (captured here, it cost a caller that alternates two buffers 5 us a call: 48 messages,
    // waited for, 47.9 us, and 42.6 without).
    if (!(flags & TDES_BATCH_NO_GRAPH) && !c->graphs[c->last_tiles <= tdes::kTeamTiles].exec)
        (void)plan_graph(c, dev_sched_table, base);
    return TDES_OK;
}

extern "C" int tdes_ecb_batch_replay(tdes_ctx *c, uint32_t flags, void *stream) {
    if (!c) return TDES_ERR_NULL;
    if (flags & ~TDES_BATCH_NO_GRAPH) return TDES_ERR_ARG;
    if (!c->have_plan) return TDES_ERR_STATE;
    if (c->last_tiles == 0) return TDES_OK;
    tdes::DeviceGuard guard(c->device);
    if (!guard.ok()) return TDES_ERR_HIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // Order after the plan kernel and the previous launch, whichever stream they ran on.
    hipEvent_t done = c->records[c->last].done;
    if (hipStreamWaitEvent(s, done, 0) != hipSuccess) return TDES_ERR_HIP;
    if (flags & TDES_BATCH_NO_GRAPH) {
        if (launch_kernel(c, c->last_sched, c->last_base, false, s) != hipSuccess) return TDES_ERR_HIP;
    } else {
        hipGraphExec_t exec = plan_graph(c, c->last_sched, c->last_base);
        if (!exec || hipGraphLaunch(exec, s) != hipSuccess) return TDES_ERR_HIP;
    }
    return hipEventRecord(done, s) == hipSuccess ? TDES_OK : TDES_ERR_HIP;
}
