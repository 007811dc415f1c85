// k_static.hip -- batched ECB that allocates nothing: tdes_ecb_batch_static.
//
// The same operation as tdes_ecb_batch (every message ECB-EDE'd on its own
// under its own key triple and direction, Abstract and Section II.A), for
// callers that cannot allocate device memory (code under HIP graph capture,
// tight serving loops, harnesses that forbid hipMalloc).  The job table is
// already in device memory, and the only working memory is one file-scope
// device array per GPU, `scratch`, whose address is looked up once per device
// with hipGetSymbolAddress and passed to the kernels from then on.
//
// Up to kSmallJobs jobs: one or two launches on the caller's stream.
//   small  -- every workgroup reads all jobs, rejects any that is malformed or reaches outside
//             [dev_base, dev_base + base_bytes) (it gets no tiles), and counts and sums their tiles in LDS:
//             wave tiles of up to 2048 blocks of one job, and lane tiles of 64 slots of up to 32 blocks, from
//             the jobs' remainders.  If there are at most kStaticTeamTiles, the workgroups work them off with their
//             eight waves (team_core.h); if not, the first workgroup leaves the plan below in scratch;
//   cipher -- launched unless the buffer's size rules out more tiles than that; ends at once if the small
//             kernel did the work.
// 512 jobs of up to 8192 blocks (658 tiles by job, 234 packed): 46 us a call by plan and cipher, 22.9 by the
// small kernel; 2048 jobs of up to 256 blocks 68 and 23.7.
//
// More jobs: two launches.
//   plan   -- one workgroup reads and checks the jobs and writes the exclusive prefix sum of wave tiles (2048
//             blocks each, a job's last one partial) per job into scratch, the tile total, the number of
//             rejected jobs, and a zeroed tile counter;
//   cipher -- persistent waves draw tiles (the first by wave index, later ones from the counter), find each
//             tile's job by binary search over the prefix sums and run the bitsliced core on it, with the
//             job's key masks in scalar registers.  A partial tile takes the core's per-block path.
// Nothing here carries state from one call to the next except scratch, which
// the plan launch rewrites before the cipher launch reads it.
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "internal.h"
#include "team_core.h"

namespace {

using namespace tdes_bs;

constexpr uint32_t kMaxJobs = TDES_STATIC_MAX_JOBS;
constexpr uint32_t kPlanThreads = 1024;
constexpr uint32_t kThreads = 256;
constexpr uint32_t kGroupsPerCU = 4;
constexpr uint64_t kMaxJobBlocks = 1ull << 40;
// Teams up to here, waves from there on: 1400 tiles 57.6 us by the small kernel and 58.1 by two, 1700 59.6 and
// 60.6, 2000 65.4 and 64.8; with smaller circuits 1100 45.1 and 50.7, 1300 54.8 and 53.5, 1500 55.6 and 55.7.
constexpr uint32_t kStaticTeamTiles = 1600;
constexpr uint32_t kSmallJobs = 4096;              // eight per thread of a team
constexpr uint32_t kLaneBlocks = 32;
constexpr uint32_t kWaveRemainder = 1800;          // a remainder of at least this many blocks is a wave tile
// Buffers for which the small kernel is launched alone are smaller than this (most_tiles below): 23 MB.  An accepted
// job has at most that many bytes, so kSmallJobs of them have fewer than 2^32 tiles or slots, whatever they share.
constexpr uint64_t kAloneBytes = 8ull * kWaveRemainder * kStaticTeamTiles;
static_assert(kSmallJobs * (kAloneBytes / (8 * kTileBlocks) + kTileBlocks / kLaneBlocks) < 1ull << 32, "sums of tiles");

// scratch: [header, 256 B][tile_start: kMaxJobs + 1 words]
struct StaticHeader {
    uint32_t n_tiles;   // wave tiles of the call (0 if the total overflowed)
    uint32_t rejected;  // jobs given no tiles because they were malformed
    uint32_t pad0[30];
    uint32_t counter;   // tile draws after each wave's first (own 128-byte line)
    uint32_t pad1[31];
};
static_assert(sizeof(StaticHeader) == 256, "header is 256 bytes");
constexpr size_t kScratchBytes = sizeof(StaticHeader) + ((size_t)(kMaxJobs + 1) * 4 + 255) / 256 * 256;

static __device__ __align__(256) uint8_t scratch[kScratchBytes];

__device__ __forceinline__ bool job_ok(const tdes_job &x, uint64_t n_scheds, uint64_t base_bytes) {
    if (x.direction > TDES_DECRYPT || x.sched_idx >= n_scheds || x.n_blocks > kMaxJobBlocks) return false;
    if ((x.in_off | x.out_off) & 7) return false;
    const uint64_t bytes = 8 * x.n_blocks;
    if (x.in_off > base_bytes || bytes > base_bytes - x.in_off) return false;
    if (x.out_off > base_bytes || bytes > base_bytes - x.out_off) return false;
    // in place, or no shared byte between input and output
    return x.in_off == x.out_off || x.in_off >= x.out_off + bytes || x.out_off >= x.in_off + bytes;
}

__global__ __launch_bounds__(kPlanThreads) void tdes_static_plan_kernel(const tdes_job *__restrict__ jobs,
                                                                        uint32_t n_jobs, uint64_t n_scheds,
                                                                        uint64_t base_bytes, uint8_t *scr,
                                                                        uint32_t *dev_rejected) {
    __shared__ uint64_t part[kPlanThreads];
    __shared__ uint32_t bad_total;
    StaticHeader *hdr = reinterpret_cast<StaticHeader *>(scr);
    uint32_t *tile_start = reinterpret_cast<uint32_t *>(scr + sizeof(StaticHeader));
    const uint32_t tid = threadIdx.x;
    if (tid == 0) bad_total = 0;
    // thread tid plans jobs [lo, hi)
    const uint32_t per = (n_jobs + kPlanThreads - 1) / kPlanThreads;
    const uint32_t lo = min(n_jobs, tid * per), hi = min(n_jobs, lo + per);
    // first pass: each job's tile count (at most 2^29) into tile_start[j]
    uint64_t sum = 0;
    uint32_t bad = 0;
    for (uint32_t j = lo; j < hi; j++) {
        const tdes_job x = jobs[j];
        uint32_t t = 0;
        if (job_ok(x, n_scheds, base_bytes))
            t = (uint32_t)((x.n_blocks + kTileBlocks - 1) / kTileBlocks);
        else
            bad++;
        tile_start[j] = t;
        sum += t;
    }
    part[tid] = sum;
    __syncthreads();
    if (bad) atomicAdd(&bad_total, bad);
    // inclusive scan of part[] (Hillis-Steele)
    for (uint32_t d = 1; d < kPlanThreads; d <<= 1) {
        const uint64_t v = tid >= d ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    const uint64_t total = part[kPlanThreads - 1];
    const bool overflow = total >= (1ull << 31);
    // second pass: counts to exclusive prefix sums, in place
    uint64_t run = part[tid] - sum;
    for (uint32_t j = lo; j < hi; j++) {
        const uint32_t t = tile_start[j];
        tile_start[j] = overflow ? 0 : (uint32_t)run;
        run += t;
    }
    if (tid == 0) {
        tile_start[n_jobs] = overflow ? 0 : (uint32_t)total;
        hdr->n_tiles = overflow ? 0 : (uint32_t)total;
        hdr->counter = 0;
    }
    __syncthreads();
    if (tid == 0) {
        const uint32_t rejected = overflow ? n_jobs : bad_total;
        hdr->rejected = rejected;
        if (dev_rejected) *dev_rejected = rejected;
    }
}

// A wave's tile after its first: n_waves + the counter's old value (none left at or past n_tiles).
__device__ __forceinline__ uint32_t next_ticket(uint32_t *counter, uint32_t n_waves, uint32_t lane) {
    uint32_t d = 0;
    if (lane == 0) d = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return n_waves + __builtin_amdgcn_readfirstlane(d);
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// A tile of the call: `count` blocks (1 .. kTileBlocks) of one job.
struct StaticTile {
    const uint32_t *ks;
    const uint8_t *in;
    uint8_t *out;
    uint32_t count;
};

__device__ __forceinline__ StaticTile find_tile(uint32_t ticket, const tdes_job *__restrict__ jobs, uint32_t n_jobs,
                                                const uint32_t *__restrict__ sched, const uint32_t *tile_start, uint8_t *base) {
    // the job j with tile_start[j] <= ticket < tile_start[j + 1] (tile_start[n_jobs] = n_tiles)
    uint32_t lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (__builtin_amdgcn_readfirstlane(tile_start[mid]) <= ticket)
            lo = mid;
        else
            hi = mid;
    }
    const tdes_job &x = jobs[lo];
    const uint64_t first = (uint64_t)(ticket - __builtin_amdgcn_readfirstlane(tile_start[lo])) * kTileBlocks;
    StaticTile t;
    t.count = tile_count(uniform64(x.n_blocks) - first);
    t.ks = sched + (uint64_t)__builtin_amdgcn_readfirstlane(x.sched_idx) * (TDES_SCHED_BYTES / 4) +
           __builtin_amdgcn_readfirstlane(x.direction) * tdes::kDirWords;
    t.in = base + uniform64(x.in_off) + 8 * first;
    t.out = base + uniform64(x.out_off) + 8 * first;
    return t;
}

__global__ __launch_bounds__(kThreads, kGroupsPerCU) void tdes_static_batch_kernel(
    const tdes_job *__restrict__ jobs, uint32_t n_jobs, const uint32_t *__restrict__ sched, uint8_t *scr,
    uint8_t *base) {
    StaticHeader *hdr = reinterpret_cast<StaticHeader *>(scr);
    const uint32_t *tile_start = reinterpret_cast<const uint32_t *>(scr + sizeof(StaticHeader));
    const uint32_t lane = threadIdx.x % kLanes;
    const uint32_t n_tiles = __builtin_amdgcn_readfirstlane(hdr->n_tiles);
    const uint32_t n_waves = gridDim.x * (blockDim.x / kLanes);
    const uint32_t wave_id = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x / kLanes) + threadIdx.x / kLanes);
    for (uint32_t ticket = wave_id; ticket < n_tiles; ticket = next_ticket(&hdr->counter, n_waves, lane)) {
        const StaticTile t = find_tile(ticket, jobs, n_jobs, sched, tile_start, base);
        if (t.count == kTileBlocks)
            wave_tile<true>(t.ks, t.in, t.out, kTileBlocks, lane);
        else
            wave_tile<false>(t.ks, t.in, t.out, t.count, lane);
    }
}

// A job's wave tiles and lane slots; both 0 if it is refused.
struct JobTiles {
    uint32_t wave, slots;
};
__device__ __forceinline__ JobTiles job_tiles(const tdes_job &x, bool ok) {
    JobTiles t{0, 0};
    if (!ok) return t;
    const uint32_t rem = (uint32_t)(x.n_blocks % kTileBlocks), wave_rem = rem >= kWaveRemainder;
    t.wave = (uint32_t)(x.n_blocks / kTileBlocks) + wave_rem;
    if (!wave_rem) t.slots = (rem + kLaneBlocks - 1) / kLaneBlocks;
    return t;
}

// The whole call by teams if its tiles are few, else its plan.  n_jobs <= kSmallJobs.  alone: no cipher kernel
// follows; scratch is not touched, and every tile is the teams' (the sums fit 32 bits: kAloneBytes).
//
// kMany: more jobs than threads.  The jobs are read by neighbouring lanes, four of a thread's in flight, and their counts
// go by way of the planes' LDS to the threads that sum consecutive jobs.  (Read by each thread for its own eight, 256
// bytes apart between lanes, and again for the plan: 4000 whole tiles 95.6 us instead of 88.4, 4096 jobs of up to 4096
// blocks, by the teams, 59.6 instead of 50.7.)  With a job per thread there is nothing to gain, and a kernel with both
// ways in it took 512 records 22.35 us instead of 22.14.
template <bool kMany>
__global__ __launch_bounds__(kTeamThreads) void tdes_static_small_kernel(const tdes_job *__restrict__ jobs, uint32_t n_jobs,
                                                                         const uint32_t *__restrict__ sched,
                                                                         uint64_t n_scheds, uint8_t *scr, uint8_t *base,
                                                                         uint64_t base_bytes, uint32_t *dev_rejected,
                                                                         bool alone) {
    __shared__ uint32_t lds[kTeamLaneWords];
    __shared__ uint32_t wave_start[kTeamThreads], lane_start[kTeamThreads];  // exclusive sums, by thread's group of jobs
    __shared__ uint64_t part_wave[8];
    __shared__ uint32_t part_lane[8], part_ragged[8], part_bad[8];
    const uint32_t tid = threadIdx.x, lane = tid % kLanes, wv = tid / kLanes;
    const uint32_t per = (n_jobs + kTeamThreads - 1) / kTeamThreads;
    uint32_t *job_wave = lds, *job_slots = lds + kSmallJobs;  // (kMany) each job's wave tiles; lane slots or kRefused
    constexpr uint32_t kRefused = 1u << 31;
    static_assert(2 * kSmallJobs <= kTeamLaneWords && kTileBlocks / kLaneBlocks < kRefused, "room for the counts");
    // the thread's jobs: wave tiles, lane slots, jobs with lane slots, refused jobs
    uint64_t wave = 0;
    uint32_t slots = 0, ragged = 0, bad = 0;
    if constexpr (kMany) {
        constexpr uint32_t kAhead = 4;  // jobs in flight
        for (uint32_t j = tid; j < n_jobs; j += kAhead * kTeamThreads) {
            tdes_job x[kAhead];
#pragma unroll
            for (uint32_t i = 0; i < kAhead; i++) x[i] = jobs[min(j + i * kTeamThreads, n_jobs - 1)];
#pragma unroll
            for (uint32_t i = 0; i < kAhead; i++) {
                const uint32_t at = j + i * kTeamThreads;
                if (at >= n_jobs) break;
                const bool ok = job_ok(x[i], n_scheds, base_bytes);
                const JobTiles t = job_tiles(x[i], ok);
                job_wave[at] = t.wave;
                job_slots[at] = ok ? t.slots : kRefused;
            }
        }
        __syncthreads();
        for (uint32_t j = tid * per; j < min(n_jobs, (tid + 1) * per); j++) {
            const uint32_t n = job_slots[j] & ~kRefused;
            wave += job_wave[j];
            slots += n;
            ragged += n != 0;
            bad += job_slots[j] / kRefused;
        }
    } else {
        for (uint32_t j = tid * per; j < min(n_jobs, (tid + 1) * per); j++) {
            const tdes_job x = jobs[j];
            const bool ok = job_ok(x, n_scheds, base_bytes);
            const JobTiles t = job_tiles(x, ok);
            wave += t.wave;
            slots += t.slots;
            ragged += t.slots != 0;
            bad += !ok;
        }
    }
    // inclusive sums over the wave's threads, then over the waves
    uint64_t w = wave;
    uint32_t s = slots, g = ragged;
#pragma unroll
    for (int d = 1; d < kLanes; d <<= 1) {
        const uint64_t pw = __shfl_up((unsigned long long)w, d);
        const uint32_t ps = __shfl_up(s, d), pg = __shfl_up(g, d);
        if ((int)lane >= d) { w += pw; s += ps; g += pg; }
    }
#pragma unroll
    for (int d = 1; d < kLanes; d <<= 1) bad += __shfl_xor(bad, d);
    if (lane == kLanes - 1) { part_wave[wv] = w; part_lane[wv] = s; part_ragged[wv] = g; part_bad[wv] = bad; }
    __syncthreads();
    uint64_t all_wave = 0;
    uint32_t all_slots = 0, all_ragged = 0, all_bad = 0;
#pragma unroll
    for (uint32_t i = 0; i < 8; i++) {
        if (i < wv) { w += part_wave[i]; s += part_lane[i]; g += part_ragged[i]; }
        all_wave += part_wave[i];
        all_slots += part_lane[i];
        all_ragged += part_ragged[i];
        all_bad += part_bad[i];
    }
    const uint64_t by_job = all_wave + all_ragged;  // the cipher kernel's tiles: a remainder is a tile of its own
    const bool overflow = by_job >= (1ull << 31);
    const uint32_t n_lane_tiles = (all_slots + kLanes - 1) / kLanes;
    const bool mine = alone || all_wave + n_lane_tiles <= kStaticTeamTiles;
    if (blockIdx.x == 0 && tid == 0 && dev_rejected) *dev_rejected = overflow ? n_jobs : all_bad;
    if (blockIdx.x == 0 && !alone) {
        StaticHeader *hdr = reinterpret_cast<StaticHeader *>(scr);
        uint32_t *tile_start = reinterpret_cast<uint32_t *>(scr + sizeof(StaticHeader));
        if (tid == 0) {
            hdr->n_tiles = mine || overflow ? 0 : (uint32_t)by_job;
            hdr->rejected = overflow ? n_jobs : all_bad;
            hdr->counter = 0;
        }
        if (!mine && !overflow) {
            uint32_t run = (uint32_t)(w - wave) + (g - ragged);
            for (uint32_t j = tid * per; j < min(n_jobs, (tid + 1) * per); j++) {
                tile_start[j] = run;
                if constexpr (kMany) {
                    run += job_wave[j] + ((job_slots[j] & ~kRefused) != 0);
                } else {
                    const tdes_job x = jobs[j];
                    if (job_ok(x, n_scheds, base_bytes)) run += (uint32_t)((x.n_blocks + kTileBlocks - 1) / kTileBlocks);
                }
            }
            if (tid == 0) tile_start[n_jobs] = (uint32_t)by_job;
        }
    }
    if (!mine) return;
    wave_start[tid] = (uint32_t)(w - wave);
    lane_start[tid] = s - slots;
    __syncthreads();

    // The job of wave tile (lane slot) `at`, and `at` within the job: the last group that starts at or before
    // it, by binary search, then along the group.
    auto find = [&](const uint32_t *start, uint32_t at, bool slots, tdes_job *job) {
        uint32_t lo = 0, hi = kTeamThreads;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) / 2;
            if (start[mid] <= at) lo = mid; else hi = mid;
        }
        at -= start[lo];
        for (uint32_t j = lo * per; j < n_jobs; j++) {
            *job = jobs[j];
            const JobTiles t = job_tiles(*job, job_ok(*job, n_scheds, base_bytes));
            const uint32_t n = slots ? t.slots : t.wave;
            if (at < n) break;
            at -= n;
        }
        return at;
    };
    const uint32_t n_tiles = n_lane_tiles + (uint32_t)all_wave;
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        if (tile < n_lane_tiles) {
            // Lanes past the last slot stay idle.
            const uint32_t slot = tile * kLanes + lane;
            const uint32_t *ks = sched;
            const uint8_t *in = base;
            uint8_t *out = base;
            uint32_t count = 0;
            if (slot < all_slots) {
                tdes_job x;
                const uint32_t at = kLaneBlocks * find(lane_start, slot, true, &x);
                const uint32_t rem = (uint32_t)(x.n_blocks % kTileBlocks);
                const uint64_t first = x.n_blocks - rem + at;
                ks = sched + (uint64_t)x.sched_idx * (TDES_SCHED_BYTES / 4) + x.direction * tdes::kDirWords;
                in = base + x.in_off + 8 * first;
                out = base + x.out_off + 8 * first;
                count = min(kLaneBlocks, rem - at);
            }
            team_tile<TileMode::kEcb, true>(ks, in, out, count, tid, 0, 0, lds);
        } else {
            tdes_job x;
            const uint64_t first = (uint64_t)__builtin_amdgcn_readfirstlane(find(wave_start, tile - n_lane_tiles, false, &x)) * kTileBlocks;
            const uint32_t *ks = sched + (uint64_t)__builtin_amdgcn_readfirstlane(x.sched_idx) * (TDES_SCHED_BYTES / 4) +
                                 __builtin_amdgcn_readfirstlane(x.direction) * tdes::kDirWords;
            team_tile<TileMode::kEcb, false>(ks, base + uniform64(x.in_off) + 8 * first, base + uniform64(x.out_off) + 8 * first,
                                             tile_count(uniform64(x.n_blocks) - first), tid, 0, 0, lds);
        }
        __syncthreads();
    }
}

// scratch's device address on each GPU, looked up on the first call there.
constexpr int kMaxDevices = 64;
std::atomic<uint8_t *> g_scratch[kMaxDevices];
std::mutex g_scratch_mu;

int scratch_for(int device, uint8_t **out) {
    if (device < 0 || device >= kMaxDevices) return TDES_ERR_ARG;
    uint8_t *p = g_scratch[device].load(std::memory_order_acquire);
    if (!p) {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        p = g_scratch[device].load(std::memory_order_relaxed);
        if (!p) {
            // device is current: the address of this GPU's copy of the array
            if (hipGetSymbolAddress(reinterpret_cast<void **>(&p), HIP_SYMBOL(scratch)) != hipSuccess || !p)
                return TDES_ERR_HIP;
            g_scratch[device].store(p, std::memory_order_release);
        }
    }
    *out = p;
    return TDES_OK;
}

}  // namespace

extern "C" int tdes_ecb_batch_static(const tdes_job *dev_jobs, uint32_t n_jobs, const void *dev_sched_table,
                                     uint64_t n_scheds, void *dev_base, uint64_t base_bytes, uint32_t *dev_rejected,
                                     void *stream) {
    if (n_jobs == 0) return TDES_OK;
    if (!dev_jobs || !dev_sched_table || !dev_base) return TDES_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(dev_jobs) & 7) || (reinterpret_cast<uintptr_t>(dev_sched_table) & 3) ||
        (reinterpret_cast<uintptr_t>(dev_base) & 7) || (reinterpret_cast<uintptr_t>(dev_rejected) & 3))
        return TDES_ERR_ALIGN;
    if (n_jobs > kMaxJobs) return TDES_ERR_SIZE;
    if (n_scheds == 0 || n_scheds > (1ull << 32) / (TDES_SCHED_BYTES / 4)) return TDES_ERR_SIZE;
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return TDES_ERR_HIP;
    uint8_t *scr = nullptr;
    int rc = scratch_for(device, &scr);
    if (rc != TDES_OK) return rc;
    tdes::DeviceInfo info;
    if (tdes::device_info(&info) != TDES_OK) return TDES_ERR_HIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    uint8_t *base = static_cast<uint8_t *>(dev_base);
    const uint32_t *table = static_cast<const uint32_t *>(dev_sched_table);
    if (n_jobs <= kSmallJobs) {
        // Outputs of different jobs share no bytes, so the buffer bounds the tiles: a wave tile has at least
        // kWaveRemainder blocks, a lane slot kLaneBlocks but for a job's last.  (If a call breaks that rule, the
        // teams still work off what they have counted.)
        const uint64_t most_tiles = base_bytes / (8 * kWaveRemainder) + n_jobs / kLanes + 2;
        const bool alone = most_tiles <= kStaticTeamTiles;
        const uint32_t resident = (uint32_t)info.cu_count * 3;  // 45 KiB of LDS per workgroup
        hipLaunchKernelGGL(n_jobs > kTeamThreads ? tdes_static_small_kernel<true> : tdes_static_small_kernel<false>,
                           dim3(most_tiles < resident ? (uint32_t)most_tiles : resident), dim3(kTeamThreads), 0, s,
                           dev_jobs, n_jobs, table, n_scheds, scr, base, base_bytes, dev_rejected, alone);
        if (hipGetLastError() != hipSuccess) return TDES_ERR_HIP;
        if (alone) return TDES_OK;
    } else {
        hipLaunchKernelGGL(tdes_static_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, dev_jobs, n_jobs, n_scheds,
                           base_bytes, scr, dev_rejected);
        if (hipGetLastError() != hipSuccess) return TDES_ERR_HIP;
    }
    hipLaunchKernelGGL(tdes_static_batch_kernel, dim3((uint32_t)info.cu_count * kGroupsPerCU), dim3(kThreads), 0, s,
                       dev_jobs, n_jobs, table, scr, base);
    return hipGetLastError() == hipSuccess ? TDES_OK : TDES_ERR_HIP;
}
