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
// Few jobs in a small buffer (kSmallJobs; the buffer bounds the tiles): one launch.  Every workgroup reads all
// jobs, counts and sums their tiles in LDS, and takes the tiles of its turn with its eight waves (team_core.h):
// wave tiles of up to 2048 blocks of one job, and lane tiles of 64 slots of up to 32 blocks, from the jobs'
// remainders.  512 jobs of up to 8192 blocks (658 tiles by job, 234 packed): 29.8 us a call with the
// launches below, 22.0 so.
//
// Otherwise three launches on the caller's stream:
//   plan   -- one workgroup reads the jobs, rejects any that is malformed or
//             reaches outside [dev_base, dev_base + base_bytes) (it gets no
//             tiles), and writes the exclusive prefix sum of wave tiles (2048
//             blocks each) per job into scratch, the tile total, the number of
//             rejected jobs, and a zeroed tile counter;
//   team   -- if there are at most kTeamTiles tiles, a workgroup per tile;
//   cipher -- otherwise persistent waves that draw tiles (the first by wave
//             index, later ones from the counter) and run the bitsliced core on them, with the
//             job's key masks in scalar registers.
// Both find each tile's job by binary search over the prefix sums; only the device knows how many tiles
// there are, so both are launched and one of them ends at once (4 us).  A job's last tile may be
// partial: its blocks take the core's per-block path.
// Nothing here carries state from one call to the next except scratch, which
// the plan launch rewrites before the cipher launch reads it.
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "batch_plan.h"
#include "internal.h"
#include "team_core.h"

namespace {

using namespace tdes_bs;

constexpr uint32_t kMaxJobs = TDES_STATIC_MAX_JOBS;
constexpr uint32_t kPlanThreads = 1024;
constexpr uint32_t kThreads = 256;
constexpr uint32_t kGroupsPerCU = 4;
constexpr uint64_t kMaxJobBlocks = 1ull << 40;
constexpr uint32_t kSmallJobs = 2 * kTeamThreads;  // two per thread
constexpr uint32_t kLaneBlocks = 32;
constexpr uint32_t kWaveRemainder = 1800;          // a remainder of at least this many blocks is a wave tile

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

__global__ __launch_bounds__(kTeamThreads) void tdes_static_team_kernel(const tdes_job *__restrict__ jobs, uint32_t n_jobs,
                                                                        const uint32_t *__restrict__ sched, uint8_t *scr,
                                                                        uint8_t *base) {
    __shared__ uint32_t lds[kTeamWords];
    const uint32_t n_tiles = reinterpret_cast<const StaticHeader *>(scr)->n_tiles;
    if (n_tiles > tdes::kTeamTiles || blockIdx.x >= n_tiles) return;
    const StaticTile t = find_tile(blockIdx.x, jobs, n_jobs, sched,
                                   reinterpret_cast<const uint32_t *>(scr + sizeof(StaticHeader)), base);
    team_tile<TileMode::kEcb, false>(t.ks, t.in, t.out, t.count, threadIdx.x, 0, 0, lds);
}

__global__ __launch_bounds__(kThreads, kGroupsPerCU) void tdes_static_batch_kernel(
    const tdes_job *__restrict__ jobs, uint32_t n_jobs, const uint32_t *__restrict__ sched, uint8_t *scr,
    uint8_t *base) {
    StaticHeader *hdr = reinterpret_cast<StaticHeader *>(scr);
    const uint32_t *tile_start = reinterpret_cast<const uint32_t *>(scr + sizeof(StaticHeader));
    const uint32_t lane = threadIdx.x % kLanes;
    const uint32_t n_tiles = __builtin_amdgcn_readfirstlane(hdr->n_tiles);
    if (n_tiles <= tdes::kTeamTiles) return;
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

// The whole call by teams, without a plan in memory.  n_jobs <= kSmallJobs, and base_bytes so small that the
// sums below fit 32 bits.
__global__ __launch_bounds__(kTeamThreads) void tdes_static_small_kernel(const tdes_job *__restrict__ jobs, uint32_t n_jobs,
                                                                         const uint32_t *__restrict__ sched,
                                                                         uint64_t n_scheds, uint8_t *base,
                                                                         uint64_t base_bytes, uint32_t *dev_rejected) {
    __shared__ uint32_t lds[kTeamLaneWords];
    __shared__ uint32_t wave_start[kSmallJobs + 1], lane_start[kSmallJobs + 1];  // exclusive sums over the jobs
    __shared__ uint32_t part_wave[8], part_lane[8], part_bad[8];
    const uint32_t tid = threadIdx.x, lane = tid % kLanes, wv = tid / kLanes;
    uint32_t wave[2], slots[2], bad = 0;
#pragma unroll
    for (int i = 0; i < 2; i++) {
        wave[i] = slots[i] = 0;
        if (2 * tid + i < n_jobs) {
            const tdes_job x = jobs[2 * tid + i];
            if (job_ok(x, n_scheds, base_bytes)) {
                const uint32_t rem = (uint32_t)(x.n_blocks % kTileBlocks), wave_rem = rem >= kWaveRemainder;
                wave[i] = (uint32_t)(x.n_blocks / kTileBlocks) + wave_rem;
                if (!wave_rem) slots[i] = (rem + kLaneBlocks - 1) / kLaneBlocks;
            } else {
                bad++;
            }
        }
    }
    // inclusive sums of both counts over the wave's threads, then over the waves
    uint32_t w = wave[0] + wave[1], s = slots[0] + slots[1];
#pragma unroll
    for (int d = 1; d < kLanes; d <<= 1) {
        const uint32_t pw = __shfl_up(w, d), ps = __shfl_up(s, d);
        if ((int)lane >= d) { w += pw; s += ps; }
    }
#pragma unroll
    for (int d = 1; d < kLanes; d <<= 1) bad += __shfl_xor(bad, d);
    if (lane == kLanes - 1) { part_wave[wv] = w; part_lane[wv] = s; part_bad[wv] = bad; }
    __syncthreads();
    uint32_t all_wave = 0, all_slots = 0, all_bad = 0;
#pragma unroll
    for (uint32_t i = 0; i < 8; i++) {
        if (i < wv) { w += part_wave[i]; s += part_lane[i]; }
        all_wave += part_wave[i];
        all_slots += part_lane[i];
        all_bad += part_bad[i];
    }
    wave_start[2 * tid + 2] = w;
    wave_start[2 * tid + 1] = w - wave[1];
    lane_start[2 * tid + 2] = s;
    lane_start[2 * tid + 1] = s - slots[1];
    if (tid == 0) {
        wave_start[0] = lane_start[0] = 0;
        if (blockIdx.x == 0 && dev_rejected) *dev_rejected = all_bad;
    }
    __syncthreads();

    const uint32_t n_lane_tiles = (all_slots + kLanes - 1) / kLanes, n_tiles = n_lane_tiles + all_wave;
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        if (tile < n_lane_tiles) {
            // The lane's slot: of the last job that starts at or before it.  Lanes past the end stay idle.
            const uint32_t slot = tile * kLanes + lane;
            const uint32_t *ks = sched;
            const uint8_t *in = base;
            uint8_t *out = base;
            uint32_t count = 0;
            if (slot < all_slots) {
                uint32_t lo = 0, hi = n_jobs;
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) / 2;
                    if (lane_start[mid] <= slot) lo = mid; else hi = mid;
                }
                const tdes_job x = jobs[lo];
                const uint32_t rem = (uint32_t)(x.n_blocks % kTileBlocks), at = kLaneBlocks * (slot - lane_start[lo]);
                const uint64_t first = x.n_blocks - rem + at;
                ks = sched + (uint64_t)x.sched_idx * (TDES_SCHED_BYTES / 4) + x.direction * tdes::kDirWords;
                in = base + x.in_off + 8 * first;
                out = base + x.out_off + 8 * first;
                count = min(kLaneBlocks, rem - at);
            }
            team_tile<TileMode::kEcb, true>(ks, in, out, count, tid, 0, 0, lds);
        } else {
            const StaticTile t = find_tile(tile - n_lane_tiles, jobs, n_jobs, sched, wave_start, base);
            team_tile<TileMode::kEcb, false>(t.ks, t.in, t.out, t.count, tid, 0, 0, lds);
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
    // Inputs and outputs of different jobs share no bytes, so the buffer bounds the tiles.  (A call that breaks
    // that rule is still worked off: the workgroups take as many turns as there are tiles.)
    const uint64_t most_tiles = base_bytes / (8 * kTileBlocks) + n_jobs;
    if (n_jobs <= kSmallJobs && most_tiles <= tdes::kTeamTiles) {
        const uint32_t resident = (uint32_t)info.cu_count * 3;  // 48 KiB of LDS per workgroup
        hipLaunchKernelGGL(tdes_static_small_kernel, dim3(most_tiles < resident ? (uint32_t)most_tiles : resident),
                           dim3(kTeamThreads), 0, s, dev_jobs, n_jobs, static_cast<const uint32_t *>(dev_sched_table),
                           n_scheds, base, base_bytes, dev_rejected);
        return hipGetLastError() == hipSuccess ? TDES_OK : TDES_ERR_HIP;
    }
    hipLaunchKernelGGL(tdes_static_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, dev_jobs, n_jobs, n_scheds,
                       base_bytes, scr, dev_rejected);
    if (hipGetLastError() != hipSuccess) return TDES_ERR_HIP;
    hipLaunchKernelGGL(tdes_static_team_kernel, dim3(tdes::kTeamTiles), dim3(kTeamThreads), 0, s, dev_jobs, n_jobs,
                       static_cast<const uint32_t *>(dev_sched_table), scr, base);
    if (hipGetLastError() != hipSuccess) return TDES_ERR_HIP;
    hipLaunchKernelGGL(tdes_static_batch_kernel, dim3((uint32_t)info.cu_count * kGroupsPerCU), dim3(kThreads), 0, s,
                       dev_jobs, n_jobs, static_cast<const uint32_t *>(dev_sched_table), scr, base);
    return hipGetLastError() == hipSuccess ? TDES_OK : TDES_ERR_HIP;
}
