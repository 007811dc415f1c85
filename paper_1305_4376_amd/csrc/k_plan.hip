// k_plan.hip -- a batch's plan written on the device from one record per message.
//
// The kernels of a batch want a slot (32 bytes) per tile or lane.  Written by the host and copied, the
// 90000 slots of 4096 messages cost about 0.3 ms of host time and a 50 us copy, and the copy engine's
// start and hand-over about 13 us of an idle GPU for any batch.  Here the host leaves one 64-byte record
// per message in pinned memory; a workgroup of one wave per record (more, strided, for long messages)
// reads it over the host link and writes the message's slots.
#include <hip/hip_runtime.h>

#include "batch_plan.h"
#include "internal.h"

namespace {

constexpr uint32_t kThreads = 64;
constexpr uint32_t kWaveBlocks = 2048, kLaneBlocks = 32;
constexpr uint32_t kMaxGridX = 1u << 16, kMaxGridY = 64;
constexpr uint32_t kTilesPerGroup = 256;  // wave slots of a message that one workgroup writes, up to kMaxGridY workgroups

__global__ __launch_bounds__(kThreads) void tdes_plan_kernel(const tdes::PlanMessage *messages, uint32_t n_messages,
                                                             tdes::PlanHeader *hdr, tdes::Slot *slots, uint32_t n_tiles,
                                                             uint32_t n_lane_slots) {
    const uint32_t n_lane_tiles = (n_lane_slots + 63) / 64;
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        if (threadIdx.x == 0) {
            hdr->n_tiles = n_tiles;
            hdr->n_lane_tiles = n_lane_tiles;
        }
        const uint32_t idle = n_lane_slots + threadIdx.x;  // at most 63 idle lanes end the last lane tile
        if (idle < 64 * n_lane_tiles) slots[idle] = tdes::Slot{0, 0, 0, 0, 0};
    }
    for (uint32_t m = blockIdx.x; m < n_messages; m += gridDim.x) {
        const tdes::PlanMessage x = messages[m];
        tdes::Slot *wave = slots + 64 * (uint64_t)n_lane_tiles + x.wave_first;
        for (uint32_t t = blockIdx.y * kThreads + threadIdx.x; t < x.wave_tiles; t += gridDim.y * kThreads) {
            const uint64_t at = (uint64_t)t * kWaveBlocks, left = x.n_blocks - at;
            wave[t] = tdes::Slot{x.in_off + 8 * at, x.out_off + 8 * at, left / kWaveBlocks ? kWaveBlocks : (uint32_t)left,
                                 x.ks_off, 0};
        }
        const uint64_t done = (uint64_t)x.wave_tiles * kWaveBlocks;
        if (blockIdx.y == 0 && done < x.n_blocks) {  // the rest: fewer than 2048 blocks, at most one slot per thread
            const uint32_t rest = (uint32_t)(x.n_blocks - done), at = kLaneBlocks * threadIdx.x;
            if (at < rest)
                slots[x.lane_first + threadIdx.x] =
                    tdes::Slot{x.in_off + 8 * (done + at), x.out_off + 8 * (done + at), min(kLaneBlocks, rest - at), x.ks_off, 0};
        }
    }
}

}  // namespace

namespace tdes {

hipError_t launch_plan(const PlanMessage *messages, uint32_t n_messages, uint32_t max_wave_tiles, PlanHeader *hdr,
                       Slot *slots, uint32_t n_tiles, uint32_t n_lane_slots, hipStream_t stream) {
    const uint32_t y = (max_wave_tiles + kTilesPerGroup - 1) / kTilesPerGroup;
    const dim3 grid(n_messages < kMaxGridX ? n_messages : kMaxGridX, y == 0 ? 1 : y < kMaxGridY ? y : kMaxGridY);
    hipLaunchKernelGGL(tdes_plan_kernel, grid, dim3(kThreads), 0, stream, messages, n_messages, hdr, slots, n_tiles,
                       n_lane_slots);
    return hipGetLastError();
}

}  // namespace tdes
