// k_plan.hip -- a batch's plan written on the device from one record per message.
//
// The kernels of a batch want a slot (32 bytes) per tile or lane.  Written by the host and copied, the
// 90000 slots of 4096 messages cost about 0.3 ms of host time and a 50 us copy, and the copy engine's
// start and hand-over about 13 us of an idle GPU for any batch.  Here the host leaves one 40-byte record
// per message in pinned memory, and this kernel reads them over the host link and writes the slots.
//
// Bound: the link.  A workgroup reads eight records in one go, as consecutive words, and each of its four
// waves writes the slots of two messages (the grid's second dimension shares out long ones).  4096 messages:
// 8.2 us; a workgroup of one wave per message, on 64-byte records, 14 us; four such waves to a workgroup, 10 us.
// 48 messages: 3.5 to 4 us, two trips over the link and the launch.
#include <hip/hip_runtime.h>

#include "batch_plan.h"
#include "internal.h"

namespace {

constexpr uint32_t kThreads = 256, kLanes = 64;
constexpr uint32_t kGroupMessages = 8;  // records that a workgroup reads at a time, two for each of its waves
constexpr uint32_t kRecordWords = sizeof(tdes::PlanMessage) / 4;
constexpr uint32_t kWaveBlocks = 2048, kLaneBlocks = 32;
constexpr uint32_t kMaxGridX = 1u << 13, kMaxGridY = 64;
constexpr uint32_t kTilesPerGroup = 256;  // wave slots of a message that one wave writes, up to kMaxGridY workgroups

// Held to 32 VGPRs (the attribute counts pairs; it takes 30 without a spill, and 34 if left alone): what four waves of
// the server's cipher kernel leave on a SIMD.  With 34 the plan of a step waited until workgroups of the step
// before retired: 156 us a plan instead of 35 to 50 (8 on an empty GPU), and the saturated server delivered 982 GB/s
// instead of 1013.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_num_vgpr(16))) void tdes_plan_kernel(
    const tdes::PlanMessage *messages, uint32_t n_messages, tdes::PlanHeader *hdr, tdes::Slot *slots, uint32_t n_tiles,
    uint32_t n_lane_slots) {
    __shared__ alignas(8) uint32_t records[kGroupMessages * kRecordWords];
    const uint32_t n_lane_tiles = (n_lane_slots + kLanes - 1) / kLanes;
    const uint32_t lane = threadIdx.x % kLanes, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    if (blockIdx.x == 0 && blockIdx.y == 0 && wave == 0) {
        if (lane == 0) {
            hdr->n_tiles = n_tiles;
            hdr->n_lane_tiles = n_lane_tiles;
        }
        const uint32_t idle = n_lane_slots + lane;  // at most 63 idle lanes end the last lane tile
        if (idle < kLanes * n_lane_tiles) slots[idle] = tdes::Slot{0, 0, 0, 0, 0};
    }
    for (uint64_t first = (uint64_t)blockIdx.x * kGroupMessages; first < n_messages;
         first += (uint64_t)gridDim.x * kGroupMessages) {
        const uint32_t count = n_messages - first < kGroupMessages ? (uint32_t)(n_messages - first) : kGroupMessages;
        if (threadIdx.x < count * kRecordWords)
            records[threadIdx.x] = reinterpret_cast<const uint32_t *>(messages + first)[threadIdx.x];
        __syncthreads();
        for (uint32_t i = wave; i < count; i += kThreads / kLanes) {
            const tdes::PlanMessage x = reinterpret_cast<const tdes::PlanMessage *>(records)[i];
            tdes::Slot *wave_slots = slots + kLanes * (uint64_t)n_lane_tiles + x.wave_first;
            for (uint32_t t = blockIdx.y * kLanes + lane; t < x.wave_tiles; t += gridDim.y * kLanes) {
                const uint64_t at = (uint64_t)t * kWaveBlocks, left = x.n_blocks - at;
                wave_slots[t] = tdes::Slot{x.in_off + 8 * at, x.out_off + 8 * at,
                                           left / kWaveBlocks ? kWaveBlocks : (uint32_t)left, x.ks_off, 0};
            }
            const uint64_t done = (uint64_t)x.wave_tiles * kWaveBlocks;
            if (blockIdx.y == 0 && done < x.n_blocks) {  // the rest: fewer than 2048 blocks, at most one slot per lane
                const uint32_t rest = (uint32_t)(x.n_blocks - done), at = kLaneBlocks * lane;
                if (at < rest)
                    slots[x.lane_first + lane] =
                        tdes::Slot{x.in_off + 8 * (done + at), x.out_off + 8 * (done + at), min(kLaneBlocks, rest - at), x.ks_off, 0};
            }
        }
        __syncthreads();
    }
}

}  // namespace

namespace tdes {

hipError_t launch_plan(const PlanMessage *messages, uint32_t n_messages, uint32_t max_wave_tiles, PlanHeader *hdr,
                       Slot *slots, uint32_t n_tiles, uint32_t n_lane_slots, hipStream_t stream) {
    const uint32_t y = (max_wave_tiles + kTilesPerGroup - 1) / kTilesPerGroup;
    const uint32_t x = (n_messages - 1) / kGroupMessages + 1;
    const dim3 grid(x < kMaxGridX ? x : kMaxGridX, y == 0 ? 1 : y < kMaxGridY ? y : kMaxGridY);
    hipLaunchKernelGGL(tdes_plan_kernel, grid, dim3(kThreads), 0, stream, messages, n_messages, hdr, slots, n_tiles,
                       n_lane_slots);
    return hipGetLastError();
}

}  // namespace tdes
