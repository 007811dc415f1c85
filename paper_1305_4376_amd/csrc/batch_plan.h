// batch_plan.h -- the device-side plan of a batch, shared by the planner (batch.cpp) and the kernel.
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>

#include "../../include/tdes.h"

namespace tdes {

// Plan buffer on the device: [PlanHeader][slots].  Slots: 64 per lane tile, then one per wave tile.
struct PlanHeader {
    uint32_t n_tiles;       // lane tiles, then wave tiles
    uint32_t n_lane_tiles;
    uint32_t pad[62];
};
static_assert(sizeof(PlanHeader) == 256, "header is one 256-byte line");

// One message as the host plans it: its first wave slot (of the wave slots), its first lane slot, and
// what of it goes where: wave_tiles runs of up to 2048 blocks, then lane slots of up to 32 for the rest.
struct PlanMessage {
    uint64_t in_off;
    uint64_t out_off;
    uint64_t n_blocks;
    uint32_t ks_off;
    uint32_t wave_first;
    uint32_t lane_first;
    uint32_t wave_tiles;
};
static_assert(sizeof(PlanMessage) == 40, "no padding: the records cross the host link");

// A run of consecutive blocks of one message: byte offsets from the batch base,
// the number of blocks (a wave tile: up to 2048; a lane slot: up to 32; 0 for
// an idle lane) and the word offset of its 96 subkey words in the schedule table.
struct Slot {
    uint64_t in_off;
    uint64_t out_off;
    uint32_t count;
    uint32_t ks_off;
    uint64_t pad;
};
static_assert(sizeof(Slot) == 32, "slot is 32 bytes");

// The slot of tile t: a lane tile's first, or a wave tile's only one.
__host__ __device__ inline uint32_t tile_slot(uint32_t t, uint32_t n_lane_tiles) {
    return t < n_lane_tiles ? 64 * t : 63 * n_lane_tiles + t;
}

// Writes the header and every slot from the messages' records, which the kernel reads from (pinned) host
// memory.  max_wave_tiles: of any message.  n_messages > 0.
hipError_t launch_plan(const PlanMessage *messages, uint32_t n_messages, uint32_t max_wave_tiles, PlanHeader *hdr,
                       Slot *slots, uint32_t n_tiles, uint32_t n_lane_slots, hipStream_t stream);

// capped: the variant held to 120 VGPRs (room for another kernel's waves beside it).
hipError_t launch_batch(const uint32_t *sched, const PlanHeader *hdr, const Slot *slots, uint32_t *counter,
                        uint8_t *base, uint32_t grid, uint32_t threads, uint32_t tiles_per_draw, bool capped,
                        hipStream_t stream);
// The capped variant alone (k_batch_capped.hip); arguments checked by launch_batch.
hipError_t launch_batch_capped(const uint32_t *sched, const PlanHeader *hdr, const Slot *slots, uint32_t *counter,
                               uint8_t *base, uint32_t grid, uint32_t threads, uint32_t tiles_per_draw,
                               hipStream_t stream);

// A batch of at most kTeamTiles tiles: a workgroup per tile (k_batch_team.hip).  Launches back to back, us, by
// teams / by waves: 1152 whole tiles 41 / -, 1400 46 / 53, 2000 58 / 60, 2300 65 / 63; with lane tiles among
// them 234 (18 of them) 22.5 / 46, 1466 (239) 48 / 55, 1949 (313) 60 / 60.  Whole calls with the present,
// smaller circuits: 1100 whole tiles 43.7 / 52.3, 1500 49.7 / 56.9, 1900 60.9 / 61.6.
constexpr uint32_t kTeamTiles = TDES_BATCH_TEAM_TILES;
hipError_t launch_batch_team(const uint32_t *sched, const PlanHeader *hdr, const Slot *slots, uint8_t *base,
                             uint32_t grid, hipStream_t stream);  // grid: at least the tiles

}  // namespace tdes
