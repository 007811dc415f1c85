// k_batch_team.hip -- a batch too small to fill the chip with one wave per tile: a workgroup per tile.
//
// A wave takes over 30 us for a tile however few there are (more for a lane tile), so a batch of up to
// kTeamTiles tiles shares each of them between the eight waves of a workgroup (team_core.h), lane tiles
// with every lane's own key too.  In a captured graph the grid is the largest, so that one graph serves
// every such batch; workgroups past the last tile end at once.
#include <hip/hip_runtime.h>

#include "batch_plan.h"
#include "internal.h"
#include "team_core.h"

namespace {

using namespace tdes_bs;

__global__ __launch_bounds__(kTeamThreads) void tdes_batch_team_kernel(const uint32_t *__restrict__ sched,
                                                                       const tdes::PlanHeader *__restrict__ hdr,
                                                                       const tdes::Slot *__restrict__ slots, uint8_t *base) {
    __shared__ uint32_t lds[kTeamLaneWords];
    const uint32_t tile = blockIdx.x, n_lane_tiles = hdr->n_lane_tiles;
    if (tile >= hdr->n_tiles) return;
    const uint32_t first_slot = tdes::tile_slot(tile, n_lane_tiles);
    if (tile < n_lane_tiles) {
        const tdes::Slot s = slots[first_slot + threadIdx.x % kLanes];
        team_tile<TileMode::kEcb, true>(sched + s.ks_off, base + s.in_off, base + s.out_off, s.count, threadIdx.x, 0, 0, lds);
    } else {
        const tdes::Slot &s = slots[first_slot];
        team_tile<TileMode::kEcb, false>(sched + s.ks_off, base + s.in_off, base + s.out_off, s.count, threadIdx.x, 0, 0, lds);
    }
}

}  // namespace

namespace tdes {

hipError_t launch_batch_team(const uint32_t *sched, const PlanHeader *hdr, const Slot *slots, uint8_t *base,
                             uint32_t grid, hipStream_t stream) {
    hipLaunchKernelGGL(tdes_batch_team_kernel, dim3(grid), dim3(kTeamThreads), 0, stream, sched, hdr, slots, base);
    return hipGetLastError();
}

}  // namespace tdes
