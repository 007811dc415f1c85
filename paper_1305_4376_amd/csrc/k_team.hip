// k_team.hip -- Triple-DES over one message of middling length (ECB, CTR, CBC decryption): a workgroup per tile.
//
// Between the lengths that fill the chip with one lane per block (k_table.hip) and those that fill it with
// one wave per tile (k_bitslice.hip), each tile of 2048 blocks is shared by the eight waves of a workgroup
// (team_core.h).  A partial last tile runs beside the others in the same launch.
//
// Measured back to back (us a launch, team / table / one wave per tile): 3 * 2^17 blocks 14.6 / 16.3 / 30.0,
// 2^19 14.9 / 16.5 / 30.5, 2^20 18.7 / 30.4 / 30.7, 3 * 2^19 23.9 / 44.0 / 31.0, 2^21 29.4 / 57.3 / 31.6.  One tile
// per CU is 2^19 blocks; a launch without rounds (loads, transposes, stores) takes 3.6 us.
#include <hip/hip_runtime.h>

#include "team_core.h"
#include "internal.h"

namespace {

using namespace tdes_bs;

template <TileMode kMode>
__global__ __launch_bounds__(kTeamThreads) void tdes_team_kernel(const uint32_t *__restrict__ ks, const uint8_t *in,
                                                                 uint8_t *out, uint64_t n_blocks, uint64_t iv) {
    __shared__ uint32_t lds[kTeamWords];
    const uint64_t first = (uint64_t)blockIdx.x * kTileBlocks;
    team_tile<kMode, false>(ks, in + 8 * first, out + 8 * first, tile_count(n_blocks - first), threadIdx.x, first, iv, lds);
}

template <TileMode kMode>
hipError_t launch(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv, hipStream_t stream) {
    const uint32_t tiles = (uint32_t)((n_blocks + kTileBlocks - 1) / kTileBlocks);  // n_blocks is below kModeTeamBelow
    hipLaunchKernelGGL(tdes_team_kernel<kMode>, dim3(tiles), dim3(kTeamThreads), 0, stream, ks, in, out, n_blocks, iv);
    return hipGetLastError();
}

}  // namespace

namespace tdes {

hipError_t launch_team_ecb(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, hipStream_t stream) {
    return launch<TileMode::kEcb>(ks, in, out, n_blocks, 0, stream);
}

hipError_t launch_team_ctr(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                           hipStream_t stream) {
    return launch<TileMode::kCtr>(ks, in, out, n_blocks, iv, stream);
}

hipError_t launch_team_cbc_decrypt(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                                   hipStream_t stream) {
    return launch<TileMode::kCbcDecrypt>(ks, in, out, n_blocks, iv, stream);
}

}  // namespace tdes
