// k_short.hip -- Triple-DES over a short message (ECB, CTR, CBC decryption): one output bit of f per lane (short_core.h).
#include <hip/hip_runtime.h>

#include "internal.h"
#include "short_core.h"

namespace {

using namespace tdes_bs;

template <TileMode kMode>
__global__ __launch_bounds__(kShortThreads) void tdes_short_kernel(const uint32_t *__restrict__ ks, const uint8_t *in,
                                                                   uint8_t *out, uint32_t n_blocks, uint64_t iv) {
    short_blocks<kMode>(ks, in, out, n_blocks, blockIdx.x, false, iv);
}

}  // namespace

namespace tdes {

namespace {

template <TileMode kMode>
hipError_t launch(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv, hipStream_t stream) {
    const uint32_t n = (uint32_t)n_blocks;
    hipLaunchKernelGGL(tdes_short_kernel<kMode>, dim3(short_groups(n)), dim3(kShortThreads), 0, stream,
                       ks, in, out, n, iv);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_short_ecb(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, hipStream_t stream) {
    return launch<TileMode::kEcb>(ks, in, out, n_blocks, 0, stream);
}

hipError_t launch_short_ctr(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                            hipStream_t stream) {
    return launch<TileMode::kCtr>(ks, in, out, n_blocks, iv, stream);
}

hipError_t launch_short_cbc_decrypt(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                                    hipStream_t stream) {
    return launch<TileMode::kCbcDecrypt>(ks, in, out, n_blocks, iv, stream);
}

}  // namespace tdes
