// k_pair.hip -- Triple-DES over a shortish message (ECB, CTR, CBC decryption): table lookups, two lanes per block.
//
// The table kernel (k_table.hip) gives a block to one lane, whose round is a chain: rotate, key, eight
// address permutes and LDS reads issued one after the other, the last read's way back, three XORs.  While a
// message leaves lanes free, that chain is the kernel's time.  Here two neighbouring lanes share a block:
// both hold both halves, the even lane looks up the boxes at the bytes of R rotated by 5 (1, 7, 5, 3), the
// odd lane those of R rotated by 9 (2, 8, 6, 4), and one exchange between the two (a DPP operand) joins their
// XORs.  A lane needs four tables, so a workgroup's copies take 32 KiB of LDS to fill instead of 64.
//
// LDS layout.  As in k_table.hip with slots for boxes: entry x of slot s (a byte position), copy c, is at
// byte (s / 2) * 16384 + x * 256 + (s % 2) * 128 + c * 4; lane l reads copy l % 32, which holds the boxes of
// l's parity, so a half-wave's lanes always hit 32 different banks.
//
// Bound: a round's chain of about 165 cycles (the table kernel's: 200), and from two waves per SIMD on the
// LDS reads, which cost as much per block as in the table kernel.  Back to back, us a launch (256 / 512
// threads / table kernel): 16384 blocks 5.5 / 5.8 / 6.2, 65536 5.7 / 5.7 / 6.4, 98304 6.8 / 7.4 / 6.6, 2^17
// 7.7 / 7.5 / 6.6, 2^18 11.8 / 11.6 / 9.8, 5 * 2^16 13.2 / 13.2 / 16.1, 3 * 2^17 16.3 / 14.7 / 16.3.
#include <hip/hip_runtime.h>

#include "bitslice_core.h"
#include "internal.h"
#include "table_core.h"

namespace {

using tdes_bs::TileMode;
using tdes_table::kCopies;

constexpr int kBox[2][4] = {{0, 6, 4, 2}, {1, 7, 5, 3}};  // the box at each byte, by the lane's parity

struct PairTables {
    uint2 v[4][64];  // [slot][entry]: even and odd lanes' word
};

constexpr PairTables make_pair_tables() {
    PairTables t{};
    for (int s = 0; s < 4; s++)
        for (uint32_t x = 0; x < 64; x++) {
            t.v[s][x].x = tdes_table::kSp.v[kBox[0][s]][x];
            t.v[s][x].y = tdes_table::kSp.v[kBox[1][s]][x];
        }
    return t;
}

__constant__ PairTables g_pair = make_pair_tables();

// What the lane's parity decides.
struct PairLane {
    uint32_t lane4;       // byte offset of its copy
    uint32_t rot;         // right rotation that brings its boxes' inputs to the bytes' low bits
    uint32_t even, odd;   // ~0 in even (odd) lanes
};

// L ^ f(R, K), all words rotated left by 5; ka, kb: the round's key words.
__device__ __forceinline__ uint32_t pair_round(uint32_t l5, uint32_t r5, uint32_t ka, uint32_t kb, const uint8_t *lds,
                                               const PairLane &p) {
    constexpr uint32_t kMask = 0x3F3F3F3Fu;
    const uint32_t k = __builtin_amdgcn_bitop3_b32(ka & p.even, kb, p.odd, 0xF8);  // even lanes ka, odd lanes kb
    const uint32_t x = __builtin_amdgcn_bitop3_b32(__builtin_amdgcn_alignbit(r5, r5, p.rot), k, kMask, 0x28);  // (R ^ k) & mask
    auto look = [&](int s) {
        const uint32_t addr = __builtin_amdgcn_perm(x, p.lane4, 0x0C0C0000u | ((4u + s) << 8));
        return *reinterpret_cast<const uint32_t *>(lds + addr + (s / 2) * 16384 + (s % 2) * 128);
    };
    const uint32_t v0 = look(0), v1 = look(1), v2 = look(2), v3 = look(3);
    const uint32_t t = __builtin_amdgcn_bitop3_b32(l5 & p.even, v0, v1, 0x96);
    const uint32_t u = __builtin_amdgcn_bitop3_b32(t, v2, v3, 0x96);
    return u ^ (uint32_t)__builtin_amdgcn_mov_dpp((int)u, 0xB1, 0xF, 0xF, true);  // 0xB1: the other lane of the pair
}

template <TileMode kMode, int kThreads>
__global__ __launch_bounds__(kThreads) void tdes_pair_kernel(const uint32_t *__restrict__ ks, const uint8_t *in,
                                                             uint8_t *out, uint32_t n_blocks, uint64_t iv) {
    __shared__ uint4 lds4[4 * 64 * kCopies / 4];
    const uint32_t parity = threadIdx.x & 1;
    const uint32_t stride = gridDim.x * (kThreads / 2);
    uint32_t b = blockIdx.x * (kThreads / 2) + threadIdx.x / 2;
    uint2 v = make_uint2(0, 0);
    auto load = [&](uint32_t at) { v = reinterpret_cast<const uint2 *>(in)[at]; };
    if (kMode != TileMode::kCtr && b < n_blocks) load(b);  // on its way while the tables are written
#pragma unroll
    for (int i = 0; i < 4 * 64 * kCopies / 4 / kThreads; i++) {
        const int c = i * kThreads + threadIdx.x, wd = 4 * c;
        const uint2 e = g_pair.v[2 * (wd / 4096) + (wd / 32) % 2][(wd / 64) % 64];
        lds4[c] = make_uint4(e.x, e.y, e.x, e.y);
    }
    __syncthreads();
    const uint8_t *lds = reinterpret_cast<const uint8_t *>(lds4);
    PairLane p;
    p.lane4 = (threadIdx.x % kCopies) * 4;
    p.rot = parity ? 28 : 0;
    p.odd = parity ? ~0u : 0u;
    p.even = ~p.odd;
    for (; b < n_blocks; b += stride) {
        uint32_t l, r;
        if constexpr (kMode == TileMode::kCtr) {
            const uint64_t t = iv + b;
            l = (uint32_t)(t >> 32);
            r = (uint32_t)t;
        } else {
            l = __builtin_bswap32(v.x);
            r = __builtin_bswap32(v.y);
        }
        // What the output word is XORed with, loaded ahead of the rounds.
        uint32_t with = 0;
        if constexpr (kMode == TileMode::kCtr) with = reinterpret_cast<const uint32_t *>(in)[2 * (uint64_t)b + parity];
        if constexpr (kMode == TileMode::kCbcDecrypt) {
            with = parity ? tdes_bs::be_lo_word(iv) : tdes_bs::be_hi_word(iv);
            if (b != 0) with = reinterpret_cast<const uint32_t *>(in)[2 * (uint64_t)b - 2 + parity];
        }
        if (kMode != TileMode::kCtr && b + stride < n_blocks) load(b + stride);
        tdes_table::initial_perm(l, r);
        uint32_t x = tdes_table::rotl(l, 5), y = tdes_table::rotl(r, 5);
#pragma unroll
        for (int i = 0; i < 48; i += 2) {
            // (between the stages only the halves swap: rounds 16..31 change y first)
            uint32_t &first = i / 16 == 1 ? y : x, &second = i / 16 == 1 ? x : y;
            first = pair_round(first, second, ks[2 * i], ks[2 * i + 1], lds, p);
            second = pair_round(second, first, ks[2 * i + 2], ks[2 * i + 3], lds, p);
        }
        l = tdes_table::rotl(x, 27);
        r = tdes_table::rotl(y, 27);
        tdes_table::final_perm(r, l);  // preoutput R16 L16
        reinterpret_cast<uint32_t *>(out)[2 * (uint64_t)b + parity] = __builtin_bswap32(parity ? l : r) ^ with;
    }
}

template <TileMode kMode>
hipError_t launch(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv, hipStream_t stream) {
    tdes::DeviceInfo info;
    if (tdes::device_info(&info) != TDES_OK) return hipErrorInvalidDevice;
    // Small workgroups reach more CUs; past one pass of the resident ones, more waves share each one's tables.
    const uint32_t n = (uint32_t)n_blocks, resident = (uint32_t)info.cu_count * 4;  // by LDS: 4 * 32 KiB a CU
    const bool small = n <= resident * (256 / 2);
    const uint32_t per = (small ? 256 : 512) / 2, groups = (n + per - 1) / per, grid = groups < resident ? groups : resident;
    if (small)
        hipLaunchKernelGGL((tdes_pair_kernel<kMode, 256>), dim3(grid), dim3(256), 0, stream, ks, in, out, n, iv);
    else
        hipLaunchKernelGGL((tdes_pair_kernel<kMode, 512>), dim3(grid), dim3(512), 0, stream, ks, in, out, n, iv);
    return hipGetLastError();
}

}  // namespace

namespace tdes {

hipError_t launch_pair_ecb(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, hipStream_t stream) {
    return launch<TileMode::kEcb>(ks, in, out, n_blocks, 0, stream);
}

hipError_t launch_pair_ctr(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                           hipStream_t stream) {
    return launch<TileMode::kCtr>(ks, in, out, n_blocks, iv, stream);
}

hipError_t launch_pair_cbc_decrypt(const uint32_t *ks, const uint8_t *in, uint8_t *out, uint64_t n_blocks, uint64_t iv,
                                   hipStream_t stream) {
    return launch<TileMode::kCbcDecrypt>(ks, in, out, n_blocks, iv, stream);
}

}  // namespace tdes
