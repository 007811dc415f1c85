// table_core.h -- what the table kernels share: the combined S-box/P tables and the block permutations.
#pragma once
#include <hip/hip_runtime.h>

#include "des_spec.h"

namespace tdes_table {

constexpr int kCopies = 32;  // of each table entry, one per LDS bank

constexpr uint32_t rotl32(uint32_t x, int n) { return n == 0 ? x : (x << n) | (x >> (32 - n)); }

struct SpTables {
    uint32_t v[8][64];
};

// SP[b][x]: f(R) word (bit 0 of f in bit 31) for box b's output S_b(x), rotated left by 5.
constexpr SpTables make_sp() {
    SpTables t{};
    for (int b = 0; b < 8; b++)
        for (uint32_t x = 0; x < 64; x++) {
            const uint32_t s = tdes_spec::sbox(b, x);
            uint32_t f = 0;
            for (int i = 0; i < 32; i++) {
                const int src = tdes_spec::kP[i];
                if (src / 4 == b) f |= ((s >> (3 - src % 4)) & 1u) << (31 - i);
            }
            t.v[b][x] = rotl32(f, 5);
        }
    return t;
}

constexpr SpTables kSp = make_sp();

__device__ __forceinline__ uint32_t rotl(uint32_t x, int n) {
    return __builtin_amdgcn_alignbit(x, x, (32 - n) & 31);
}

// Exchange bits (a >> n) & m with b & m.
__device__ __forceinline__ void exchange(uint32_t &a, uint32_t &b, int n, uint32_t m) {
    const uint32_t t = ((a >> n) ^ b) & m;
    b ^= t;
    a ^= t << n;
}

// IP on a block held as (hi, lo) = bits 0..31, 32..63 of the standard's numbering.
__device__ __forceinline__ void initial_perm(uint32_t &hi, uint32_t &lo) {
    exchange(hi, lo, 4, 0x0F0F0F0Fu);
    exchange(hi, lo, 16, 0x0000FFFFu);
    exchange(lo, hi, 2, 0x33333333u);
    exchange(lo, hi, 8, 0x00FF00FFu);
    exchange(hi, lo, 1, 0x55555555u);
}

__device__ __forceinline__ void final_perm(uint32_t &hi, uint32_t &lo) {
    exchange(hi, lo, 1, 0x55555555u);
    exchange(lo, hi, 8, 0x00FF00FFu);
    exchange(lo, hi, 2, 0x33333333u);
    exchange(hi, lo, 16, 0x0000FFFFu);
    exchange(hi, lo, 4, 0x0F0F0F0Fu);
}

}  // namespace tdes_table
