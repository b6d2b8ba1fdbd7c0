// 8 x 8 bit transposition in registers, shared by the bit-plane packer and the first layer's product.
#pragma once

#include "bnn_internal.h"

namespace bnn {

__device__ inline uint32_t bit_select(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }

// One stage of the transposition below: exchanges the K-bit fields of registers b and b + K.
template <int K, uint32_t MASK>
__device__ inline void exchange_fields(uint32_t (&p)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int b = (i / K) * 2 * K + i % K;
        const uint32_t a = p[b], c = p[b + K];
        p[b] = bit_select(MASK, a, c << K);
        p[b + K] = bit_select(MASK, a >> K, c);
    }
}

// In each byte column: in p[b] bit 8j + s -> out p[s] bit 8j + b (its own inverse; 48 vector operations).
__device__ inline void transpose_bits_8x8(uint32_t (&p)[8]) {
    exchange_fields<4, 0x0F0F0F0Fu>(p);
    exchange_fields<2, 0x33333333u>(p);
    exchange_fields<1, 0x55555555u>(p);
}

// Lane l with bit m of word x -> lane m with bit l, in each half wavefront of 32 lanes (every lane active): five exchanges with
// the lane 16, 8, 4, 2, 1 away, each a rotation and a select.
__device__ inline uint32_t transpose_bits_32_lanes(uint32_t x) {
    int lane = int(threadIdx.x);
    asm volatile("" : "+v"(lane));           // the masks below are made here, not kept in registers for a kernel's life
    auto join = [&](uint32_t own, uint32_t partner, int s, uint32_t low) {
        const bool upper = lane & s;
        return bit_select(upper ? ~low : low, own, __builtin_amdgcn_alignbit(partner, partner, upper ? s : 32 - s));
    };
    const auto sw = __builtin_amdgcn_permlane16_swap(x, x, false, false);               // what lanes 0-15 / 16-31 of a half have
    x = join(x, (lane & 16) ? sw[0] : sw[1], 16, 0x0000FFFFu);
    x = join(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x128, 0xF, 0xF, true)), 8, 0x00FF00FFu);      // row_ror:8
    const int mirror = __builtin_amdgcn_update_dpp(0, int(x), 0x141, 0xF, 0xF, true);                          // lane ^ 7
    x = join(x, uint32_t(__builtin_amdgcn_update_dpp(0, mirror, 0x1B, 0xF, 0xF, true)), 4, 0x0F0F0F0Fu);       // ... ^ 3
    x = join(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x4E, 0xF, 0xF, true)), 2, 0x33333333u);
    return join(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0xB1, 0xF, 0xF, true)), 1, 0x55555555u);
}

}  // namespace bnn
