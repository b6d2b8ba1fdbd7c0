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

}  // namespace bnn
