// Morton (Z-order) keys for quadtree positions.
//
// A node or block at (row r, column c) of a level gets the key with the bits
// of c at even positions and the bits of r at odd positions. The two lowest
// bits of a key are then the quadrant q = 2*m + n of the position inside its
// parent (m = row half, n = column half), matching the child order
// C_11, C_12, C_21, C_22 of the quadtree, and sorting by key lists every
// subtree contiguously.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace qt {

__host__ __device__ inline uint64_t spread_bits(uint32_t x) {
    uint64_t v = x;
    v = (v | (v << 16)) & 0x0000FFFF0000FFFFull;
    v = (v | (v << 8)) & 0x00FF00FF00FF00FFull;
    v = (v | (v << 4)) & 0x0F0F0F0F0F0F0F0Full;
    v = (v | (v << 2)) & 0x3333333333333333ull;
    v = (v | (v << 1)) & 0x5555555555555555ull;
    return v;
}

__host__ __device__ inline uint32_t compact_bits(uint64_t v) {
    v &= 0x5555555555555555ull;
    v = (v | (v >> 1)) & 0x3333333333333333ull;
    v = (v | (v >> 2)) & 0x0F0F0F0F0F0F0F0Full;
    v = (v | (v >> 4)) & 0x00FF00FF00FF00FFull;
    v = (v | (v >> 8)) & 0x0000FFFF0000FFFFull;
    v = (v | (v >> 16)) & 0x00000000FFFFFFFFull;
    return (uint32_t)v;
}

__host__ __device__ inline uint64_t morton_key(uint32_t r, uint32_t c) {
    return (spread_bits(r) << 1) | spread_bits(c);
}
__host__ __device__ inline uint32_t morton_row(uint64_t k) { return compact_bits(k >> 1); }
__host__ __device__ inline uint32_t morton_col(uint64_t k) { return compact_bits(k); }

// Swaps index bits a > b of a 64-bit mask (bit i of the result is the bit of
// the mask whose index has these two bits of i exchanged). pos: the mask of
// all indices with bit b set and bit a clear.
__device__ __forceinline__ uint64_t swap_index_bits(uint64_t m, int a, int b, uint64_t pos) {
    const int sh = (1 << a) - (1 << b);
    const uint64_t d = ((m >> sh) ^ m) & pos;
    return m ^ d ^ (d << sh);
}

// A leaf's occupancy in Morton order (index bits r2 c2 r1 c1 r0 c0) as
// row-major (r2 r1 r0 c2 c1 c0), and that transposed as column-major; leaves
// of 4 x 4 and 2 x 2 blocks have the lower four and two index bits only.
__device__ __forceinline__ uint64_t morton_to_rowmajor(uint64_t m, int lb_log) {
    if (lb_log == 3) {
        m = swap_index_bits(m, 4, 3, 0x0000FF000000FF00ull);   // r2 r1 c2 c1 r0 c0
        m = swap_index_bits(m, 2, 1, 0x0C0C0C0C0C0C0C0Cull);   // r2 r1 c2 r0 c1 c0
        return swap_index_bits(m, 3, 2, 0x00F000F000F000F0ull);
    }
    return lb_log == 2 ? swap_index_bits(m, 2, 1, 0x0C0Cull) : m;
}
__device__ __forceinline__ uint64_t rowmajor_to_colmajor(uint64_t m, int lb_log) {
    if (lb_log == 3) {
        m = swap_index_bits(m, 5, 2, 0x00000000F0F0F0F0ull);
        m = swap_index_bits(m, 4, 1, 0x0000CCCC0000CCCCull);
        return swap_index_bits(m, 3, 0, 0x00AA00AA00AA00AAull);
    }
    if (lb_log == 2) return swap_index_bits(swap_index_bits(m, 3, 1, 0x00CCull), 2, 0, 0x0A0Aull);
    return lb_log == 1 ? swap_index_bits(m, 1, 0, 0x2ull) : m;
}

}  // namespace qt
