// Byte offsets into a layer's packed values and positions.  A layer may hold almost 4 GiB of values, so they are formed in
// unsigned 32-bit arithmetic throughout.  Integer arithmetic only, so that it also runs in a host test.
#pragma once
#include <cstdint>

namespace crisp {

// Value `slot` of row `row` of kept block `block` (16 x 16 blocks, `slots` values a row).
__host__ __device__ __forceinline__ constexpr uint32_t b16_value_at(int block, int row, int slots, int slot) {
    return (((uint32_t)block * 16u + (uint32_t)row) * (uint32_t)slots + (uint32_t)slot) * 2u;
}
// The position words of that row (`words` each).
__host__ __device__ __forceinline__ constexpr uint32_t b16_words_at(int block, int row, int words) {
    return ((uint32_t)block * 16u + (uint32_t)row) * (uint32_t)words * 4u;
}

}  // namespace crisp
