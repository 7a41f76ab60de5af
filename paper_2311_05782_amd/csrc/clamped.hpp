// Addresses of rows and columns that a tile has and the problem has not.
#pragma once

#include <stdint.h>

namespace fi {

// Byte offset of element (row, col) of an [M][N] array of 32-bit words (less than 4 GiB) without padding.
// Beyond the last row or column it is the last one's: a load there stays inside the array whatever the
// hardware's range check does with the parts of an address.
__host__ __device__ __forceinline__ uint32_t clamped_word_offset(int row, int col, int M, int N) {
  return ((uint32_t)(row < M ? row : M - 1) * (uint32_t)N + (uint32_t)(col < N ? col : N - 1)) * 4u;
}

}  // namespace fi
