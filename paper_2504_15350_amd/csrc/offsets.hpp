// 32-bit byte offsets of a lane from a uniform base in the FP32 passes, and the leading dimensions
// up to which they hold (host and device).
#pragma once

#include <stdint.h>

namespace rpod {

// S^T Q: column c < 16 of a block of FP32 columns ld apart, 16-byte chunk k < 16 of a unit of rows; with
// k = 0 and 4 i added, row i < ld
constexpr uint32_t chunk_offset(int c, int64_t ld, int k) { return (uint32_t)c * (uint32_t)(4 * ld) + 16u * (uint32_t)k; }
constexpr bool chunk_offset_fits(int64_t ld) { return ld < ((int64_t)1 << 26); }

// S X: row i <= ld + 255 of column 8 g, g < 4
constexpr uint32_t row_offset(int g, int64_t ld, int64_t i) {
    return (uint32_t)(8 * g) * (uint32_t)(4 * ld) + (uint32_t)(4 * i);
}
constexpr bool row_offset_fits(int64_t ld) { return ld < ((int64_t)1 << 25); }

}  // namespace rpod
