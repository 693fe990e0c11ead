// Offsets of the predictors' feature loads within a tile's buffer resource of rows * row_bytes bytes.
// Rows of a partial tile past its last stage must read zeros and touch no memory, so the whole offset
// of a lane goes into the per-lane register, which the hardware compares with the buffer's size, and
// the scalar offset stays 0: whether that one is added before the comparison, or taken off the size
// (which wraps when it exceeds the size of a short tile), the same loads are dropped. Plain C++, so that
// a host program can walk every lane of every tile height.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define MAESTRO_LANE_FN __device__ __host__
#else
#define MAESTRO_LANE_FN
#endif

namespace maestro {

constexpr int kFeatureRow = 512;         // bytes: 256 bfloat16 features

// Large batches, one row group: load q (of eight) of feature chunk j brings tile rows 64 j + 2 i + h,
// i = wave + 4 q, half a wavefront a row; 16-byte unit u of row r is stored at u ^ (r % 16).
MAESTRO_LANE_FN constexpr uint32_t feature_offset_rows(int j, int q, int wave, int lane) {
  const int row = 64 * j + 2 * (wave + 4 * q) + (lane >> 5);
  return (uint32_t)(row * kFeatureRow + (((lane & 31) ^ (row & 15)) << 4));
}

// Large batches, two row groups: load q of chunk j brings K-slice j (128 bytes) of tile rows 8 i ..
// 8 i + 7, i = wave + 4 q; unit u of row r is stored at u ^ ((r / 2) % 8).
MAESTRO_LANE_FN constexpr uint32_t feature_offset_slice(int j, int q, int wave, int lane) {
  const int row = 8 * (wave + 4 * q) + (lane >> 3);
  return (uint32_t)(row * kFeatureRow + 128 * j + (((lane & 7) ^ ((row >> 1) & 7)) << 4));
}

// Small batches: load q brings tile rows 2 i + h, i = wave + 4 q, stored as with one row group.
MAESTRO_LANE_FN constexpr uint32_t feature_offset_split(int q, int wave, int lane) {
  return feature_offset_rows(0, q, wave, lane);
}

}  // namespace maestro
