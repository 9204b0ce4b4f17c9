// The evaluation kernels that score one order per lane: their LDS, and the calls that take them.
// Plain arithmetic, with no HIP but the function attributes.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace sa {

constexpr int kLaneOrders = 64;                   // orders of a tile, one per lane of a wave
constexpr int kLaneInvStride = kLaneOrders + 4;  // bytes per request, padded across the banks

// LDS one wave needs to validate and replay one (order, layout) row: order, flags, the
// replay's staging and the validity bitmap.
__host__ __device__ __forceinline__ size_t sized_row_bytes(int n) {
  return (((size_t)n * 2 + 15) & ~size_t(15)) + (((size_t)n + 15) & ~size_t(15)) + 64 * 16 + 32 * 4;
}

__host__ __device__ __forceinline__ size_t lane_inv_bytes(int n) {
  return ((size_t)(n + 1) * kLaneInvStride + 15) / 16 * 16;  // a spare row takes ids out of range
}
__host__ __device__ __forceinline__ int lane_words(int n) { return ((n + 31) / 32) | 1; }
// LDS shared by a workgroup: the three sorted tables, and the requests by id for layouts.
__host__ __device__ __forceinline__ size_t lane_shared_bytes(int n, bool layout) { return (size_t)n * (layout ? 64 : 48); }
// LDS of one wave: inv, the entries (U, W) and T0 of mcap batches and a spare, and for
// layouts the start bits with their running counts and the rows' flags.
__host__ __device__ __forceinline__ size_t lane_wave_bytes(int n, int mcap, bool layout) {
  const size_t own = lane_inv_bytes(n) + (size_t)(mcap + 1) * (kLaneOrders * 12) +
                     (layout ? (size_t)kLaneOrders * lane_words(n) * 8 + kLaneOrders * 4 : 0);
  return layout && own < sized_row_bytes(n) ? sized_row_bytes(n) : own;
}

constexpr int kContStage = 32;               // positions staged at a time
constexpr int kContIdStride = kContStage + 2;  // u16 entries per lane

// LDS of one wave under continuous admission: slots (8 B), staged ids and the bitmap, per lane.
__host__ __device__ __forceinline__ size_t cont_lane_wave_bytes(int n, int cap) {
  return (size_t)kLaneOrders * (cap * 8 + kContIdStride * 2 + ((n + 31) / 32) * 4);
}

// Rows from which evaluation runs with one order per lane, where that becomes the faster one of the
// two. A tile of 64 orders takes a lone wave about as long as the one-order-per-wave kernels take
// for all rows, so the crossing lies well before every SIMD has a tile (65536 rows): at 32768 rows
// 128 of the 256 CUs hold the 512 tiles. Measured (us, lanes against waves): static, 128 requests,
// batches of 16: 33 against 34 at 32768 rows, 35 against 51 at 65536, but batches of 4 only 37
// against 41 at 65536 (38 against 32 at 32768); layouts, the same queue: 39 against 52 at 16384;
// continuous, 32 running: 58 against 43 at 16384 rows of 128 requests and 58 against 82 at 32768,
// while with long queues the scans' LDS leaves the other kernel few waves (1024 requests: 1.8 times
// its rate at 8192 rows) and short ones are over in a few events.
inline int64_t eval_lane_rows(int n, int B, bool layout) {
  return layout ? 16384 : (n <= 64 || B >= 16 ? 32768 : 65536);
}
inline int64_t eval_cont_lane_rows(int n) { return n >= 768 ? 8192 : (n >= 320 || n <= 24 ? 16384 : 32768); }

// How a call takes the kernels: waves per workgroup (0: not at all), their LDS, and `cap`: the
// batches a lane's entries hold, or the registers of the running set under continuous admission.
struct LaneShape {
  int waves;
  size_t lds;
  int cap;
};

// Static batches, of the maximum size or by layout: four waves per workgroup or not at all, which
// the LDS allows for 431 requests at most (static, batches of 64; 306 of 16, 144 of 4; with layouts
// 256, 144 and 52).
inline LaneShape eval_lane_shape(int n, int B, bool layout, int64_t rows, int lim) {
  const int M = (n + B - 1) / B, cap = layout ? std::min(n, 3 * M + 4) : M;
  const size_t lds = lane_shared_bytes(n, layout) + 4 * lane_wave_bytes(n, cap, layout);
  if (n < 2 || rows < eval_lane_rows(n, B, layout) || cap > 254 || lds > (size_t)lim) return LaneShape{0, 0, 0};
  return LaneShape{4, lds, cap};
}
// Continuous admission: the running requests in 8, 16, 32 or 64 registers.
inline LaneShape eval_cont_lane_shape(int n, int B, int64_t rows, int lim) {
  if (rows < eval_cont_lane_rows(n)) return LaneShape{0, 0, 0};
  const int n0 = std::min(B, n), cap = n0 <= 8 ? 8 : (n0 <= 16 ? 16 : (n0 <= 32 ? 32 : 64));
  const size_t shared = (size_t)n * 16, per = cont_lane_wave_bytes(n, cap);
  int waves = 4;
  while (waves > 0 && shared + waves * per > (size_t)lim) --waves;
  return LaneShape{waves, shared + waves * per, cap};
}

}  // namespace sa
