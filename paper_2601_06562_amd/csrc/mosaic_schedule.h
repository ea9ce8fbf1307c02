// How a launch of the fused pass divides its rows and its vocabulary, from the number of rows it really finds.
//
// The host plans for a bound on the masked rows; the number itself is known on the device only.  Every kernel of a
// pass therefore works the division out itself, with the function below, from the same few numbers: a plan for 16
// row tiles that finds 9 of them in use spreads those over all compute units instead of leaving 7/16 of its units
// empty (4096 positions planned, 2077 masked: 2621 -> 1569 us).  What a pass computes does not depend on the
// division (see Fold in mosaic_logits.hip), so neither do its results.
#ifndef MOSAIC_SCHEDULE_H_
#define MOSAIC_SCHEDULE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mosaic.h"

namespace mosaic {

struct Schedule {
  int32_t row_tiles;   // row tiles that hold rows
  int32_t splits;      // vocabulary ranges of every row tile
  int32_t stride;      // rows of one split in the partial arrays
};

struct ScheduleInput {
  uint32_t vocab_tiles;   // tiles to divide (without the ragged last one where a second launch covers it)
  uint32_t grid;          // workgroups of the launch
  uint32_t extra;         // partial slots per row beyond the splits (1 where a second launch adds its own)
  uint32_t slots64;       // rows x splits the partial arrays hold, in units of 64
};

__host__ __device__ inline uint32_t ceil_div(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

// Rows of one split in the partial arrays.
__host__ __device__ inline int32_t partial_stride(int32_t rows) { return (rows + 63) & ~63; }

// The candidate that uses `extra_rounds` rounds of the grid more than the fewest possible, as (cost, splits) packed
// into one integer: the smaller one is the better one.  A round lasts as long as its longest unit, a unit costs half
// a tile on top of its tiles (pipeline fill, merge); of the split counts that fit the same rounds the largest has the
// shortest units, and of those with equally long units the smallest makes the fewest partial results.  At least four
// splits where vocabulary and memory allow: the 32 workgroups that share an L2 then work on 8 row tiles x 4 splits
// (256 row tiles in one split each: 62 ms; in four: 47 ms).
constexpr int kScheduleRounds = 64;   // candidates looked at: the rounds' quantisation is below 2% beyond
__host__ __device__ inline uint64_t schedule_candidate(const ScheduleInput& in, int32_t rows, uint32_t extra_rounds) {
  // 32-bit throughout (rows < 2^31, so at most 2^23 row tiles and 2^31 units): a wide division costs the device 10x
  const uint32_t row_tiles = ceil_div((uint32_t)rows, MOSAIC_ROW_TILE);
  const uint32_t fit = in.slots64 / ((uint32_t)partial_stride(rows) >> 6);
  uint32_t most = in.vocab_tiles < MOSAIC_MAX_VOCAB_SPLITS ? in.vocab_tiles : MOSAIC_MAX_VOCAB_SPLITS;
  if (fit < most + in.extra) most = fit <= in.extra + 1 ? 1 : fit - in.extra;
  const uint32_t least = most < 4 ? most : 4;
  const uint32_t first = ceil_div(row_tiles * least, in.grid);
  uint32_t s = (first + extra_rounds) * in.grid / row_tiles;
  if (s > most) s = most;
  const uint32_t longest = ceil_div(in.vocab_tiles, s);
  uint32_t splits = ceil_div(in.vocab_tiles, longest);
  if (splits < least) splits = least;
  const uint32_t rounds = ceil_div(row_tiles * splits, in.grid);
  return (uint64_t)rounds * (2 * longest + 1) << 16 | splits;
}

__host__ __device__ inline Schedule schedule_of(int32_t rows, uint64_t best) {
  return Schedule{(int32_t)ceil_div((uint32_t)rows, MOSAIC_ROW_TILE), (int32_t)(best & 0xffff), partial_stride(rows)};
}

// On the host: for the bound the plan was made for, handed to the kernels so that they need not search when the
// count turns out to be that bound.
inline Schedule choose_schedule(const ScheduleInput& in, int32_t rows) {
  uint64_t best = ~(uint64_t)0;
  for (int32_t r = 0; r < kScheduleRounds; ++r) {
    const uint64_t c = schedule_candidate(in, rows, (uint32_t)r);
    best = c < best ? c : best;
  }
  return schedule_of(rows, best);
}

// On the device: one candidate per lane, the same result in every wave (~1 us).
__device__ __forceinline__ Schedule choose_schedule_wave(const ScheduleInput& in, int32_t rows) {
  uint64_t best = schedule_candidate(in, rows, threadIdx.x & 63);
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) {
    const uint64_t other = __shfl_xor((unsigned long long)best, x, 64);
    best = other < best ? other : best;
  }
  Schedule s = schedule_of(rows, best);
  s.splits = __builtin_amdgcn_readfirstlane(s.splits);
  return s;
}

}  // namespace mosaic
#endif
