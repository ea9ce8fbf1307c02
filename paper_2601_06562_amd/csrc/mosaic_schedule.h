// How a launch of the fused pass divides its rows and its vocabulary, from the number of rows it really finds.
//
// The host plans for a bound on the masked rows; the number itself is known on the device only.  Every kernel of a
// pass therefore works the division out itself, with the function below, from the same few numbers: a plan for 16
// row tiles that finds 9 of them in use spreads those over all compute units instead of leaving 7/16 of its units
// empty (4096 positions planned, 2077 masked: 2621 -> 1569 us).  What a pass computes does not depend on the
// division but for a last bit here and there (see Fold in mosaic_logits.hip).
#ifndef MOSAIC_SCHEDULE_H_
#define MOSAIC_SCHEDULE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mosaic.h"

namespace mosaic {

struct Schedule {
  int32_t width;       // of a row tile, in units of 32 rows
  int32_t row_tiles;   // row tiles that hold rows
  int32_t splits;      // vocabulary ranges of every row tile
  int32_t stride;      // rows of one split in the partial arrays
};

struct ScheduleInput {
  uint32_t vocab_tiles;   // tiles to divide (without the ragged last one where a second launch covers it)
  uint32_t k_tiles;       // K-tiles of a vocabulary tile
  uint32_t widths;        // bit w - 1: row tiles of 32*w rows are on offer
  uint32_t sampling;      // 1: the reduction draws, too
  uint32_t grid;          // workgroups of the launch
  uint32_t extra;         // partial slots per row beyond the splits (1 where a second launch adds its own)
  uint32_t slots64;       // rows x splits the partial arrays hold, in units of 64
};

__host__ __device__ inline uint32_t ceil_div(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

// Rows of one split in the partial arrays.
__host__ __device__ inline int32_t partial_stride(int32_t rows) { return (rows + 63) & ~63; }

// Row tiles scheduled side by side: the workgroups behind one L2 share the LM-head tiles of that many, and the hidden
// tiles of as many splits as are left of them.  Eight tiles of 256 rows (8 x 4 of the 32 workgroups; the plan's tile_panel
// if that is less), sixteen of the narrow ones, whose traffic is nearly all LM head; evenly deep panels, since a lone row
// tile streams the whole LM head once more (280 rows as 8 + 1 tiles of 32: 861 us, as 9: 595 us; 6672 rows as 8 + 8 + 8 + 3
// tiles of 256: 4545 us, as 7 + 7 + 7 + 6: 4519).
__host__ __device__ inline uint32_t panel_depth(uint32_t row_tiles, uint32_t width, uint32_t widest = 8) {
  const uint32_t side = width <= 4 ? 16 : width <= 7 || widest > 8 ? 8 : widest;
  return ceil_div(row_tiles, ceil_div(row_tiles, side));
}

// Workgroups are dealt to the 8 XCDs round-robin by id, and the workgroups of one XCD share an L2.  This maps
// workgroup b of a grid of G to a position such that each XCD's workgroups hold one contiguous range of positions
// (XCD x owns ceil((G - x) / 8) of them), so that consecutive work units -- which share LM-head and hidden tiles --
// meet in one L2.  A bijection on [0, G) for any G.
__host__ __device__ inline int xcd_contiguous_position(int b, int G) {
  const int x = b & 7;
  int first = 0;
  for (int y = 0; y < x; ++y) first += (G - y + 7) >> 3;
  return first + (b >> 3);
}

// The unit with which workgroup b of the grid begins (`units`: it has none).  A grid of more workgroups than units leaves
// the last ones idle, a few on every XCD: the positions are those of the workgroups that work.  With the whole grid's
// positions the units sat on the first XCDs (32 of 256 rows found, 32000 x 1024: 125 units of 256 workgroups on four of them
// 32.7 us, on all 25.6; 152064 x 3584, 198 units: 72 rows 202 -> 189, 100 rows 208 -> 200).
__host__ __device__ inline int first_unit(int b, int grid, int units) {
  const int working = grid < units ? grid : units;
  return b < working ? xcd_contiguous_position(b, working) : units;
}

// What a unit's parts take, in units of 10 ns, fitted to measurements at widths 1..8 and 32..4096 rows of a 126464 x 4096
// and a 32000 x 1024 LM head (most within 10%).  A K-tile: bound by the copies into LDS up to four token blocks a wave
// (0.64 to 0.76 us), by the matrix cores beyond (1.26 us at eight); or by memory, which brings the 32 KiB of LM head
// for all compute units in 1.48 us, shared by the panel's row tiles; the shorter of the two hides but for a sixth.  A lone
// row tile's workgroups all wait for bytes of their own: 1.26 us for 256 of them and less for fewer, down to what one can
// have under way (594 vocabulary tiles, 100 rows: 198 workgroups on three tiles each 200 us, two row tiles in 119 splits
// of five, which 1.48 us a K-tile for any number of workgroups preferred, 257; 240 rows 249 against 299; over 176 steps of
// up to 256 rows of eight LM heads, greedy and drawn, the choice is 0.8% off the best width, over the 22 of 594 tiles it is
// the best).  The reduction of a tile: 0.56 us per token block, with a draw 1.66 us and, in a unit's first tiles, where
// nothing bounds the scores yet, 2.5 us more (1.9 where a lone row tile waits for memory meanwhile), fitted at temperature
// 0.7 (2700 rows of 32000 x 1024 take 280 us at 0.3, 257 at 0.7, 245 at 1.0): 6000 rows of 65536 x 2048 1545 us as two rounds
// of short units of 256 rows, 1335 as one round, which it now takes; 2700 rows of 32000 x 1024 287 -> 261; over 157 sizes of
// 33 to 9000 rows the choice is 0.9% off the best width at each of the three temperatures, without that term 1.8% at 0.7.
// A further round of units (pipeline fill, merge): half a tile and 4 us.  With the K-loop in pair order the wide tiles are
// 5% faster throughout; at 21 row counts from 280 to 3500 of 126464 x 4096 no other width beats the one this picks by more
// than 1.4%.
__host__ __device__ inline uint32_t k_tile_time(uint32_t width, uint32_t share, uint32_t workgroups) {
  const uint32_t compute = width <= 4 ? 60 + 4 * width : (36 + 27 * width) / 2;
  const uint32_t alone = workgroups < 128 ? 62 : workgroups * 126 / 256, memory = share == 1 ? alone : 148 / share;
  return compute > memory ? compute + memory / 6 : memory + compute / 6;
}
__host__ __device__ inline uint32_t reduction_time(uint32_t width, uint32_t sampling) {
  return (sampling != 0 ? 166 : 56) * width;
}

// The candidate with row tiles of 32*width rows that uses `extra_rounds` rounds of the grid more than the fewest
// possible, as (cost, width, splits) packed into one integer: the smaller one is the better one.  A round lasts as
// long as its longest unit; of the split counts that fit the same rounds the largest has the shortest units, and of
// those with equally long units the smallest makes the fewest partial results.  At least four splits where vocabulary
// and memory allow: the 32 workgroups that share an L2 then work on 8 row tiles x 4 splits (256 row tiles in one
// split each: 62 ms; in four: 47 ms).
constexpr uint32_t kScheduleRounds = 32;       // candidates per width: the rounds' quantisation is below 3% beyond
constexpr int32_t kNarrowRows = 1 << 20;       // beyond, the widest tile always pays (and 32 bits hold its units)
struct SplitRange {
  uint32_t row_tiles, least, most;   // splits on offer (most = 0: the width is not)
  uint32_t first;                    // the fewest rounds
};
__host__ __device__ inline SplitRange split_range(const ScheduleInput& in, int32_t rows, uint32_t width) {
  SplitRange range{0, 0, 0, 0};
  if ((in.widths >> (width - 1) & 1) == 0 || (width < 8 && rows > kNarrowRows)) return range;
  // 32-bit throughout (rows < 2^31, so at most 2^23 row tiles and 2^31 units): a wide division costs the device 10x
  range.row_tiles = ceil_div((uint32_t)rows, 32 * width);
  const uint32_t fit = in.slots64 / ((uint32_t)partial_stride(rows) >> 6);
  range.most = in.vocab_tiles < MOSAIC_MAX_VOCAB_SPLITS ? in.vocab_tiles : MOSAIC_MAX_VOCAB_SPLITS;
  if (fit < range.most + in.extra) range.most = fit <= in.extra + 1 ? 1 : fit - in.extra;
  range.least = range.most < 4 ? range.most : 4;
  range.first = ceil_div(range.row_tiles * range.least, in.grid);
  return range;
}
__host__ __device__ inline uint32_t splits_in(const ScheduleInput& in, const SplitRange& range, uint32_t extra_rounds) {
  return (range.first + extra_rounds) * in.grid / range.row_tiles;   // (may be more than `most`)
}
__host__ __device__ inline uint64_t schedule_candidate(const ScheduleInput& in, const SplitRange& range, uint32_t width,
                                                       uint32_t extra_rounds) {
  if (range.most == 0) return ~(uint64_t)0;
  uint32_t s = splits_in(in, range, extra_rounds);
  if (s > range.most) s = range.most;
  const uint32_t longest = ceil_div(in.vocab_tiles, s);
  uint32_t splits = ceil_div(in.vocab_tiles, longest);
  if (splits < range.least) splits = range.least;
  const uint32_t rounds = ceil_div(range.row_tiles * splits, in.grid);
  const uint32_t workgroups = range.row_tiles * splits < in.grid ? range.row_tiles * splits : in.grid;
  const uint32_t tile = in.k_tiles * k_tile_time(width, panel_depth(range.row_tiles, width), workgroups) +
                        reduction_time(width, in.sampling);
  const uint32_t first_tiles = in.sampling == 0 ? 0 : range.row_tiles == 1 ? 187 * width : 250 * width;
  uint64_t cost = (rounds * ((uint64_t)longest * tile + first_tiles) + (uint64_t)(rounds - 1) * (tile / 2 + 400)) >> 3;
  // a narrower tile has to win by more than the model is off (5748 rows of 32000 x 1024: 36 x 7 units of 160 rows 300 us,
  // 23 x 11 of 256 rows 294 us); where drawn the more, the narrower (600 rows of 126464 x 4096: five token blocks 590 us,
  // seven 562, 0.6% apart in the model)
  if (in.sampling != 0) cost += cost * (8 - width) >> 8;
  else if (width < 8) cost += cost >> 6;
  return cost << 20 | (uint64_t)(8 - width) << 16 | splits;
}

__host__ __device__ inline Schedule schedule_of(int32_t rows, uint64_t best) {
  const int32_t width = 8 - (int32_t)(best >> 16 & 15);
  return Schedule{width, (int32_t)ceil_div((uint32_t)rows, 32 * (uint32_t)width), (int32_t)(best & 0xffff),
                  partial_stride(rows)};
}

// Whether the units of a draw share the best scores of their rows (shared bounds, mosaic_logits.hip).  A unit of one tile has
// nothing to take over.  One of two does at row tiles of 64 rows and more (40 rows of 126464 x 4096 177.1 -> 174.1 us, 1000
// rows of 8192 x 512 33.9 -> 31.5), at 32 rows it gains less than the runs differ (20 rows of 126464 x 4096 169.7 -> 168.6);
// three tiles of 32 rows gain (32 rows of 152064 x 3584 181.8 -> 180.5).
constexpr int32_t kShareAtTwo = 2;   // widths from which on units of two tiles share, too
__host__ __device__ inline bool units_share(uint32_t vocab_tiles, int32_t width, int32_t splits) {
  return vocab_tiles > (width < kShareAtTwo ? 2u : 1u) * (uint32_t)splits;
}

// The splits that a launch says it settled on, for the launches behind it.  The word lies in the caller's workspace (or in
// the library's one array per GPU, which calls share): whatever another call leaves there, nobody is to be led beyond
// the partial arrays by it.
__host__ __device__ inline int32_t held_splits(const ScheduleInput& in, int32_t rows, int32_t found) {
  const uint32_t column = (uint32_t)partial_stride(rows) >> 6;
  return found >= 1 && ((uint64_t)(uint32_t)found + in.extra) * column <= in.slots64 ? found : 1;
}

// On the host: for the bound the plan was made for, handed to the kernels so that they need not search when the
// count turns out to be that bound.  A width whose most splits fit one round has one candidate (all of the smallest
// steps, whose host side this is a part of: 256 candidates took 2.5 us).
inline Schedule choose_schedule(const ScheduleInput& in, int32_t rows) {
  uint64_t best = ~(uint64_t)0;
  for (uint32_t w = 1; w <= 8; ++w) {
    const SplitRange range = split_range(in, rows, w);
    for (uint32_t r = 0; r < kScheduleRounds; ++r) {
      const uint64_t c = schedule_candidate(in, range, w, r);
      best = c < best ? c : best;
      if (range.most == 0 || splits_in(in, range, r) >= range.most) break;   // further rounds change nothing
    }
  }
  return schedule_of(rows, best);
}

// On the device: eight lanes per width, the same result in every wave (1.8 us where it runs cold, in a launch of few tiles;
// 2.3 with all rounds searched).
__device__ __forceinline__ Schedule choose_schedule_wave(const ScheduleInput& in, int32_t rows) {
  const uint32_t lane = threadIdx.x & 63;
  const SplitRange range = split_range(in, rows, 1 + (lane >> 3));
  uint64_t best = ~(uint64_t)0;
  for (uint32_t r = lane & 7; r < kScheduleRounds; r += 8) {
    const uint64_t c = schedule_candidate(in, range, 1 + (lane >> 3), r);
    best = c < best ? c : best;
    if (range.most == 0 || splits_in(in, range, r) >= range.most) break;   // as on the host
  }
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) {
    const uint64_t other = __shfl_xor((unsigned long long)best, x, 64);
    best = other < best ? other : best;
  }
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)best);   // width and splits sit there
  return schedule_of(rows, lo);
}

}  // namespace mosaic
#endif
