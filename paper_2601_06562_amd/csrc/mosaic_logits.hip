// Fused gather-GEMM + vocabulary reduction for mask-only logits on gfx950 (MI355X).
//
// Paper section 4.2 describes a gather-GEMM: the kernel gets the hidden states of all positions
// plus the indices of the masked ones, computes row addresses by pointer arithmetic, stages the
// scattered rows in on-chip memory, multiplies, accumulates, and discards each tile -- no gathered
// copy in global memory.  This kernel keeps that idea (the gather is folded into the global->LDS
// copy, one address per lane) and, unlike the paper's kernel, never writes logits either: every
// 256x256 tile of logits lives only in MFMA accumulators and is reduced on the spot to a running
// (max, sum-exp, arg-max) per token row.
//
// Shape of the computation.  The MFMA "A" operand is the LM-head tile (vocabulary ids along the
// instruction's rows), "B" is the gathered hidden tile (token rows along the instruction's columns).
// A lane then owns ONE token per accumulator block (column lane%16 with v_mfma_f32_16x16x32_bf16 in the
// 4-wave kernel, lane%32 with v_mfma_f32_32x32x16_bf16 in the general one) and several vocabulary ids,
// so the reduction over the vocabulary is almost entirely in-register; the cross-lane steps and the
// cross-wave step happen once per work unit, not per tile.
//
// Work decomposition.  A unit is (row tile of 256 masked tokens, vocabulary split); a workgroup (4 waves
// in the hand-scheduled kernel, 8 in the general one) walks the 256-wide vocabulary tiles of its split,
// folding each finished tile into a running triple in registers, and writes one partial triple per row at the
// end.  A second tiny kernel merges the S partials per row and emits token, confidence and log-sum-exp.  How many
// splits there are is decided on the device from the rows found (mosaic_schedule.h); the fold makes the results
// independent of it.
//
// Sampling.  The SAMPLE instantiations of both kernels draw the token by the Gumbel-max form of categorical
// sampling at temperature tau (paper section 2.1 leaves the sampler open): arg-max of x + tau*g with g from a
// Philox4x32-10 stream keyed by (seed, position, vocabulary id), next to the unperturbed max / sum-exp.
//
// Data movement.  Global->LDS copies use the direct-to-LDS 16-byte loads of gfx950; both tiles are
// K-contiguous ([256 rows][64 k] bf16 = 128 B per row, i.e. whole 128-byte lines per request) and
// 16-byte chunks are XOR-swizzled by row so that the ds_read_b128 operand fetches of 32 consecutive
// rows spread over all LDS banks.  Each operand has its own ring of 32 KiB slots: three for the LM-head
// tiles (two K-tiles ahead), two for the hidden tiles (one ahead) -- 160 KiB, all of a CU's LDS; the
// merge scratch aliases slot 0 at the end of a unit.  One workgroup barrier per K-tile.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>
#include <stdlib.h>

#include "mosaic_internal.h"
#include "mosaic_schedule.h"

namespace mosaic {

using bf16x8 = __attribute__((ext_vector_type(8))) __bf16;
using f32x16 = __attribute__((ext_vector_type(16))) float;
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gbl_ptr_t;

constexpr int kTileRows = MOSAIC_ROW_TILE;     // masked tokens per tile (MFMA N side)
constexpr int kTileVocab = MOSAIC_VOCAB_TILE;  // vocabulary ids per tile (MFMA M side)
constexpr int kThreads = 512;                  // 8 waves: 2 (vocabulary halves) x 4 (token quarters)
// "Minus infinity" that survives subtraction.  A power of two: its product with log2 e is then exact, so that a lane
// whose ids all lie past the vocabulary holds a plain finite sum relative to it, which every merge scales to zero.
constexpr float kNeg = -0x1p100f;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct KernelParams {
  const char* hidden;
  int64_t ldh_bytes;
  const char* w;
  int32_t d;
  int32_t V;
  const int32_t* idx;        // hidden row to read, per masked row
  const int32_t* noise_idx;  // sampling: the position that keys the row's noise (idx unless the gather is shifted)
  const int32_t* count;
  int32_t T;           // rows of hidden: gather entries are clamped to [0, T)
  int32_t row0;        // first compacted row of this chunk
  int32_t chunk_rows;  // capacity of the chunk (C)
  int32_t max_rows;
  int32_t panel;       // row tiles scheduled side by side
  int32_t stream_w;    // the LM head is larger than kStreamBytes
  ScheduleInput sched; // what the division of the work is made from (of a pair of launches: the first one's)
  Schedule bound;      // ... and the division for bound_rows rows
  int32_t bound_rows;
  int32_t ragged_tile; // second launch of a pair: it covers this vocabulary tile alone, behind the other splits; else -1
  int32_t id_bits;     // bits of V, which a vocabulary id has in a packed partial
  float* part_m;       // largest logit per row and split
  uint64_t* part_si;   // the sum of exponentials and the id (pack_sum_id)
  int32_t* out_token;
  float* out_conf;
  float* out_lse;
  // sampling with temperature (tau > 0): two more partial planes and the generator key
  float tau;
  uint32_t seed_lo, seed_hi;
  float* part_ym;   // best perturbed score x + tau*g (the id in part_si is then this score's)
  float* part_xa;   // the unperturbed logit at that arg-max
  int32_t* sync;    // round counters of the persistent grid (cleared before the launch), sync_slots of them
  int32_t sync_slots;
  int32_t* found_splits;   // the splits of the division a launch found, for a pair's second one and the merge kernel
  // Hidden tensors of 4 GiB or more.  The 4-wave kernel addresses the rows a wave copies (8 times the width) by 32-bit
  // offsets from the lowest of them, which works unless those rows lie 4 GiB or more apart; a small kernel looks for such
  // a group in the list and raises *wide_flag, and of the two launches that follow (4-wave kernel, general kernel) the one
  // whose wide_run_if differs from the flag returns at once.  nullptr: no such check (the launch always runs).
  const int32_t* wide_flag;
  int32_t wide_run_if;
};

// Fold.  The running state of a row is (m, s, i): the largest logit, the sum of exponentials, and the lowest id that
// attains m.  s is kept relative to 2^E, E = ceil(m log2 e), in double precision: a change of m only ever scales s by
// an exact power of two, and what a tile adds depends on the tile alone.  Any order and any grouping of the tiles
// then gives the same sum to ~2^-50 within a unit, and a unit's sum is rounded once more, to the 58 - id_bits mantissa
// bits of its packed partial (2^-42 for 126464 ids).  So the outputs, rounded to fp32, are those of one pass over the
// vocabulary however it was split, but for the last bit of a row whose sum lies that close to a rounding boundary (of
// random rows 0.7 in a million at 126464 ids, 7 at 2^20), and the division of the work is free to follow the number of
// rows.  A scale factor exp(m - m') rounded in fp32 at each step, as the state once had, makes the last bits follow the
// split count everywhere.
__device__ __forceinline__ float ref_exponent(float m) { return __builtin_ceilf(m * kLog2e); }
__device__ __forceinline__ int scale_steps(float d) { return (int)fmaxf(d, -2000.f); }   // 2^-2000 is 0 either way

// One tile's triple (s relative to exp(m), fp32) as a folded sum, relative to 2^ref_exponent(m).
__device__ __forceinline__ double tile_sum(float m, float s) {
  return (double)(s * __builtin_amdgcn_exp2f(__builtin_fmaf(m, kLog2e, -ref_exponent(m))));
}

// Folded sums added; m becomes the larger maximum.
__device__ __forceinline__ void merge_sum(float& m, double& s, float m2, double s2) {
  const float e = ref_exponent(m), e2 = ref_exponent(m2), en = fmaxf(e, e2);
  s = __builtin_ldexp(s, scale_steps(e - en)) + __builtin_ldexp(s2, scale_steps(e2 - en));
  m = fmaxf(m, m2);
}
__device__ __forceinline__ void merge_triple(float& m, double& s, int& i, float m2, double s2, int i2) {
  const bool keep = (m > m2) || (m == m2 && i < i2);
  i = keep ? i : i2;
  merge_sum(m, s, m2, s2);
}

// A partial result is 12 bytes: m, and one 64-bit word with the id in its low id_bits bits and above them s as a
// floating-point number of 6 exponent bits (s lies between 1/2 and the number of ids) and the remaining
// 58 - id_bits mantissa bits (41 for 126464 ids), rounded to nearest.  0 stands for an empty sum, the largest exponent
// for one that is not a number (a NaN or an infinity among the logits); logits so large that the rounding of m log2 e
// moves s out of those bounds (10^8 and more) have s clamped.  id_bits hold the number of ids, so that all ones are no
// id: they stand for INT_MAX, the id of a state that no logit has entered.
constexpr int kSumBias = 1019;   // exponent field of a double that is stored as 0
constexpr int kNoSum = 63;       // stored exponent of a sum that is not a number
__device__ __forceinline__ uint64_t pack_sum_id(double s, int i, int id_bits) {
  const int drop = id_bits > 6 ? id_bits - 6 : 0;       // mantissa bits of the double that do not fit
  uint64_t b = (uint64_t)__double_as_longlong(__builtin_fmin(__builtin_fmax(s, 0x1p-3), 0x1p57));
  if (drop > 0) b += (uint64_t)1 << (drop - 1);
  b = (b >> drop) - ((uint64_t)kSumBias << (52 - drop));
  if (!(s > 0.0)) b = s == 0.0 ? 0 : ~(uint64_t)0;
  return b << id_bits | ((uint64_t)(uint32_t)i & (((uint64_t)1 << id_bits) - 1));
}
__device__ __forceinline__ void unpack_sum_id(uint64_t w, int id_bits, double& s, int& i) {
  const int drop = id_bits > 6 ? id_bits - 6 : 0;
  const uint64_t no_id = ((uint64_t)1 << id_bits) - 1, b = w >> id_bits;
  i = (w & no_id) == no_id ? INT_MAX : (int)(w & no_id);
  s = b == 0 ? 0.0 : __longlong_as_double((long long)((b + ((uint64_t)kSumBias << (52 - drop))) << drop));
  if (b >> (52 - drop) >= kNoSum) s = __builtin_nan("");
}

// Sampled candidate: best perturbed score, the plain logit there, its id (lowest id on equal scores).
__device__ __forceinline__ void merge_pick(float& ym, float& xa, int& i, float ym2, float xa2, int i2) {
  const bool keep = (ym > ym2) || (ym == ym2 && i < i2);
  ym = keep ? ym : ym2;
  xa = keep ? xa : xa2;
  i = keep ? i : i2;
}

// tau * Gumbel noise for the four vocabulary ids 4*v4 .. 4*v4+3 of one position.  Philox4x32-10 (Salmon et
// al., SC'11), key = seed, counter = (v4, position, 0, 0); word j -> u = ((word >> 9) + 1/2) * 2^-23 (exact in
// fp32, never 0 or 1); g = -ln(-ln u).  Near u = 1 the inner logarithm comes from the series of -ln(1 - e)
// (e = 1 - u is exact too), where the hardware log2 loses relative accuracy.
__device__ __forceinline__ void gumbel4(uint32_t k0, uint32_t k1, uint32_t pos, uint32_t v4, float tau, float (&n)[4]) {
  uint32_t c0 = v4, c1 = pos, c2 = 0u, c3 = 0u;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    if (round > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  const uint32_t w[4] = {c0, c1, c2, c3};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t k = w[j] >> 9;
    const float u = ((float)k + 0.5f) * 0x1p-23f;
    const float e = ((float)(8388607u - k) + 0.5f) * 0x1p-23f;   // 1 - u
    const float by_log = -__builtin_amdgcn_logf(u) * kLn2;
    const float by_series = e * (1.0f + e * (0.5f + e * (1.0f / 3.0f)));
    const float inner = (e < 0x1p-8f) ? by_series : by_log;       // -ln u  > 0
    n[j] = -__builtin_amdgcn_logf(inner) * kLn2 * tau;
  }
}

// Shared bounds of a draw.  A score that any unit has reached for a row bounds what can still win it, and the units of a
// row (its vocabulary splits, and the two halves of a tile) run side by side, so they publish their rows' best scores and
// take the others' into their own running best.  The exact path, which ids that the bound lets pass go through, was more
// than half of what the draw costs (a timing variant that never takes it: 4096 rows of 126464 x 4096 2786 -> 2644 us, 280
// rows 347 -> 307).  Without sharing and with it, temperature 0.7: 280 rows 331 -> 309 us, 205 rows 253 -> 241, 1004 rows
// 835 -> 777, 4096 rows at temperature 1 2938 -> 2836; 6554 rows of 152064 x 3584 5298 -> 5039; 500 and 2700 rows of 65536 x
// 2048 162 -> 144 and 701 -> 601; 900 and 16000 rows of 32000 x 1024 106 -> 88 and 1139 -> 997; 1000 and 9000 rows of 8192 x
// 512 33.9 -> 31.5 and 174 -> 143.  What is left is mostly the units' first tiles.  The scores are taken over between a
// tile's products and its draw, so that a unit's second tile finds what the first ones of all units reached; ahead of the
// products all are still at it (units of two tiles: 205 rows 246 -> 236 us by the later point, 500 rows of 65536 x 2048 160 -> 148).
// Which units share follows from the division found (units_share, mosaic_schedule.h).
//
// The bounds lie in out_conf, which holds nothing else until the merge writes it.  Every unit clears the words of its rows
// itself, at its start, and each lane reads only words that it has stored to (but for lanes that pad a row tile, whose draw
// nobody sees): what it finds there was written by this launch.  So the store need be seen by no other (at the scope of the
// workgroup it stays behind the XCD's own L2; through to memory, where all units of a row queue for the same lines, 500 rows
// of 65536 x 2048 take 146 us instead of 141, 8 rows of 152064 x 3584, 198 units on one line, 185 instead of 175), and a unit
// that starts late and wipes what others have published costs them a bound and no result.  A launch ahead of the pass that
// cleared the rows cost every draw whose bound has units that share 2 us, also where the units found do not: 16 rows of
// 32000 x 1024 under a bound of 512 27.0 -> 29.0 us, of 8192 x 512 under 4096 19.1 -> 21.0 (without it 26.4 and 18.5).
// What is taken over is a float below (two steps: one below +0 is -0, its equal): an id of another unit with the very same
// score still counts, and the merge then finds the lowest of them as it does without.  The lane's id and logit stay those of
// its own best, which no longer matters: the unit that published the score holds it, or a better one, in its partial result.
// The words are integers in the scores' order (score_order).  As the scores' own bits, which are in order from 0 on up only,
// they left rows whose best score is below zero unshared, at the cost of the exchange: with all logits 300 lower 32 rows of
// 152064 x 3584 take 183.3 us so, 182.0 without any sharing, 180.1 in this order; 280 rows 319 -> 299; 900 rows of 32000 x 1024 103 -> 84.
// (Taking over is the sampling statements' own: take_published in gen_w4_loop.py.)

// Largest of a token's four lanes (l, l ^ 16, l ^ 32, l ^ 48).
__device__ __forceinline__ float token_max(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Rows of this launch's chunk, and the division of the work for them.
__device__ __forceinline__ int chunk_rows_found(const KernelParams& p) {
  int total = *p.count;
  if (total > p.max_rows) total = p.max_rows;
  const int rows = total - p.row0;
  return rows > p.chunk_rows ? p.chunk_rows : rows;
}
__device__ __forceinline__ Schedule launch_schedule(const KernelParams& p, int rows) {
  const Schedule sched = rows == p.bound_rows ? p.bound : choose_schedule_wave(p.sched, rows);
  if (blockIdx.x == 0 && threadIdx.x == 0) *p.found_splits = sched.splits;
  return sched;
}

// The second launch of a pair stores behind the splits of the launch that ran before it, whichever of two that was:
// its division is that launch's word, not a choice of its own (the 4-wave kernel and the general kernel in its place
// settle on different counts, 40 and 49 splits for 769 rows of 50257 ids).
__device__ __forceinline__ Schedule division_found(const KernelParams& p, int rows) {
  return Schedule{8, (rows + kTileRows - 1) / kTileRows, held_splits(p.sched, rows, *p.found_splits), partial_stride(rows)};
}

__device__ __forceinline__ int choose_width(const KernelParams& p, int rows) {
  return rows == p.bound_rows ? p.bound.width : choose_schedule_wave(p.sched, rows).width;
}

// Round alignment of the persistent grid.  A workgroup that takes more than one unit meets the others before each
// further one: the workgroups behind one L2 share LM-head and hidden tiles only while they walk their units in
// step, and once they have drifted apart (units end at slightly different times) every tile is fetched several
// times over; measured on 229 row tiles x 19 splits, 17 rounds: 43.6 ms without, 41.5 ms with the meeting.  It is a
// hint, not a synchronisation anything depends on: the wait is bounded (a workgroup that is not resident, or a
// counter that was never cleared, costs time, never a hang and never a wrong result), and rounds beyond the
// counters provided simply do not meet.
constexpr int kRoundSpins = 256;
__device__ __forceinline__ void meet_before_round(const KernelParams& p, int round, int n_units, int G, int tid) {
  if (p.sync != nullptr && round < p.sync_slots) {
    if (tid == 0) {
      const int left = n_units - G * round;
      const int expect = left > G ? G : left;            // workgroups that have a unit in this round
      int* ctr = p.sync + round;
      __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int spin = 0; spin < kRoundSpins; ++spin) {
        if (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= expect) break;
        __builtin_amdgcn_s_sleep(2);
      }
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void clear_round_counters_kernel(int32_t* sync, int n) {
  if ((int)threadIdx.x < n) sync[threadIdx.x] = 0;
}

// For hidden tensors of 4 GiB or more: raises *flag when some group of consecutive rows of the chunk's list that one
// wave of the 4-wave kernel copies (8 times the width found; the last group padded with the last row as that kernel
// does) spans rows whose byte offsets differ by 4 GiB or more.  One wave per group.
__device__ __forceinline__ bool group_spans_4gib(const KernelParams& p, int rows, int group, int group_rows) {
  const int lane = (int)threadIdx.x & 63;
  int j = group * group_rows + (lane < group_rows ? lane : group_rows - 1);
  if (j > rows - 1) j = rows - 1;
  int t = p.idx[p.row0 + j];
  t = t < 0 ? 0 : (t > p.T - 1 ? p.T - 1 : t);
  int lo = t, hi = t;
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) {
    const int a = __shfl_xor(lo, x, 64), b = __shfl_xor(hi, x, 64);
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
  }
  // the offset of a row from the group's lowest, plus the 16-byte chunk inside the row's K-tile, must fit 32 bits
  return (uint64_t)(hi - lo) * (uint64_t)p.ldh_bytes >= ((uint64_t)1 << 32) - 256;
}
__global__ __launch_bounds__(256) void span_check_kernel(const KernelParams p, int32_t* flag) {
  const int rows = chunk_rows_found(p);
  if (rows <= 0) return;
  const int group_rows = 8 * choose_width(p, rows);
  for (int group = (int)blockIdx.x * 4 + ((int)threadIdx.x >> 6); group * group_rows < rows; group += (int)gridDim.x * 4)
    if (group_spans_4gib(p, rows, group, group_rows) && ((int)threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

// Few rows: one block clears the round counters and checks the list, a launch (~5 us) less than the two kernels above.
constexpr int64_t kOneBlockCheckRows = 4096;   // at most four groups a wave
__global__ __launch_bounds__(1024) void clear_and_check_kernel(const KernelParams p, int32_t* counters, int n, int32_t* flag) {
  if ((int)threadIdx.x < n) counters[threadIdx.x] = 0;
  const int rows = chunk_rows_found(p);
  bool far = false;
  if (rows > 0) {
    const int group_rows = 8 * choose_width(p, rows);
    for (int group = (int)threadIdx.x >> 6; group * group_rows < rows; group += 16)
      far |= group_spans_4gib(p, rows, group, group_rows);
  }
  const int any = __syncthreads_or(far);
  if (threadIdx.x == 0) *flag = any ? 1 : 0;
}

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// exp(x - mn) as exp2.  Full tiles fold the subtraction into one fma against nml = -mn*log2(e).  Tail
// tiles hold the kNeg sentinel, whose magnitude would turn the rounding of nml into a huge exponent, so
// they subtract first (exact zero when x == mn).
template <bool TAIL>
__device__ __forceinline__ float exp_rel(float x, float mn, float nml) {
  if constexpr (TAIL) return __builtin_amdgcn_exp2f((x - mn) * kLog2e);
  else return __builtin_amdgcn_exp2f(__builtin_fmaf(x, kLog2e, nml));
}

// Reduce one finished 256x256 logits tile (this wave's 128 vocabulary ids x 64 tokens) into the
// lane's triples of the tile.  vb = vocabulary id of this lane's element (block 0, register 0).
template <bool TAIL>
__device__ __forceinline__ void reduce_tile(f32x16 (&acc)[4][2], float (&m)[2], float (&s)[2], int (&ix)[2], int vb,
                                            int V) {
#pragma unroll
  for (int bj = 0; bj < 2; ++bj) {
    float mt = kNeg;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int code = bi * 32 + 8 * (r >> 2) + (r & 3);
        if (TAIL) {
          if (vb + code >= V) acc[bi][bj][r] = kNeg;
        }
        mt = fmaxf(mt, acc[bi][bj][r]);
      }
    }
    int sel = 0;
#pragma unroll
    for (int bi = 3; bi >= 0; --bi) {
#pragma unroll
      for (int r = 15; r >= 0; --r) {
        const int code = bi * 32 + 8 * (r >> 2) + (r & 3);
        sel = (acc[bi][bj][r] == mt) ? code : sel;  // descending scan: the lowest id wins
      }
    }
    const bool upd = mt > m[bj];  // strict: an equal maximum in a later tile has a higher id
    ix[bj] = upd ? vb + sel : ix[bj];
    const float mn = fmaxf(m[bj], mt);
    const float nml = -mn * kLog2e;
    float p0 = 0.f, p1 = 0.f, p2 = 0.f, p3 = 0.f;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi) {
#pragma unroll
      for (int r = 0; r < 16; r += 4) {
        p0 += exp_rel<TAIL>(acc[bi][bj][r + 0], mn, nml);
        p1 += exp_rel<TAIL>(acc[bi][bj][r + 1], mn, nml);
        p2 += exp_rel<TAIL>(acc[bi][bj][r + 2], mn, nml);
        p3 += exp_rel<TAIL>(acc[bi][bj][r + 3], mn, nml);
      }
    }
    s[bj] = s[bj] * __builtin_amdgcn_exp2f((m[bj] - mn) * kLog2e) + ((p0 + p1) + (p2 + p3));
    m[bj] = mn;
  }
}

// Separate rings for the two operands: NW slots of W K-tiles, NH slots of H K-tiles (32 KiB each).
// The shallow ring runs one K-tile ahead, the deep one two; the shallow operand is issued first in
// every iteration so that the in-order vmcnt wait can leave the deep ring's newest tile in flight.
// Same tile under sampling: also tracks the arg-max of x + tau*g and the plain logit there.
template <bool TAIL>
__device__ __forceinline__ void reduce_tile_sample(f32x16 (&acc)[4][2], float (&m)[2], float (&s)[2], float (&ym)[2],
                                                   float (&xa)[2], int (&ix)[2], int vb, int V, const int (&pos)[2],
                                                   uint32_t k0, uint32_t k1, float tau) {
#pragma unroll
  for (int bj = 0; bj < 2; ++bj) {
    float mt = kNeg, yt = kNeg, xsel = 0.f;
    int sel = 0;
#pragma unroll
    for (int bi = 3; bi >= 0; --bi) {
#pragma unroll
      for (int r4 = 3; r4 >= 0; --r4) {
        const int code0 = bi * 32 + 8 * r4;
        float n[4];
        gumbel4(k0, k1, (uint32_t)pos[bj], (uint32_t)(vb + code0) >> 2, tau, n);
#pragma unroll
        for (int r = 3; r >= 0; --r) {
          // ids past the vocabulary: selects, not branches (a branch per element makes the compiler move whole
          // accumulator vectors through scratch)
          const bool past = TAIL && vb + code0 + r >= V;
          const float x = past ? kNeg : acc[bi][bj][4 * r4 + r];
          if (TAIL) acc[bi][bj][4 * r4 + r] = x;
          const float y = past ? kNeg : x + n[r];
          mt = fmaxf(mt, x);
          const bool better = y >= yt;   // descending scan: on equal scores the lower id replaces the higher
          sel = better ? code0 + r : sel;
          xsel = better ? x : xsel;
          yt = better ? y : yt;
        }
      }
    }
    const bool upd = yt > ym[bj];
    ix[bj] = upd ? vb + sel : ix[bj];
    xa[bj] = upd ? xsel : xa[bj];
    ym[bj] = upd ? yt : ym[bj];
    const float mn = fmaxf(m[bj], mt);
    const float nml = -mn * kLog2e;
    float p0 = 0.f, p1 = 0.f, p2 = 0.f, p3 = 0.f;
#pragma unroll
    for (int bi = 0; bi < 4; ++bi) {
#pragma unroll
      for (int r = 0; r < 16; r += 4) {
        p0 += exp_rel<TAIL>(acc[bi][bj][r + 0], mn, nml);
        p1 += exp_rel<TAIL>(acc[bi][bj][r + 1], mn, nml);
        p2 += exp_rel<TAIL>(acc[bi][bj][r + 2], mn, nml);
        p3 += exp_rel<TAIL>(acc[bi][bj][r + 3], mn, nml);
      }
    }
    s[bj] = s[bj] * __builtin_amdgcn_exp2f((m[bj] - mn) * kLog2e) + ((p0 + p1) + (p2 + p3));
    m[bj] = mn;
  }
}

template <int NW, int NH, bool SAMPLE>
__global__ __launch_bounds__(kThreads) void masked_logits_kernel(const KernelParams p) {
  static_assert((NW == 2 || NW == 3) && (NH == 2 || NH == 3) && NW + NH <= 5, "ring shape");
  constexpr int kTileK = 64;
  constexpr int kRowBytes = 128;
  constexpr int kOperandBytes = 256 * kRowBytes;        // 32 KiB
  constexpr int kSwzShift = 1;
  constexpr int kSubSteps = 4;
  constexpr int kDW = NW - 1, kDH = NH - 1;             // prefetch distance in K-tiles
  constexpr int kRing = (NW + NH) * kOperandBytes;
  constexpr int kLds = (NW + NH == 5) ? kRing : kRing + 6 * 256 * 4;
  constexpr int kRedOff = (NW + NH == 5) ? 0 : kRing;   // 5 slots fill the LDS: merge scratch aliases slot 0
  __shared__ __attribute__((aligned(1024))) char smem[kLds];
  double* red_s = reinterpret_cast<double*>(smem + kRedOff);
  float* red_m = reinterpret_cast<float*>(red_s + 256);
  int* red_i = reinterpret_cast<int*>(red_m + 256);
  float* red_ym = reinterpret_cast<float*>(red_i + 256);   // sampling only
  float* red_xa = red_ym + 256;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wv = wave & 1;   // vocabulary half of the tile
  const int wt = wave >> 1;  // token quarter of the tile
  const int l32 = lane & 31, lhalf = lane >> 5;

  if (p.wide_flag != nullptr && *p.wide_flag != p.wide_run_if) return;   // the other kernel of the two serves this list
  const int rows = chunk_rows_found(p);
  if (rows <= 0) return;
  const bool ragged_only = p.ragged_tile >= 0;
  const Schedule sched = ragged_only ? division_found(p, rows) : launch_schedule(p, rows);
  const int n_tt = (rows + kTileRows - 1) / kTileRows;   // its row tiles have the one width

  const int G = gridDim.x;
  const int S = ragged_only ? 1 : sched.splits;
  const int n_units = n_tt * S;
  const int pos = first_unit((int)blockIdx.x, G, n_units);
  const int A = p.panel < n_tt ? p.panel : n_tt;
  const int full_panel_units = A * S;
  const int n_panels = (n_tt + A - 1) / A;

  const int drow = wave * 32 + (lane >> 3);
  int src_chunk_bytes[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) src_chunk_bytes[i] = (((lane & 7) ^ (((drow + 8 * i) >> kSwzShift) & 7))) * 16;
  int rd_off[kSubSteps];
#pragma unroll
  for (int ks = 0; ks < kSubSteps; ++ks) rd_off[ks] = l32 * kRowBytes + (((2 * ks + lhalf) ^ ((l32 >> kSwzShift) & 7)) * 16);

  const int nk = p.d / kTileK;

  for (int u = pos, round = 0; u < n_units; u += G, ++round) {
    if (round > 0) meet_before_round(p, round, n_units, G, tid);
    int pnl = u / full_panel_units;
    if (pnl >= n_panels) pnl = n_panels - 1;
    const int ul = u - pnl * full_panel_units;
    const int hp = (n_tt - pnl * A) < A ? (n_tt - pnl * A) : A;
    const int sp = ul / hp;
    const int tt = pnl * A + ul % hp;
    const int vt0 = ragged_only ? p.ragged_tile : (int)(((int64_t)sp * p.sched.vocab_tiles) / S);
    const int vt1 = ragged_only ? p.ragged_tile + 1 : (int)(((int64_t)(sp + 1) * p.sched.vocab_tiles) / S);
    const int ntile = vt1 - vt0;
    const int total_steps = ntile * nk;

    const char* hptr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int j = tt * kTileRows + drow + 8 * i;
      if (j > rows - 1) j = rows - 1;
      int t = p.idx[p.row0 + j];
      t = t < 0 ? 0 : (t > p.T - 1 ? p.T - 1 : t);   // a bad entry of a caller-built list reads a valid row
      hptr[i] = p.hidden + (int64_t)t * p.ldh_bytes + src_chunk_bytes[i];
    }
    const char* wptr[4];

    // W loader: global step w_g = (vocab tile, k); slot w_g % NW.
    int w_g = 0, w_vt = vt0, w_k = 0, w_slot = 0;
    auto issue_w = [&]() {
      if (__builtin_expect(w_k == 0, 0)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          int v = w_vt * kTileVocab + drow + 8 * i;
          if (v > p.V - 1) v = p.V - 1;
          wptr[i] = p.w + (int64_t)v * ((int64_t)p.d * 2) + src_chunk_bytes[i];
        }
      }
      char* dst = smem + w_slot * kOperandBytes + (wave * 32) * kRowBytes;
      const int koff = w_k * kRowBytes;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_global_load_lds((gbl_ptr_t)(wptr[i] + koff), (lds_ptr_t)(dst + i * 1024), 16, 0, 0);
      w_k += 1;
      if (w_k == nk) { w_k = 0; w_vt += 1; }
      w_slot = (w_slot + 1 == NW) ? 0 : w_slot + 1;
      w_g += 1;
    };
    int h_g = 0, h_k = 0, h_slot = 0;
    auto issue_h = [&]() {
      char* dst = smem + (NW + h_slot) * kOperandBytes + (wave * 32) * kRowBytes;
      const int koff = h_k * kRowBytes;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_global_load_lds((gbl_ptr_t)(hptr[i] + koff), (lds_ptr_t)(dst + i * 1024), 16, 0, 0);
      h_k = (h_k + 1 == nk) ? 0 : h_k + 1;
      h_slot = (h_slot + 1 == NH) ? 0 : h_slot + 1;
      h_g += 1;
    };
    // One scheduling slot: at (virtual) iteration it, bring in W step it+kDW and H step it+kDH,
    // shallow ring first.  The compiler is told that steps copy: taken for rare, a hidden row's pointer went to scratch,
    // and its reload in every step waited for the copies under way (4096 rows greedy 3831 us, with it in registers 3635).
    auto issue_pair = [&](int it) {
      if constexpr (kDW <= kDH) {
        if (__builtin_expect(it + kDW >= 0 && it + kDW < total_steps, 1)) issue_w();
        if (__builtin_expect(it + kDH >= 0 && it + kDH < total_steps, 1)) issue_h();
      } else {
        if (__builtin_expect(it + kDH >= 0 && it + kDH < total_steps, 1)) issue_h();
        if (__builtin_expect(it + kDW >= 0 && it + kDW < total_steps, 1)) issue_w();
      }
    };
    constexpr int kDMax = kDW > kDH ? kDW : kDH;
    constexpr int kDMin = kDW < kDH ? kDW : kDH;

    float run_m[2] = {kNeg, kNeg};
    double run_s[2] = {0.0, 0.0};
    int run_i[2] = {INT_MAX, INT_MAX};
    float run_ym[2] = {kNeg, kNeg};   // sampling: best x + tau*g, the plain logit there
    float run_xa[2] = {0.f, 0.f};
    int pos[2] = {0, 0};              // sampling: the position whose row this lane's column holds
    if constexpr (SAMPLE) {
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        int j = tt * kTileRows + wt * 64 + bj * 32 + l32;
        if (j > rows - 1) j = rows - 1;
        pos[bj] = p.noise_idx[p.row0 + j];
      }
    }

    wait_vm<0>();
#pragma unroll
    for (int it = -kDMax; it < 0; ++it) issue_pair(it);

    int ws = 0, hs = 0, step = 0;
    for (int n = 0; n < ntile; ++n) {
      f32x16 acc[4][2];
#pragma unroll
      for (int bi = 0; bi < 4; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[bi][bj][r] = 0.f;

      for (int kt = 0; kt < nk; ++kt, ++step) {
        // Both operands of `step` must have landed.  The only loads issued after them are the deep
        // ring's tile step+kDMax... (one tile, 4 loads) when the rings differ in depth by one.
        if (kDMax > kDMin && step + kDMax - kDMin < total_steps && kDMin == 1) wait_vm<4>();
        else wait_vm<0>();
        __builtin_amdgcn_s_barrier();
        issue_pair(step);

        const char* wbase = smem + ws * kOperandBytes + (wv * 128) * kRowBytes;
        const char* hbase = smem + (NW + hs) * kOperandBytes + (wt * 64) * kRowBytes;
#pragma unroll
        for (int ks = 0; ks < kSubSteps; ++ks) {
          bf16x8 a[4], b[2];
#pragma unroll
          for (int bi = 0; bi < 4; ++bi) a[bi] = *reinterpret_cast<const bf16x8*>(wbase + bi * 32 * kRowBytes + rd_off[ks]);
#pragma unroll
          for (int bj = 0; bj < 2; ++bj) b[bj] = *reinterpret_cast<const bf16x8*>(hbase + bj * 32 * kRowBytes + rd_off[ks]);
#pragma unroll
          for (int bi = 0; bi < 4; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
              acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[bi], b[bj], acc[bi][bj], 0, 0, 0);
        }
        ws = (ws + 1 == NW) ? 0 : ws + 1;
        hs = (hs + 1 == NH) ? 0 : hs + 1;
      }

      const int v_tile0 = (vt0 + n) * kTileVocab;
      const int vb = v_tile0 + wv * 128 + 4 * lhalf;
      float tile_m[2] = {kNeg, kNeg}, tile_s[2] = {0.f, 0.f};   // this tile's own triple, folded in below
      int tile_i[2] = {INT_MAX, INT_MAX};
      if constexpr (SAMPLE) {
        if (v_tile0 + kTileVocab > p.V)
          reduce_tile_sample<true>(acc, tile_m, tile_s, run_ym, run_xa, run_i, vb, p.V, pos, p.seed_lo, p.seed_hi, p.tau);
        else
          reduce_tile_sample<false>(acc, tile_m, tile_s, run_ym, run_xa, run_i, vb, p.V, pos, p.seed_lo, p.seed_hi, p.tau);
      } else {
        if (v_tile0 + kTileVocab > p.V) reduce_tile<true>(acc, tile_m, tile_s, tile_i, vb, p.V);
        else reduce_tile<false>(acc, tile_m, tile_s, tile_i, vb, p.V);
      }
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        const double ts = tile_sum(tile_m[bj], tile_s[bj]);
        if constexpr (SAMPLE) merge_sum(run_m[bj], run_s[bj], tile_m[bj], ts);
        else merge_triple(run_m[bj], run_s[bj], run_i[bj], tile_m[bj], ts, tile_i[bj]);
      }
    }

#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      const float m2 = __shfl_xor(run_m[bj], 32, 64);
      const double s2 = __shfl_xor(run_s[bj], 32, 64);
      const int i2 = __shfl_xor(run_i[bj], 32, 64);
      if constexpr (SAMPLE) {
        merge_sum(run_m[bj], run_s[bj], m2, s2);
        merge_pick(run_ym[bj], run_xa[bj], run_i[bj], __shfl_xor(run_ym[bj], 32, 64), __shfl_xor(run_xa[bj], 32, 64), i2);
      } else {
        merge_triple(run_m[bj], run_s[bj], run_i[bj], m2, s2, i2);
      }
    }
    __syncthreads();  // every wave is done reading the ring (the merge scratch may alias it)
    if (wv == 1 && lhalf == 0) {
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        const int e = (wt * 2 + bj) * 32 + l32;
        red_m[e] = run_m[bj];
        red_s[e] = run_s[bj];
        red_i[e] = run_i[bj];
        if constexpr (SAMPLE) {
          red_ym[e] = run_ym[bj];
          red_xa[e] = run_xa[bj];
        }
      }
    }
    __syncthreads();
    if (wv == 0 && lhalf == 0) {
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) {
        const int e = (wt * 2 + bj) * 32 + l32;
        if (tt * kTileRows + e >= rows) continue;
        const int64_t slot = (int64_t)(ragged_only ? sched.splits : sp) * sched.stride + tt * kTileRows + e;
        if constexpr (SAMPLE) {
          merge_sum(run_m[bj], run_s[bj], red_m[e], red_s[e]);
          merge_pick(run_ym[bj], run_xa[bj], run_i[bj], red_ym[e], red_xa[e], red_i[e]);
          p.part_ym[slot] = run_ym[bj];
          p.part_xa[slot] = run_xa[bj];
        } else {
          merge_triple(run_m[bj], run_s[bj], run_i[bj], red_m[e], red_s[e], red_i[e]);
        }
        p.part_m[slot] = run_m[bj];
        p.part_si[slot] = pack_sum_id(run_s[bj], run_i[bj], p.id_bits);
      }
    }
    __syncthreads();  // the scratch is read before the next unit's copies may overwrite it
  }
}

// ---- 4-wave fast path: one wave per SIMD, 128 (vocab) x 16*NB (token) per wave as 8 x NB blocks of
// v_mfma_f32_16x16x32_bf16 (the more power-efficient bf16 shape on this part), accumulators in AGPRs.
// A vocabulary tile is one hand-scheduled inline-asm statement (mosaic_w4_tile.inc greedy, mosaic_w4_tile_sample.inc
// sampling; both generated): the K-loop, then the tile's reduction to a triple per column.  Up to NB = 4 the LDS reads,
// direct-to-LDS copies and scalars are spread evenly behind the MFMAs (two instructions each at NB = 3 and 4, up to six at
// NB = 1, which waits for memory), fragments are double-buffered in fixed VGPRs, the LM-head ring runs two K-tiles ahead
// and the hidden ring one (three and two at NB <= 2).
// From NB = 5 on (kW4PairsFrom), where the matrix cores under the power cap are the bound, the two K-halves of a block's
// products go back to back, which costs the least energy (the generator says how; the waves that copy vocabulary blocks 0..3
// of a half run three K-tiles ahead there, and at NB = 7 and 8 not all token fragments have two buffers): 4096 rows
// 2641 -> 2535 us.
// NB sets the width of the row tile, 32*NB tokens.  The widest, 256, has the fewest LDS and L2 bytes per product and is
// the one for many rows; a list that does not fill its last row tile takes the width that pads it least
// (mosaic_schedule.h): 280 rows as two tiles of 160 take 278 us, as two of 256 375 us; 32 rows
// as one of 32 take 170 us (the LM head at 6.1 TB/s), as one of 256 211 us.
// A vocabulary that is no multiple of 256 ends in a tile over its last 256 ids, of which those that the tile before it
// has counted are taken out before the reduction; the general kernel on that tile alone, as a second launch, cost
// 100 to 130 us for four row tiles.
// Preconditions (checked by the launcher): V % 256 == 0, or V >= 256, five K-tiles and, sampling, V % 4 == 0;
// 256*d*2 < 4 GiB; and, in a hidden tensor of 4 GiB or more,
// no wave's 8*NB consecutive rows of the list 4 GiB apart (checked on the device, see KernelParams::wide_flag).
// Streaming.  A single row tile reads the LM head once, and one of more than the 256 MiB of the memory-side cache finds
// nothing of it there from the step before: its copies then carry the nt bit, by which they pass that cache by (copies
// alone: 6.6 instead of 5.9 TB/s).  126464 x 4096: 32 rows 204 -> 184 us a pass, 205 rows 223 -> 192, 256 rows 249 -> 237.
// Not where it is smaller (64 rows of 65536 x 2048, 256 MiB: 55 -> 72 us; 81920 x 2048, 320 MiB: 82 -> 77), and not
// where several row tiles share it behind an L2 (280 rows in two: 337 -> 349 us, 4096 rows 2551 -> 2592).
constexpr int64_t kStreamBytes = (int64_t)288 << 20;
constexpr int kRowBytes = 128;                       // one K-tile of a row
constexpr int kLmHeadSlot = 256 * kRowBytes;         // 32 KiB
constexpr int kLdsBytes = 160 * 1024;
#include "mosaic_w4_pieces.inc"
// Exchanges come after 1, 2, 4, 8, ... tiles, since a bound from n tiles lets pass half of what one from n / 2 does
// (after every tile: 4096 rows 2779 -> 2787 us, of 11 sizes none faster than its runs differ).  Of a row's splits at most about
// kPublishers publish, since atomics on one word take turns and a few are nearly as good a bound as all (205 rows 252.9 us with
// 8, 250.5 with 32, 250.6 with 64, 253.8 with all 247; 900 rows of 32000 x 1024, 125 splits, 88.6, 85.7, 85.0, 84.7).  The read may be served by any cache: an old bound is a bound.
// The columns that pad a row tile hold the last row once more and publish nothing: their atomics all went to that one row's
// word, up to 256 a publisher, and the next copies wait behind them (4105 rows 3114 -> 3006 us, 2700 rows of 65536 x 2048
// 659 -> 619, 16000 rows of 32000 x 1024 1037 -> 971).
constexpr int kPublishers = 32;
// The lane, anew: what these few lines derive from it is not to be kept in registers from one tile to the next.
__device__ __forceinline__ int fresh_lane() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
}
__device__ __forceinline__ int score_order(float x) {
  const int b = __float_as_int(x);
  return b ^ (int)((uint32_t)(b >> 31) >> 1);
}
// Lane group q clears, publishes and reads columns q and q + 4 of a wave.
__device__ __forceinline__ int32_t* row_best_at(const KernelParams& p, int row) {
  return reinterpret_cast<int32_t*>(p.out_conf + p.row0) + (uint32_t)row;
}
template <int NB>
__device__ __forceinline__ void clear_best(const KernelParams& p, int first_row, int rows) {
  const int lane = fresh_lane(), q = lane >> 4;
#pragma unroll
  for (int k = 0; k < (NB + 3) / 4; ++k) {
    const int column = 4 * k + q, row = first_row + column * 16 + (lane & 15);
    if (column < NB && row < rows)   // a padding column's draw is of no account, whatever it finds
      __hip_atomic_store(row_best_at(p, row), score_order(kNeg), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}
template <int NB>
__device__ __forceinline__ void publish_best(const KernelParams& p, const float (&ym)[NB], int first_row, int rows) {
  const int lane = fresh_lane(), q = lane >> 4;
#pragma unroll
  for (int k = 0; k < (NB + 3) / 4; ++k) {
    float own = kNeg;
#pragma unroll
    for (int tb = 4 * k; tb < NB && tb < 4 * k + 4; ++tb) {
      const float t = token_max(ym[tb]);
      own = q == (tb & 3) ? t : own;
    }
    const int column = 4 * k + q, row = first_row + column * 16 + (lane & 15);
    if (column < NB && row < rows)   // a padding column holds the last row
      __hip_atomic_fetch_max(row_best_at(p, row), score_order(own), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
// A prologue copy's address as a scalar base and a 32-bit offset a lane, which the copy's instruction takes as they are.  Left
// alone the compiler widens the offsets ahead of the units and spills the 64-bit addresses: a unit's start then waited for a
// reload, and the copies ahead of it, up to eight times (16000 rows of 32000 x 1024 drawn 1037 -> 1002 us, 9000 rows of
// 8192 x 512 drawn 165 -> 161, greedy 88.1 -> 87.0; vector registers spilled 69 -> 19 sampling, 10 -> 3 greedy).
__device__ __forceinline__ const char* scalar_pointer(const char* x) {
  const uint64_t a = (uint64_t)x;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
  return (const char*)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ uint32_t local_offset(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

template <bool SAMPLE, int NB, bool STREAM>
__device__ __forceinline__ void w4_units(const KernelParams& p, const Schedule& sched, int rows, int first, char* smem) {
  constexpr int kDepth = NB <= 2 ? 3 : 2;            // K-tiles under way, as the generator's depth()
  constexpr bool kPairs = NB >= kW4PairsFrom;        // the K-loop in pair order
  constexpr int kLatePieces = w4_late_pieces(NB);    // of eight LM-head copies, those a step issues behind its sync
  constexpr int NW = kDepth + 1, NH = kDepth;
  constexpr int kHiddenSlot = 32 * NB * kRowBytes;
  constexpr int kTokens = 32 * NB;
  constexpr int kAuxW = STREAM ? 2 : 0;              // the nt bit of the LM head's copies
  constexpr int kTileK = 64;
  constexpr int kSwzShift = 1;
  static_assert(NW * kLmHeadSlot + NH * kHiddenSlot <= kLdsBytes, "rings");
  // merge scratch, over the rings at unit end: eight entries per token
  double* red_s = reinterpret_cast<double*>(smem);
  float* red_m = reinterpret_cast<float*>(red_s + 8 * kTokens);
  int* red_i = reinterpret_cast<int*>(red_m + 8 * kTokens);
  float* red_ym = reinterpret_cast<float*>(red_i + 8 * kTokens);   // sampling only
  float* red_xa = red_ym + 8 * kTokens;
  static_assert(8 * kTokens * 24 <= NW * kLmHeadSlot + NH * kHiddenSlot, "merge scratch");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wv = wave & 1;   // vocabulary half of the tile
  const int wt = wave >> 1;  // token half of the tile
  const bool odd_wave = (__builtin_amdgcn_readfirstlane(wave) & 1) != 0;
  const int l16 = lane & 15, q = lane >> 4;   // MFMA 16x16x32: row/column lane%16, k group lane/16

  const int n_tt = sched.row_tiles;

  const int G = (int)p.sched.grid;   // (gridDim would make the launch carry 256 bytes more of arguments)
  const int S = sched.splits;
  const int n_units = n_tt * S;
  const int A = (int)panel_depth((uint32_t)n_tt, NB, (uint32_t)p.panel);
  const int full_panel_units = A * S;
  const int n_panels = (n_tt + A - 1) / A;

  // Direct-to-LDS copy: instruction i of this wave fills rows first + 8*i + lane/8 of the tile, first = 64*wave for
  // the LM head (i = 0..7), 8*NB*wave for the hidden rows (i = 0..NB-1); 16-byte chunks are swizzled by row.  (wlane: a
  // wave's row sub of an even and of an odd piece.)
  const int sub = lane >> 3;
  auto chunk_of = [&](int row) { return (uint32_t)(((lane & 7) ^ ((row >> kSwzShift) & 7)) * 16); };
  const int nk = p.d / kTileK;
  const uint32_t w_row_bytes = (uint32_t)p.d * 2u;

  // LDS read offsets per half K-tile: row (lane%16) of this wave's first 16-row block, swizzled chunk.
  uint32_t rdw[2], rdh[2], wlane[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const uint32_t o = (uint32_t)(l16 * kRowBytes + (((4 * ks + q) ^ ((l16 >> kSwzShift) & 7)) * 16));
    rdw[ks] = o + (uint32_t)(wv * 128 * kRowBytes);
    rdh[ks] = o + (uint32_t)(NW * kLmHeadSlot + wt * (kTokens / 2) * kRowBytes);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) wlane[i] = (uint32_t)(wave * 64 + sub) * w_row_bytes + chunk_of(wave * 64 + 8 * i + sub);

  // sampling: the generator's key (the statement derives the round keys from it), its multipliers, 1/tau and tau
  const uint32_t seed_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)p.seed_lo);
  const uint32_t seed_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)p.seed_hi);
  const uint32_t philox_m0 = 0xD2511F53u, philox_m1 = 0xCD9E8D57u;
  const float tau_s = p.tau;
  const float inv_tau_log2e = SAMPLE ? kLog2e / p.tau : 0.f;
  const uint32_t u_nk = (uint32_t)nk;
  // from a vocabulary tile's last K-tile to the next tile's first: 256 rows on, or, into the ragged last tile, V % 256
  const uint32_t u_wwrap = 256u * w_row_bytes - (uint32_t)(nk - 1) * 128u;
  const int ragged_rows = p.V % kTileVocab, ragged_tile = ragged_rows != 0 ? p.V / kTileVocab : -1;
  const uint32_t u_wwrap_ragged = (uint32_t)ragged_rows * w_row_bytes - (uint32_t)(nk - 1) * 128u;
  auto first_id = [&](int vt) { return vt == ragged_tile ? p.V - kTileVocab : vt * kTileVocab; };
  const uint32_t u_hwrap = (uint32_t)(nk - 1) * 128u;
  const uint32_t w_dst = (uint32_t)wave * 64u * kRowBytes, h_dst = (uint32_t)(wave * 8 * NB) * kRowBytes;

  for (int u = first, round = 0; u < n_units; u += G, ++round) {
    if (round > 0) meet_before_round(p, round, n_units, G, tid);
    int pnl = u / full_panel_units;
    if (pnl >= n_panels) pnl = n_panels - 1;
    const int ul = u - pnl * full_panel_units;
    const int hp = (n_tt - pnl * A) < A ? (n_tt - pnl * A) : A;
    const int sp = ul / hp;
    const int tt = pnl * A + ul % hp;
    const int vt0 = (int)(((int64_t)sp * p.sched.vocab_tiles) / S);
    const int vt1 = (int)(((int64_t)(sp + 1) * p.sched.vocab_tiles) / S);
    const int ntile = vt1 - vt0;
    const int total_steps = ntile * nk;
    const uint32_t u_total = (uint32_t)total_steps;

    // The row tiles that share an LM-head tile copy its pieces in orders of their own (a wave's piece i, to its place in LDS,
    // is its copy i ^ turn): in the same order all of them wait for the same lines, in different ones each finds half of them
    // asked for by another a quarter of a step before.  280 rows 277.6 -> 273.6 us, drawn 320.5 -> 308.8, 340 rows 313 -> 310,
    // 2077 1428 -> 1413.  Not at the widest tile, which waits for the matrix cores (4096 rows 2580 -> 2593, drawn 2776 -> 2802).
    const int turn = NB < 8 ? (tt & 1) * 4 + (tt & 2) : 0;
    uint32_t woff[8];
    auto w_source = [&](int gw) {   // past the end: the last one
      const int g = gw < total_steps ? gw : total_steps - 1;
      return p.w + (int64_t)first_id(vt0 + g / nk) * (int64_t)w_row_bytes + (g % nk) * kRowBytes;
    };
    auto copy_w = [&](int gw, int pieces = 8) {
      const char* src = scalar_pointer(w_source(gw));
      char* dst = smem + (gw % NW) * kLmHeadSlot + w_dst;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (i < pieces) __builtin_amdgcn_global_load_lds((gbl_ptr_t)(src + local_offset(woff[i])), (lds_ptr_t)(dst + (i ^ turn) * 1024), 16, 0, kAuxW);
    };
    // The list's entries are asked for first, then the first LM-head tile, which does not depend on them (the two latencies
    // one after the other: 1.0 us of a unit's start).
    wait_vm<0>();
    int trow[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      int j = tt * kTokens + wave * 8 * NB + 8 * i + sub;
      if (j > rows - 1) j = rows - 1;
      trow[i] = p.idx[p.row0 + j];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) woff[i] = wlane[i & 1] + (uint32_t)(8 * (i ^ turn)) * w_row_bytes;
    copy_w(0);

    [[maybe_unused]] const int first_row = tt * kTokens + wt * (kTokens / 2);   // this wave's columns
    [[maybe_unused]] int exchange = 0;   // 1: the unit takes shared bounds over; 2: it publishes, too
    if constexpr (SAMPLE) {
      if (units_share(p.sched.vocab_tiles, NB, S)) {
        exchange = sp % ((S + kPublishers - 1) / kPublishers) == 0 ? 2 : 1;
        clear_best<NB>(p, first_row, rows);
      }
      exchange = __builtin_amdgcn_readfirstlane(exchange);
    }

    // Gather: 32-bit byte offsets of the NB hidden rows this lane copies, from the lowest of the 8*NB rows this wave
    // copies (rows past the end of the chunk re-read the last valid row; their results are never stored).  The
    // offsets fit 32 bits when the hidden tensor is smaller than 4 GiB, and otherwise because this launch only
    // runs when no wave's rows lie that far apart (span_check_kernel).
    int tmin = INT_MAX;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      int t = trow[i];
      t = t < 0 ? 0 : (t > p.T - 1 ? p.T - 1 : t);   // a bad entry of a caller-built list reads a valid row
      trow[i] = t;
      tmin = t < tmin ? t : tmin;
    }
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) {
      const int other = __shfl_xor(tmin, x, 64);
      tmin = other < tmin ? other : tmin;
    }
    tmin = __builtin_amdgcn_readfirstlane(tmin);
    const char* hidden_wave = p.hidden + (int64_t)tmin * p.ldh_bytes;
    uint32_t hoff[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
      hoff[i] = (uint32_t)(trow[i] - tmin) * (uint32_t)p.ldh_bytes + chunk_of(wave * 8 * NB + 8 * i + sub);

    // Prologue copies: W0 and H0, which are needed first, then what else the rings hold.
    auto copy_h = [&](int gh) {
      const char* src = scalar_pointer(hidden_wave + (gh % nk) * kRowBytes);
      char* dst = smem + NW * kLmHeadSlot + (gh % NH) * kHiddenSlot + h_dst;
#pragma unroll
      for (int i = 0; i < NB; ++i)
        __builtin_amdgcn_global_load_lds((gbl_ptr_t)(src + local_offset(hoff[i])), (lds_ptr_t)(dst + i * 1024), 16, 0, 0);
    };
    // What the rings hold.  In pair order the waves that copy a half's vocabulary blocks 4..7 run a K-tile behind the
    // others, and the copies that may be under way at the first sync, the eight youngest, are the LM head's.
    const int lead = kPairs && odd_wave ? NW - 1 : NW;   // K-tiles of the LM head ahead of the step
    copy_h(0);
    if constexpr (kPairs) {
      if (!odd_wave && total_steps > 1) copy_w(1);
      if (total_steps > 1) copy_h(1);
      copy_w(lead - 1, kLatePieces);   // the first step copies the others
      if (total_steps < NW) wait_vm<0>();
      else if (odd_wave) wait_vm<kLatePieces + NB>();
      else wait_vm<kLatePieces + 8 + NB>();
    } else {
#pragma unroll
      for (int g = 1; g < NW; ++g)
        if (g < total_steps) copy_w(g);
#pragma unroll
      for (int g = 1; g < NH; ++g)
        if (g < total_steps) copy_h(g);
      if (total_steps >= NW && total_steps >= NH) wait_vm<8 * (NW - 1) + NB * (NH - 1)>(); else wait_vm<0>();
    }
    __builtin_amdgcn_s_barrier();

    // State of the asm loop: next tiles to copy are W(gw) and H(NH).  Never issued if past the end, or, in pair order, into
    // slots that nobody reads any more: the last LM-head tile again, and the front of the hidden rows.
    const int gw = kPairs ? lead - 1 : NW, gh = NH;
    const uint64_t wsrc0 = (uint64_t)(kPairs ? w_source(gw) : p.w + (int64_t)first_id(vt0 + gw / nk) * (int64_t)w_row_bytes + (gw % nk) * kRowBytes);
    const uint64_t hsrc0 = (uint64_t)(hidden_wave + (gh % nk) * kRowBytes);
    uint32_t st_wsrc_lo = (uint32_t)wsrc0, st_wsrc_hi = (uint32_t)(wsrc0 >> 32);
    uint32_t st_hsrc_lo = (uint32_t)hsrc0, st_hsrc_hi = (uint32_t)(hsrc0 >> 32);
    uint32_t st_wrd = 0, st_hrd = 0;
    uint32_t st_wdst = (uint32_t)((gw % NW) * kLmHeadSlot) + w_dst + (uint32_t)turn * 1024u;
    uint32_t st_hdst = (uint32_t)((gh % NH) * kHiddenSlot) + h_dst;
    uint32_t st_wk = (uint32_t)((kPairs && gw >= total_steps ? total_steps - 1 : gw) % nk), st_hk = (uint32_t)(gh % nk);
    uint32_t st_g = 0;

    float run_m[NB], run_ym[NB], run_xa[NB];
    double run_s[NB];
    int run_i[NB], pos[NB];
#pragma unroll
    for (int tb = 0; tb < NB; ++tb) {
      run_m[tb] = kNeg; run_s[tb] = 0.0; run_i[tb] = INT_MAX; run_ym[tb] = kNeg; run_xa[tb] = 0.f; pos[tb] = 0;
      if constexpr (SAMPLE) {   // the position whose row this lane's column tb holds
        int j = tt * kTokens + wt * (kTokens / 2) + tb * 16 + l16;
        if (j > rows - 1) j = rows - 1;
        pos[tb] = p.noise_idx[p.row0 + j];
      }
    }

#pragma unroll 1
    for (int n = 0; n < ntile; ++n) {
      if constexpr (SAMPLE) asm volatile("" : "+s"(exchange));   // one loop, not one for each of its values
      st_wsrc_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_wsrc_lo);
      st_wsrc_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_wsrc_hi);
      st_hsrc_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_hsrc_lo);
      st_hsrc_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_hsrc_hi);
      st_wrd = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_wrd);
      st_hrd = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_hrd);
      st_wdst = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_wdst);
      st_hdst = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_hdst);
      st_wk = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_wk);
      st_hk = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_hk);
      st_g = (uint32_t)__builtin_amdgcn_readfirstlane((int)st_g);
      {
      const uint32_t st_total = (uint32_t)__builtin_amdgcn_readfirstlane((int)u_total);
      const uint32_t st_nk = (uint32_t)__builtin_amdgcn_readfirstlane((int)u_nk);
      const bool ragged_next = vt0 + n + 1 == ragged_tile, ragged = vt0 + n == ragged_tile;
      const uint32_t st_wwrap = (uint32_t)__builtin_amdgcn_readfirstlane((int)(ragged_next ? u_wwrap_ragged : u_wwrap));
      int tile_first = 0;   // what the statement does ahead of the reduction: nothing, the ids counted before, or
      if (ragged) tile_first = ragged_tile * kTileVocab;
      else if (SAMPLE && exchange > 0 && n > 0 && (n & (n - 1)) == 0) tile_first = kW4Take;   // the shared bounds, behind 1, 2, 4, ... tiles
      const uint32_t st_first = (uint32_t)__builtin_amdgcn_readfirstlane(tile_first);
      const uint32_t st_hwrap = (uint32_t)__builtin_amdgcn_readfirstlane((int)u_hwrap);
        [[maybe_unused]] const uint32_t st_wnext = (uint32_t)__builtin_amdgcn_readfirstlane(lead);
        uint32_t addr_tmp0, addr_tmp1;
        [[maybe_unused]] uint32_t addr_tmp2, addr_tmp3;
        const int vb = first_id(vt0 + n) + wv * 128 + 4 * q;   // vocabulary id of this lane's element 0
        float tile_m[NB], tile_s[NB];   // this tile's own triples
        int tile_i[NB];
        if constexpr (SAMPLE) {
          // the shared bounds of the wave's rows, and how many follow the first (a padding column takes the last one's; a wave
          // of nothing else begins there)
          const int from = first_row < rows ? first_row : rows - 1;
          const uint64_t row_best = (uint64_t)scalar_pointer((const char*)(p.out_conf + p.row0 + (int64_t)from));
          const int last_row = __builtin_amdgcn_readfirstlane(rows - 1 - from);
          // sampling: the same, with the Gumbel-max draw in the reduction (round keys by number too).  The drawn
          // candidate is carried from tile to tile: it bounds what can still win
#include "mosaic_w4_tile_sample.inc"
        } else {
          // greedy: one statement clears the accumulators (the AGPR file, by number), runs the K-loop and reduces
          // the tile to a triple per column (fragments and temporaries by number), so nothing of it is left to the
          // compiler's scheduling
#include "mosaic_w4_tile.inc"
        }
        if constexpr (SAMPLE)
          if (exchange > 1 && (n & (n + 1)) == 0)
            publish_best<NB>(p, run_ym, first_row, rows);
        // the fold, ~25 instructions per column and tile of 64 K-tiles: 0.5% of the tile
#pragma unroll
        for (int tb = 0; tb < NB; ++tb) {
          if constexpr (!SAMPLE) run_i[tb] = tile_m[tb] > run_m[tb] ? tile_i[tb] : run_i[tb];   // ascending tiles
          merge_sum(run_m[tb], run_s[tb], tile_m[tb], tile_sum(tile_m[tb], tile_s[tb]));
        }
      }
    }

    // Unit end: a token's state lies in eight lanes (four of a wave, times the two vocabulary halves).  All of them go to
    // LDS, and one thread per token merges its eight in a loop: a tenth of the code of a tree of shuffles over NB
    // columns, and it is code that runs once a unit, cold.
    if constexpr (kPairs) wait_vm<0>();   // the copies that the last steps made for nobody
    __syncthreads();  // every wave is done with the ring (the merge scratch aliases it)
#pragma unroll
    for (int tb = 0; tb < NB; ++tb) {
      const int e = (wv * 4 + q) * kTokens + wt * (kTokens / 2) + tb * 16 + l16;
      red_m[e] = run_m[tb];
      red_s[e] = run_s[tb];
      red_i[e] = run_i[tb];
      if constexpr (SAMPLE) {
        red_ym[e] = run_ym[tb];
        red_xa[e] = run_xa[tb];
      }
    }
    __syncthreads();
    if (tid < kTokens && tt * kTokens + tid < rows) {
      float m = red_m[tid], ym = kNeg, xa = 0.f;
      double s = red_s[tid];
      int i = red_i[tid];
      if constexpr (SAMPLE) { ym = red_ym[tid]; xa = red_xa[tid]; }
#pragma unroll 1
      for (int e = tid + kTokens; e < 8 * kTokens; e += kTokens) {
        if constexpr (SAMPLE) {
          merge_sum(m, s, red_m[e], red_s[e]);
          merge_pick(ym, xa, i, red_ym[e], red_xa[e], red_i[e]);
        } else {
          merge_triple(m, s, i, red_m[e], red_s[e], red_i[e]);
        }
      }
      const int64_t slot = (int64_t)sp * sched.stride + tt * kTokens + tid;
      if constexpr (SAMPLE) {
        p.part_ym[slot] = ym;
        p.part_xa[slot] = xa;
      }
      p.part_m[slot] = m;
      p.part_si[slot] = pack_sum_id(s, i, p.id_bits);
    }
    __syncthreads();
  }
}

template <bool SAMPLE, bool STREAM>
__device__ __forceinline__ void w4_units_of(const KernelParams& p, const Schedule& sched, int rows, int first, char* smem) {
  switch (sched.width) {
    case 1: w4_units<SAMPLE, 1, STREAM>(p, sched, rows, first, smem); break;
    case 2: w4_units<SAMPLE, 2, STREAM>(p, sched, rows, first, smem); break;
    case 3: w4_units<SAMPLE, 3, STREAM>(p, sched, rows, first, smem); break;
    case 4: w4_units<SAMPLE, 4, STREAM>(p, sched, rows, first, smem); break;
    case 5: w4_units<SAMPLE, 5, STREAM>(p, sched, rows, first, smem); break;
    case 6: w4_units<SAMPLE, 6, STREAM>(p, sched, rows, first, smem); break;
    case 7: w4_units<SAMPLE, 7, STREAM>(p, sched, rows, first, smem); break;
    default: w4_units<SAMPLE, 8, STREAM>(p, sched, rows, first, smem); break;
  }
}

// Asks for all lines of a launch's arguments at once: read where they are used, one line waits for the other (268 rows of
// 8192 x 512, a step of three launches: 19.3 -> 19.0 us).
__device__ __forceinline__ void fetch_arguments() {
  static_assert(sizeof(KernelParams) > 192 && sizeof(KernelParams) <= 256, "four lines");
  uint32_t a, b, c, d;
  asm volatile("s_load_dword %0, %4, 0x0\n\ts_load_dword %1, %4, 0x40\n\ts_load_dword %2, %4, 0x80\n\ts_load_dword %3, %4, 0xc0\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&s"(a), "=&s"(b), "=&s"(c), "=&s"(d) : "s"(__builtin_amdgcn_kernarg_segment_ptr()));
}

template <bool SAMPLE>
__global__ __launch_bounds__(256) void masked_logits_kernel_w4(const KernelParams p) {
  __shared__ __attribute__((aligned(1024))) char smem[kLdsBytes];
  fetch_arguments();
  if (p.wide_flag != nullptr && *p.wide_flag != p.wide_run_if) return;   // the other kernel of the two serves this list
  const int rows = chunk_rows_found(p);
  if (rows <= 0) return;
  const Schedule sched = launch_schedule(p, rows);
  const int units = sched.row_tiles * sched.splits, first = first_unit((int)blockIdx.x, (int)p.sched.grid, units);
  if (first >= units) return;
  if (p.stream_w != 0 && sched.row_tiles == 1) w4_units_of<SAMPLE, true>(p, sched, rows, first, smem);
  else w4_units_of<SAMPLE, false>(p, sched, rows, first, smem);
}

// Merge the S partial results of every row and emit the outputs.  A wave handles ROWS rows with G = 64 / ROWS lanes
// each, without a barrier: the largest logit of the row first, by a butterfly of shuffles, so that every sum is scaled
// once and the sums meet in a second butterfly of plain additions.  Few splits: four rows a wave; many (one row tile
// spread over ~250 of them, where this kernel is a visible part of the step): one.  Bound by latency: a launch, the
// loads of count and splits, the partials, twelve shuffles.
constexpr int kWideMergeSplits = 64;   // from this many splits on, a wave per row
__host__ __device__ inline int combine_blocks(int rows) { return rows < 4 * 4096 ? (rows + 3) / 4 : 4096; }
template <int ROWS>
__device__ __forceinline__ void combine_rows(const KernelParams& p, int splits, int rows) {
  constexpr int G = 64 / ROWS;
  constexpr int kMost = ROWS == 1 ? MOSAIC_MAX_VOCAB_SPLITS + 1 : kWideMergeSplits - 1;
  constexpr int kPerLane = (kMost + G - 1) / G;   // splits one lane loads at most
  const bool sample = p.tau > 0.f;   // sampling: the token is the arg-max of the perturbed scores
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int lr = lane % ROWS, g = lane / ROWS;
  for (int r0 = ((int)blockIdx.x * 4 + wave) * ROWS; r0 < rows; r0 += combine_blocks(p.bound_rows) * 4 * ROWS) {
    const bool valid = r0 + lr < rows;
    const int r = valid ? r0 + lr : rows - 1;
    float lm[kPerLane], lym[kPerLane], lxa[kPerLane];
    uint64_t lsi[kPerLane];
#pragma unroll
    for (int k = 0; k < kPerLane; ++k) {
      const int sp = g + k * G;
      const bool on = sp < splits;
      const int64_t slot = (int64_t)(on ? sp : 0) * partial_stride(rows) + r;
      lm[k] = on ? p.part_m[slot] : kNeg;        // beyond S: the neutral element
      lsi[k] = on ? p.part_si[slot] : 0;
      lym[k] = (on && sample) ? p.part_ym[slot] : kNeg;
      lxa[k] = (on && sample) ? p.part_xa[slot] : 0.f;
    }
    float m = kNeg;
#pragma unroll
    for (int k = 0; k < kPerLane; ++k) m = fmaxf(m, lm[k]);
#pragma unroll
    for (int x = ROWS; x < 64; x <<= 1) m = fmaxf(m, __shfl_xor(m, x, 64));
    const float e = ref_exponent(m);
    double s = 0.0;
    float best = kNeg, xa = 0.f;     // what the token is the arg-max of; its plain logit
    int i = INT_MAX;
#pragma unroll
    for (int k = 0; k < kPerLane; ++k) {
      double s2;
      int i2;
      unpack_sum_id(lsi[k], p.id_bits, s2, i2);
      s += __builtin_ldexp(s2, scale_steps(ref_exponent(lm[k]) - e));
      if (g + k * G < splits) merge_pick(best, xa, i, sample ? lym[k] : lm[k], lxa[k], i2);
    }
#pragma unroll
    for (int x = ROWS; x < 64; x <<= 1) {
      s += __shfl_xor(s, x, 64);
      merge_pick(best, xa, i, __shfl_xor(best, x, 64), __shfl_xor(xa, x, 64), __shfl_xor(i, x, 64));
    }
    if (g == 0 && valid) {
      // back from 2^E to exp(m)
      const float rel = (float)(s / (double)__builtin_amdgcn_exp2f(__builtin_fmaf(m, kLog2e, -e)));
      p.out_token[p.row0 + r] = i;
      p.out_lse[p.row0 + r] = m + __builtin_amdgcn_logf(rel) * kLn2;
      p.out_conf[p.row0 + r] = sample ? __builtin_amdgcn_exp2f((xa - m) * kLog2e) / rel : 1.0f / rel;
    }
  }
}
__global__ __launch_bounds__(256) void combine_kernel(const KernelParams p) {
  const int rows = chunk_rows_found(p);
  if (rows <= 0) return;
  const int splits = held_splits(p.sched, rows, *p.found_splits) + (int)p.sched.extra;   // a pair's second launch adds one
  if (splits >= kWideMergeSplits) combine_rows<1>(p, splits, rows);
  else combine_rows<4>(p, splits, rows);
}

int launch_masked_logits(const LogitsArgs& a, const mosaic_plan& plan, hipStream_t stream) {
  KernelParams p;
  p.hidden = static_cast<const char*>(a.hidden);
  p.ldh_bytes = a.ld_h * 2;
  p.w = static_cast<const char*>(a.w);
  p.d = a.d;
  p.V = a.V;
  p.idx = a.idx;
  p.noise_idx = a.noise_idx != nullptr ? a.noise_idx : a.idx;
  p.count = a.count;
  p.T = (int32_t)a.T;
  p.chunk_rows = plan.rows_per_chunk;
  p.max_rows = (int32_t)a.max_rows;
  p.panel = plan.tile_panel;
  p.stream_w = (int64_t)a.V * a.d * 2 > kStreamBytes ? 1 : 0;
  const int64_t slots = (int64_t)plan.vocab_splits * plan.rows_per_chunk;   // a multiple of 256
  p.part_si = static_cast<uint64_t*>(a.workspace);
  p.part_m = reinterpret_cast<float*>(p.part_si + slots);
  p.id_bits = 32 - __builtin_clz((unsigned)a.V);
  p.out_token = a.out_token;
  p.out_conf = a.out_conf;
  p.out_lse = a.out_lse;
  const bool sample = a.temperature > 0.f;
  p.tau = sample ? a.temperature : 0.f;
  p.seed_lo = (uint32_t)a.seed;
  p.seed_hi = (uint32_t)(a.seed >> 32);
  p.part_ym = p.part_m + slots;
  p.part_xa = p.part_ym + slots;
  // the round counters sit behind the partial planes (three for a greedy pass, five for a sampling one)
  constexpr int kSyncSlots = MOSAIC_SYNC_BYTES / 4 - 2;   // then the division found, and the flag of the span check
  p.sync = reinterpret_cast<int32_t*>(sample ? p.part_xa + slots : p.part_ym);
  p.sync_slots = kSyncSlots;
  p.wide_flag = nullptr;
  p.wide_run_if = 0;

  const KernelChoice choice = choose_kernel(a.T, a.ld_h, a.d, a.V, plan, sample);
  const bool fast = choice.fast, paired = choice.paired, wide = choice.wide;
  p.found_splits = p.sync + kSyncSlots;
  int32_t* const flag = p.found_splits + 1;
  const int32_t vocab_tiles = (a.V + kTileVocab - 1) / kTileVocab;
  p.sched.vocab_tiles = (uint32_t)(paired ? vocab_tiles - 1 : vocab_tiles);
  p.sched.k_tiles = (uint32_t)(a.d / MOSAIC_K_TILE);
  p.sched.widths = fast || paired ? 0xff : 0x80;   // the general kernel has the one width
  p.sched.sampling = sample ? 1 : 0;
  // never more workgroups than the plan has units of 64 rows, whatever its field says; with that many the
  // division's products stay below 2^32 (a larger one could only be refused by the launch)
  const int64_t units = (int64_t)(plan.rows_per_chunk / 64) * plan.vocab_splits;
  const int32_t grid = plan.grid < units ? plan.grid : (int32_t)units;
  p.sched.grid = (uint32_t)(grid < 1 << 24 ? grid : 1 << 24);
  p.sched.extra = paired ? 1 : 0;
  p.sched.slots64 = (uint32_t)(slots / 64 < INT32_MAX ? slots / 64 : INT32_MAX);
  p.ragged_tile = -1;
  KernelParams tail = p;   // the second launch of a pair
  if (paired) {
    tail.ragged_tile = vocab_tiles - 1;
    p.sync_slots = tail.sync_slots = kSyncSlots / 2;   // each launch of the pair meets on its own counters
    tail.sync = p.sync + kSyncSlots / 2;
  }
  int32_t* const counters = p.sync;
  // A hidden tensor of 4 GiB or more: the 4-wave launch and a general-kernel launch of the same work both go out,
  // and the flag of the span check decides on the device which of the two does it.
  if (wide) p.wide_flag = flag;
  int rc = 0;
  for (int c = 0; c < plan.num_chunks; ++c) {
    const int64_t row0 = (int64_t)c * plan.rows_per_chunk;
    if (row0 >= a.max_rows) break;
    int64_t cap = a.max_rows - row0;
    if (cap > plan.rows_per_chunk) cap = plan.rows_per_chunk;
    p.row0 = tail.row0 = (int32_t)row0;
    p.bound_rows = tail.bound_rows = (int32_t)cap;
    p.bound = tail.bound = choose_schedule(p.sched, (int32_t)cap);
    const int64_t tiles = (cap + kTileRows - 1) / kTileRows;
    const bool several_rounds = (int64_t)p.bound.row_tiles * p.bound.splits > grid || (paired && tiles > grid);
    if (!several_rounds) p.sync = tail.sync = nullptr;   // nobody meets (fewer rows may still take two rounds)
    else p.sync = counters, tail.sync = counters + kSyncSlots / 2;
    if (wide && cap <= kOneBlockCheckRows) {
      rc |= launch_kernel(clear_and_check_kernel, dim3(1), dim3(1024), stream, p, counters, kSyncSlots + 1, flag);
    } else {
      if (several_rounds || wide)
        rc |= launch_kernel(clear_round_counters_kernel, dim3(1), dim3(256), stream, counters, kSyncSlots + 2);
      if (wide)
        rc |= launch_kernel(span_check_kernel, dim3((unsigned)((cap + 255) / 256)), dim3(256), stream, p, flag);
    }
    auto launch_general = [&](const KernelParams& kp, int64_t blocks) {
      return sample ? launch_kernel(masked_logits_kernel<3, 2, true>, dim3((unsigned)blocks), dim3(kThreads), stream, kp)
                    : launch_kernel(masked_logits_kernel<3, 2, false>, dim3((unsigned)blocks), dim3(kThreads), stream, kp);
    };
    if (fast || paired) {
      rc |= sample ? launch_kernel(masked_logits_kernel_w4<true>, dim3((unsigned)grid), dim3(256), stream, p)
                   : launch_kernel(masked_logits_kernel_w4<false>, dim3((unsigned)grid), dim3(256), stream, p);
      if (wide) {   // the same work on the general kernel, for lists the span check flags
        KernelParams fallback = p;
        fallback.wide_run_if = 1;
        fallback.sched.widths = 0x80;
        fallback.bound = choose_schedule(fallback.sched, (int32_t)cap);
        rc |= launch_general(fallback, grid);
      }
    } else {
      rc |= launch_general(p, grid);
    }
    if (paired) rc |= launch_general(tail, tiles < grid ? tiles : grid);
    rc |= launch_kernel(combine_kernel, dim3((unsigned)combine_blocks((int)cap)), dim3(256), stream, p);
    if (rc != 0) break;
  }
  return rc;
}

}  // namespace mosaic
