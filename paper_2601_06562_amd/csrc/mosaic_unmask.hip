// The tail of a denoising step, after mask-only logits: pick the positions to unmask and write their
// tokens (paper section 2.1: a step's drawn tokens replace a chosen subset of the still-masked positions;
// which subset is left open), and the index shift of Dream-style prediction (section 4.5, last paragraph).
// Integer / byte work: results are bit-exact by construction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mosaic_internal.h"

namespace mosaic {

constexpr int kUnmaskThreads = 1024;

// First row j in [0, n) with idx[j] >= pos (idx ascending): a binary search whose next ten levels are probed at once,
// one node of the decision tree per thread (thread h - 1 holds node h of the heap), so that a list of up to 10^6 rows
// takes two dependent memory latencies where the search alone took twenty (~0.6 us each).  It walks exactly the nodes
// that the search would, whatever the list holds.
constexpr int kSearchNodes = 1023;
static_assert(kSearchNodes < kUnmaskThreads, "one thread per node");
__device__ __forceinline__ int lower_bound_rows(const int32_t* __restrict__ idx, int n, int pos, uint64_t* below_bits) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int node = (int)threadIdx.x + 1;
    int l = lo, r = hi;
    for (int b = 30 - __clz(node); b >= 0; --b) {   // the path to the node: the bits behind its leading one
      const int mid = (l + r) >> 1;
      if ((node >> b) & 1) l = mid + 1; else r = mid;
    }
    const bool below = node <= kSearchNodes && l < r && idx[(l + r) >> 1] < pos;
    const uint64_t wave = __ballot(below);
    if ((threadIdx.x & 63) == 0) below_bits[threadIdx.x >> 6] = wave;
    __syncthreads();
    for (int h = 1; lo < hi && h <= kSearchNodes;) {
      const int mid = (lo + hi) >> 1;
      const bool right = (below_bits[(h - 1) >> 6] >> ((h - 1) & 63)) & 1;
      if (right) lo = mid + 1; else hi = mid;
      h = 2 * h + (right ? 1 : 0);
    }
    __syncthreads();   // below_bits is reused
  }
  return lo;
}

// Exclusive scan of one 0/1 flag per thread over the block, in thread order.  Returns the exclusive
// prefix; *total receives the block total.  wave_tot: LDS, one int per wave.
__device__ __forceinline__ int block_exclusive_scan_flag(int flag, int* wave_tot, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t ballot = __ballot(flag);
  const int excl = __popcll(ballot & ((1ull << lane) - 1ull));
  if (lane == 0) wave_tot[wave] = __popcll(ballot);
  __syncthreads();
  int before = 0, tot = 0;
  for (int w = 0; w < kUnmaskThreads / 64; ++w) {
    const int t = wave_tot[w];
    if (w < wave) before += t;
    tot += t;
  }
  __syncthreads();  // wave_tot is reused by the next call
  *total = tot;
  return before + excl;
}

// Bins 0..255 of `hist`, read by the first wave (four bins per lane): the largest bin whose "at least" count reaches
// `need`, and what of `need` is left inside it.  One wave-wide suffix sum; one thread walking the bins took ~10 us.
__device__ __forceinline__ void find_threshold_bin(const int* hist, int need, int* bin, int* left) {
  const int lane = threadIdx.x;   // of the first wave
  int c[4], sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) { c[k] = hist[4 * lane + k]; sum += c[k]; }
  int at_least = sum;             // inclusive suffix sum over the lanes
#pragma unroll
  for (int x = 1; x < 64; x <<= 1) {
    const int other = __shfl_down(at_least, x, 64);
    at_least += lane + x < 64 ? other : 0;
  }
  const int above = at_least - sum;
  if (above < need && need <= at_least) {   // exactly one lane
    int a = above, k = 3;
    while (k > 0 && a + c[k] < need) a += c[k--];
    *bin = 4 * lane + k;
    *left = need - a;
  }
}

// One block per sequence: exact top-n by confidence (ties: lower position).  Confidences are non-negative, so their
// bit patterns order like the values.  Up to kRankRows rows (a block of a block-wise decoder): one thread per row
// counts the rows that come before it.  More: a radix select of the threshold key, four passes of eight bits.
// Bound by latency (a chain of barriers and dependent reads by one block): 24 rows 46 -> 6 us, 1004 rows 33 -> 10 us.
constexpr int kRankRows = 256;   // the count is 64 LDS reads of four keys there, ~1 us; a radix pass ~2 us
__global__ __launch_bounds__(kUnmaskThreads) void unmask_topn_kernel(
    const float* __restrict__ conf, const int32_t* __restrict__ token, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ count, int32_t max_rows, const int32_t* __restrict__ seq_starts,
    const int32_t* __restrict__ n_per_seq, int32_t* __restrict__ tokens, uint8_t* __restrict__ mask, int32_t T) {
  __shared__ __attribute__((aligned(16))) int hist[256];   // bin counts, or the keys of up to kRankRows rows
  __shared__ int wave_tot[kUnmaskThreads / 64];
  __shared__ int sh_bin, sh_need;
  __shared__ uint64_t below_bits[kUnmaskThreads / 64];
  static_assert(kRankRows <= 256, "the keys share the bins' memory");
  const int b = blockIdx.x, tid = threadIdx.x;
  int total = *count;
  if (total > max_rows) total = max_rows;
  const int lo = lower_bound_rows(idx, total, seq_starts[b], below_bits);
  const int hi = lower_bound_rows(idx, total, seq_starts[b + 1], below_bits);
  const int m = hi - lo;
  int n = n_per_seq[b];
  if (n > m) n = m;
  if (n <= 0) return;
  const uint32_t* keys = reinterpret_cast<const uint32_t*>(conf);
  auto unmask_row = [&](int j) {
    const int t = idx[j];
    if (t >= 0 && t < T) {   // an entry outside [0, T) of a caller-built list is skipped, never written through
      tokens[t] = token[j];
      mask[t] = 0;
    }
  };

  if (m <= kRankRows) {
    const uint32_t key = tid < m ? keys[lo + tid] : 0u;
    if (tid < 256) hist[tid] = (int)key;
    __syncthreads();
    if (tid < m) {
      int before = 0;                       // rows taken ahead of this one
      for (int j = 0; j < m; j += 4) {      // rows past m hold key 0 behind every real row: they count for nobody
        const uint4 k = *reinterpret_cast<const uint4*>(hist + j);
        before += (k.x > key || (k.x == key && j + 0 < tid)) ? 1 : 0;
        before += (k.y > key || (k.y == key && j + 1 < tid)) ? 1 : 0;
        before += (k.z > key || (k.z == key && j + 2 < tid)) ? 1 : 0;
        before += (k.w > key || (k.w == key && j + 3 < tid)) ? 1 : 0;
      }
      if (before < n) unmask_row(lo + tid);
    }
    return;
  }

  uint32_t prefix = 0;   // bytes of the threshold key decided so far
  int need = n;          // rows still to find among keys matching the prefix
  if (n < m) {
    for (int pass = 3; pass >= 0; --pass) {
      const int shift = 8 * pass;
      const uint32_t high_mask = (pass == 3) ? 0u : (0xffffffffu << (shift + 8));
      if (tid < 256) hist[tid] = 0;
      __syncthreads();
      for (int j = lo + tid; j < hi; j += kUnmaskThreads) {
        const uint32_t k = keys[j];
        const int bin = (int)((k >> shift) & 0xffu);
        if (pass == 3) {   // a handful of exponents: one addition per distinct bin of the wave, not one per row
          uint64_t open = __ballot(1);
          while (open != 0) {
            const int lead = __ffsll((unsigned long long)open) - 1;
            const uint64_t same = __ballot(bin == __builtin_amdgcn_readlane(bin, lead)) & open;
            if (((int)threadIdx.x & 63) == lead) atomicAdd(&hist[bin], (int)__popcll(same));
            open &= ~same;
          }
        } else if ((k & high_mask) == prefix) {
          atomicAdd(&hist[bin], 1);
        }
      }
      __syncthreads();
      if (tid < 64) find_threshold_bin(hist, need, &sh_bin, &sh_need);
      __syncthreads();
      prefix |= (uint32_t)sh_bin << shift;
      need = sh_need;
    }
  }
  // Rows above the threshold key are taken; of the rows equal to it, the first `need` in position order.
  int base = 0;
  for (int j0 = lo; j0 < hi; j0 += kUnmaskThreads) {
    const int j = j0 + tid;
    const bool valid = j < hi;
    const uint32_t k = valid ? keys[j] : 0u;
    const bool all = (n == m);
    const int eq = (valid && !all && k == prefix) ? 1 : 0;
    int eq_total;
    const int rank = base + block_exclusive_scan_flag(eq, wave_tot, &eq_total);
    base += eq_total;
    if (valid && (all || k > prefix || (eq && rank < need))) unmask_row(j);
  }
}

// gather[j] = idx[j] - 1, except where idx[j] is the first position of its sequence.
__global__ __launch_bounds__(256) void shift_indices_kernel(const int32_t* __restrict__ idx,
                                                            const int32_t* __restrict__ count, int32_t max_rows,
                                                            const int32_t* __restrict__ seq_starts, int32_t num_seqs,
                                                            int32_t* __restrict__ gather) {
  int total = *count;
  if (total > max_rows) total = max_rows;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= total) return;
  const int pos = idx[j];
  int lo = 0, hi = num_seqs;            // largest b with seq_starts[b] <= pos
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (seq_starts[mid] <= pos) lo = mid; else hi = mid;
  }
  int g = (seq_starts[lo] == pos) ? pos : pos - 1;
  const int last = seq_starts[num_seqs] - 1;   // T - 1: an out-of-range entry is clamped, never passed on
  g = g > last ? last : g;
  gather[j] = g < 0 ? 0 : g;
}

int launch_unmask_topn(const float* conf, const int32_t* token, const int32_t* idx, const int32_t* count,
                       int64_t max_rows, const int32_t* seq_starts, int32_t num_seqs, const int32_t* n_per_seq,
                       int32_t* tokens, uint8_t* mask, int64_t T, hipStream_t stream) {
  return launch_kernel(unmask_topn_kernel, dim3((unsigned)num_seqs), dim3(kUnmaskThreads), stream, conf, token, idx,
                       count, (int32_t)max_rows, seq_starts, n_per_seq, tokens, mask, (int32_t)T);
}

int launch_shift_indices(const int32_t* idx, const int32_t* count, int64_t max_rows, const int32_t* seq_starts,
                         int32_t num_seqs, int32_t* gather, hipStream_t stream) {
  return launch_kernel(shift_indices_kernel, dim3((unsigned)((max_rows + 255) / 256)), dim3(256), stream, idx, count,
                       (int32_t)max_rows, seq_starts, num_seqs, gather);
}

}  // namespace mosaic
