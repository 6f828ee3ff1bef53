// Stable ordering of token positions by index, for the sorted embedding backward: a radix
// sort, least significant digit first, written for what it sorts here - indices below a
// vocabulary size (15 bits for 30522 words: two digits) that come straight from the caller's
// array, so that the first pass makes its keys as it reads them and the positions need not be
// stored before they are moved.
//
// What bounds it is the number of dependent launches and memory round trips, not the traffic (21 MB
// for half a million entries and two digits): a merge sort took 22 launches and 135 us, this takes 6
// and 35 us (3 launches per digit of about 5, 4 and 10 us: the tiles of 2048 entries count their
// digits, one workgroup per digit value sums the counts over the tiles, the tiles place their entries).
//   * up to kSortSmall entries: everything in one workgroup and one launch;
//   * up to kSortSumInPlace tiles: the placing workgroup sums the counts of the tiles before
//     its own itself (at most 32 loads per thread; 9 us with whole lines read, 12 without, for 32
//     tiles) and the launch in between goes away;
//   * digits of 10 bits, with workgroups of 1024 threads, where they are one fewer than of 8 bits:
//     indices below 250000 in two passes instead of three 32 -> 18 us for 16000 entries, 50 -> 39 for
//     527340; below 300 in one instead of two 20.5 -> 8.7 and 31 -> 19.
// The place of an entry among the entries of its wavefront with the same digit comes from
// one ballot per digit bit; wavefronts and tiles follow each other in order: stable, and the
// same result in every run.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fmha {

constexpr int kSortTile = 2048;                             // entries per workgroup
constexpr int kSortDigits = 256;                            // values of a digit of 8 bits
constexpr int kSortWideDigits = 1024;                       // of 10
constexpr int kSortSumInPlace = 32;                         // tiles
constexpr int kSortSmallRounds = 4;
constexpr int kSortSmall = 1024 * kSortSmallRounds;         // 4096 entries: one workgroup of 1024 threads
constexpr int kSortTiny = 256 * kSortSmallRounds;           // or of 256, with fewer wavefronts to sum over

struct SortArgs {
  const int32_t* indices;  // first pass: the caller's indices; nullptr: read `in`
  const int32_t* n_rows;   // device, may be null: entries that count
  const uint2* in;         // {key, position}
  uint2* out;
  uint32_t* counts;        // [digit values][tiles], then their totals; or [tiles][digit values]
  int32_t tile_stride, digit_stride;  // which of the two
  int32_t rows, vocab, padding_idx;
  int32_t tiles;
  int32_t shift, bits;     // this pass's digit, at most 8 bits (wide: 10)
};

// key of entry t: its index if the token counts (in range, not the padding index, t < n), else
// vocab (sorted last)
static __device__ __forceinline__ uint2 sort_entry(const SortArgs& a, int t, int n) {
  if (!a.indices) return a.in[t];
  const int v = t < n ? a.indices[t] : -1;
  return make_uint2((v >= 0 && v < a.vocab && v != a.padding_idx) ? (uint32_t)v : (uint32_t)a.vocab, (uint32_t)t);
}
static __device__ __forceinline__ int sort_rows(const SortArgs& a) {
  return a.n_rows ? min(max(*a.n_rows, 0), a.rows) : a.rows;
}

// Where this lane's entry stands among the wavefront's entries of the same digit so far;
// `count` (the wavefront's own counters in LDS) moves on.  All 64 lanes must be active.
static __device__ __forceinline__ uint32_t sort_rank(uint32_t digit, bool valid, int bits, int lane,
                                                     volatile uint32_t* count) {
  uint64_t same = __ballot(valid);
  for (int b = 0; b < bits; b++) {  // uniform
    const bool bit = (digit >> b) & 1u;
    const uint64_t ones = __ballot(bit);
    same &= bit ? ones : ~ones;
  }
  const uint32_t ahead = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
  uint32_t base = 0;
  if (valid) base = count[digit];
  __builtin_amdgcn_wave_barrier();  // every lane has read before the first of each digit writes
  if (valid && ahead == 0) count[digit] = base + (uint32_t)__popcll(same);
  __builtin_amdgcn_wave_barrier();
  return base + ahead;
}

// Exclusive prefix sum over the values of the first 64 WAVES threads of the workgroup (every
// thread of the workgroup must call it; the others pass 0).
template <int WAVES>
static __device__ __forceinline__ uint32_t sort_scan(uint32_t mine, int tid, uint32_t (&wave_sum)[WAVES]) {
  const int lane = tid & 63, wave = tid >> 6;
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (wave < WAVES && lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int w = 0; w < WAVES - 1; w++) before += w < wave ? wave_sum[w] : 0u;
  return before + incl - mine;
}

// DIGITS: values of a digit, and threads of a workgroup.
template <int DIGITS>
__global__ __launch_bounds__(DIGITS) void sort_count_kernel(const SortArgs a) {
  __shared__ uint32_t count[DIGITS];
  const int tid = threadIdx.x, n = sort_rows(a);
  count[tid] = 0;
  __syncthreads();
  const uint32_t mask = (1u << a.bits) - 1u;
  const int base = blockIdx.x * kSortTile + tid;
#pragma unroll
  for (int r = 0; r < kSortTile / DIGITS; r++) {
    const int t = base + r * DIGITS;
    if (t < a.rows) atomicAdd(&count[(sort_entry(a, t, n).x >> a.shift) & mask], 1u);
  }
  __syncthreads();
  a.counts[(int64_t)tid * a.digit_stride + (int64_t)blockIdx.x * a.tile_stride] = count[tid];
}

constexpr int kSortTilesThreads = 256;

// One workgroup per digit: its counts over the tiles <- their exclusive prefix sums, and the total.
template <int DIGITS>
__global__ __launch_bounds__(kSortTilesThreads) void sort_tiles_kernel(const SortArgs a) {
  __shared__ uint32_t wave_sum[kSortTilesThreads / 64];
  const int tid = threadIdx.x;
  uint32_t* c = a.counts + (int64_t)blockIdx.x * a.tiles;
  uint32_t run = 0;
  for (int b0 = 0; b0 < a.tiles; b0 += kSortTilesThreads) {
    const int b = b0 + tid;
    const uint32_t mine = b < a.tiles ? c[b] : 0u;
    const uint32_t excl = sort_scan(mine, tid, wave_sum);
    if (b < a.tiles) c[b] = run + excl;
    run += wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
    __syncthreads();
  }
  if (tid == 0) a.counts[(int64_t)DIGITS * a.tiles + blockIdx.x] = run;
}

// SUM: the counts are as the counting kernel left them, tile by tile (a tile's counts side by
// side, so that the sums below read whole lines).
template <int DIGITS, bool SUM>
__global__ __launch_bounds__(DIGITS) void sort_place_kernel(const SortArgs a) {
  constexpr int kWaves = DIGITS / 64, kRounds = kSortTile / DIGITS;
  __shared__ uint32_t count[kWaves][DIGITS];
  __shared__ uint32_t wave_sum[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = sort_rows(a);
  const uint32_t mask = (1u << a.bits) - 1u;
  // every wavefront takes 64 kRounds consecutive entries, 64 at a time
  const int base = blockIdx.x * kSortTile + wave * (64 * kRounds) + lane;
  uint2 e[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; r++) e[r] = base + 64 * r < a.rows ? sort_entry(a, base + 64 * r, n) : make_uint2(0u, 0u);
  uint32_t before = 0, total = 0;  // entries of digit tid in earlier tiles, and in all
  if (SUM) {
#pragma unroll 8
    for (int b = 0; b < a.tiles; b++) {
      const uint32_t x = a.counts[b * DIGITS + tid];
      total += x;
      before += b < (int)blockIdx.x ? x : 0u;
    }
  } else {
    before = a.counts[(int64_t)tid * a.tiles + blockIdx.x];
    total = a.counts[(int64_t)DIGITS * a.tiles + tid];
  }
#pragma unroll
  for (int w = 0; w < kWaves; w++) count[w][tid] = 0;
  before += sort_scan(total, tid, wave_sum);  // (holds a barrier: the counters are zero)
  uint32_t at[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; r++)
    at[r] = sort_rank((e[r].x >> a.shift) & mask, base + 64 * r < a.rows, a.bits, lane, count[wave]);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; w++) {
    const uint32_t c = count[w][tid];
    count[w][tid] = before;
    before += c;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRounds; r++)
    if (base + 64 * r < a.rows) a.out[count[wave][(e[r].x >> a.shift) & mask] + at[r]] = e[r];
}

// All passes in one workgroup: rows <= THREADS * kSortSmallRounds, `passes` digits of `bits` bits.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void sort_small_kernel(const SortArgs a, int passes) {
  constexpr int kWaves = THREADS / 64;
  __shared__ uint32_t count[kWaves][kSortDigits];
  __shared__ uint2 entries[THREADS * kSortSmallRounds];
  __shared__ uint32_t wave_sum[kSortDigits / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = sort_rows(a);
  const uint32_t mask = (1u << a.bits) - 1u;
  const int base = wave * (64 * kSortSmallRounds) + lane;
  uint2 e[kSortSmallRounds];
#pragma unroll
  for (int r = 0; r < kSortSmallRounds; r++) e[r] = base + 64 * r < a.rows ? sort_entry(a, base + 64 * r, n) : make_uint2(0u, 0u);
  for (int p = 0; p < passes; p++) {
    const int shift = p * a.bits;
    for (int i = tid; i < kWaves * kSortDigits; i += THREADS) (&count[0][0])[i] = 0;
    __syncthreads();
    uint32_t at[kSortSmallRounds];
#pragma unroll
    for (int r = 0; r < kSortSmallRounds; r++)
      at[r] = sort_rank((e[r].x >> shift) & mask, base + 64 * r < a.rows, a.bits, lane, count[wave]);
    __syncthreads();
    uint32_t total = 0;
    if (tid < kSortDigits)
#pragma unroll
      for (int w = 0; w < kWaves; w++) total += count[w][tid];
    uint32_t run = sort_scan(total, tid, wave_sum);
    if (tid < kSortDigits)
#pragma unroll
      for (int w = 0; w < kWaves; w++) {
        const uint32_t c = count[w][tid];
        count[w][tid] = run;
        run += c;
      }
    __syncthreads();
    const bool last = p == passes - 1;
#pragma unroll
    for (int r = 0; r < kSortSmallRounds; r++)
      if (base + 64 * r < a.rows) {
        const uint32_t to = count[wave][(e[r].x >> shift) & mask] + at[r];
        if (last)
          a.out[to] = e[r];
        else
          entries[to] = e[r];
      }
    __syncthreads();
    if (!last) {
#pragma unroll
      for (int r = 0; r < kSortSmallRounds; r++) e[r] = base + 64 * r < a.rows ? entries[base + 64 * r] : make_uint2(0u, 0u);
    }
  }
}

}  // namespace fmha
