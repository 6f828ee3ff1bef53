// Stable ordering of token positions by index, for the sorted embedding backward: a radix
// sort, least significant digit first, written for what it sorts here - indices below a
// vocabulary size (15 bits for 30522 words: two digits) that come straight from the caller's
// array, so that the first pass makes its keys as it reads them and the positions need not be
// stored before they are moved.
//
// What bounds it is the number of dependent launches and memory round trips, not the 4 - 8 MB
// moved: for half a million pairs a merge sort took 22 launches and 135 us, this takes 6 and
// 43 us (3 launches per digit of about 5, 4 and 10 us: the tiles of 2048 entries count their
// digits, one workgroup per digit sums the counts over the tiles, the tiles place their entries).
//   * up to kSortSmall entries: everything in one workgroup and one launch;
//   * up to kSortSumInPlace tiles: the placing workgroup sums the counts of the tiles before
//     its own itself (at most 32 loads per thread; 9 us with whole lines read, 12 without, for 32
//     tiles) and the launch in between goes away.
// The place of an entry among the entries of its wavefront with the same digit comes from
// one ballot per digit bit; wavefronts and tiles follow each other in order: stable, and the
// same result in every run.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fmha {

constexpr int kSortThreads = 256;
constexpr int kSortRounds = 8;                              // entries per thread
constexpr int kSortTile = kSortThreads * kSortRounds;       // 2048 entries per workgroup
constexpr int kSortDigits = 256;
constexpr int kSortSumInPlace = 32;                         // tiles
constexpr int kSortSmallRounds = 4;
constexpr int kSortSmall = 1024 * kSortSmallRounds;         // 4096 entries: one workgroup of 1024 threads
constexpr int kSortTiny = 256 * kSortSmallRounds;           // or of 256, with fewer wavefronts to sum over

struct SortArgs {
  const int32_t* indices;  // first pass: the caller's indices; nullptr: read `in`
  const int32_t* n_rows;   // device, may be null: entries that count
  const uint2* in;         // {key, position}
  uint2* out;
  uint32_t* counts;        // [kSortDigits][tiles], then kSortDigits totals; or [tiles][kSortDigits]
  int32_t tile_stride, digit_stride;  // which of the two
  int32_t rows, vocab, padding_idx;
  int32_t tiles;
  int32_t shift, bits;     // this pass's digit; bits <= 8
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

// Exclusive prefix sum over the kSortDigits values of the first kSortDigits threads of the
// workgroup (every thread of the workgroup must call it; the others pass 0).
static __device__ __forceinline__ uint32_t sort_scan256(uint32_t mine, int tid, uint32_t (&wave_sum)[4]) {
  const int lane = tid & 63, wave = tid >> 6;
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = __shfl_up(incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (wave < 4 && lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int w = 0; w < 3; w++) before += w < wave ? wave_sum[w] : 0u;
  return before + incl - mine;
}

__global__ __launch_bounds__(kSortThreads) void sort_count_kernel(const SortArgs a) {
  __shared__ uint32_t count[kSortDigits];
  const int tid = threadIdx.x, n = sort_rows(a);
  count[tid] = 0;
  __syncthreads();
  const uint32_t mask = (1u << a.bits) - 1u;
  const int base = blockIdx.x * kSortTile + tid;
#pragma unroll
  for (int r = 0; r < kSortRounds; r++) {
    const int t = base + r * kSortThreads;
    if (t < a.rows) atomicAdd(&count[(sort_entry(a, t, n).x >> a.shift) & mask], 1u);
  }
  __syncthreads();
  a.counts[(int64_t)tid * a.digit_stride + (int64_t)blockIdx.x * a.tile_stride] = count[tid];
}

// One workgroup per digit: its counts over the tiles <- their exclusive prefix sums, and the total.
__global__ __launch_bounds__(kSortThreads) void sort_tiles_kernel(const SortArgs a) {
  __shared__ uint32_t wave_sum[4];
  const int tid = threadIdx.x;
  uint32_t* c = a.counts + (int64_t)blockIdx.x * a.tiles;
  uint32_t run = 0;
  for (int b0 = 0; b0 < a.tiles; b0 += kSortThreads) {
    const int b = b0 + tid;
    const uint32_t mine = b < a.tiles ? c[b] : 0u;
    const uint32_t excl = sort_scan256(mine, tid, wave_sum);
    if (b < a.tiles) c[b] = run + excl;
    run += wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
    __syncthreads();
  }
  if (tid == 0) a.counts[(int64_t)kSortDigits * a.tiles + blockIdx.x] = run;
}

// SUM: the counts are as the counting kernel left them, tile by tile (a tile's 256 counts side by
// side, so that the sums below read whole lines).
template <bool SUM>
__global__ __launch_bounds__(kSortThreads) void sort_place_kernel(const SortArgs a) {
  __shared__ uint32_t count[kSortThreads / 64][kSortDigits];
  __shared__ uint32_t wave_sum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = sort_rows(a);
  const uint32_t mask = (1u << a.bits) - 1u;
  // every wavefront takes 512 consecutive entries, 64 at a time
  const int base = blockIdx.x * kSortTile + wave * (64 * kSortRounds) + lane;
  uint2 e[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; r++) e[r] = base + 64 * r < a.rows ? sort_entry(a, base + 64 * r, n) : make_uint2(0u, 0u);
  uint32_t before = 0, total = 0;  // entries of digit tid in earlier tiles, and in all
  if (SUM) {
#pragma unroll 8
    for (int b = 0; b < a.tiles; b++) {
      const uint32_t x = a.counts[b * kSortDigits + tid];
      total += x;
      before += b < (int)blockIdx.x ? x : 0u;
    }
  } else {
    before = a.counts[(int64_t)tid * a.tiles + blockIdx.x];
    total = a.counts[(int64_t)kSortDigits * a.tiles + tid];
  }
#pragma unroll
  for (int w = 0; w < kSortThreads / 64; w++) count[w][tid] = 0;
  before += sort_scan256(total, tid, wave_sum);  // (holds a barrier: the counters are zero)
  uint32_t at[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; r++)
    at[r] = sort_rank((e[r].x >> a.shift) & mask, base + 64 * r < a.rows, a.bits, lane, count[wave]);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kSortThreads / 64; w++) {
    const uint32_t c = count[w][tid];
    count[w][tid] = before;
    before += c;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortRounds; r++)
    if (base + 64 * r < a.rows) a.out[count[wave][(e[r].x >> a.shift) & mask] + at[r]] = e[r];
}

// All passes in one workgroup: rows <= THREADS * kSortSmallRounds, `passes` digits of `bits` bits.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void sort_small_kernel(const SortArgs a, int passes) {
  constexpr int kWaves = THREADS / 64;
  __shared__ uint32_t count[kWaves][kSortDigits];
  __shared__ uint2 entries[THREADS * kSortSmallRounds];
  __shared__ uint32_t wave_sum[4];
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
    uint32_t run = sort_scan256(total, tid, wave_sum);
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
