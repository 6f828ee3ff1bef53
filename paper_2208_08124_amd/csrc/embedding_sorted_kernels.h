// Embedding backward without atomics, for callers that know the indices before the gradient
// arrives (the paper computes its index tensors once per mini-batch, Section IV-B-2, and
// names the colliding additions of Section IV-C-3 as the cost of this step): the token
// positions are ordered by index once (position_sort_kernels.h, a call of its own), and the
// gradient rows of an index are then summed in fp32 in that order and written as ONE row.
//
// The sorted positions are cut into chunks of 256 entries, one workgroup each.  A workgroup
// walks its chunk run by run (a run = consecutive entries with the same index).  A run that
// begins and ends inside the chunk is finished on the spot: weight row = old row + sum,
// rounded once.  A run that reaches into the chunk from before ("head") or out of it at the
// end ("tail") leaves its fp32 partial sum in the workspace; a second kernel adds the partial
// sums of each such run in chunk order and writes the row.  Every weight row has exactly one
// writer and every sum a fixed order: results are identical from run to run.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fmha {

constexpr int kEmbChunk = 256;    // sorted entries per workgroup
constexpr int kEmbSortThreads = 128;

// What the two kernels pass through the workspace, per chunk.
struct EmbChunkInfo {
  int32_t head_key;    // index of the run that reaches in from the chunk before, or -1
  int32_t head_whole;  // 1 if that run covers the whole chunk and goes on into the next one
  int32_t tail_key;    // index of the run that goes on into the next chunk and began in this one, or -1
  int32_t pad;
};

struct EmbSortedArgs {
  const uint32_t* dy;     // [rows, pairs] packed pairs of 16-bit values
  const uint2* sorted;    // [rows] {index, or vocab for entries that are skipped (sorted last); token position}
  EmbChunkInfo* info;     // [chunks]
  float* partial;         // [chunks][2][2 * pairs]: head and tail partial sums
  uint32_t* dw;           // [vocab, pairs]
  int32_t rows, pairs, vocab;
  int32_t accumulate;     // 1: add onto the weight rows that are there, 0: they count as zero
  int32_t clear;          // workgroups of the chunk kernel that clear the rows nothing is added onto (0 if accumulate)
};

// x (eight 16-bit values in four dwords) added onto eight fp32 sums
template <bool BF16>
static __device__ __forceinline__ void emb_add8(const uint4& x, float (&s)[8]) {
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int i = 0; i < 4; i++) {
    if (BF16) {
      s[2 * i] += __builtin_bit_cast(float, w[i] << 16);
      s[2 * i + 1] += __builtin_bit_cast(float, w[i] & 0xffff0000u);
    } else {
      s[2 * i] += (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] & 0xffffu));
      s[2 * i + 1] += (float)__builtin_bit_cast(_Float16, (uint16_t)(w[i] >> 16));
    }
  }
}

// the sums (plus the old weight values, if they count) rounded once to the 16-bit type
template <bool BF16>
static __device__ __forceinline__ uint4 emb_finish8(const uint4& old, float (&s)[8], bool accumulate) {
  if (accumulate) emb_add8<BF16>(old, s);
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    if (BF16) {
      typedef __bf16 b2 __attribute__((ext_vector_type(2)));
      w[i] = __builtin_bit_cast(uint32_t, b2{(__bf16)s[2 * i], (__bf16)s[2 * i + 1]});
    } else {
      typedef _Float16 h2 __attribute__((ext_vector_type(2)));
      w[i] = __builtin_bit_cast(uint32_t, h2{(_Float16)s[2 * i], (_Float16)s[2 * i + 1]});
    }
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// Weight rows first .. first + kEmbClearRows - 1 that no sorted entry names <- zeros (the others
// are written whole by their one writer, so clearing all of them ahead of the sums would move
// most of dw twice and cost a launch: 9 us for 30522 x 768 weights).  A thread looks its row up
// in the sorted entries by bisection; these workgroups come first in the grid, so that their
// chains of loads run beside the sums.  (Narrow rows of large vocabularies: see clear_ahead.)
constexpr int kEmbClearRows = 64;
static __device__ void emb_clear_rows(const EmbSortedArgs& a, int first, uint32_t* s_absent) {
  const int tid = threadIdx.x, n = min(kEmbClearRows, a.vocab - first);
  if (tid < n) {
    const uint32_t row = (uint32_t)(first + tid);
    int lo = 0, hi = a.rows;  // first entry whose index is not below `row`
    while (lo < hi) {
      const int mid = lo + ((hi - lo) >> 1);
      if (a.sorted[mid].x < row)
        lo = mid + 1;
      else
        hi = mid;
    }
    s_absent[tid] = lo == a.rows || a.sorted[lo].x != row;
  }
  __syncthreads();
  const int pieces = a.pairs >> 2;  // of 16 bytes
  for (int r = 0; r < n; r++) {
    if (!s_absent[r]) continue;  // uniform
    uint4* w = reinterpret_cast<uint4*>(a.dw) + (int64_t)(first + r) * pieces;
    for (int i = tid; i < pieces; i += kEmbSortThreads) w[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  __syncthreads();  // s_absent may be written again
}

constexpr int kEmbAhead = 16;  // rows a thread has in flight

// One workgroup per chunk of `chunk` (<= kEmbChunk) sorted entries; thread i owns the columns
// 8i .. 8i+7 (and 8(i + 128) .. for rows wider than 1024 values) and walks the chunk's rows in
// order, sixteen 16-byte loads in flight.  What happens at the end of a run is worked out once
// per chunk (one entry per thread) and kept in LDS as index * 4 + action.
template <bool BF16>
__global__ __launch_bounds__(kEmbSortThreads) void emb_chunk_kernel(const EmbSortedArgs a, const int chunk) {
  __shared__ uint32_t s_code[kEmbChunk];  // index * 4 + {0: the run goes on, 1: head partial, 2: tail partial, 3: final row}
  __shared__ uint32_t s_pos[kEmbChunk];
  __shared__ int s_live;                  // entries of the chunk that count (skipped ones are sorted last)
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < a.clear) {
    for (int64_t first = (int64_t)blockIdx.x * kEmbClearRows; first < a.vocab; first += (int64_t)a.clear * kEmbClearRows)
      emb_clear_rows(a, (int)first, s_pos);
    return;
  }
  const int c = blockIdx.x - a.clear;
  const int base = c * chunk;
  const int n = min(chunk, a.rows - base);
  const uint32_t none = (uint32_t)a.vocab;
  const uint32_t first = a.sorted[base].x, last = a.sorted[base + n - 1].x;
  const uint32_t before = base > 0 ? a.sorted[base - 1].x : none, after = base + n < a.rows ? a.sorted[base + n].x : none;
  const bool head = first != none && before == first;  // the first run began before this chunk
  const bool tail = last != none && after == last;     // the last run goes on after it
  if (tid == 0) {
    EmbChunkInfo inf;
    inf.head_key = head ? (int32_t)first : -1;
    inf.head_whole = head && tail && first == last;
    inf.tail_key = (tail && !(head && first == last)) ? (int32_t)last : -1;
    inf.pad = 0;
    a.info[c] = inf;
    s_live = 0;
  }
  __syncthreads();
  for (int r = tid; r < n; r += kEmbSortThreads) {
    const uint2 entry = a.sorted[base + r];
    const uint32_t key = entry.x;
    const uint32_t next = r + 1 < n ? a.sorted[base + r + 1].x : after;
    uint32_t action = 0;
    if (key != none && (r == n - 1 || next != key)) {  // the run ends here, or leaves the chunk
      if (head && key == first)
        action = 1;  // (sorted: the run of `first` is the chunk's first run)
      else if (r == n - 1 && tail)
        action = 2;
      else
        action = 3;
    }
    s_code[r] = key * 4u + action;
    s_pos[r] = entry.y;
    if (key != none && (r == n - 1 || next == none)) s_live = r + 1;  // exactly one entry qualifies
  }
  __syncthreads();
  const int live = s_live;
  const int hidden = 2 * a.pairs;
  float* part = a.partial + (int64_t)c * 2 * hidden;  // [head | tail][hidden]
  const uint16_t* dy = reinterpret_cast<const uint16_t*>(a.dy);
  uint16_t* dw = reinterpret_cast<uint16_t*>(a.dw);
  for (int col = 8 * tid; col < hidden; col += 8 * kEmbSortThreads) {
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int r0 = 0; r0 < live; r0 += kEmbAhead) {  // (uniform over the workgroup)
      uint4 x[kEmbAhead];
#pragma unroll
      for (int u = 0; u < kEmbAhead; u++)
        x[u] = *reinterpret_cast<const uint4*>(dy + (int64_t)s_pos[min(r0 + u, live - 1)] * hidden + col);
#pragma unroll
      for (int u = 0; u < kEmbAhead; u++) {
        const int r = r0 + u;
        if (r >= live) break;
        emb_add8<BF16>(x[u], s);
        const uint32_t code = s_code[r];
        if (code & 3u) {
          if ((code & 3u) == 3u) {
            uint4* w = reinterpret_cast<uint4*>(dw + (int64_t)(code >> 2) * hidden + col);
            *w = emb_finish8<BF16>(a.accumulate ? *w : make_uint4(0u, 0u, 0u, 0u), s, a.accumulate != 0);
          } else {
            float4* p = reinterpret_cast<float4*>(part + ((code & 3u) == 2u ? hidden : 0) + col);
            p[0] = make_float4(s[0], s[1], s[2], s[3]);
            p[1] = make_float4(s[4], s[5], s[6], s[7]);
          }
#pragma unroll
          for (int i = 0; i < 8; i++) s[i] = 0.f;
        }
      }
    }
  }
}

// One workgroup (or wavefront) per chunk in which a run begins that goes on into later chunks: its partial
// sums are added in chunk order and the row is written.  Where the run ends is found first (the
// first later chunk that it does not cover whole, 128 chunks at a time, by each wavefront for
// itself), so that the partial sums - up to a few hundred for the most frequent index of a large
// batch, and its one workgroup is what the kernel waits for - can then be fetched kEmbCombineAhead
// at a time and added in order (527340 Zipf-distributed rows of 768: 60 us with four at a time
// behind a binary search for the end, 18 so).  Runs of few partial sums, the usual ones of a uniform
// distribution, fetch no more than kEmbCombineFew: 65536 rows of 128, 8192 indices, both
// kernels, 15.5 us without that and with the end agreed on in LDS, 13.8 so.  The loads in flight take
// 154 registers, six workgroups per compute unit: on rows of up to kEmbCombineNarrow columns, which
// leave one of their two wavefronts idle, each wavefront takes a chunk of its own (500000 rows of 128,
// uniform over 8192 indices, accumulating: 63.4 us without, 56.3 so; rows of 512 the same either way).
constexpr int kEmbCombineAhead = 16, kEmbCombineFew = 4, kEmbCombineNarrow = 256;
template <bool BF16, bool NARROW>
__global__ __launch_bounds__(kEmbSortThreads) void emb_combine_kernel(const EmbSortedArgs a, const int chunk) {
  const int chunks = (a.rows - 1) / chunk + 1, lane = threadIdx.x & 63;
  const int c = NARROW ? 2 * blockIdx.x + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : blockIdx.x;  // (uniform)
  if (NARROW && c >= chunks) return;
  const int key = a.info[c].tail_key;
  if (key < 0) return;
  int d_last;
  for (int d0 = c + 1;; d0 += 128) {  // (a run ends in the last chunk at the latest)
    const uint64_t near = __ballot(!a.info[min(d0 + lane, chunks - 1)].head_whole);
    const uint64_t far = __ballot(!a.info[min(d0 + 64 + lane, chunks - 1)].head_whole);
    if (near | far) {
      d_last = min(d0 + (near ? __builtin_ctzll(near) : 64 + __builtin_ctzll(far)), chunks - 1);
      break;
    }
  }
  const int hidden = 2 * a.pairs;
  uint16_t* dw = reinterpret_cast<uint16_t*>(a.dw);
  for (int col = 8 * (NARROW ? lane : threadIdx.x); col < hidden; col += 8 * kEmbSortThreads) {
    const float4* p = reinterpret_cast<const float4*>(a.partial + ((int64_t)c * 2 + 1) * hidden + col);
    float s[8] = {p[0].x, p[0].y, p[0].z, p[0].w, p[1].x, p[1].y, p[1].z, p[1].w};
    // (both forms written out: as one function of the number the longer one took 2 - 7 % more)
    if (d_last - c <= kEmbCombineFew) {
      const int d0 = c + 1;
      float4 t[kEmbCombineFew][2];
#pragma unroll
      for (int u = 0; u < kEmbCombineFew; u++) {
        const float4* q = reinterpret_cast<const float4*>(a.partial + (int64_t)min(d0 + u, d_last) * 2 * hidden + col);
        t[u][0] = q[0];
        t[u][1] = q[1];
      }
#pragma unroll
      for (int u = 0; u < kEmbCombineFew; u++) {
        if (d0 + u <= d_last) {
          s[0] += t[u][0].x, s[1] += t[u][0].y, s[2] += t[u][0].z, s[3] += t[u][0].w;
          s[4] += t[u][1].x, s[5] += t[u][1].y, s[6] += t[u][1].z, s[7] += t[u][1].w;
        }
      }
    } else {
      for (int d0 = c + 1; d0 <= d_last; d0 += kEmbCombineAhead) {
        float4 t[kEmbCombineAhead][2];
#pragma unroll
        for (int u = 0; u < kEmbCombineAhead; u++) {
          const float4* q = reinterpret_cast<const float4*>(a.partial + (int64_t)min(d0 + u, d_last) * 2 * hidden + col);
          t[u][0] = q[0];
          t[u][1] = q[1];
        }
#pragma unroll
        for (int u = 0; u < kEmbCombineAhead; u++) {
          if (d0 + u <= d_last) {
            s[0] += t[u][0].x, s[1] += t[u][0].y, s[2] += t[u][0].z, s[3] += t[u][0].w;
            s[4] += t[u][1].x, s[5] += t[u][1].y, s[6] += t[u][1].z, s[7] += t[u][1].w;
          }
        }
      }
    }
    uint4* w = reinterpret_cast<uint4*>(dw + (int64_t)key * hidden + col);
    *w = emb_finish8<BF16>(a.accumulate ? *w : make_uint4(0u, 0u, 0u, 0u), s, a.accumulate != 0);
  }
}

}  // namespace fmha
