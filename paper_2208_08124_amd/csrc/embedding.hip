// Host side of fmha_embedding_bwd (include/fmha_varlen.h): argument checks (host memory
// only) and launches on the caller's stream.  Nothing here allocates, copies to the host or waits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "../../include/fmha_varlen.h"
#include "embedding_kernels.h"
#include "embedding_sorted_kernels.h"
#include "host_error.h"
#include "position_sort_kernels.h"

namespace {
using fmha_host::fail;
bool misaligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }
size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Chunk of sorted entries per workgroup: small batches get smaller chunks so that they still
// spread over the chip.
int sort_chunk(int rows) { return rows >= (1 << 17) ? fmha::kEmbChunk : 32; }

// Bits of the sort key: indices 0 .. vocab (vocab itself stands for "skipped").
unsigned key_bits(int vocab) {
  unsigned b = 1;
  while (b < 32 && ((uint64_t)1 << b) <= (uint64_t)vocab) b++;
  return b;
}

// Layout of the workspace of the sorted embedding backward (offsets in bytes).
struct SortSpace {
  size_t moved, sorted, info, partial, counts, bytes;
  int chunks, tiles;
};
SortSpace sort_space(int rows, int hidden) {
  SortSpace s;
  const size_t n = (size_t)(rows > 0 ? rows : 1);
  s.chunks = (int)((n + sort_chunk(rows) - 1) / sort_chunk(rows));
  s.tiles = (int)((n + fmha::kSortTile - 1) / fmha::kSortTile);
  size_t at = 256;
  s.moved = at, at = round_up(at + 8 * n, 256);  // the entries between two passes of the sort
  s.sorted = at, at = round_up(at + 8 * n, 256);
  s.info = at, at = round_up(at + sizeof(fmha::EmbChunkInfo) * (size_t)s.chunks, 256);
  s.partial = at, at = round_up(at + sizeof(float) * 2 * (size_t)hidden * (size_t)s.chunks, 256);
  s.counts = at, at = round_up(at + sizeof(uint32_t) * fmha::kSortWideDigits * ((size_t)s.tiles + 1), 256);
  s.bytes = at;
  return s;
}

// Whether all of dw is cleared ahead of the sums, instead of beside them the rows that no entry names
// (emb_clear_rows).  Beside them costs a bisection in the sorted entries per weight row, ahead of them a
// launch and the writing of every row: narrow rows of large vocabularies are cheaper to write than to
// look up.  Backward with f16 rows, us beside / ahead: 16000 x 128 of 30522 weight rows 17 / 19, of
// 120000 20.6 / 23.3 (uniform indices 17.7 / 21.2), of 250000 30.9 / 27.6; 40000 x 128 of 120000 29.3 /
// 26.7, x 256 29.4 / 31.6; 527340 x 128 of 30522 77 / 79, of 120000 104 / 85, x 256 114 / 106, x 512 187 /
// 181 (uniform 168 / 171), x 768 254 / 279; 300 x 8 of 250000 22.8 / 13.6.  Where the sums' workgroups fit on
// the chip at once and only the clearing ones beside them do not, the last sums wait for a second
// round: 600000 x 128 of 30522 92 / 83 (uniform 79 / 68; x 256 103 / 102 and 89 / 85, left as it is).
constexpr int64_t kSumsResident = 2560;  // workgroups of the chunk kernel: ten per compute unit
int64_t clear_groups(int vocab) { return ((int64_t)vocab + fmha::kEmbClearRows - 1) / fmha::kEmbClearRows; }
bool clear_ahead(int rows, int hidden, int vocab) {
  int64_t steps = 0;
  for (int64_t n = rows; n > 0; n >>= 1) steps += vocab;
  if (steps > 1750000 && hidden < (rows >= (1 << 18) ? 384 : 192)) return true;
  const int64_t sums = ((int64_t)rows + sort_chunk(rows) - 1) / sort_chunk(rows);
  return rows >= (1 << 17) && hidden < 192 && sums <= kSumsResident && sums + clear_groups(vocab) > kSumsResident;
}

template <int DIGITS>
void sort_pass(const fmha::SortArgs& a, bool sum_in_place, hipStream_t st) {
  fmha::sort_count_kernel<DIGITS><<<(unsigned)a.tiles, DIGITS, 0, st>>>(a);
  if (sum_in_place) {
    fmha::sort_place_kernel<DIGITS, true><<<(unsigned)a.tiles, DIGITS, 0, st>>>(a);
  } else {
    fmha::sort_tiles_kernel<DIGITS><<<DIGITS, fmha::kSortTilesThreads, 0, st>>>(a);
    fmha::sort_place_kernel<DIGITS, false><<<(unsigned)a.tiles, DIGITS, 0, st>>>(a);
  }
}
}  // namespace

extern "C" size_t fmha_embedding_sort_workspace_size(int32_t rows, int32_t hidden) {
  if (rows < 0 || hidden <= 0) return 0;
  return sort_space(rows, hidden).bytes;
}

extern "C" int fmha_embedding_sort(const int32_t* indices, const int32_t* n_rows, int32_t rows, int32_t hidden,
                                   int32_t vocab, int32_t padding_idx, void* workspace, size_t workspace_bytes,
                                   void* stream) {
  if (rows < 0 || vocab <= 0) return fail(FMHA_ERR_INVALID_ARG, "rows=%d must not be negative and vocab=%d must be positive", rows, vocab);
  if (hidden <= 0 || (hidden & 7)) return fail(FMHA_ERR_INVALID_ARG, "hidden=%d must be a positive multiple of 8", hidden);
  if (rows > 0 && (!indices || misaligned(indices, 4))) return fail(FMHA_ERR_INVALID_ARG, "indices null or not 4-byte aligned");
  if (n_rows && misaligned(n_rows, 4)) return fail(FMHA_ERR_INVALID_ARG, "n_rows must be 4-byte aligned");
  const SortSpace s = sort_space(rows, hidden);
  if (!workspace || misaligned(workspace, 256)) return fail(FMHA_ERR_WORKSPACE, "workspace is null or not 256-byte aligned (%zu bytes needed)", s.bytes);
  if (workspace_bytes < s.bytes) return fail(FMHA_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, s.bytes);
  fmha_host::g_err[0] = 0;
  if (rows == 0) return FMHA_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* w = static_cast<char*>(workspace);
  uint2* buffers[2] = {reinterpret_cast<uint2*>(w + s.sorted), reinterpret_cast<uint2*>(w + s.moved)};
  // Digits of at most 8 bits, or of 10 where that saves a pass (position_sort_kernels.h has the figures);
  // what fits into one workgroup has no launches to save.
  const int key_size = (int)key_bits(vocab);
  const bool wide = rows > fmha::kSortSmall && (key_size + 9) / 10 < (key_size + 7) / 8;
  const int passes = wide ? (key_size + 9) / 10 : (key_size + 7) / 8, digits = wide ? fmha::kSortWideDigits : fmha::kSortDigits;
  fmha::SortArgs a;
  a.indices = indices;
  a.n_rows = n_rows;
  a.in = nullptr;
  a.counts = reinterpret_cast<uint32_t*>(w + s.counts);
  a.rows = rows;
  a.vocab = vocab;
  a.padding_idx = padding_idx;
  a.tiles = s.tiles;
  const bool sum_in_place = s.tiles <= fmha::kSortSumInPlace;
  a.tile_stride = sum_in_place ? digits : 1;
  a.digit_stride = sum_in_place ? 1 : s.tiles;
  a.bits = (key_size + passes - 1) / passes;
  if (rows <= fmha::kSortSmall) {
    a.out = buffers[0];
    a.shift = 0;
    if (rows <= fmha::kSortTiny)
      fmha::sort_small_kernel<256><<<1, 256, 0, st>>>(a, passes);
    else
      fmha::sort_small_kernel<1024><<<1, 1024, 0, st>>>(a, passes);
  } else {
    for (int p = 0; p < passes; p++) {
      a.out = buffers[(passes - 1 - p) & 1];  // the last pass writes the result
      a.shift = p * a.bits;
      if (wide)
        sort_pass<fmha::kSortWideDigits>(a, sum_in_place, st);
      else
        sort_pass<fmha::kSortDigits>(a, sum_in_place, st);
      a.indices = nullptr;
      a.in = a.out;
    }
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FMHA_ERR_HIP, "position sort launch failed: %s", hipGetErrorString(e));
  return FMHA_OK;
}

extern "C" int fmha_embedding_bwd_sorted(const void* dy, void* workspace, size_t workspace_bytes, int32_t rows,
                                         int32_t hidden, int32_t vocab, int32_t dtype, uint32_t flags, void* dw,
                                         void* stream) {
  if (dtype != FMHA_F16 && dtype != FMHA_BF16) return fail(FMHA_ERR_UNSUPPORTED, "dtype=%d is neither FMHA_F16 nor FMHA_BF16", dtype);
  if (rows < 0 || vocab <= 0) return fail(FMHA_ERR_INVALID_ARG, "rows=%d must not be negative and vocab=%d must be positive", rows, vocab);
  if (hidden <= 0 || (hidden & 7)) return fail(FMHA_ERR_INVALID_ARG, "hidden=%d must be a positive multiple of 8", hidden);
  if (flags & ~FMHA_EMB_ZERO_FIRST) return fail(FMHA_ERR_INVALID_ARG, "flags=%u: only FMHA_EMB_ZERO_FIRST applies to the sorted variant", flags);
  if (!dw || misaligned(dw, 16)) return fail(FMHA_ERR_INVALID_ARG, "dw is null or not 16-byte aligned");
  if (rows > 0 && (!dy || misaligned(dy, 16))) return fail(FMHA_ERR_INVALID_ARG, "dy null or not 16-byte aligned");
  const SortSpace s = sort_space(rows, hidden);
  if (!workspace || misaligned(workspace, 256)) return fail(FMHA_ERR_WORKSPACE, "workspace is null or not 256-byte aligned (%zu bytes needed)", s.bytes);
  if (workspace_bytes < s.bytes) return fail(FMHA_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", workspace_bytes, s.bytes);
  fmha_host::g_err[0] = 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipError_t e;
  const bool fill = (flags & FMHA_EMB_ZERO_FIRST) && (rows == 0 || clear_ahead(rows, hidden, vocab));
  if (fill) {
    const int64_t n16 = (int64_t)vocab * hidden * 2 / 16;
    int64_t g = (n16 + 255) / 256;
    if (g > 256 * 16) g = 256 * 16;
    fmha::zero_fill_kernel<<<(unsigned)g, 256, 0, st>>>(static_cast<uint4*>(dw), n16);
    if ((e = hipGetLastError()) != hipSuccess) return fail(FMHA_ERR_HIP, "zero fill launch failed: %s", hipGetErrorString(e));
  }
  if (rows == 0) return FMHA_OK;
  char* w = static_cast<char*>(workspace);
  fmha::EmbSortedArgs a;
  a.dy = static_cast<const uint32_t*>(dy);
  a.sorted = reinterpret_cast<const uint2*>(w + s.sorted);
  a.info = reinterpret_cast<fmha::EmbChunkInfo*>(w + s.info);
  a.partial = reinterpret_cast<float*>(w + s.partial);
  a.dw = static_cast<uint32_t*>(dw);
  a.rows = rows;
  a.pairs = hidden / 2;
  a.vocab = vocab;
  a.accumulate = (flags & FMHA_EMB_ZERO_FIRST) ? 0 : 1;
  a.clear = (flags & FMHA_EMB_ZERO_FIRST) && !fill ? (int)std::min<int64_t>(clear_groups(vocab), 65536) : 0;  // (they stride)
  const int chunk = sort_chunk(rows);
  const unsigned grid = (unsigned)(a.clear + s.chunks);
  if (dtype == FMHA_BF16) {
    fmha::emb_chunk_kernel<true><<<grid, fmha::kEmbSortThreads, 0, st>>>(a, chunk);
    if (hidden <= fmha::kEmbCombineNarrow)
      fmha::emb_combine_kernel<true, true><<<((unsigned)s.chunks + 1) / 2, fmha::kEmbSortThreads, 0, st>>>(a, chunk);
    else
      fmha::emb_combine_kernel<true, false><<<(unsigned)s.chunks, fmha::kEmbSortThreads, 0, st>>>(a, chunk);
  } else {
    fmha::emb_chunk_kernel<false><<<grid, fmha::kEmbSortThreads, 0, st>>>(a, chunk);
    if (hidden <= fmha::kEmbCombineNarrow)
      fmha::emb_combine_kernel<false, true><<<((unsigned)s.chunks + 1) / 2, fmha::kEmbSortThreads, 0, st>>>(a, chunk);
    else
      fmha::emb_combine_kernel<false, false><<<(unsigned)s.chunks, fmha::kEmbSortThreads, 0, st>>>(a, chunk);
  }
  if ((e = hipGetLastError()) != hipSuccess) return fail(FMHA_ERR_HIP, "sorted embedding backward launch failed: %s", hipGetErrorString(e));
  return FMHA_OK;
}

extern "C" int fmha_embedding_bwd(const void* dy, const int32_t* indices, const int32_t* n_rows, int32_t rows,
                                  int32_t hidden, int32_t vocab, int32_t padding_idx, int32_t dtype, uint32_t flags,
                                  void* dw, void* stream) {
  if (dtype != FMHA_F16 && dtype != FMHA_BF16) return fail(FMHA_ERR_UNSUPPORTED, "dtype=%d is neither FMHA_F16 nor FMHA_BF16", dtype);
  if (rows < 0 || vocab <= 0) return fail(FMHA_ERR_INVALID_ARG, "rows=%d must not be negative and vocab=%d must be positive", rows, vocab);
  if (hidden <= 0 || (hidden & 7)) return fail(FMHA_ERR_INVALID_ARG, "hidden=%d must be a positive multiple of 8", hidden);
  if (!dw || misaligned(dw, 16)) return fail(FMHA_ERR_INVALID_ARG, "dw is null or not 16-byte aligned");
  if (rows > 0 && (!dy || !indices || misaligned(dy, 4) || misaligned(indices, 4)))
    return fail(FMHA_ERR_INVALID_ARG, "dy / indices null or not 4-byte aligned");
  if (n_rows && misaligned(n_rows, 4)) return fail(FMHA_ERR_INVALID_ARG, "n_rows must be 4-byte aligned");
  fmha_host::g_err[0] = 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (flags & FMHA_EMB_ZERO_FIRST) {
    const int64_t n16 = (int64_t)vocab * hidden * 2 / 16;
    int64_t g = (n16 + 255) / 256;
    if (g > 256 * 16) g = 256 * 16;
    fmha::zero_fill_kernel<<<(unsigned)g, 256, 0, st>>>(static_cast<uint4*>(dw), n16);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FMHA_ERR_HIP, "zero fill launch failed: %s", hipGetErrorString(e));
  }
  if (rows == 0) return FMHA_OK;
  fmha::EmbArgs a;
  a.dy = static_cast<const uint32_t*>(dy);
  a.indices = indices;
  a.n_rows = n_rows;
  a.dw = static_cast<uint32_t*>(dw);
  a.rows = rows;
  a.pairs = hidden / 2;
  a.vocab = vocab;
  a.padding_idx = padding_idx;
  const int per = fmha::kEmbThreads / 64;
  const bool bf16 = dtype == FMHA_BF16;
  if (flags & FMHA_EMB_PLAIN_SPLIT) {
    int64_t g = ((int64_t)rows + per - 1) / per;
    if (g > 256 * 8) g = 256 * 8;
    if (bf16)
      fmha::embedding_bwd_kernel<true><<<(unsigned)g, fmha::kEmbThreads, 0, st>>>(a);
    else
      fmha::embedding_bwd_kernel<false><<<(unsigned)g, fmha::kEmbThreads, 0, st>>>(a);
  } else {
    // 64-token windows while the batch is small (more workgroups), 256-token windows once
    // there are enough of them to fill the chip several times over (more merging; 128 and 512
    // were both slower on 527 340 Zipf-distributed rows: 0.74 / 0.65 / 0.82 ms)
    const int nw = rows >= (1 << 17) ? 4 : 1;
    const int window = 64 * nw;
    const bool die = !(flags & FMHA_EMB_NO_DIE_SPLIT);
    int64_t g = ((int64_t)rows + window - 1) / window;  // one window per workgroup and trip (per die, if split)
    const int64_t cap = die ? 256 : 256 * 8;
    if (g > cap) g = cap;
    if (g < 1) g = 1;
    if (die) g *= 8;
    const unsigned grid = (unsigned)g;
#define FMHA_EMB_LAUNCH(BF, DIE)                                                                          \
  do {                                                                                                    \
    if (nw == 4)                                                                                          \
      fmha::embedding_bwd_window_kernel<BF, DIE, 4><<<grid, fmha::kEmbThreads, 0, st>>>(a);               \
    else                                                                                                  \
      fmha::embedding_bwd_window_kernel<BF, DIE, 1><<<grid, fmha::kEmbThreads, 0, st>>>(a);               \
  } while (0)
    if (bf16) {
      if (die) FMHA_EMB_LAUNCH(true, true); else FMHA_EMB_LAUNCH(true, false);
    } else {
      if (die) FMHA_EMB_LAUNCH(false, true); else FMHA_EMB_LAUNCH(false, false);
    }
#undef FMHA_EMB_LAUNCH
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FMHA_ERR_HIP, "embedding backward launch failed: %s", hipGetErrorString(e));
  return FMHA_OK;
}
