// Host side of the C ABI declared in include/fmha_varlen.h: argument checks
// (host memory only), workspace carving, and the launches.  One launch per
// direction and kernel on the caller's stream; nothing here allocates,
// copies to the host or waits for the device.
#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>

#include "../../include/fmha_varlen.h"
#include "host_error.h"
#include "bwd_fused_kernel.h"
#include "bwd_kernels.h"
#include "fwd64_kernel.h"
#include "fwd_kernel.h"
#include "keep_mask_kernel.h"
#include "schedule.h"

namespace fmha_host {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

}  // namespace fmha_host

namespace {

using fmha_host::fail;
using fmha_host::g_err;

constexpr size_t kAlign = 256;
size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Tiles of 128 rows: sum_i ceil(L_i/128) <= T/128 + B for any lengths.
int64_t tile_capacity(int64_t batch, int64_t total_tokens) {
  return total_tokens / fmha::kTileRows + batch;
}

struct Workspace {
  int32_t* count;
  uint32_t* feed;  // the item feed's counters (item_feed.h)
  fmha::TileItem* list;
  float* dsum;
  float* lse2;
  fmha::TileItem* seqs;  // the sequences, for the one-pass backward
  float* slab;           // its fp32 dQ between sweeps
  size_t count_off, feed_off, list_off, seqs_off, dsum_off, lse2_off, slab_off, bytes_list, bytes_fwd, bytes_bwd;
};

// Workgroups of the one-pass backward at most, and rows of fp32 dQ that each may be given.
constexpr int64_t kFusedGrid = 256, kFusedSlabRows = 2048;

// Workgroups of the one-pass backward for `items` items and at most `units` of them: a multiple of 8.
int64_t fused_grid(int64_t items, int64_t units = kFusedGrid) { return ((items < units ? items : units) + 7) / 8 * 8; }

Workspace carve(void* base, int64_t batch, int64_t total_tokens, int64_t heads) {
  Workspace w;
  w.count_off = 0;
  w.feed_off = kAlign;
  w.list_off = w.feed_off + sizeof(uint32_t) * fmha::kFeedWords;
  const size_t list_bytes = sizeof(fmha::TileItem) * (size_t)(tile_capacity(batch, total_tokens) + 1);
  w.bytes_list = w.list_off + list_bytes;
  w.seqs_off = round_up(w.bytes_list, kAlign);
  w.dsum_off = round_up(w.seqs_off + sizeof(fmha::TileItem) * (size_t)batch, kAlign);
  w.bytes_fwd = w.dsum_off;
  // one float per (token, head) plus one pad entry
  const size_t stat_bytes = round_up(sizeof(float) * ((size_t)total_tokens * (size_t)heads + 1), kAlign);
  w.lse2_off = w.dsum_off + stat_bytes;
  // dQ between sweeps: a workgroup needs no more rows than a sequence has, and there are no more
  // workgroups on long sequences than there are rows in all heads; but 256 rows for every workgroup
  // in any case (what is stated of the longest sequence may be wrong)
  w.slab_off = w.lse2_off + stat_bytes;
  const int64_t rows = ((int64_t)total_tokens + 255) / 256 * 256;
  int64_t slab = kFusedGrid * (rows < kFusedSlabRows ? rows : kFusedSlabRows);
  if (slab > rows * heads) slab = rows * heads;
  if (slab < fused_grid(batch * heads) * fmha::kFusedKeys) slab = fused_grid(batch * heads) * fmha::kFusedKeys;
  if (total_tokens <= fmha::kFusedKeys) slab = 0;
  w.bytes_bwd = w.slab_off + (size_t)slab * fmha::kHeadDim * sizeof(float);
  // (base is null when only the sizes are wanted: no pointer arithmetic on it then)
  const uintptr_t b = reinterpret_cast<uintptr_t>(base);
  auto at = [b](size_t off) { return b ? reinterpret_cast<void*>(b + off) : nullptr; };
  w.count = static_cast<int32_t*>(at(w.count_off));
  w.feed = static_cast<uint32_t*>(at(w.feed_off));
  w.list = static_cast<fmha::TileItem*>(at(w.list_off));
  w.dsum = static_cast<float*>(at(w.dsum_off));
  w.lse2 = static_cast<float*>(at(w.lse2_off));
  w.seqs = static_cast<fmha::TileItem*>(at(w.seqs_off));
  w.slab = static_cast<float*>(at(w.slab_off));
  return w;
}

bool misaligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

int check_stride(const char* name, int64_t s, int64_t dense, int64_t* out) {
  if (s == 0) s = dense;
  if (s < dense || (s & 7)) return fail(FMHA_ERR_INVALID_ARG, "%s_stride=%lld must be 0 or a multiple of 8 that is >= heads*64=%lld",
                                        name, (long long)s, (long long)dense);
  // the kernels address the 64 rows of a block with 32-bit byte offsets from a 64-bit base
  if (s > ((int64_t)1 << 24)) return fail(FMHA_ERR_INVALID_ARG, "%s_stride=%lld exceeds 2^24 elements", name, (long long)s);
  *out = s;
  return FMHA_OK;
}

int check_common(const fmha_varlen_params_t* p, bool bwd, bool list_only = false) {
  if (!p) return fail(FMHA_ERR_INVALID_ARG, "params is null");
  if (p->head_dim != fmha::kHeadDim) return fail(FMHA_ERR_UNSUPPORTED, "head_dim=%d, only 64 is supported", p->head_dim);
  if (p->dtype != FMHA_F16 && p->dtype != FMHA_BF16) return fail(FMHA_ERR_UNSUPPORTED, "dtype=%d is neither FMHA_F16 nor FMHA_BF16", p->dtype);
  if (p->batch < 0) return fail(FMHA_ERR_INVALID_ARG, "batch=%d is negative", p->batch);
  if (p->total_tokens < 0) return fail(FMHA_ERR_INVALID_ARG, "total_tokens=%d is negative", p->total_tokens);
  if (p->heads <= 0) return fail(FMHA_ERR_INVALID_ARG, "heads=%d must be positive", p->heads);
  if ((int64_t)p->total_tokens * p->heads > (int64_t)1 << 40) return fail(FMHA_ERR_INVALID_ARG, "total_tokens*heads too large");
  if (!(p->scale == p->scale) || p->scale - p->scale != 0.f) return fail(FMHA_ERR_INVALID_ARG, "scale is not finite");
  if (!p->cu_seqlens) return fail(FMHA_ERR_INVALID_ARG, "cu_seqlens is null");
  if (misaligned(p->cu_seqlens, 4) || (p->seqused && misaligned(p->seqused, 4)))
    return fail(FMHA_ERR_INVALID_ARG, "cu_seqlens/seqused must be 4-byte aligned");
  if (p->cu_seqlens_host) {
    const int32_t* cu = p->cu_seqlens_host;
    if (cu[0] != 0) return fail(FMHA_ERR_INVALID_ARG, "cu_seqlens_host[0]=%d, expected 0", cu[0]);
    for (int i = 0; i < p->batch; i++) {
      if (cu[i + 1] < cu[i]) return fail(FMHA_ERR_INVALID_ARG, "cu_seqlens_host decreases at %d (%d -> %d)", i, cu[i], cu[i + 1]);
      if (p->max_seqlen > 0 && cu[i + 1] - cu[i] > p->max_seqlen)
        return fail(FMHA_ERR_INVALID_ARG, "sequence %d has %d tokens, more than max_seqlen=%d", i, cu[i + 1] - cu[i], p->max_seqlen);
    }
    if (cu[p->batch] != p->total_tokens)
      return fail(FMHA_ERR_INVALID_ARG, "cu_seqlens_host[batch]=%d differs from total_tokens=%d", cu[p->batch], p->total_tokens);
  }
  // (a backward without room for fp32 dQ between sweeps takes the two passes, which use none)
  const Workspace sizes = carve(nullptr, p->batch, p->total_tokens, p->heads);
  const size_t need = list_only ? sizes.bytes_list : bwd ? sizes.slab_off : sizes.bytes_fwd;
  if (!p->workspace) return fail(FMHA_ERR_WORKSPACE, "workspace is null (%zu bytes needed)", need);
  if (misaligned(p->workspace, kAlign)) return fail(FMHA_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (p->workspace_bytes < need) return fail(FMHA_ERR_WORKSPACE, "workspace has %zu bytes, %zu needed", p->workspace_bytes, need);
  return FMHA_OK;
}

int check_ptr(const char* name, const void* ptr) {
  if (!ptr) return fail(FMHA_ERR_INVALID_ARG, "%s is null", name);
  if (misaligned(ptr, 16)) return fail(FMHA_ERR_INVALID_ARG, "%s is not 16-byte aligned", name);
  return FMHA_OK;
}

// Compute units of the current device (host query, cached per device).
int compute_units() {
  thread_local int cached_dev = -1, cached_cus = 0;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (dev != cached_dev) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached_dev = dev;
    cached_cus = n;
  }
  return cached_cus;
}

// Workgroups launched: persistent, `per_cu` per compute unit, but never more than
// the (tile, head) items that can exist.  max_seqlen, when given, tightens that
// bound; the kernels stride over the list, so a wrong bound costs time, never
// correctness.
unsigned grid_for(const fmha_varlen_params_t* p, int per_cu) {
  int64_t tiles = tile_capacity(p->batch, p->total_tokens);
  if (p->max_seqlen > 0) {
    const int64_t per_seq = (p->max_seqlen + fmha::kTileRows - 1) / fmha::kTileRows;
    if (per_seq * p->batch < tiles) tiles = per_seq * p->batch;
  }
  int64_t g = tiles * p->heads;
  const int64_t resident = (int64_t)compute_units() * per_cu;
  if (g > resident) g = resident;
  if (g < 1) g = 1;
  return (unsigned)g;
}

int launch_schedule(const fmha_varlen_params_t* p, const Workspace& w, hipStream_t st) {
  if (p->flags & FMHA_FLAG_REUSE_SCHEDULE) return FMHA_OK;
  const int cap = (int)tile_capacity(p->batch, p->total_tokens);
  fmha::schedule_kernel<<<w.seqs ? 2 : 1, fmha::kSchedThreads, 0, st>>>(p->cu_seqlens, p->seqused, p->batch, p->total_tokens,
                                                                       w.count, w.list, cap, w.feed, w.seqs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FMHA_ERR_HIP, "schedule launch failed: %s", hipGetErrorString(e));
  return FMHA_OK;
}

fmha::Problem problem_of(const fmha_varlen_params_t* p, const Workspace& w) {
  fmha::Problem pb;
  pb.n_tiles = w.count;
  pb.tiles = w.list;
  pb.heads = p->heads;
  pb.total_tokens = p->total_tokens;
  pb.scale = p->scale;
  return pb;
}

// Upper bound on the number of (tile, head) items, from host-visible sizes only.
int64_t items_bound(const fmha_varlen_params_t* p) {
  int64_t tiles = tile_capacity(p->batch, p->total_tokens);
  if (p->max_seqlen > 0) {
    const int64_t per_seq = (p->max_seqlen + fmha::kTileRows - 1) / fmha::kTileRows;
    if (per_seq * p->batch < tiles) tiles = per_seq * p->batch;
  }
  return tiles * p->heads;
}

// Persistent grid of `per_cu` workgroups per compute unit (a multiple of 8, never more than
// there can be items), and the item feed's chunk size for it: about 24 chunks per workgroup
// on large batches, single items on small ones.
unsigned feed_grid(const fmha_varlen_params_t* p, int per_cu, const Workspace& w, fmha::FeedArgs* feed) {
  const int64_t items = items_bound(p);
  int64_t g = (int64_t)compute_units() * per_cu;
  if (g > items) g = items;
  g = (g + 7) / 8 * 8;
  if (g < 8) g = 8;
  int64_t chunk = items / (g * 24);
  if (chunk < 1) chunk = 1;
  if (chunk > 256) chunk = 256;
  feed->counters = w.feed;
  feed->chunk = (int32_t)chunk;
  return (unsigned)g;
}

// Workgroups of the one-pass backward that run at a time: one per compute unit.
int64_t fused_units() { return compute_units() < kFusedGrid ? compute_units() : kFusedGrid; }

// Rows of fp32 dQ for each workgroup of the one-pass backward.
// (a multiple of 256: the sweeps of a sequence that needs more begin at multiples of eight blocks)
int32_t fused_slab_rows(const fmha_varlen_params_t* p) {
  int64_t rows = p->max_seqlen > 0 && p->max_seqlen < p->total_tokens ? p->max_seqlen : p->total_tokens;
  rows = (rows + 255) / 256 * 256;
  return (int32_t)(rows < kFusedSlabRows ? rows : kFusedSlabRows);
}

// Whether the backward runs as one pass (bwd_fused_kernel.h) or as two (bwd_kernels.h).  The figures are
// two passes' time over one's, without / with dropout, from 750 batches of 1 - 16 heads, 24 - 2048 tokens and lengths
// equal, uniform, mostly long and mostly short, and 250 more with key counts of their own.
//
// The one pass is 1.1 - 1.5 / 1.1 - 1.8 times as fast while all compute units are busy, but its items are
// whole sequences, where the two passes have tiles of 128 rows to deal out.  A compute unit's share of the
// work is estimated from below by what the batch would be with all sequences as long (in steps of 256 keys by 32
// queries), and held against the longest sequence.
//  - More rows than the fp32 dQ between sweeps has room for: the scores would be formed twice after all.
//    Nor without that room in the workspace, whatever the lengths (the longest may have been stated too small).
//  - Up to 256 tokens (one sweep an item) it pays from a fifth of the longest sequence on: 0.98 / 0.99 at
//    0.12 - 0.15, 1.04 - 1.5 / 1.06 - 1.7 from 0.2 on, even where a second round of items is nearly empty.
//    Equal lengths of 65 - 80 leave a wavefront in four without a key: 0.93 - 0.97 / 0.97 - 1.09.
//  - Longer sequences that are (nearly) all equal take whole rounds: 0.72 - 1.1 / 0.69 - 1.2 where the rounds are 0.5 - 0.65 full,
//    0.96 - 1.4 / 0.92 - 1.3 from 0.7 on (0.93 - 1.0 / 0.86 - 1.06 above 1024 tokens at 0.79 - 0.88).  With few keys in a second sweep
//    that sweep costs more than it saves: 257 - 320 tokens 0.85 - 1.03 / 0.85 - 1.0 in more than one round, with
//    dropout 0.93 - 1.04 up to 416.
//  - Longer sequences of mixed lengths: up to 512 tokens 0.8 - 1.2 / 0.7 - 1.1 at 0.2 - 0.4 of the longest, 0.97 - 1.0 / 0.96 - 1.02 at
//    0.62 - 0.64, 1.0 - 1.2 / 0.98 - 1.12 from 0.65 on; up to 1024 one batch of 33 0.90 / 0.87 at 0.76 (another, of 34, 0.81 / 1.02 at
//    0.67), 1.05 - 1.2 from 0.8 on; above, 0.95 - 1.02 / 0.86 - 0.95 at 0.5 - 0.64.  Where most are short the squares of the longer ones make
//    the share larger than it is estimated here: 1.0 - 1.3 / 1.0 - 1.35 from 0.3 on up to 1024 tokens.
//  - Sequences of up to 64 (128) tokens are taken four (two) heads at a time, and places without a head cost as
//    much as others.  Heads 1 / 2 / 3 / 5 / 6, without dropout: up to 64 tokens 0.47 / 0.87 / 1.09 / 0.89 / 1.02, up to 128
//    0.6 - 0.86 / 0.96 - 1.06 / 0.8 - 0.95 / 0.94 - 0.99 / 1.0, up to 160 0.79 / 1.12 / 0.97, up to 256 1.0 / 1.17 / 0.94; with dropout (where an
//    empty place makes no mask) 0.6 / 1.1 / 1.4 / 1.16 / 1.34, 0.67 - 0.87 / 1.12 - 1.2 / 0.8 - 1.03 / 1.07 - 1.13 / 1.19, 0.92 / 1.21 / 1.07,
//    1.07 / 1.2 / 1.0.  The length that counts is twice the mean where that is less than the longest.
//  - With key counts of their own (seqused) all sequences are taken one head at a time, and the work goes by counts that the
//    host does not know: rows of up to 64 tokens 0.44 - 0.75 / 0.54 - 0.83, up to 128 0.6 - 0.97 / 0.64 - 0.9, 129 - 256 1.0 - 1.4 / 0.98 - 1.37;
//    longer ones in full rounds 0.96 - 1.5 / 0.98 - 1.4 from a share as large as the longest sequence on.
bool one_pass(const fmha_varlen_params_t* p, const Workspace& w, bool dropout) {
  if (p->flags & (FMHA_FLAG_BWD_ONLY_DQ | FMHA_FLAG_BWD_ONLY_DKV)) return false;
  const int64_t total = p->total_tokens;
  const int h = p->heads, n = (int)(p->max_seqlen < total ? p->max_seqlen : total);
  if (n <= 0 || p->batch <= 0 || n > kFusedSlabRows) return false;
  const size_t slab = (size_t)fused_grid((int64_t)p->batch * h, fused_units()) * (size_t)fused_slab_rows(p) * fmha::kHeadDim * sizeof(float);
  const size_t given = p->workspace_bytes < w.bytes_bwd ? p->workspace_bytes : w.bytes_bwd;
  if (total > fmha::kFusedKeys && given - w.slab_off < slab) return false;
  const int64_t units = fused_units(), items = (int64_t)p->batch * h, rounds = (items + units - 1) / units;
  const double mean = (double)total / p->batch, full = (double)items / (double)(rounds * units);
  const double longest = (double)((n + 255) / 256) * ((n + 31) / 32);
  const double share = (double)total * mean * h / (256. * 32. * (double)units) / longest;
  if (p->seqused) return mean > 128 && (n <= fmha::kFusedKeys ? share >= 0.2 : share >= 1. && full >= 0.85);
  const double len = 2 * mean < n ? 2 * mean : n;
  if (dropout) {
    if (h == 1 && len <= 192) return false;
    if (h == 3 && len > 64 && len <= 128) return false;
  } else {
    if (len <= 128 && h < 0.75 * ((h + 3) / 4 * 4)) return false;
    if (len > 64 && len <= fmha::kFusedKeys && h < 0.8 * ((h + 1) / 2 * 2)) return false;
  }
  const bool equal = mean >= 0.9 * n;
  if (n <= fmha::kFusedKeys) return share >= 0.2 && !(equal && !dropout && n > 64 && n <= 80);
  if (equal) {
    if (dropout ? n <= 416 : n <= 320 && rounds > 1) return false;
    return full >= (n > 1024 ? 0.85 : dropout ? 0.75 : 0.7);
  }
  if (n <= 1024 && mean < 0.3 * n) return share >= 0.3;
  return share >= (n <= 512 ? 0.65 : n <= 1024 ? 0.8 : 0.9);
}

// Dropout arguments for the kernels; d == nullptr means no dropout.
int drop_args(const fmha_dropout_t* d, bool required, fmha::DropArgs* out) {
  *out = fmha::DropArgs{0u, 0u, 0u, 1.f};
  if (!d) return required ? fail(FMHA_ERR_INVALID_ARG, "dropout is null") : FMHA_OK;
  if (!(d->p >= 0.f && d->p < 1.f)) return fail(FMHA_ERR_INVALID_ARG, "dropout p=%g is not in [0, 1)", (double)d->p);
  int t = (int)(256.f * d->p + 0.5f);  // p is exactly representable times 256: no double rounding
  if (t > 255) t = 255;
  out->thr = (uint32_t)t;
  out->k0 = (uint32_t)(d->seed & 0xffffffffu);
  out->k1 = (uint32_t)(d->seed >> 32);
  out->rp = 256.f / (float)(256 - t);
  return FMHA_OK;
}

// ---- the library's own scratch memory, for fmha_varlen_fwd_static -----------------
// `scratch` is a device array: in host code its name is only a handle for
// hipGetSymbolAddress, never an address to hand to a kernel.  Every GPU holds its own copy
// at its own address, looked up once per device (with that device current) and kept.
constexpr size_t kStaticScratchBytes = (size_t)1 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(FMHA_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return fail(FMHA_ERR_HIP, "device index %d is outside [0, %d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(FMHA_ERR_HIP, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return FMHA_OK;
}

int run_fwd(const fmha_varlen_params_t* p, const fmha_dropout_t* d, bool with_dropout, const void* q,
            const void* k, const void* v, void* o, float* lse, void* stream, bool list_only = false);
int run_bwd(const fmha_varlen_params_t* p, const fmha_dropout_t* d, bool with_dropout, const void* q,
            const void* k, const void* v, const void* o, const void* d_o, const float* lse, void* dq,
            void* dk, void* dv, void* stream);

}  // namespace

extern "C" {

const char* fmha_last_error(void) { return g_err; }

size_t fmha_varlen_workspace_size(int32_t batch, int32_t total_tokens, int32_t heads, int32_t need_bwd) {
  if (batch < 0 || total_tokens < 0 || heads <= 0) return 0;
  Workspace w = carve(nullptr, batch, total_tokens, heads);
  return need_bwd ? w.bytes_bwd : w.bytes_fwd;
}

int32_t fmha_varlen_schedule_info(int32_t batch, int32_t total_tokens, int32_t max_seqlen,
                                  size_t* count_offset, size_t* list_offset) {
  if (batch < 0 || total_tokens < 0) return -1;
  Workspace w = carve(nullptr, batch, total_tokens, 1);
  if (count_offset) *count_offset = w.count_off;
  if (list_offset) *list_offset = w.list_off;
  (void)max_seqlen;
  return (int32_t)tile_capacity(batch, total_tokens);
}

int fmha_varlen_fwd(const fmha_varlen_params_t* p, const void* q, const void* k, const void* v,
                    void* o, float* lse, void* stream) {
  return run_fwd(p, nullptr, false, q, k, v, o, lse, stream);
}

int fmha_varlen_fwd_dropout(const fmha_varlen_params_t* p, const fmha_dropout_t* dropout, const void* q,
                            const void* k, const void* v, void* o, float* lse, void* stream) {
  return run_fwd(p, dropout, true, q, k, v, o, lse, stream);
}

size_t fmha_varlen_static_scratch_bytes(void) { return kStaticScratchBytes; }

int fmha_varlen_fwd_static(const fmha_varlen_params_t* p, const void* q, const void* k, const void* v,
                           void* o, float* lse, void* stream) {
  if (!p) return fail(FMHA_ERR_INVALID_ARG, "params is null");
  if (p->batch < 0 || p->total_tokens < 0 || p->heads <= 0)
    return fail(FMHA_ERR_INVALID_ARG, "batch=%d, total_tokens=%d, heads=%d: invalid sizes", p->batch, p->total_tokens, p->heads);
  const size_t need = carve(nullptr, p->batch, p->total_tokens, p->heads).bytes_list;
  if (need > kStaticScratchBytes)
    return fail(FMHA_ERR_WORKSPACE,
                "a batch of %d sequences and %d tokens needs %zu bytes for its tile list, the built-in scratch "
                "holds %zu: use fmha_varlen_fwd with a workspace",
                p->batch, p->total_tokens, need, kStaticScratchBytes);
  void* ptr = nullptr;
  int rc = static_scratch(&ptr);
  if (rc) return rc;
  fmha_varlen_params_t local = *p;
  local.workspace = ptr;
  local.workspace_bytes = kStaticScratchBytes;
  return run_fwd(&local, nullptr, false, q, k, v, o, lse, stream, true);
}

int fmha_varlen_bwd(const fmha_varlen_params_t* p, const void* q, const void* k, const void* v,
                    const void* o, const void* d_o, const float* lse, void* dq, void* dk,
                    void* dv, void* stream) {
  return run_bwd(p, nullptr, false, q, k, v, o, d_o, lse, dq, dk, dv, stream);
}

int fmha_varlen_bwd_dropout(const fmha_varlen_params_t* p, const fmha_dropout_t* dropout, const void* q,
                            const void* k, const void* v, const void* o, const void* d_o,
                            const float* lse, void* dq, void* dk, void* dv, void* stream) {
  return run_bwd(p, dropout, true, q, k, v, o, d_o, lse, dq, dk, dv, stream);
}

int32_t fmha_varlen_bwd_passes(const fmha_varlen_params_t* p, const fmha_dropout_t* dropout) {
  int rc = check_common(p, true);
  if (rc) return -rc;
  fmha::DropArgs da;
  if ((rc = drop_args(dropout, false, &da))) return -rc;
  g_err[0] = 0;
  return one_pass(p, carve(p->workspace, p->batch, p->total_tokens, p->heads), da.thr != 0) ? 1 : 2;
}

int fmha_dropout_keep_mask(const fmha_varlen_params_t* p, const fmha_dropout_t* dropout, int32_t orientation,
                           int32_t row_bytes, uint8_t* mask, void* stream) {
  int rc = check_common(p, false);
  if (rc) return rc;
  fmha::DropArgs da;
  if ((rc = drop_args(dropout, true, &da))) return rc;
  if (!mask) return fail(FMHA_ERR_INVALID_ARG, "mask is null");
  if (orientation != 0 && orientation != 1) return fail(FMHA_ERR_INVALID_ARG, "orientation=%d is neither 0 nor 1", orientation);
  if (row_bytes <= 0) return fail(FMHA_ERR_INVALID_ARG, "row_bytes=%d must be positive", row_bytes);
  if (p->max_seqlen > row_bytes) return fail(FMHA_ERR_INVALID_ARG, "row_bytes=%d is smaller than max_seqlen=%d", row_bytes, p->max_seqlen);
  g_err[0] = 0;
  if (p->batch == 0 || p->total_tokens == 0) return FMHA_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  Workspace w = carve(p->workspace, p->batch, p->total_tokens, p->heads);
  if ((rc = launch_schedule(p, w, st))) return rc;
  const fmha::Problem pb = problem_of(p, w);
  const unsigned grid = grid_for(p, 4);
  if (orientation == 0)
    fmha::keep_mask_kernel<false><<<grid, fmha::kThreads, 0, st>>>(pb, da, mask, row_bytes);
  else
    fmha::keep_mask_kernel<true><<<grid, fmha::kThreads, 0, st>>>(pb, da, mask, row_bytes);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FMHA_ERR_HIP, "keep-mask launch failed: %s", hipGetErrorString(e));
  return FMHA_OK;
}

}  // extern "C"

namespace {

int run_fwd(const fmha_varlen_params_t* p, const fmha_dropout_t* d, bool with_dropout, const void* q,
            const void* k, const void* v, void* o, float* lse, void* stream, bool list_only) {
  int rc = check_common(p, false, list_only);
  if (rc) return rc;
  fmha::DropArgs da;
  if ((rc = drop_args(d, with_dropout, &da))) return rc;
  if ((rc = check_ptr("q", q)) || (rc = check_ptr("k", k)) || (rc = check_ptr("v", v)) ||
      (rc = check_ptr("o", o)) || (rc = check_ptr("lse", lse)))
    return rc;
  const int64_t dense = (int64_t)p->heads * fmha::kHeadDim;
  fmha::FwdArgs a;
  if ((rc = check_stride("q", p->q_stride, dense, &a.q_stride)) ||
      (rc = check_stride("k", p->k_stride, dense, &a.k_stride)) ||
      (rc = check_stride("v", p->v_stride, dense, &a.v_stride)) ||
      (rc = check_stride("o", p->o_stride, dense, &a.o_stride)))
    return rc;
  g_err[0] = 0;
  if (p->batch == 0 || p->total_tokens == 0) return FMHA_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  Workspace w = carve(p->workspace, p->batch, p->total_tokens, p->heads);
  if (list_only) w.seqs = nullptr;  // (no backward follows)
  // Small batches work out the tile list in the forward kernel (SELF): one lane per sequence,
  // and every item resident from the start (4 workgroups per compute unit).  The order still
  // decides which items share a compute unit, so it is the list's once there are more items than
  // compute units (fwd64_kernel.h has the figures).
  const bool self = da.thr == 0 && !(p->flags & FMHA_FLAG_REUSE_SCHEDULE) && p->batch <= fmha::kSelfListBatch &&
                    items_bound(p) <= (int64_t)compute_units() * 4;
  if (!self && (rc = launch_schedule(p, w, st))) return rc;
  a.pb = problem_of(p, w);
  a.list = fmha::ListArgs{p->cu_seqlens, p->seqused, p->batch, (int32_t)tile_capacity(p->batch, p->total_tokens),
                          items_bound(p) > (int64_t)compute_units(), w.count, w.list, w.seqs};
  a.feed = fmha::FeedArgs{w.feed, 1};
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.o = static_cast<uint16_t*>(o);
  a.lse = lse;
  const unsigned grid = grid_for(p, 3);
  a.drop = da;
  // p = 0 (threshold 0) keeps everything: the plain kernels serve it
  if (self) {
    const unsigned grid_self = (unsigned)items_bound(p) + 1;  // one writes the list
    if (p->dtype == FMHA_F16)
      fmha::fmha_fwd64_kernel<_Float16, true><<<grid_self, fmha::kF64Threads, 0, st>>>(a);
    else
      fmha::fmha_fwd64_kernel<__bf16, true><<<grid_self, fmha::kF64Threads, 0, st>>>(a);
  } else if (da.thr == 0) {
    // persistent: 4 workgroups of 2 wavefronts per compute unit
    const unsigned grid64 = feed_grid(p, 4, w, &a.feed);
    if (p->dtype == FMHA_F16)
      fmha::fmha_fwd64_kernel<_Float16, false><<<grid64, fmha::kF64Threads, 0, st>>>(a);
    else
      fmha::fmha_fwd64_kernel<__bf16, false><<<grid64, fmha::kF64Threads, 0, st>>>(a);
  } else {
    if (p->dtype == FMHA_F16)
      fmha::fmha_fwd_kernel<_Float16, true><<<grid, fmha::kThreads, 0, st>>>(a);
    else
      fmha::fmha_fwd_kernel<__bf16, true><<<grid, fmha::kThreads, 0, st>>>(a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FMHA_ERR_HIP, "forward launch failed: %s", hipGetErrorString(e));
  return FMHA_OK;
}

int run_bwd(const fmha_varlen_params_t* p, const fmha_dropout_t* d, bool with_dropout, const void* q,
            const void* k, const void* v, const void* o, const void* d_o, const float* lse, void* dq,
            void* dk, void* dv, void* stream) {
  int rc = check_common(p, true);
  if (rc) return rc;
  fmha::DropArgs da;
  if ((rc = drop_args(d, with_dropout, &da))) return rc;
  if ((p->flags & FMHA_FLAG_BWD_ONLY_DQ) && (p->flags & FMHA_FLAG_BWD_ONLY_DKV))
    return fail(FMHA_ERR_INVALID_ARG, "FMHA_FLAG_BWD_ONLY_DQ and FMHA_FLAG_BWD_ONLY_DKV exclude each other");
  if ((rc = check_ptr("q", q)) || (rc = check_ptr("k", k)) || (rc = check_ptr("v", v)) ||
      (rc = check_ptr("o", o)) || (rc = check_ptr("d_o", d_o)) || (rc = check_ptr("lse", lse)) ||
      (rc = check_ptr("dq", dq)) || (rc = check_ptr("dk", dk)) || (rc = check_ptr("dv", dv)))
    return rc;
  const int64_t dense = (int64_t)p->heads * fmha::kHeadDim;
  fmha::BwdArgs a;
  if ((rc = check_stride("q", p->q_stride, dense, &a.q_stride)) ||
      (rc = check_stride("k", p->k_stride, dense, &a.k_stride)) ||
      (rc = check_stride("v", p->v_stride, dense, &a.v_stride)) ||
      (rc = check_stride("o", p->o_stride, dense, &a.o_stride)) ||
      (rc = check_stride("do", p->do_stride, dense, &a.do_stride)) ||
      (rc = check_stride("dq", p->dq_stride, dense, &a.dq_stride)) ||
      (rc = check_stride("dk", p->dk_stride, dense, &a.dk_stride)) ||
      (rc = check_stride("dv", p->dv_stride, dense, &a.dv_stride)))
    return rc;
  g_err[0] = 0;
  if (p->batch == 0 || p->total_tokens == 0) return FMHA_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  Workspace w = carve(p->workspace, p->batch, p->total_tokens, p->heads);
  if ((rc = launch_schedule(p, w, st))) return rc;
  a.pb = problem_of(p, w);
  a.feed = fmha::FeedArgs{w.feed, 1};
  a.drop = da;
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.o = static_cast<const uint16_t*>(o);
  a.d_o = static_cast<const uint16_t*>(d_o);
  a.lse = lse;
  a.dsum = w.dsum;
  a.lse2 = w.lse2;
  a.dq = static_cast<uint16_t*>(dq);
  a.dk = static_cast<uint16_t*>(dk);
  a.dv = static_cast<uint16_t*>(dv);
  if (one_pass(p, w, da.thr != 0)) {
    const int64_t grid = fused_grid((int64_t)p->batch * p->heads, fused_units());
    a.seqs = w.seqs;
    a.slab = w.slab;
    a.slab_rows = fused_slab_rows(p);
    if (da.thr == 0) {
      if (p->dtype == FMHA_F16)
        fmha::bwd_fused_kernel<_Float16, false><<<(unsigned)grid, fmha::kFusedThreads, 0, st>>>(a);
      else
        fmha::bwd_fused_kernel<__bf16, false><<<(unsigned)grid, fmha::kFusedThreads, 0, st>>>(a);
    } else {
      if (p->dtype == FMHA_F16)
        fmha::bwd_fused_kernel<_Float16, true><<<(unsigned)grid, fmha::kFusedThreads, 0, st>>>(a);
      else
        fmha::bwd_fused_kernel<__bf16, true><<<(unsigned)grid, fmha::kFusedThreads, 0, st>>>(a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(FMHA_ERR_HIP, "backward launch failed: %s", hipGetErrorString(e));
    return FMHA_OK;
  }
  // persistent grids with their own hand-out chunk sizes: 3 workgroups per compute unit for
  // the dQ pass (2 with dropout), 2 for the dK/dV pass
  fmha::BwdArgs a_dq = a, a_dkv = a;
  const unsigned grid_dq = feed_grid(p, da.thr == 0 ? 3 : 2, w, &a_dq.feed);
  const unsigned grid_dkv = feed_grid(p, 2, w, &a_dkv.feed);
  const bool run_dq = !(p->flags & FMHA_FLAG_BWD_ONLY_DKV);
  const bool run_dkv = !(p->flags & FMHA_FLAG_BWD_ONLY_DQ);
  if (da.thr == 0) {
    if (p->dtype == FMHA_F16) {
      if (run_dq) fmha::bwd_dq_kernel<_Float16, false><<<grid_dq, fmha::kThreads, 0, st>>>(a_dq);
      if (run_dkv) fmha::bwd_dkv_kernel<_Float16, false><<<grid_dkv, fmha::kThreads, 0, st>>>(a_dkv);
    } else {
      if (run_dq) fmha::bwd_dq_kernel<__bf16, false><<<grid_dq, fmha::kThreads, 0, st>>>(a_dq);
      if (run_dkv) fmha::bwd_dkv_kernel<__bf16, false><<<grid_dkv, fmha::kThreads, 0, st>>>(a_dkv);
    }
  } else {
    if (p->dtype == FMHA_F16) {
      if (run_dq) fmha::bwd_dq_kernel<_Float16, true><<<grid_dq, fmha::kThreads, 0, st>>>(a_dq);
      if (run_dkv) fmha::bwd_dkv_kernel<_Float16, true><<<grid_dkv, fmha::kThreads, 0, st>>>(a_dkv);
    } else {
      if (run_dq) fmha::bwd_dq_kernel<__bf16, true><<<grid_dq, fmha::kThreads, 0, st>>>(a_dq);
      if (run_dkv) fmha::bwd_dkv_kernel<__bf16, true><<<grid_dkv, fmha::kThreads, 0, st>>>(a_dkv);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(FMHA_ERR_HIP, "backward launch failed: %s", hipGetErrorString(e));
  return FMHA_OK;
}

}  // namespace
