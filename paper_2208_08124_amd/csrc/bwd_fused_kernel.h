// Backward of Eq. 1 in one pass over the scores: S and dP are formed once per (query, key) and
// dQ, dK and dV all come from them (5 products and one exponential per score; the two passes of
// bwd_kernels.h execute 7 and two).
//
// One workgroup of 8 wavefronts has a compute unit to itself and takes a work item: one
// sequence and NH heads, NH = 1, 2 or 4 so that the item's keys fill the workgroup's 256 key
// places (sequences of more than 64 keys get 2 heads at most, of more than 128 one).  Each
// wavefront owns 32 keys of one head; K and V as B operands and the accumulators of dK^T and
// dV^T stay in its registers.  The queries go by in blocks of 32 (Q, dO, O and the log-sum-exp
// through a ring of LDS places, several blocks ahead), one barrier per block:
//   S = Q K^T,  dP = dO V^T             (rows = queries, column = this lane's key)
//   P = exp(S - LSE),  dS = P o (dP - D)
//   dV^T += dO^T P,  dK^T += Q^T dS     (P and dS straight from the result registers)
// dQ = dS K contracts over keys, which lie across the lanes and wavefronts: dS goes through LDS
// (16 KB a block, two buffers).  During the next block's step every wavefront computes one
// 16 x 16 part of that block's dQ over ALL keys of the item (its K^T operand, 16 channels of up
// to 256 keys, stays in registers too), so no sums cross wavefronts, and these products stand
// beside the exponentials of the step instead of waiting for them.
//
// Sequences of more than 256 keys are swept once per 256 keys; dQ is carried from sweep to sweep
// in fp32 through a buffer of the workgroup's own in the workspace, each lane reading back what
// it wrote itself.  (A sequence longer than that buffer, possible only if max_seqlen was stated
// too small, is done in more sweeps: first dK and dV, then dQ for as many rows as fit at a time.)
//
// What bounds it: the issue of instructions.  A step takes about 3400 cycles; of those the matrix cores of a
// SIMD work 2 x 640 for its two wavefronts, each of which has 24 products, 16 exponentials and about 130
// other vector instructions to issue beside them (the products of one and the vector instructions of
// the other hardly overlap), and a sweep has some 17 000 cycles outside its steps (K and V in, operands
// transposed, the first step, dK and dV out).  So an instruction less per step counts: with the products of
// dK ahead of those of dV (dS is used up before its successor is packed, without copies), dS in runs that
// need no XOR per place, and no scratch memory in any instance (a reload waits for all transfers under
// way), a backward pass of 65 536 tokens and 16 heads took 339 for 361 us at length 256, 262 for 272 at
// 512, 264 for 288 at 128 and 238 for 257 at 64; with dropout 423 for 492, 353 for 395, 312 for 356, 264 for 313.
// Two passes / one, 32 768 tokens, 16 heads, us, without and with dropout: length 64 194 / 129, 220 / 144; 128
// 196 / 147, 219 / 172; 256 242 / 174, 295 / 223; 512 339 / 267, 460 / 368.
//
// Every sum is formed in a fixed order: results are identical from run to run.  With dropout dK and dV
// are those of the two passes bit for bit; without, dP - D is summed from -D on (16 subtractions and 8
// registers less a step), which rounds otherwise.
#pragma once
#include "bwd_kernels.h"
#include "dropout.h"
#include "kernel_args.h"
#include "mfma_tiles.h"

namespace fmha {

constexpr int kFusedThreads = 512;
constexpr int kFusedKeys = 256;   // key places of a workgroup
constexpr int kFusedSlots = 8;    // (head, block of 32 queries) units in the LDS ring
constexpr int kCarry = 4;         // blocks of fp32 dQ on their way in

struct FusedLds {
  uint16_t q[kFusedSlots][32 * 64];
  uint16_t g[kFusedSlots][32 * 64];  // dO
  union {
    uint16_t o[kFusedSlots][32 * 64];       // O, in an item's first sweep
    u32x4 carry[kCarry][kFusedThreads];     // in the others: dQ of the sweeps before, on its way in
  };
  uint16_t ds[2][kFusedKeys * 32];   // dS of a block: [key][query]; K tiles at the start, rows on their way out at the end
  uint16_t rows[2][2][32 * 64];      // finished dQ of a block (of two heads), on its way out
  float lse[kFusedSlots][64];
  float stat[kFusedSlots][128];      // LSE * log2(e) of 32 rows, -D of 32 rows; then +inf and 0, for keys that do not exist
  u32x4 record;   // the next item's sequence
  int mail[2];    // the next item, and its sequence's place among those of the section
};

// (referred to as what it is, LDS: an address taken through a generic reference is checked for null)
typedef __attribute__((address_space(3))) FusedLds FusedShared;
static __device__ __forceinline__ uint32_t lds_at(const __attribute__((address_space(3))) void* p) {
  return (uint32_t)(uintptr_t)p;
}

// The kernel's arguments, read anew: what is taken from them here is not held in registers from one
// use to the next (there are more than the scalar registers hold, and the compiler would keep them
// in lanes of vector registers through the steps).
static __device__ __forceinline__ const BwdArgs& fused_args() {
  auto p = (const __attribute__((address_space(4))) BwdArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const BwdArgs*)p;
}

// Per lane one of two arrays: x in lanes 0..31, y in the others.  (Both addresses are brought into
// scalar registers first: the compiler would fetch the address itself by lane, and wait for that
// together with all the transfers under way.)
typedef __attribute__((address_space(1))) float* GlobalFloat;
static __device__ __forceinline__ GlobalFloat per_half(const float* x, const float* y, int64_t offset, int lane) {
  uint64_t u = (uint64_t)(uintptr_t)(x + offset), v = (uint64_t)(uintptr_t)(y + offset);
  asm volatile("" : "+s"(u), "+s"(v));
  return (GlobalFloat)(uintptr_t)(lane < 32 ? u : v);
}

template <typename T>
struct Mfma16;
template <>
struct Mfma16<_Float16> {
  static __device__ __forceinline__ f32x4 mul(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <>
struct Mfma16<__bf16> {
  static __device__ __forceinline__ f32x4 mul(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};

// One sweep: 256 key places over the item's queries.
struct FusedPhase {
  int r0, len, nk;   // the sequence
  int head;          // first head
  int kt, n_kt;      // key tile, and how many there are
  int q0, q1;        // first and last + 1 block of 32 queries
  int want;          // 1: dK, dV;  2: dQ
  int step, steps;   // of the item's sweeps
  // (all of it is uniform over the workgroup, which the compiler does not always see)
  __device__ __forceinline__ FusedPhase scalar() const {
    auto s = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    return FusedPhase{s(r0), s(len), s(nk), s(head), s(kt), s(n_kt), s(q0), s(q1), s(want), s(step), s(steps)};
  }
};

// LDS by byte address: what a lane reads lies at a wave-uniform base plus an offset of the lane's
// own, of which one register per kind is kept (the others differ from it by one XOR).
template <typename V>
static __device__ __forceinline__ V lds_get(uint32_t addr) {
  return *(const __attribute__((address_space(3))) V*)addr;
}
template <typename V>
static __device__ __forceinline__ void lds_put(uint32_t addr, V v) {
  *(__attribute__((address_space(3))) V*)addr = v;
}
static __device__ __forceinline__ u32x2 lds_get_tr16(uint32_t addr) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)addr));
}

// dS byte offset of (key row, piece of four queries): per 32 keys four runs of 512 bytes, of eight
// queries each, key by key.  A wavefront's write fills a run; the transposing reads (four keys by four
// pieces per 16 lanes) take two runs at a time, of which the second has its groups of eight keys
// exchanged so that they do not meet in a bank.
static __device__ __forceinline__ uint32_t ds_off(int row, int piece) {
  const int run = piece >> 1;
  return (row >> 5) * 2048 + run * 512 + (((row & 31) ^ ((run & 1) << 3)) << 4) + ((piece & 1) << 3);
}

// Sum over 16 neighbouring lanes, the same in all of them: pairs, quads, halves, all.
template <int CTRL>
static __device__ __forceinline__ float dpp_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}
static __device__ __forceinline__ float sum16(float x) {
  x = dpp_add<0xB1>(x);    // lane ^ 1
  x = dpp_add<0x4E>(x);    // lane ^ 2
  x = dpp_add<0x141>(x);   // mirrored in eight
  return dpp_add<0x140>(x);  // mirrored in sixteen
}

static __device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// 4 bytes per lane, wave-uniform base and byte offset per lane (see dma16s)
static __device__ __forceinline__ void dma4s(const void* sbase, uint32_t voff, uint32_t lds_byte_addr, uint32_t more) {
  const void* base;
  asm volatile("s_add_u32 m0, %1, %4\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dword %2, %0"
               : "=&s"(base)
               : "s"(lds_byte_addr), "v"(voff), "s"(sbase), "s"(more)
               : "memory", "scc");
}

// 4 KB of LDS for wavefront (or group of keys) w between two sweeps.  NH == 1: the ring's last four places,
// which the next sweep's first blocks leave free (sweeps begin at blocks that are multiples of eight); else
// where dS was.
template <int NH>
static __device__ __forceinline__ uint32_t fused_tile(const FusedShared& lds, int w) {
  constexpr uint32_t kToG = offsetof(FusedLds, g) - offsetof(FusedLds, q);
  static_assert(kFusedSlots == 8 && kToG == 8 * 4096, "");
  return NH == 1 ? lds_at(&lds.q[4][0]) + 4096 * w + (w >= 4 ? kToG - 4 * 4096 : 0) : lds_at(&lds.ds[0][0]) + 4096 * w;
}

template <int NH>
struct FusedShape {
  static constexpr int KG = 8 / NH;            // wavefronts (groups of 32 keys) per head
  static constexpr int D = kFusedSlots / NH;   // blocks in the ring
  static constexpr int NCH = NH == 4 ? 2 : 1;  // a wavefront's part of a block's dQ: channel blocks of 16 ...
  static constexpr int NQH = NH == 1 ? 1 : 2;  // ... by query halves of 16 ...
  static constexpr int KS = KG;                // ... over KS steps of 32 keys
  static constexpr int kAhead = NH == 4 ? 2 : 3;  // blocks that are requested before a sweep begins
};

// A sweep of one wavefront.
template <typename T, int NH, bool DROP>
struct FusedWave {
  using S = FusedShape<NH>;
  const BwdArgs& a;
  FusedShared& lds;
  const FusedPhase& ph;
  const int wave, kg, hd;  // this wavefront, its group of keys and head within the item
  const u32x4 (&kb)[4];    // K and V as B operands
  const u32x4 (&vb)[4];

  // per lane, bytes
  uint32_t row_rd;   // Q, dO as A operands of the scores
  uint32_t col_rd;   // the same transposed
  uint32_t ds_rd;    // dS for the dQ products (query half 0 of them, or this wavefront's)
  uint32_t ds_wr;    // this lane's key's row of dS
  uint32_t stat_rd;  // LSE and D of the rows this lane's registers hold; what stands for them if its key does not exist
  uint32_t sum_rd;   // this lane's four channels of dO and O of the row it helps to sum
  uint32_t sum_wr;   // where this lane's result goes (one lane in sixteen the LSE, the others D); the lower 128: the row's entry
  uint32_t carry_lane;  // this lane's place in a block of fp32 dQ
  uint32_t out_wr;      // in a block of dQ on its way out
  uint32_t out_lane;    // and in memory: of fp32 dQ, or of the rows that are read back whole
  // wave-uniform
  char *dq_first, *dq_at;  // the first block of dQ, and the next to go out (or to the buffer between sweeps)
  int64_t dq_step;   // bytes from block to block
  bool to_slab;      // not the last sweep
  float scale, c2;

  f32x16 dk[2], dv[2];       // dK^T, dV^T: column = key ln, rows = channels
  u32x4 kT[S::NCH][S::KS];   // K^T operands of the dQ products
  f32x16 s, dp;              // S and dP of a block: rows = queries, column = key ln
  uint32_t keep[4];          // DROP: its mask bytes
  u32x4 p[2], ds[2];         // P and dS of the block before as B operands
  f32x4 acc[S::NCH][S::NQH];  // dQ of a block: column = query, rows = channels

  __device__ __forceinline__ FusedWave(const BwdArgs& a_, FusedShared& lds_, const FusedPhase& ph_, int w, const u32x4 (&kb_)[4], const u32x4 (&vb_)[4], u32x4* slab)
      : a(a_), lds(lds_), ph(ph_), wave(w), kg(w % S::KG), hd(w / S::KG), kb(kb_), vb(vb_) {
    const int lane = lane_id(), g = lane >> 5, ln = lane & 31;
    const int e = (lane >> 2) & 3, pc = lane & 3, g4 = lane >> 4, c = lane & 15;
    row_rd = 2 * tile_off(ln, 8 * g);
    col_rd = 2 * tile_off(4 * g + e, 16 * (g4 & 1) + 4 * pc);
    ds_rd = ds_off(4 * g4 + e, (NH == 1 ? 4 * (wave & 1) : 0) + pc) + hd * (S::KG * 2048);
    ds_wr = ds_off(32 * wave + ln, g);
    // A key place without a key holds a copy of the last key, and draws a mask of its own: its dS belongs to no score, and
    // one that overflows the 16-bit type would be inf * 0 in the dQ products.  Its probabilities are zeros, by the LSE
    // that it reads (any of 32; not from the banks that its neighbours read); V is cleared in fused_sweep.
    stat_rd = ph.kt * kFusedKeys + 32 * kg + ln < ph.nk ? 16 * g : 272 - 16 * g;
    const int row = kg * 4 * NH + g4;
    sum_rd = 2 * tile_off(row, 4 * c);
    sum_wr = 128 * min(c, 1) + 4 * row;
    to_slab = NH == 1 && ph.kt + 1 < ph.n_kt;
    scale = a.pb.scale;
    c2 = scale * kLog2e;
    const uint16_t* dq0 = a.dq + uniform_i64((int64_t)(ph.r0 + 32 * ph.q0) * a.dq_stride + (ph.head + hd) * kHeadDim);
    carry_lane = (64 * wave + lane) * 16;
    if (to_slab) {
      dq_at = reinterpret_cast<char*>(slab);
      dq_step = kFusedThreads * 16;
    } else {
      dq_at = reinterpret_cast<char*>(const_cast<uint16_t*>(dq0));
      dq_step = a.dq_stride * 64;
    }
    dq_first = dq_at;
    // (16 channels of 16 rows; NH == 2: of both halves)
    const int qrow = (NH == 1 ? 16 * (wave & 1) : 0) + c, cq = NH == 1 ? wave >> 1 : kg;
    out_wr = hd * 4096 + 2 * tile_off(qrow, 16 * cq + 4 * g4);
    const int orow = 8 * (wave & 3) + (lane >> 3);
    out_lane = to_slab ? carry_lane : (orow * (uint32_t)a.dq_stride + ((lane & 7) ^ swz(orow)) * 8) * 2u;
  }
  __device__ __forceinline__ uint32_t slot(int j) const { return (j & (S::D - 1)) * NH + hd; }

  // S = Q K^T, dP - D = dO V^T - D of block j (DROP: dP, of which the mask comes first)
  __device__ __forceinline__ void scores(int j) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const uint32_t q = lds_at(&lds.q[0][0]) + slot(j) * 4096 + row_rd;
    constexpr uint32_t kToG = offsetof(FusedLds, g) - offsetof(FusedLds, q);
    u32x4 qa[4], ga[4];
#pragma unroll
    for (int t = 0; t < 4; t++) {
      qa[t] = lds_get<u32x4>(q ^ (t << 5));
      ga[t] = lds_get<u32x4>((q ^ (t << 5)) + kToG);
    }
    f32x16 minus_d;
    if (!DROP) {
      const uint32_t st = lds_at(&lds.stat[0][0]) + slot(j) * 512 + stat_rd + 128;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const f32x4 d = lds_get<f32x4>(st + 32 * i);
#pragma unroll
        for (int e = 0; e < 4; e++) minus_d[4 * i + e] = d[e];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 4; t++) {
      s = Op<T>::mfma(qa[t], kb[t], t == 0 ? zero : s);
      dp = Op<T>::mfma(ga[t], vb[t], t > 0 ? dp : DROP ? zero : minus_d);
    }
    if (DROP) {  // (independent of the products just issued)
      const int lane = lane_id(), ln = lane & 31;
      const int krow = ph.kt * kFusedKeys + 32 * kg + ln;
      keep_bytes<true>(keep, krow >> 2, 8 * j + (lane >> 5), ln, ph.r0, ph.head + hd, a.drop);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // A operand of product i (0..7) of dK^T += Q^T dS (first), dV^T += dO^T P; `q` = Q of the block + col_rd
  __device__ __forceinline__ u32x4 operand(uint32_t q, int i) const {
    constexpr uint32_t kToG = offsetof(FusedLds, g) - offsetof(FusedLds, q);
    const uint32_t at = (q ^ ((i & 1) << 6)), off = (i < 4 ? 0 : kToG) + ((i >> 1) & 1) * 2048;
    const u32x2 lo = lds_get_tr16(at + off), hi = lds_get_tr16((at ^ 32) + off + 1024);
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  }
  __device__ __forceinline__ void multiply(int i, u32x4 x) {
    const int t2 = (i >> 1) & 1, cb = i & 1;
    if (i < 4)
      dk[cb] = Op<T>::mfma(x, ds[t2], dk[cb]);
    else
      dv[cb] = Op<T>::mfma(x, p[t2], dv[cb]);
  }
  // B operand of product i (0..7) of the dQ part; `d` = dS of the block + ds_rd
  __device__ __forceinline__ u32x4 dq_operand(uint32_t d, int i) const {
    const int h = (i / S::NCH) % S::NQH, k = i / (S::NCH * S::NQH);
    const u32x2 lo = lds_get_tr16(d + 1024 * h + 2048 * k), hi = lds_get_tr16(d + 1024 * h + 2048 * k + 256);
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  }
  __device__ __forceinline__ void dq_multiply(int i, u32x4 x) {
    const int c = i % S::NCH, h = (i / S::NCH) % S::NQH, k = i / (S::NCH * S::NQH);
    acc[c][h] = Mfma16<T>::mul(kT[c][k], x, acc[c][h]);
  }
  __device__ __forceinline__ uint32_t ds_base(int j) const { return lds_at(&lds.ds[0][0]) + (j & 1) * 16384; }

  // One step for a wavefront with live keys: P and dS of block j from its scores, beside the dV,
  // dK and dQ products of block j - 1 (none in a sweep's first step).
  template <bool FIRST, bool LATE>
  __device__ __forceinline__ void step(int j) {
    const uint32_t q = lds_at(&lds.q[0][0]) + slot(j + S::D - 1) * 4096 + col_rd;
    const uint32_t d = ds_base(j - 1) + ds_rd, w = ds_base(j) + ds_wr;
    const uint32_t st = lds_at(&lds.stat[0][0]) + slot(j) * 512 + stat_rd;
    // operands, fetched two groups ahead (DROP: one, whose groups are longer; two would not fit the registers)
    constexpr int kAhead = DROP ? 1 : 2, kOps = kAhead + 1;
    u32x4 x[kOps], y[kOps];
    f32x4 l4[2], d4[2];
    auto stats = [&](int i) {
      l4[i & 1] = lds_get<f32x4>(st + 32 * i);
      if (DROP) d4[i & 1] = lds_get<f32x4>(st + 32 * i + 128);
    };
    auto fetch = [&](int i) {
      if (FIRST) return;
      x[i % kOps] = operand(q, i);
      y[i % kOps] = dq_operand(d, i);
    };
    fetch(0);
    stats(0);
    if (kAhead == 2) fetch(1);
    __builtin_amdgcn_sched_barrier(0);
    // (dS of the block before is used up by the fourth product, P by the last: new ones are packed behind
    // that, into the same registers)
    float pe[16], de[4];
    u32x4 pn[2];
#pragma unroll
    for (int i = 0; i < 8; i++) {
      if (LATE && i == 2) __builtin_amdgcn_s_setprio(0);
      if (LATE && i == 7) __builtin_amdgcn_s_setprio(1);
      if (i + kAhead < 8) fetch(i + kAhead);
      if (i & 1 && i < 7) stats((i + 1) >> 1);
      if (!FIRST) {
        multiply(i, x[i % kOps]);
        dq_multiply(i, y[i % kOps]);
      }
      const f32x4 l = l4[(i >> 1) & 1], dd = d4[(i >> 1) & 1];
      const float lv[2] = {l[2 * (i & 1)], l[2 * (i & 1) + 1]};
      const float dvv[2] = {dd[2 * (i & 1)], dd[2 * (i & 1) + 1]};
#pragma unroll
      for (int e = 0; e < 2; e++) {
        const int r = 2 * i + e;
        const float x0 = fast_exp2(__builtin_fmaf(s[r], c2, -lv[e]));
        if (DROP) {
          const bool on = kept(keep, r, a.drop.thr);
          pe[r] = on ? x0 : 0.f;
          de[r & 3] = x0 * ((on ? dp[r] * a.drop.rp : 0.f) + dvv[e]);
        } else {
          pe[r] = x0;
          de[r & 3] = x0 * dp[r];
        }
      }
      if (DROP) {  // (chosen in fp32: the compiler would convert one by one and choose halves)
        asm volatile("" : "+v"(pe[2 * i]), "+v"(pe[2 * i + 1]));
        pn[i >> 2][i & 3] = Op<T>::pack2(pe[2 * i], pe[2 * i + 1]);
      }
      if (i & 1) {  // dS of this block, also for the dQ products of the next step
        const u32x2 x = {Op<T>::pack2(de[0], de[1]), Op<T>::pack2(de[2], de[3])};
        ds[i >> 2][(i & 3) - 1] = x[0];
        ds[i >> 2][i & 3] = x[1];
        lds_put((w ^ (((i >> 1) & 1) << 7)) + (i >> 1) * 512, x);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 8; i++) p[i >> 2][i & 3] = DROP ? pn[i >> 2][i & 3] : Op<T>::pack2(pe[2 * i], pe[2 * i + 1]);
  }
  // dV and dK of the last block
  __device__ __forceinline__ void last_products(int j) {
    const uint32_t q = lds_at(&lds.q[0][0]) + slot(j) * 4096 + col_rd;
#pragma unroll
    for (int i = 0; i < 8; i++) multiply(i, operand(q, i));
  }
  // The dQ products of block j by themselves.
  __device__ __forceinline__ void dq_products(int j) {
    const uint32_t d = ds_base(j) + ds_rd;
#pragma unroll
    for (int i = 0; i < 8; i++) dq_multiply(i, dq_operand(d, i));
  }
  // A wavefront without live keys has zeros for dS.
  __device__ __forceinline__ void no_scores(int j) const {
    const uint32_t w = ds_base(j) + wave * 2048 + 32 * lane_id();
    lds_put(w, u32x4{0, 0, 0, 0});
    lds_put(w + 16, u32x4{0, 0, 0, 0});
  }
  // What the sweeps before left of a block's dQ, or zeros.
  __device__ __forceinline__ void dq_begin(uint32_t place, bool carry) {
#pragma unroll
    for (int c = 0; c < S::NCH; c++)
#pragma unroll
      for (int h = 0; h < S::NQH; h++) acc[c][h] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (NH == 1 && carry) acc[0][0] = lds_get<f32x4>(lds_at(&lds.carry[0][0]) + place + carry_lane);
  }
  __device__ __forceinline__ uint32_t out_base(int j) const {
    return lds_at(&lds.rows[0][0][0]) + (j & 1) * 8192;
  }
  // dQ of block j as it now is: on to the next sweep, or finished and into LDS (`out`: out).
  __device__ __forceinline__ void dq_finish(int j, bool out = NH == 4) {
    if (to_slab) {
      *reinterpret_cast<u32x4*>(dq_at + out_lane) = __builtin_bit_cast(u32x4, acc[0][0]);
      dq_at += dq_step;
      return;
    }
    const uint32_t to = out_base(j) + out_wr;
#pragma unroll
    for (int h = 0; h < S::NQH; h++)
#pragma unroll
      for (int c = 0; c < S::NCH; c++) {
        const f32x4 x = acc[c][h];
        const u32x2 o = {Op<T>::pack2(x[0] * scale, x[1] * scale), Op<T>::pack2(x[2] * scale, x[3] * scale)};
        if (!out) {
          lds_put(to + 2048 * h, o);
          continue;
        }
        const int lane = lane_id(), row = 16 * (NH == 1 ? wave & 1 : h) + (lane & 15);
        const int col = NH == 1 ? 16 * (wave >> 1) : 32 * kg + 16 * c;
        if (row < ph.len - 32 * j && ph.head + hd < a.pb.heads)
          *reinterpret_cast<u32x2*>(dq_at + ((uint32_t)row * (uint32_t)a.dq_stride + col + 4 * (lane >> 4)) * 2u) = o;
      }
    if (out) dq_at += dq_step;
  }
  // Finished dQ of block j out of LDS, a quarter of the rows for each of four wavefronts.
  __device__ __forceinline__ void dq_out(int j) {
    if (NH == 4 || (NH == 2 && ph.head + hd >= a.pb.heads)) return;
    const u32x4 x = lds_get<u32x4>(out_base(j) + hd * 4096 + (wave & 3) * 1024 + 16 * lane_id());
    const int rows = ph.len - 32 * j;  // left in the sequence
    if (rows >= 32 || 8 * (wave & 3) + (lane_id() >> 3) < rows) *reinterpret_cast<u32x4*>(dq_at + out_lane) = x;
    dq_at += dq_step;
  }
  // -D and LSE * log2(e) of block j, from its O, dO and LSE in the ring: 16 threads per row.
  __device__ __forceinline__ void statistics(int j) const {
    const uint32_t u = slot(j), sum_row = sum_wr & 127;
    const uint32_t from = lds_at(&lds.g[0][0]) + u * 4096 + sum_rd, lse = lds_at(&lds.lse[0][0]) + u * 256 + sum_row;
    const uint32_t to = lds_at(&lds.stat[0][0]) + u * 512 + sum_wr;
    const int left = 4 * (ph.len - 32 * j);
#pragma unroll
    for (int it = 0; it < NH; it++) {
      // (four rows on: 512 bytes, and the swizzle's bit 1 of row / 2 flips; eight: its bit 2)
      const uint32_t at = (from ^ (((it & 1) ? 16u : 0u) | ((it & 2) ? 32u : 0u))) + 512 * it;
      const u32x2 gv = lds_get<u32x2>(at);
      const u32x2 ov = lds_get<u32x2>(at + (uint32_t)(offsetof(FusedLds, o) - offsetof(FusedLds, g)));
      const float l = lds_get<float>(lse + 16 * it);
      const float d = sum16(Op<T>::dot2(gv[1], ov[1], Op<T>::dot2(gv[0], ov[0], 0.f)));
      const bool in = (int)sum_row + 16 * it < left;
      const float x = in ? l * kLog2e : INFINITY, y = in ? -d : 0.f;
      lds_put(to + 16 * it, sum_wr < 128 ? x : y);
    }
  }
  // The statistics of block j stay in the workspace, for the sweeps that follow and as the two
  // passes leave them (lanes 0..31 the LSE's, the others D's).
  __device__ __forceinline__ void keep_statistics(int j) const {
    const int lane = lane_id(), row = lane & 31;
    const BwdArgs& b = fused_args();
#pragma unroll
    for (int h = 0; h < NH; h++)
      if ((NH == 1 || ph.head + h < b.pb.heads) && 32 * j + row < ph.len)
        per_half(b.lse2, b.dsum, uniform_i64((int64_t)(ph.head + h) * b.pb.total_tokens + ph.r0 + 32 * j), lane)[row] =
            lds_get<float>(lds_at(&lds.stat[0][0]) + ((j & (S::D - 1)) * NH + h) * 512 + 4 * lane);
  }
  // dK and dV of this wavefront's keys (zeros where a key is masked), and zeros for the keys behind
  // the last tile, which are all masked.
  __device__ __forceinline__ void store_keys(const BwdArgs& a) {
    if (ph.head + hd >= a.pb.heads) return;
    const int head = ph.head + hd;
    const int row0 = ph.kt * kFusedKeys + 32 * kg;
    uint16_t* scratch = (uint16_t*)(__attribute__((address_space(3))) uint16_t*)fused_tile<NH>(lds, wave);
    if (row0 < ph.len) {
      if (!(row0 + (lane_id() & 31) < ph.nk)) {
#pragma unroll
        for (int cb = 0; cb < 2; cb++)
#pragma unroll
          for (int r = 0; r < 16; r++) dv[cb][r] = dk[cb][r] = 0.f;
      }
      const int64_t tok = ph.r0 + row0;
      store_rows32<T>(dk, a.pb.scale, scratch, a.dk, tok * a.dk_stride + head * kHeadDim, a.dk_stride, ph.len - row0);
      store_rows32<T>(dv, DROP ? a.drop.rp : 1.f, scratch, a.dv, tok * a.dv_stride + head * kHeadDim, a.dv_stride, ph.len - row0);
    }
    if (ph.kt + 1 < ph.n_kt) return;
#pragma unroll 1
    for (int r = ph.n_kt * kFusedKeys / NH + 32 * kg; r < ph.len; r += 32 * S::KG) {
      const int lane = lane_id();
      char* kz = reinterpret_cast<char*>(a.dk + uniform_i64((int64_t)(ph.r0 + r) * a.dk_stride + head * kHeadDim));
      char* vz = reinterpret_cast<char*>(a.dv + uniform_i64((int64_t)(ph.r0 + r) * a.dv_stride + head * kHeadDim));
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int row = 8 * i + (lane >> 3);
        if (r + row < ph.len) {
          *reinterpret_cast<u32x4*>(kz + ((uint32_t)row * (uint32_t)a.dk_stride * 2u + 16u * (lane & 7))) = u32x4{0, 0, 0, 0};
          *reinterpret_cast<u32x4*>(vz + ((uint32_t)row * (uint32_t)a.dv_stride * 2u + 16u * (lane & 7))) = u32x4{0, 0, 0, 0};
        }
      }
    }
  }
};

// This wavefront's transfers of query blocks, one block after the other (the last one again when
// there are no more: every step issues the same number, so that the waits are constants).
// NH == 1: wavefronts 0..3 a quarter of Q and of O, 4..7 a quarter of dO, and the LSE.  NH == 2:
// a quarter of each and the LSE; NH == 4: two quarters of each.  AGAIN (NH == 1): a sweep after the
// first, which finds LSE * log2(e) and D in the workspace and needs no O.
template <int NH, bool FIRST, bool AGAIN>
struct FusedPull {
  static constexpr int KG = 8 / NH, D = kFusedSlots / NH, kParts = NH == 1 ? (FIRST && !AGAIN ? 2 : 1) : 3;
  static constexpr bool kTail = NH > 1 || !FIRST;  // the LSE, or (AGAIN) both statistics
  static constexpr int kGroup = kParts * (NH == 4 ? 2 : 1) + kTail;
  const char *src[kParts], *tail;
  int64_t step[kParts];  // bytes from block to block
  uint32_t lane[kParts], tail_lane;
  uint32_t to[kParts], tail_to;  // place 0 of the ring
  GlobalFloat stat;              // AGAIN: per lane
  int left;                      // rows of the sequence from the next block on

  // (only handed to the transfers, which take any address in scalar registers)
  static __device__ __forceinline__ const char* scalar(const void* p) {
    return reinterpret_cast<const char*>(uniform_i64((int64_t)(uintptr_t)p));
  }
  static __device__ __forceinline__ int piece(int wave) { return NH == 1 ? wave & 3 : wave % KG; }
  __device__ __forceinline__ void part(int i, const uint16_t* base, int64_t stride, int64_t row0, int head, const __attribute__((address_space(3))) uint16_t* place, int wave) {
    const int l = lane_id(), r = 8 * piece(wave) + (l >> 3);
    src[i] = scalar(base + row0 * stride + head * kHeadDim);
    step[i] = uniform_i64(stride * 64);
    lane[i] = ((uint32_t)r * (uint32_t)stride + ((l & 7) ^ swz(r)) * 8) * 2u;
    to[i] = __builtin_amdgcn_readfirstlane(lds_at(place) + 1024u * piece(wave));
  }
  __device__ __forceinline__ FusedPull(const BwdArgs& a, FusedShared& lds, const FusedPhase& ph, int j, int wave) {
    const int hd = wave / KG, head = min(ph.head + hd, a.pb.heads - 1);
    const int64_t row0 = (int64_t)ph.r0 + 32 * j;
    left = ph.len - 32 * j;
    if (NH > 1) {
      part(0, a.q, a.q_stride, row0, head, &lds.q[hd][0], wave);
      part(1, a.d_o, a.do_stride, row0, head, &lds.g[hd][0], wave);
      part(2, a.o, a.o_stride, row0, head, &lds.o[hd][0], wave);
    } else if (FIRST) {
      part(0, a.q, a.q_stride, row0, head, &lds.q[0][0], wave);
      if (!AGAIN) part(kParts - 1, a.o, a.o_stride, row0, head, &lds.o[0][0], wave);
    } else {
      part(0, a.d_o, a.do_stride, row0, head, &lds.g[0][0], wave);
    }
    if (kTail) {
      const int l = lane_id();
      if (AGAIN) {
        stat = per_half(a.lse2, a.dsum, uniform_i64((int64_t)head * a.pb.total_tokens + row0), l) + (l & 31);
        tail_to = __builtin_amdgcn_readfirstlane(lds_at(&lds.stat[0][0]));
      } else {
        tail = scalar(a.lse + (int64_t)head * a.pb.total_tokens + row0);
        tail_lane = 4u * (l & 31);
        tail_to = __builtin_amdgcn_readfirstlane(lds_at(&lds.lse[hd][0]));
      }
    }
    if (left < 32) last(a, wave);
  }
  // The next block is the sequence's last and not whole: what lies behind its rows repeats the last
  // one (the statistics: the entries that stand for no row).
  __device__ __forceinline__ void last(const BwdArgs& a, int wave) {
    const int l = lane_id(), over = max(8 * piece(wave) + (l >> 3) - (left - 1), 0);
#pragma unroll
    for (int i = 0; i < kParts; i++) lane[i] -= (uint32_t)over * (uint32_t)(step[i] >> 5);
    if (!kTail) return;
    if (AGAIN) {
      const GlobalFloat none = per_half(a.lse2, a.dsum, uniform_i64((int64_t)a.pb.heads * a.pb.total_tokens), l);
      stat = (l & 31) >= left ? none : stat;
    } else {
      tail_lane = min(tail_lane, 4u * (left - 1));
    }
  }
  // The next block, into the place of block j.
  __device__ __forceinline__ void fetch(const BwdArgs& a, int j, int wave) {
    const uint32_t place = (j & (D - 1)) * NH;
#pragma unroll
    for (int i = 0; i < kParts; i++) {
      dma16s(src[i], lane[i], to[i], 4096u * place);
      if (NH == 4) {  // sixteen rows on
        const int r = 8 * piece(wave) + (lane_id() >> 3);
        const int more = min(16, max(left - 1 - r, 0));
        dma16s(src[i], lane[i] + (uint32_t)more * (uint32_t)(step[i] >> 5), to[i], 4096u * place + 2048u);
      }
    }
    if (kTail) {
      if (AGAIN)
        dma4((const float*)stat, tail_to + 512u * place);
      else
        dma4s(tail, tail_lane, tail_to, 256u * place);
    }
    if (left > 32) {
#pragma unroll
      for (int i = 0; i < kParts; i++) src[i] += step[i];
      if (kTail) {
        if (AGAIN)
          stat += 32;
        else
          tail += 128;
      }
      left -= 32;
      if (left < 32) last(a, wave);
    }
  }
};

// Rows of K and of V of this wavefront's keys, whole lines per instruction (8 rows each); keys at or
// beyond nk repeat the last one.
template <int NH>
static __device__ __forceinline__ void fused_load_kv(const BwdArgs& a, const FusedPhase& ph, int wave, u32x4 (&kb)[4], u32x4 (&vb)[4]) {
  constexpr int KG = 8 / NH;
  const int lane = lane_id();
  const int head = min(ph.head + wave / KG, a.pb.heads - 1);
  const int first = min(ph.kt * kFusedKeys + 32 * (wave % KG), max(ph.nk - 1, 0));
  const int room = max(ph.nk - 1, 0) - first;
  const char* kp = reinterpret_cast<const char*>(a.k + uniform_i64((int64_t)(ph.r0 + first) * a.k_stride + head * kHeadDim));
  const char* vp = reinterpret_cast<const char*>(a.v + uniform_i64((int64_t)(ph.r0 + first) * a.v_stride + head * kHeadDim));
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const uint32_t row = min(8 * i + (lane >> 3), room);
    kb[i] = *reinterpret_cast<const u32x4*>(kp + (row * (uint32_t)a.k_stride * 2u + 16u * (lane & 7)));
    vb[i] = *reinterpret_cast<const u32x4*>(vp + (row * (uint32_t)a.v_stride * 2u + 16u * (lane & 7)));
  }
}
// The same through 4 KB of LDS of the wavefront's own into B operands: column = key ln, slots =
// channels 16t + 8g .. +7.  The tile stays behind.
static __device__ __forceinline__ void fused_operands(uint32_t tile, uint32_t row_rd, u32x4 (&x)[4]) {
  const int lane = lane_id();
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int row = 8 * i + (lane >> 3);
    lds_put(tile + row * 128 + (((lane & 7) ^ swz(row)) << 4), x[i]);
  }
  __builtin_amdgcn_wave_barrier();  // (the wavefront's LDS operations execute in order)
#pragma unroll
  for (int t = 0; t < 4; t++) x[t] = lds_get<u32x4>((tile + row_rd) ^ (t << 5));
  __builtin_amdgcn_wave_barrier();
}

// The first query blocks of a sweep.
template <int NH>
static __device__ __forceinline__ void fused_begin(const BwdArgs& a, const FusedPhase& phase, FusedShared& lds, int wave) {
  const FusedPhase ph = phase.scalar();
  auto two = [&](auto first, auto again) {
    FusedPull<NH, decltype(first)::value, decltype(again)::value> pull(a, lds, ph, ph.q0, wave);
#pragma unroll
    for (int j = 0; j < FusedShape<NH>::kAhead; j++) pull.fetch(a, ph.q0 + j, wave);
  };
  if (NH > 1)
    two(std::true_type{}, std::false_type{});
  else if (ph.step == 0)
    wave < 4 ? two(std::true_type{}, std::false_type{}) : two(std::false_type{}, std::false_type{});
  else
    wave < 4 ? two(std::true_type{}, std::integral_constant<bool, NH == 1>{}) : two(std::false_type{}, std::integral_constant<bool, NH == 1>{});
}

// A sweep of at least so many blocks finds the next item's sequence in LDS before its last products: it is
// requested after the first step, and has landed when the step so many less one opens.  (NH == 1: the
// four groups of transfers that follow it leave three under way then.)
template <int NH>
constexpr int kFusedNext = NH == 1 ? 4 : NH == 2 ? 3 : 2;

// The steps of a sweep, for wavefronts 0..3 (LATE = false) and 4..7.  The former form the scores of
// block j + 1 at the end of step j, the latter those of block j at its start: the two of a SIMD then
// have their products and their exponentials at different times.  Of two wavefronts of one priority the
// SIMD favours the older, and wavefronts 4..7 came a quarter of a step late to every barrier; raised
// outside the middle of their steps the two arrive together (sequences of 256: 388 -> 358 us for a
// backward pass of 65 536 tokens and 16 heads; lowered from the fourth group on 359, from the sixth 367).
// AGAIN: a sweep after the item's first.
template <typename T, int NH, bool DROP, bool LATE, bool AGAIN, typename Publish>
static __device__ __forceinline__ void fused_steps(FusedWave<T, NH, DROP>& fw, const BwdArgs& a, const FusedPhase& ph, FusedShared& lds, int wave,
                                                   bool wave_on, u32x4* slab, Publish publish) {
  using S = FusedShape<NH>;
  using Pull = FusedPull<NH, NH == 1 ? !LATE : true, AGAIN>;
  const int q0 = ph.q0, q1 = ph.q1;
  const bool want_dq = ph.want & 2;
  const bool carry_in = AGAIN && ph.kt > 0 && want_dq;
  if (LATE) __builtin_amdgcn_s_setprio(1);
  // fp32 dQ of the sweeps before: read kCarry blocks ahead, into the place that has just been used
  const char* carry_src = reinterpret_cast<const char*>(slab);
  const uint32_t carry_to = __builtin_amdgcn_readfirstlane(lds_at(&lds.carry[0][64 * wave]));
  uint32_t place = 0;
  int carry_left = q1 - q0;
  auto carry_fetch = [&]() {
    dma16s(carry_src, fw.carry_lane, carry_to, place);
    if (--carry_left > 0) carry_src += kFusedThreads * 16;
    place = (place + kFusedThreads * 16) & (kCarry * kFusedThreads * 16 - 1);
  };
  // Blocks are requested one a step from the third step on, into the place of block j - 2; the ring's
  // free places are filled by two a step before that (NH == 1; else all at once).
  Pull pull(a, lds, ph, min(q0 + S::kAhead, q1 - 1), wave);
  int want = q0 + S::kAhead;  // next block to request
  if (NH > 1) {
#pragma unroll
    for (; want < q0 + S::D; want++) pull.fetch(a, want, wave);
  }
  // Opens step j.  Block j + 2 has landed (its statistics are formed in this step; AGAIN: block
  // j + 1), and what is carried into block j - 1's dQ.  A step issues, in this order, the transfers
  // of block j + 6, that of the carry for block j + 3 (from the second step on, four in the first) and
  // a store of dQ; so from the fourth step on at least the block's three successors have been
  // requested since (AGAIN: four), and after the carry three blocks and carries; before, one block
  // and three carries.  (What else is among them only makes a wait longer.)
  auto open = [&](int j) {
    if (NH > 1) {
      if (j == q0) wait_vmem<0>();  // (the ring holds all there is)
      if (!LATE && wave == 0 && j == q0 + kFusedNext<NH> - 1) wait_vmem<0>();  // (the next item's sequence)
    } else if (j > q0 + 2) {
      if (AGAIN && carry_in)
        wait_vmem<3 * (Pull::kGroup + 1)>();
      else
        wait_vmem<3 * Pull::kGroup>();
    } else if (j > q0) {
      if (AGAIN)
        wait_vmem<3>();
      else
        wait_vmem<Pull::kGroup>();
    }
    lds_barrier();
    if (NH == 1) {
      if (j < q0 + 3) pull.fetch(a, want++, wave);
      pull.fetch(a, want++, wave);
    }
  };
  auto close = [&](int j) {
    if (AGAIN) return;
    if (j + 2 < q1) fw.statistics(j + 2);
    if ((j & 7) == wave) fw.keep_statistics(j);
  };
  auto dq_step = [&](int j) {
    if (carry_in) carry_fetch();
    if (want_dq) {
      fw.dq_finish(j - 1);
      if (LATE || NH == 2)
        if (!fw.to_slab && j > q0 + 1) fw.dq_out(j - 2);
    }
  };
  open(q0);
  if (carry_in) {
#pragma unroll
    for (int i = 0; i < kCarry; i++) carry_fetch();
  }
  if (wave_on) {
    fw.scores(q0);
    fw.template step<true, LATE>(q0);
    if (!LATE && q0 + 1 < q1) fw.scores(q0 + 1);
  } else {
    fw.no_scores(q0);
    fw.no_scores(q0 + 1);
  }
  close(q0);
  publish();
  if (wave_on) {
#pragma unroll 1
    for (int j = q0 + 1; j < q1; j++) {
      open(j);
      fw.dq_begin(place, carry_in);
      if (LATE) fw.scores(j);
      fw.template step<false, LATE>(j);
      if (!LATE && j + 1 < q1) fw.scores(j + 1);
      close(j);
      dq_step(j);
    }
  } else {
#pragma unroll 1
    for (int j = q0 + 1; j < q1; j++) {
      open(j);
      fw.dq_begin(place, carry_in);
      fw.dq_products(j - 1);
      close(j);
      dq_step(j);
    }
  }
}

// A sweep from "its first transfers have landed" to its results and to the first transfers of the one
// after it.  `publish` is called once in it, behind its first step; `next` then finds out whether
// there is another sweep and puts it into nx.  Returns that.
template <typename T, int NH, bool DROP, typename Publish, typename Next>
static __device__ __forceinline__ bool fused_sweep(const FusedPhase& phase, const FusedPhase& nx, FusedShared& lds, int wave, u32x4* slab,
                                                   u32x4 (&kb)[4], u32x4 (&vb)[4], Publish publish, Next next) {
  using S = FusedShape<NH>;
  const BwdArgs& a = fused_args();
  const FusedPhase ph = phase.scalar();
  FusedWave<T, NH, DROP> fw(a, lds, ph, wave, kb, vb, slab);
  const int key0 = ph.kt * kFusedKeys;
  const bool wave_on = key0 + 32 * fw.kg < ph.nk && ph.head + fw.hd < a.pb.heads;
  const int q0 = ph.q0, q1 = ph.q1;
  {
    const uint32_t tile = fused_tile<NH>(lds, wave);
    fused_operands(tile, fw.row_rd, vb);
    fused_operands(tile, fw.row_rd, kb);  // (read back transposed by all wavefronts below)
  }
  if (key0 + 32 * fw.kg + 32 > ph.nk) {  // (dP of a key that does not exist is 0, whatever its copy of V gives)
    const uint32_t on = key0 + 32 * fw.kg + (lane_id() & 31) < ph.nk ? 0xffffffffu : 0u;
#pragma unroll
    for (int t = 0; t < 4; t++) vb[t] &= u32x4{on, on, on, on};
  }
  lds_barrier();
  {
    const int lane = lane_id();
    const int e = (lane >> 2) & 3, pc = lane & 3, g4 = lane >> 4;
    const int nkeys = min(ph.nk - key0, kFusedKeys);
#pragma unroll
    for (int c = 0; c < S::NCH; c++) {
      const int cq = NH == 1 ? (wave >> 1) : fw.kg * S::NCH + c;
      const uint32_t at = fused_tile<NH>(lds, 0) + fw.hd * (S::KG * 4096);
      const uint32_t lo_off = 2 * tile_off(4 * g4 + e, 16 * cq + 4 * pc), hi_off = 2 * tile_off(4 * g4 + e + 16, 16 * cq + 4 * pc);
#pragma unroll
      for (int k = 0; k < S::KS; k++) {
        const uint32_t tile = fused_tile<NH>(lds, k) - fused_tile<NH>(lds, 0);
        const u32x2 lo = lds_get_tr16(at + lo_off + tile), hi = lds_get_tr16(at + hi_off + tile);
        fw.kT[c][k] = u32x4{lo[0], lo[1], hi[0], hi[1]};
      }
    }
    // keys that do not exist take no part
    if (nkeys < 32 * S::KS) {
#pragma unroll
      for (int k = 0; k < S::KS; k++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const int key = 32 * k + 4 * g4 + 16 * (i >> 1) + 2 * (i & 1);
          const uint32_t m = key + 1 < nkeys ? 0xffffffffu : key < nkeys ? 0xffffu : 0u;
#pragma unroll
          for (int c = 0; c < S::NCH; c++) fw.kT[c][k][i] &= m;
        }
    }
  }
  const bool again = NH == 1 && ph.step > 0;
  if (!again) {
    fw.statistics(q0);
    if (q0 + 1 < q1) fw.statistics(q0 + 1);
  }
#pragma unroll
  for (int cb = 0; cb < 2; cb++)
#pragma unroll
    for (int r = 0; r < 16; r++) fw.dk[cb][r] = fw.dv[cb][r] = 0.f;
  if (wave < 4) {
    if (again)
      fused_steps<T, NH, DROP, false, NH == 1>(fw, a, ph, lds, wave, wave_on, slab, publish);
    else
      fused_steps<T, NH, DROP, false, false>(fw, a, ph, lds, wave, wave_on, slab, publish);
  } else {
    if (again)
      fused_steps<T, NH, DROP, true, NH == 1>(fw, a, ph, lds, wave, wave_on, slab, publish);
    else
      fused_steps<T, NH, DROP, true, false>(fw, a, ph, lds, wave, wave_on, slab, publish);
  }
  const bool want_dq = ph.want & 2, rows_out = want_dq && !fw.to_slab && (NH == 2 || wave >= 4);
  // The next sweep's K and V are requested now (their registers are free), its first query blocks
  // behind the barrier.
  const bool few = q1 - q0 < kFusedNext<NH>;  // (then what was published is only seen behind the barrier)
  bool more = !few && next();
  if (more) fused_load_kv<NH>(fused_args(), nx.scalar(), wave, kb, vb);
  if (wave_on) fw.last_products(q1 - 1);
  if (more)
    wait_vmem<8>();
  else
    wait_vmem<0>();
  // (read ahead of the barrier: the next sweep's transfers may go to the same place)
  if (want_dq) fw.dq_begin(((q1 - 1 - q0) & (kCarry - 1)) * (kFusedThreads * 16), again && ph.kt > 0);
  lds_barrier();
  if (few) {
    more = next();
    if (more) fused_load_kv<NH>(fused_args(), nx.scalar(), wave, kb, vb);
  }
  if (rows_out && q1 - q0 > 1) fw.dq_out(q1 - 2);
  if (more) fused_begin<NH>(fused_args(), nx, lds, wave);
  if (want_dq) {
    fw.dq_products(q1 - 1);
    // (NH == 1: straight out, which saves a barrier; early wavefronts have not followed dq_at)
    if (NH == 1 && !fw.to_slab) fw.dq_at = fw.dq_first + (int64_t)(q1 - 1 - q0) * fw.dq_step;
    fw.dq_finish(q1 - 1, NH != 2);
  }
  if (NH > 1) lds_barrier();
  if (NH == 2 && rows_out) fw.dq_out(q1 - 1);
  // The next sweep's K, V and first blocks have to have landed at the end.  Behind them there are at
  // least the 8 stores of a whole tile of keys, which need not be awaited.
  if (ph.want & 1) fw.store_keys(fused_args());
  if ((ph.want & 1) && key0 + 32 * fw.kg + 32 <= ph.len && ph.head + fw.hd < a.pb.heads)
    wait_vmem<8>();
  else
    wait_vmem<0>();
#pragma unroll
  for (int t = 0; t < 4; t++) asm volatile("" : "+v"(kb[t]), "+v"(vb[t]));
  return more;
}

// The items of one kind (NH heads at a time), from `item` on: the first is item `begin` of the
// whole list, the last lies before `end`.  Returns the first item of the workgroup that is not.
template <typename T, int NH, bool DROP>
static __device__ __forceinline__ int fused_items(const BwdArgs& a, FusedShared& lds, int wave, int item, int begin, int end, int record) {
  item = __builtin_amdgcn_readfirstlane(item);
  if (item >= end) return item;
  const int groups = (a.pb.heads + NH - 1) / NH;
  const int cls = blockIdx.x & 7, per_class = gridDim.x >> 3;
  const int fit = (a.slab_rows >> 5) & ~7;  // blocks of fp32 dQ that can be kept
  u32x4* slab = reinterpret_cast<u32x4*>(a.slab) + (int64_t)blockIdx.x * a.slab_rows * 16;
  uint32_t* counter = a.feed.counters + cls * kFeedClassWords;
  auto set_step = [&](FusedPhase& ph, int step) {
    const int nq = (ph.len + 31) >> 5;
    ph.step = step;
    ph.kt = NH == 1 ? step % ph.n_kt : 0;
    ph.q0 = 0;
    ph.q1 = nq;
    ph.want = 3;
    if (NH == 1 && ph.steps > ph.n_kt) {
      ph.want = step < ph.n_kt ? 1 : 2;
      if (step >= ph.n_kt) {
        ph.q0 = (step / ph.n_kt - 1) * fit;
        ph.q1 = min(nq, ph.q0 + fit);
      }
    }
  };
  auto phase_of = [&](int i, int rec, int r0, int len, int nk) {
    FusedPhase ph;
    ph.head = NH * (i - begin - rec * groups);
    ph.r0 = r0;
    ph.len = len;
    ph.nk = nk;
    ph.n_kt = NH > 1 ? 1 : max((ph.nk + kFusedKeys - 1) / kFusedKeys, 1);
    const int nq = (ph.len + 31) >> 5;
    ph.steps = ph.n_kt == 1 || nq <= fit ? ph.n_kt : ph.n_kt * (1 + (nq + fit - 1) / fit);
    set_step(ph, 0);
    return ph.scalar();
  };
  const int rec0 = (item - begin) / groups;
  ConstInt p = (ConstInt)(uintptr_t)(a.seqs + record + rec0);
  FusedPhase ph = phase_of(item, rec0, p[0], p[1], p[2]);
  u32x4 kb[4], vb[4];
  fused_load_kv<NH>(a, ph, wave, kb, vb);
  fused_begin<NH>(a, ph, lds, wave);
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
#pragma unroll
  for (int t = 0; t < 4; t++) asm volatile("" : "+v"(kb[t]), "+v"(vb[t]));
  while (true) {
    const bool last = NH > 1 || ph.step + 1 == ph.steps;
    uint32_t claimed = 0;
    if (last && threadIdx.x == 0)
      claimed = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    FusedPhase nx = ph;
    auto publish = [&]() {
      if (!last || wave != 0) return;
      const int it = (per_class + __builtin_amdgcn_readfirstlane((int)claimed)) * kFeedClasses + cls;
      const int rec = (it - begin) / groups;
      if (lane_id() == 0) {
        lds.mail[0] = it;
        lds.mail[1] = rec;
        if (it < end) dma16s((const void*)(uintptr_t)uniform_i64((int64_t)(uintptr_t)(fused_args().seqs + record + rec)), 0, lds_at(&lds.record));
      }
    };
    auto next = [&]() {
      if (NH > 1 || last) {
        auto s = [](uint32_t x) { return __builtin_amdgcn_readfirstlane((int)x); };
        item = s(lds.mail[0]);
        if (item >= end) return false;
        const u32x4 r = lds_get<u32x4>(lds_at(&lds.record));
        nx = phase_of(item, s(lds.mail[1]), s(r[0]), s(r[1]), s(r[2]));
      } else {
        set_step(nx, ph.step + 1);
        nx = nx.scalar();
      }
      return true;
    };
    const bool more = fused_sweep<T, NH, DROP>(ph, nx, lds, wave, slab, kb, vb, publish, next);
    if (!more) {
      if (NH == 1) lds_barrier();  // (what follows uses the LDS in another way)
      return item;
    }
    ph = nx;
  }
}

template <typename T, bool DROP>
__global__ __launch_bounds__(kFusedThreads, 2) void bwd_fused_kernel(const BwdArgs a) {
  __shared__ __align__(1024) FusedLds lds;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (the entries behind the statistics that stand for no row; every workgroup reads its own write)
  if (threadIdx.x == 0) {
    a.lse2[(int64_t)a.pb.heads * a.pb.total_tokens] = INFINITY;
    a.dsum[(int64_t)a.pb.heads * a.pb.total_tokens] = 0.f;
  }
  // Items: those of sequences taken one head at a time first, then two, then four.  Position k
  // of a class (die) is item 8 k + class; a workgroup's first one is its rank in the class, all others
  // are claimed while the item before is computed.
  ConstInt sec = (ConstInt)(uintptr_t)(a.pb.n_tiles + 1);
  const int n1 = sec[0], n2 = sec[1], n4 = sec[2];
  const int i1 = n1 * a.pb.heads, i2 = i1 + n2 * ((a.pb.heads + 1) >> 1), i4 = i2 + n4 * ((a.pb.heads + 3) >> 2);
  const int cls = blockIdx.x & 7, per_class = gridDim.x >> 3;
  int item = (int)(blockIdx.x >> 3) * kFeedClasses + cls;
  FusedShared& shared = *(FusedShared*)&lds;
  static_assert(kFusedThreads == 64 * kFusedSlots, "one thread per entry");
  lds.stat[threadIdx.x >> 6][64 + (threadIdx.x & 63)] = (threadIdx.x & 32) ? 0.f : INFINITY;
  item = fused_items<T, 1, DROP>(a, shared, wave, item, 0, i1, 0);
  item = fused_items<T, 2, DROP>(a, shared, wave, item, i1, i2, n1);
  item = fused_items<T, 4, DROP>(a, shared, wave, item, i2, i4, n1 + n2);
  // the last workgroup of a class leaves its counters zero
  if (threadIdx.x == 0) {
    uint32_t* counter = a.feed.counters + cls * kFeedClassWords;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (__hip_atomic_fetch_add(counter + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)per_class - 1u) {
      __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(counter + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

}  // namespace fmha
