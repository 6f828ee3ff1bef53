// Stand-ins with which the backward kernels compile for the CPU: a lane is a fiber, and what
// crosses lanes is a meeting of the wavefront's fibers (backward.cpp).
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __restrict__
#define __align__(x)
#define __ATOMIC_RELAXED 0
#define __HIP_MEMORY_SCOPE_AGENT 0

using std::max;
using std::min;

struct Index {
  unsigned x;
};
struct float4 {
  float x, y, z, w;
};

namespace emu {

enum Meeting { kFirstLane, kDpp, kSwapHalves, kReadTr16, kMfma32F16, kMfma32Bf16, kMfma16F16, kMfma16Bf16, kWave, kWorkgroup };

extern Index block, grid;
extern unsigned char* lds;   // below 4 GiB, so that 32 bits hold an LDS address
extern const void* kernarg;
Index& thread();
unsigned char* in();         // 64 bytes each of the lane's own
unsigned char* out();
void meet(Meeting what, int imm = 0);
void dma(const void* from, uint32_t lds_address, int bytes_per_lane);

template <typename T, typename U>
inline T exchange(Meeting what, const U& x, int imm = 0) {
  memcpy(in(), &x, sizeof x);
  meet(what, imm);
  T r;
  memcpy(&r, out(), sizeof r);
  return r;
}
template <typename A, typename C>
inline C mfma(Meeting what, A a, A b, C c) {
  memcpy(in(), &a, 16);
  memcpy(in() + 16, &b, 16);
  meet(what);
  C d;
  memcpy(&d, out(), sizeof d);
  return c + d;
}
struct Pair {
  uint32_t v[2];
  uint32_t operator[](int i) const { return v[i]; }
};
typedef short Four __attribute__((__vector_size__(8)));
template <typename V>
inline float dot2(V a, V b, float c, bool) {
  return fmaf((float)a[0], (float)b[0], fmaf((float)a[1], (float)b[1], c));
}
inline uint32_t align_bits(uint32_t hi, uint32_t lo, uint32_t s) {
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> (s & 31));
}
inline uint32_t permute(uint32_t hi, uint32_t lo, uint32_t select) {
  const uint64_t v = ((uint64_t)hi << 32) | lo;
  uint32_t r = 0;
  for (int i = 0; i < 4; i++) r |= (uint32_t)((v >> (8 * ((select >> (8 * i)) & 7))) & 255) << (8 * i);
  return r;
}
inline uint32_t fetch_add(uint32_t* p, uint32_t v) {
  const uint32_t old = *p;
  *p += v;
  return old;
}

}  // namespace emu

#define threadIdx (emu::thread())
#define blockIdx (emu::block)
#define gridDim (emu::grid)
#define __syncthreads() emu::meet(emu::kWorkgroup)
#define __hip_atomic_fetch_add(p, v, order, scope) emu::fetch_add((p), (v))
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))

#define __builtin_amdgcn_readfirstlane(x) ((decltype(+(x)))emu::exchange<uint32_t>(emu::kFirstLane, (uint32_t)(x)))
#define __builtin_amdgcn_update_dpp(old, x, ctrl, rows, banks, bound) emu::exchange<int>(emu::kDpp, (int)(x), (ctrl))
#define __builtin_amdgcn_permlane32_swap(a, b, fi, bc) emu::exchange<emu::Pair>(emu::kSwapHalves, (uint32_t)(a))
#define __builtin_amdgcn_ds_read_tr16_b64_v4i16(p) emu::exchange<emu::Four>(emu::kReadTr16, (uint64_t)(uintptr_t)(p))
#define __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, x, y, z) emu::mfma(emu::kMfma32F16, (a), (b), (c))
#define __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, x, y, z) emu::mfma(emu::kMfma32Bf16, (a), (b), (c))
#define __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, x, y, z) emu::mfma(emu::kMfma16F16, (a), (b), (c))
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) emu::mfma(emu::kMfma16Bf16, (a), (b), (c))
#define __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_fdot2 emu::dot2
#define __builtin_amdgcn_fdot2_f32_bf16 emu::dot2
#define __builtin_amdgcn_wave_barrier() emu::meet(emu::kWave)
#define __builtin_amdgcn_s_waitcnt(x) emu::meet(emu::kWave)
#define __builtin_amdgcn_sched_barrier(x)
#define __builtin_amdgcn_s_setprio(x)
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_mbcnt_lo(mask, below) (below)
#define __builtin_amdgcn_mbcnt_hi(mask, below) (emu::thread().x & 63)
#define __builtin_amdgcn_alignbit(hi, lo, s) emu::align_bits(hi, lo, s)
#define __builtin_amdgcn_perm(hi, lo, s) emu::permute(hi, lo, s)
#define __builtin_amdgcn_bitop3_b32(a, b, c, table) ((a) ^ (b) ^ (c))
#define __builtin_amdgcn_kernarg_segment_ptr() (emu::kernarg)
