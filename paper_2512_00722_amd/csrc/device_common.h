// Device helpers shared by the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spec {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// bf16 bit pattern -> fp32 (exact: bf16 is the high half of a binary32).
__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Unpack 8 bf16 (one 16-byte load) to fp32.
__device__ __forceinline__ void unpack8(const uint4& v, float* f) {
  f[0] = bf16lo(v.x); f[1] = bf16hi(v.x);
  f[2] = bf16lo(v.y); f[3] = bf16hi(v.y);
  f[4] = bf16lo(v.z); f[5] = bf16hi(v.z);
  f[6] = bf16lo(v.w); f[7] = bf16hi(v.w);
}

__device__ __forceinline__ uint4 ldg16(const uint16_t* p) {
  return *reinterpret_cast<const uint4*>(p);
}

// Four floats in one 16-byte load from a 4-byte aligned address.
__device__ __forceinline__ float4 read16(const float* p) {
  typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
  const floatx4u v = *reinterpret_cast<const floatx4u*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}

// Streaming 16-byte load: data read once, hint the caches not to keep it.
__device__ __forceinline__ uint4 ldg16_stream(const uint16_t* p) {
  const uint4* q = reinterpret_cast<const uint4*>(p);
  uint4 r;
  r.x = __builtin_nontemporal_load(&q->x);
  r.y = __builtin_nontemporal_load(&q->y);
  r.z = __builtin_nontemporal_load(&q->z);
  r.w = __builtin_nontemporal_load(&q->w);
  return r;
}

// Order-preserving map of an fp32 to uint32 (larger float -> larger key).
__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ int clampi(int x, int lo, int hi) {
  return x < lo ? lo : (x > hi ? hi : x);
}

// ---- cross-lane reductions inside a 16-lane DPP row (no LDS traffic) ----
// DPP controls: quad_perm [1,0,3,2] = 0xB1, quad_perm [2,3,0,1] = 0x4E,
// row_half_mirror = 0x141, row_mirror = 0x140.  After the four steps every
// lane of the row holds the reduction over its 16 lanes (8 lanes: three).
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <int N>  // N in {2, 4, 8, 16}
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_f<0xB1>(v);
  if (N >= 4) v += dpp_f<0x4E>(v);
  if (N >= 8) v += dpp_f<0x141>(v);
  if (N >= 16) v += dpp_f<0x140>(v);
  return v;
}
template <int N>
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp_f<0xB1>(v));
  if (N >= 4) v = fmaxf(v, dpp_f<0x4E>(v));
  if (N >= 8) v = fmaxf(v, dpp_f<0x141>(v));
  if (N >= 16) v = fmaxf(v, dpp_f<0x140>(v));
  return v;
}

// Combine two (max, sum-of-exp2) pairs; -inf max marks an empty pair.
__device__ __forceinline__ void ms_combine(float& m, float& s, float m2, float s2) {
  if (m2 == -INFINITY) return;
  if (m == -INFINITY) { m = m2; s = s2; return; }
  const float mn = fmaxf(m, m2);
  s = s * exp2f(m - mn) + s2 * exp2f(m2 - mn);
  m = mn;
}

}  // namespace spec
