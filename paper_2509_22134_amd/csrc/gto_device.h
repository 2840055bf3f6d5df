// Device-side helpers shared by the GTO kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gto {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr float kLog2e = 1.44269504088896340736f;   // fp32(log2 e)
constexpr double kLn2 = 0.693147180559945309417232121458;
constexpr int kNoId = 0x7fffffff;                   // id of an empty top-k entry (loses every tie)

__device__ __forceinline__ float neg_inf() { return -__builtin_inff(); }

__device__ __forceinline__ int lane_id() {
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// lane i receives the value of lane i-1; lane 0 receives `fill`.
__device__ __forceinline__ int wave_shr1(int v, int fill) {
  return __builtin_amdgcn_update_dpp(fill, v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}
__device__ __forceinline__ float wave_shr1(float v, float fill) {
  return __int_as_float(wave_shr1(__float_as_int(v), __float_as_int(fill)));
}

__device__ __forceinline__ float readlane(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ int readlane(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
  return v;
}
__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = min(v, __shfl_xor(v, off, kWave));
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// (value, id) ordering used everywhere: larger value first, lower id first among equals.
__device__ __forceinline__ bool better(float v, int id, float w, int jd) {
  return (v > w) || (v == w && id < jd);
}

// Monotone map of an fp32 score to uint32 (larger float -> larger uint); -0 and +0 coincide.
__device__ __forceinline__ uint32_t ordered_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_ordered_bits(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// Packed ranking key: (score descending, index ascending) is descending key order.  Keys are unique and never 0.
__device__ __forceinline__ uint64_t rank_key(float score, int index) {
  return ((uint64_t)ordered_bits(score) << 32) | (uint32_t)(0xffffffffu - (uint32_t)index);
}
__device__ __forceinline__ float key_score(uint64_t key) { return from_ordered_bits((uint32_t)(key >> 32)); }
__device__ __forceinline__ int key_index(uint64_t key) { return (int)(0xffffffffu - (uint32_t)key); }

// s * 2^e for an integer-valued e (far below the exponent range: zero); exact but for underflow.
__device__ __forceinline__ double scale_pow2(double s, float e) { return __builtin_amdgcn_ldexp(s, (int)fmaxf(e, -4000.f)); }

// Number of set lanes below this one.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Wave reductions in DPP moves (rows of 16, then across rows): the result is the same in every lane.
template <int CTRL>
__device__ __forceinline__ float dpp(float v, float fill) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(fill), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {      // lanes without a source receive 0
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
__device__ __forceinline__ float wave_max_dpp(float v) {
  const float f = neg_inf();
  v = fmaxf(v, dpp<kRowShr + 1>(v, f));
  v = fmaxf(v, dpp<kRowShr + 2>(v, f));
  v = fmaxf(v, dpp<kRowShr + 4>(v, f));
  v = fmaxf(v, dpp<kRowShr + 8>(v, f));
  v = fmaxf(v, dpp<kRowBcast15>(v, f));
  v = fmaxf(v, dpp<kRowBcast31>(v, f));
  return readlane(v, 63);
}
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v += dpp<kRowShr + 1>(v);
  v += dpp<kRowShr + 2>(v);
  v += dpp<kRowShr + 4>(v);
  v += dpp<kRowShr + 8>(v);
  v += dpp<kRowBcast15>(v);
  v += dpp<kRowBcast31>(v);
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, 63), hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 63);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ uint32_t wave_max_dpp(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowShr + 1, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowShr + 2, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowShr + 4, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowShr + 8, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowBcast15, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowBcast31, 0xf, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Value of lane `lane ^ M`: DPP moves inside a row of 16, a permute through LDS beyond.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  const int x = (int)v;
  if constexpr (M == 1) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xb1 /* quad 1,0,3,2 */, 0xf, 0xf, true);
  else if constexpr (M == 2) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x4e /* quad 2,3,0,1 */, 0xf, 0xf, true);
  else if constexpr (M == 4)      // ^7 within eight lanes, then ^3 within four
    return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true), 0x1b, 0xf, 0xf, true);
  else if constexpr (M == 8) return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x128 /* row_ror:8 */, 0xf, 0xf, true);
  else return (uint32_t)__shfl_xor(x, M, kWave);
}
template <int M>
__device__ __forceinline__ double lane_xor(double v) {
  const uint64_t u = __double_as_longlong(v);
  return __longlong_as_double(((uint64_t)lane_xor<M>((uint32_t)(u >> 32)) << 32) | lane_xor<M>((uint32_t)u));
}

// 16 bytes of logits -> fp32 values.
template <typename T> struct Elem;
template <> struct Elem<uint16_t> {           // bf16 storage
  static constexpr int kPerVec = 8;
  __device__ static __forceinline__ void unpack(const u32x4 &q, float *x) {
    x[0] = __uint_as_float(q.x << 16); x[1] = __uint_as_float(q.x & 0xffff0000u);
    x[2] = __uint_as_float(q.y << 16); x[3] = __uint_as_float(q.y & 0xffff0000u);
    x[4] = __uint_as_float(q.z << 16); x[5] = __uint_as_float(q.z & 0xffff0000u);
    x[6] = __uint_as_float(q.w << 16); x[7] = __uint_as_float(q.w & 0xffff0000u);
  }
  __device__ static __forceinline__ float load1(const uint16_t *p) {
    return __uint_as_float(((uint32_t)*p) << 16);
  }
};
template <> struct Elem<float> {
  static constexpr int kPerVec = 4;
  __device__ static __forceinline__ void unpack(const u32x4 &q, float *x) {
    x[0] = __uint_as_float(q.x); x[1] = __uint_as_float(q.y);
    x[2] = __uint_as_float(q.z); x[3] = __uint_as_float(q.w);
  }
  __device__ static __forceinline__ float load1(const float *p) { return *p; }
};

// Offset (in elements) of slot (l, j) of root r, and the index of its statistics entry.
__device__ __forceinline__ int64_t stat_index(int r, int l, int j, int d, int k) {
  return ((int64_t)r * d + l) * k + j;
}

}  // namespace gto
