// Device-side helpers shared by the libmtla kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mtla {

constexpr int kWave = 64;          // CDNA wavefront width
constexpr int kBlock = 256;        // threads per workgroup in the VALU kernels (4 waves)
constexpr int kHeaderBytes = 256;  // workspace header, cleared once: int32[0] is the sticky device status,
constexpr int kArrivalWord = 8;    // from here on the counters of a decode step in one launch (zeros between launches)

// Storage element types.  bf16 is carried as its 16-bit pattern.
struct bf16 {
  uint16_t bits;
};

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return __uint_as_float(uint32_t(v.bits) << 16); }

// fp32 -> bf16, round to nearest, ties to even: gfx950's v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}
// Two fp32 values to a packed bf16 pair (lo in bits 0..15), one instruction.
// One int32 at a wavefront-uniform address, from memory that nothing writes while the kernel runs (a page
// table): read through the constant address space, so that it is a scalar load and has a wait counter of its
// own.  As an ordinary load it is a vector load, and waiting for it means waiting for every tile load in flight.
__device__ __forceinline__ int32_t load_uniform_i32(const int32_t* p, int idx) {
  typedef const int32_t __attribute__((address_space(4))) * const_i32_ptr;
  return reinterpret_cast<const_i32_ptr>(reinterpret_cast<uintptr_t>(p))[idx];
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
// Two fp32 values to a packed IEEE-half pair (lo in bits 0..15), round to nearest even.
__device__ __forceinline__ uint32_t pack_f16x2(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));
}
// ... and back.
__device__ __forceinline__ float f16_lo_to_f32(uint32_t v) {
  return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(v & 0xffffu)));
}
__device__ __forceinline__ float f16_hi_to_f32(uint32_t v) {
  return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(v >> 16)));
}

// 8 consecutive stored elements as fp32.
__device__ __forceinline__ void load8(const bf16* p, float (&o)[8]) {
  const uint4 v = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[2 * i] = __uint_as_float(w[i] << 16);
    o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ void load8(const float* p, float (&o)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
  o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}

// fp32 pair -> bf16 pair hi plus bf16 pair lo with hi + lo ~ value to about 16 mantissa bits.
__device__ __forceinline__ void split_bf16x2(float a, float b, uint32_t& hi, uint32_t& lo) {
  hi = pack_bf16x2(a, b);
  lo = pack_bf16x2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

template <typename T>
__device__ __forceinline__ T from_f32(float v);
template <>
__device__ __forceinline__ float from_f32<float>(float v) {
  return v;
}
template <>
__device__ __forceinline__ bf16 from_f32<bf16>(float v) {
  return bf16{f32_to_bf16_bits(v)};
}

// Cross-lane reductions on the vector ALU: row permutations (DPP) inside 16 lanes, v_permlane16_swap and
// v_permlane32_swap between them.  __shfl_xor goes through the LDS unit instead, about 120 cycles a step: a sum over a
// wavefront was 0.3 us of decode kernels that last 2.5 to 4.5.
struct LaneSum {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct LaneMax {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
template <int CTRL>
__device__ __forceinline__ float row_permuted(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// Over aligned groups of N lanes (N a power of two up to the wavefront); every lane gets its group's value.
template <int N, class Op>
__device__ __forceinline__ float group_reduce(float v, Op op) {
  if constexpr (N >= 2) v = op(v, row_permuted<0xb1>(v));   // lane ^ 1
  if constexpr (N >= 4) v = op(v, row_permuted<0x4e>(v));   // lane ^ 2
  if constexpr (N >= 8) v = op(v, row_permuted<0x141>(v));  // mirrored within 8: the other four, all alike by now
  if constexpr (N >= 16) v = op(v, row_permuted<0x140>(v)); // mirrored within 16: the other eight
  if constexpr (N >= 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  if constexpr (N >= 64) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  return v;
}
template <int CTRL>
__device__ __forceinline__ float row_rotated(float v) {  // inside 16 lanes
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + CTRL, 0xf, 0xf, true));
}
// Over the four lanes l16, l16 + 16, + 32, + 48 (the lanes that share a row or column of a matrix tile).
template <class Op>
__device__ __forceinline__ float quarter_reduce(float v, Op op) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(t[0]), __uint_as_float(t[1]));
}
// Inclusive running sum over the wavefront.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // inside 16 lanes: from 1, 2, 4 and 8 lanes below
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // lane 15 to the row above, lane 47 likewise
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // lane 31 to the upper half
  return v;
}
__device__ __forceinline__ float wave_sum(float v) { return group_reduce<kWave>(v, LaneSum()); }
__device__ __forceinline__ float wave_max(float v) { return group_reduce<kWave>(v, LaneMax()); }

// (cos, sin) of pos * freq, freq = base^(-2k/d) (a double, from the host: positions reach tens of thousands of radians, so the
// product and its reduction to a quarter turn are done in double).  Taylor series in float from there: what they leave out is
// below 2e-9 at pi / 4.  Some forty instructions without a branch, where the library's pair of any argument is several hundred
// that a cold launch fetches first (a short prompt's projections 9.1 us with the library's pair, 8.6 with this one); largest error against 64 bits over 200000 positions
// 6.9e-8, the library's behind a reduction to a whole turn 1.3e-7.
__device__ __forceinline__ float2 rope_angle(int pos, double freq) {
  const double ang = (double)pos * freq, q = rint(ang * 0.63661977236758134308);
  const float x = (float)fma(q, -1.57079632679489661923, ang), z = x * x;
  const float sp = fmaf(z, fmaf(z, fmaf(z, 1.f / 362880, -1.f / 5040), 1.f / 120), -1.f / 6);
  const float cp = fmaf(z, fmaf(z, fmaf(z, fmaf(z, -1.f / 3628800, 1.f / 40320), -1.f / 720), 1.f / 24), -0.5f);
  const float sn = fmaf(x * z, sp, x), cs = fmaf(z, cp, 1.f);
  const int k = (int)q;  // quarter turns
  const float c = (k & 1) ? sn : cs, s = (k & 1) ? cs : sn;
  return make_float2(((k + 1) & 2) ? -c : c, (k & 2) ? -s : s);
}

// A pair of elements (2k, 2k + 1) of a vector, turned by that angle.
__device__ __forceinline__ float2 rope_turn(float2 v, float2 cs) { return make_float2(v.x * cs.x - v.y * cs.y, v.x * cs.y + v.y * cs.x); }

}  // namespace mtla
