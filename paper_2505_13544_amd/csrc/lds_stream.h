// fp16 operands of the prefill kernels (gfx950): memory -> LDS without registers, swizzles, waits, conversions.
#pragma once
#include "mtla_device.h"

namespace mtla {

namespace {

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));  // staging registers (a plain vector type: promoted reliably)
typedef short4_t __attribute__((address_space(3))) * lds_short4_ptr;

// 8 bf16 values, each times `scale` -> 8 fp16 values
__device__ __forceinline__ u32x4_t bf16x8_to_f16x8(u32x4_t v, float scale = 1.f) {
  u32x4_t o;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    o[i] = pack_f16x2(__uint_as_float(v[i] << 16) * scale, __uint_as_float(v[i] & 0xffff0000u) * scale);
  return o;
}

// ---- memory -> LDS without registers --------------------------------------------------------
//
// The prefill kernels stream their operands from memory straight into LDS: 16 bytes per lane, 64
// lanes fill 1 KB of consecutive LDS, several tiles ahead of the one being multiplied, so no
// register carries a tile and one barrier per tile is enough.  Rows are stored without padding;
// each 16-byte piece j of row `row` sits at position j ^ swizzle(row), chosen per region so that
// the reads of the matrix-core operands are free of bank conflicts:
//   swz_rows16   ds_read_b128, 16 lanes = 16 consecutive rows, same logical piece
//   swz_tr       transposing 8-byte reads, 32 lanes = 8 consecutive rows x 32 bytes
// The swizzle is applied on the way in: a lane asks memory for the piece that belongs at its place.
// (PC pieces per row; 16 / PC short rows share 256 bytes, rows of 16 pieces and more start at the same bank.)
template <int PC>
__device__ __forceinline__ int swz_rows16(int row) {
  constexpr int P = PC < 16 ? PC : 16;
  // A read is served 16 lanes at a time: rows 0-3 and 12-15 of one piece with 4-11 of the next.  With four pieces a row the
  // rows' own order would put two of each such group in every bank (half of the LDS time of the matrix products).
  const int i = row / (16 / P);
  return (PC == 4 ? -i : i) & (P - 1);
}
template <int PC>
__device__ __forceinline__ int swz_tr(int row) {
  constexpr int P = PC < 16 ? PC : 16;
  return ((row / (16 / P)) & (P / 2 - 1)) << 1;
}

typedef __attribute__((address_space(3))) unsigned char* lds_byte_ptr;

// 64 lanes x 16 bytes from memory to 1 KB of LDS starting at byte address `lds_addr` (the same in
// every lane); lane i's 16 bytes land at lds_addr + 16 i.  Counted by vmcnt like any load.  Written
// as an instruction of its own so that the compiler keeps no account of it: the waits for these
// loads are the explicit ones below, and ordinary LDS reads are not held back by loads in flight
// into another buffer.
__device__ __forceinline__ void load_to_lds_16(const void* src, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(src) : "memory", "m0");
}
// The same with the address as a wavefront-uniform base and a 32-bit byte offset per lane: a loop that only moves the
// base pays no vector instruction for the addresses of its loads.
__device__ __forceinline__ void load_to_lds_16(const void* base, uint32_t off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(off), "s"(base) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_loads_but() {  // until at most N of this wavefront's loads are in flight
  static_assert(N >= 0 && N <= 63, "vmcnt field");
  if constexpr (N == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
// workgroup barrier without a fence: callers order their own memory traffic around it
__device__ __forceinline__ void barrier_only() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// <x, y> of 8 fp16 pairs, summed in fp32
__device__ __forceinline__ float dot8(u32x4_t x, u32x4_t y, float c) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t xi = x[i], yi = y[i];  // (a bit_cast of a vector element takes element 0)
    c = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2_t, xi), __builtin_bit_cast(f16x2_t, yi), c, false);
  }
  return c;
}

}  // namespace

}  // namespace mtla
