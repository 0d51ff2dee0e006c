// Absorbed query on the matrix cores (bf16 storage): the body of one workgroup, shared by the
// stand-alone absorb kernel and the fused front kernel of a decode step.
#pragma once
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

// Rows (tokens) one workgroup walks, 16 per MFMA.  Few rows (a decode step): short walks and many
// workgroups, since a walk is a chain of load -> multiply -> store round trips (256 rows in one
// workgroup took 17 us at batch 256); many rows (prefill): long walks that keep W_K^(h) in registers.
__host__ __device__ constexpr int absorb_rows_per_block(int rows) { return rows >= 4096 ? 256 : 32; }
__host__ __device__ constexpr int absorb_col_blocks(int r) { return (r + 127) / 128; }

// ---------------------------------------------------------------------------
// absorb, bf16 on the matrix cores.  Block coordinates (bx, h, bz) span (absorb_col_blocks(r) + 1, n_heads, row groups).
// Workgroups x < absorb_col_blocks(r): wavefront w owns output columns n0 = (4x + w) * 32 .. + 31 of
// head h and walks the rows 16 at a time: D[n, row] = sum_k W[n, k] q[row, k], two matrix tiles side by side.  Row i of
// tile t is column n0 + 8 (i / 4) + 4 t + i % 4, so that a lane ends up with eight consecutive columns: it stores 16 bytes
// per plane and a row's 64 at once (with one tile per wavefront the rows went out in pieces of 32 bytes, and the front of a
// decode step of 256 sequences, 16 heads, r = 512 needed 1408 workgroups, more than are resident: 12.6 us, now 10.2).
// The last workgroup of a head copies (and scales) the RoPE query part.  The operand row is written
// as two bf16 planes, hi and lo (a.plane elements apart): the logits are then formed from an
// almost-fp32 query at the price of a second MFMA per K step, which removes the largest
// avoidable error of the bf16 path (rounding the absorbed query) for sequences of few slots.
// ---------------------------------------------------------------------------
// Weights and queries come memory -> LDS, four neighbouring lanes to 64 bytes of a row, and are read from there in the operand layout: loaded
// straight into it, where neighbouring lanes are 16 rows, they keep the address path of the unit for 66 cycles a load, and every wavefront
// fetched the queries for itself.
// QF32 (= a.q_f32, fixed at compile time so that the registers of the other form do not count against the
// kernel's occupancy: with both forms compiled in, d_head = 128 took 160 registers and a decode step at
// batch 256 ran its 1408 workgroups in almost three rounds).
template <int KK, bool QF32>  // d_head / 32
struct AbsorbLds {
  static constexpr int W = 2 * KK * 1024;                           // a wavefront's weights: [matrix tile][K step][16 rows][64 bytes]
  static constexpr int Q = KK * (QF32 ? 2048 : 1024);               // 16 rows: [K step][row][64 bytes, fp32: 128]
  static constexpr int bytes = (kBlock / kWave) * W + 2 * Q;
};

template <int KK, bool QF32>
__device__ __forceinline__ void absorb_mfma_block(const AbsorbArgs& a, int bx, int h, int bz, unsigned char* lds) {
  typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
  constexpr int kWaves = kBlock / kWave;
  constexpr int DH = 32 * KK;
  using L = AbsorbLds<KK, QF32>;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int r = a.r, dR = a.d_rope, E = r + dR;
  const int per_block = absorb_rows_per_block(a.rows);
  const int row_lo = bz * per_block;
  const int row_hi = row_lo + per_block < a.rows ? row_lo + per_block : a.rows;
  uint16_t* qcat = reinterpret_cast<uint16_t*>(a.qcat);

  if (bx == absorb_col_blocks(r)) {  // RoPE part: qcat[row, h, r + j] = scale * q_rope[row, h, j]
    const uint16_t* qr = reinterpret_cast<const uint16_t*>(a.q_rope);
    const int per_row = dR / 8;
    for (int idx = tid; idx < (row_hi - row_lo) * per_row; idx += kBlock) {
      const int row = row_lo + idx / per_row, j8 = idx % per_row;
      float v[8];
      if (QF32) load8(reinterpret_cast<const float*>(a.q_rope) + ((size_t)row * a.n_heads + h) * dR + 8 * j8, v);
      else load8(reinterpret_cast<const bf16*>(qr) + ((size_t)row * a.n_heads + h) * dR + 8 * j8, v);
      uint32_t hi[4], lo[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) split_bf16x2(v[2 * i] * a.scale_log2, v[2 * i + 1] * a.scale_log2, hi[i], lo[i]);
      uint16_t* dst = qcat + ((size_t)row * a.n_heads + h) * E + r + 8 * j8;
      *reinterpret_cast<uint4*>(dst) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
      *reinterpret_cast<uint4*>(dst + a.plane) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    }
    return;
  }

  const int n0 = (bx * kWaves + wv) * 32;
  const bool mine = n0 < r;  // (the others help with the queries)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_ptr)lds;
  const int q4 = lane >> 2, p4 = (lane & 3) ^ swz_rows16<4>(q4);  // row and 16 bytes of the 64 that a lane brings in
  if (mine) {
    const uint16_t* w = reinterpret_cast<const uint16_t*>(a.w_uk) + ((size_t)h * r + n0) * DH;
    const uint32_t at = (uint32_t)((8 * (q4 >> 2) + (q4 & 3)) * DH * 2 + 16 * p4);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) load_to_lds_16(w + 4 * nt * DH + 32 * kk, at, lds0 + (uint32_t)(wv * L::W + (nt * KK + kk) * 1024));
  }
  unsigned char* sQ = lds + kWaves * L::W;
  // the queries of rows row0 .. row0 + 31, a KB at a time by the wavefronts in turn; rows past the last one: copies of it
  auto request = [&](int row0) {
    constexpr int N = 2 * KK * (QF32 ? 2 : 1);
#pragma unroll
    for (int i = 0; i < (N + kWaves - 1) / kWaves; ++i) {
      const int c = wv + kWaves * i;
      if (c >= N) break;
      const int t = c / (N / 2), in_tile = c % (N / 2);
      if (row0 + 16 * t >= row_hi) break;  // (the tiles follow one another)
      if constexpr (QF32) {
        const int kk = in_tile >> 1, u = in_tile & 1, i16 = 8 * u + (lane >> 3), row = row0 + 16 * t + i16;
        const float* src = reinterpret_cast<const float*>(a.q) + ((size_t)(row < row_hi ? row : row_hi - 1) * a.n_heads + h) * DH + 32 * kk +
                           4 * ((lane & 7) ^ swz_rows16<8>(i16));
        load_to_lds_16(src, lds0 + (uint32_t)(kWaves * L::W + c * 1024));
      } else {
        const int row = row0 + 16 * t + q4;
        const uint16_t* src = reinterpret_cast<const uint16_t*>(a.q) + ((size_t)(row < row_hi ? row : row_hi - 1) * a.n_heads + h) * DH + 32 * in_tile + 8 * p4;
        load_to_lds_16(src, lds0 + (uint32_t)(kWaves * L::W + c * 1024));
      }
    }
  };
  request(row_lo);
  const uint32_t frag = (uint32_t)(l16 * 64 + ((g ^ swz_rows16<4>(l16)) << 4));
  u32x4_t wa[2][KK];
  // two 16-row tiles per pass, their operands requested together
  for (int row0 = row_lo; row0 < row_hi; row0 += 32) {
    if (row0 > row_lo) {
      __syncthreads();  // the rows before have been read
      request(row0);
    }
    wait_loads_but<0>();
    __syncthreads();
    if (!mine) continue;
    if (row0 == row_lo) {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) wa[nt][kk] = *reinterpret_cast<const u32x4_t*>(lds + wv * L::W + (nt * KK + kk) * 1024 + frag);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (row0 + 16 * t >= row_hi) break;  // wavefront-uniform
      float4_t acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
      const unsigned char* qt = sQ + t * L::Q;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        if constexpr (QF32) {  // unrounded queries: hi + lo planes, two matrix instructions per K step
          const float4_t v0 = *reinterpret_cast<const float4_t*>(qt + 2048 * kk + l16 * 128 + (((2 * g) ^ swz_rows16<8>(l16)) << 4));
          const float4_t v1 = *reinterpret_cast<const float4_t*>(qt + 2048 * kk + l16 * 128 + (((2 * g + 1) ^ swz_rows16<8>(l16)) << 4));
          uint4 hi, lo;
          split_bf16x2(v0[0], v0[1], hi.x, lo.x);
          split_bf16x2(v0[2], v0[3], hi.y, lo.y);
          split_bf16x2(v1[0], v1[1], hi.z, lo.z);
          split_bf16x2(v1[2], v1[3], hi.w, lo.w);
#pragma unroll
          for (int nt = 0; nt < 2; ++nt) {
            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wa[nt][kk]),
                                                              __builtin_bit_cast(bf16x8_t, hi), acc[nt], 0, 0, 0);
            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wa[nt][kk]),
                                                              __builtin_bit_cast(bf16x8_t, lo), acc[nt], 0, 0, 0);
          }
        } else {
          const bf16x8_t q8 = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(qt + 1024 * kk + frag));
#pragma unroll
          for (int nt = 0; nt < 2; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wa[nt][kk]), q8, acc[nt], 0, 0, 0);
        }
      }
      const int row = row0 + 16 * t + l16;
      if (row < row_hi) {  // lane holds columns n0 + 8g .. + 7 of its row
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          split_bf16x2(acc[i >> 1][2 * (i & 1)] * a.scale_log2, acc[i >> 1][2 * (i & 1) + 1] * a.scale_log2, hi[i], lo[i]);
        uint16_t* dst = qcat + ((size_t)row * a.n_heads + h) * E + n0 + 8 * g;
        *reinterpret_cast<uint4*>(dst) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        *reinterpret_cast<uint4*>(dst + a.plane) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
      }
    }
  }
}

}  // namespace mtla
