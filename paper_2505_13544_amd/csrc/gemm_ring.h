// Matrix products of few rows, D[n, row] = sum_k W[n, k] x[row, k] (gfx950): a workgroup owns TN x 16 outputs for TM x 16 rows, its
// wavefronts a share of the contraction each, so that nothing is fetched twice inside a workgroup and no barrier is needed before
// their sums meet.  For the projections of a decode step (layer.hip) and the products of short prompts (gemm_ring.hip).
//
// Operands go memory -> LDS -> operand layout, through a ring of the wavefront's own.  Straight into the operand layout the
// neighbouring lanes of a load are 16 rows, and a unit takes such a load one lane a cycle: 38 GB/s whatever is in flight.  With four
// neighbouring lanes to 64 bytes of a row it takes 115 (both with all units at it, operands in the L2s).
#pragma once
#include <type_traits>

#include "lds_stream.h"
#include "mtla_device.h"

namespace mtla {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// TM x 16 rows by TN x 16 outputs a workgroup of NW wavefronts, each with a ring of D K steps (of 32).  W and x are bf16 or fp16, or W is bf16
// and x fp32, which enters as bf16 hi + lo planes (two matrix instructions a step).
enum RingType { kRingBf16, kRingF16, kRingF32 };
template <int TM_, int TN_, int NW_, int D_, RingType TYPE_>
struct RingTile {
  static constexpr int TM = TM_, TN = TN_, NW = NW_, D = D_, NT = 64 * NW_, kTiles = TM_ * TN_;
  static constexpr RingType TYPE = TYPE_;
  static constexpr bool F32 = TYPE_ == kRingF32;
  static constexpr int XL = F32 ? 2 : 1, LOADS = TN_ + TM_ * XL;  // loads (1 KB) of 16 rows, of a step
  static constexpr int STAGE = 1024 * LOADS, LDS = NW_ * D_ * STAGE;
  static constexpr int CH = kTiles < 4 ? kTiles : 4;               // 16 x 16 tiles summed at a time
  static constexpr int kRow = 17;                                  // floats per output row: a column of four rows apart lies in other banks
  static constexpr int SUMS = NW_ * CH * 16 * kRow * 4;
  static constexpr int BYTES = LDS > SUMS ? LDS : SUMS;
  static_assert(kTiles % CH == 0 && D_ >= 3 && LOADS * (D_ - 2) <= 63 && BYTES <= 160 * 1024, "rounds, wait counts, LDS");
};

template <int N, class F>
__device__ __forceinline__ void each_down(F f) {  // f(N), f(N - 1), .. f(0)
  f(std::integral_constant<int, N>());
  if constexpr (N > 0) each_down<N - 1>(f);
}

// A wavefront's share of the contraction, `n` K steps from element `lo` on: acc[i][j] = D[n_j + 4g + v, row_i + l16], v = 0..3.
// Addresses: the tiles' first rows (wb; xb of the first row tile), and from there the lane's 16 bytes (w_at, x_at); `ring`: this
// wavefront's part of the LDS.
template <class C>
__device__ __forceinline__ void contract(float4_t (&acc)[C::TM][C::TN], const unsigned char* const (&wb)[C::TN], const uint32_t (&w_at)[C::TN], const unsigned char* xb,
                                         const uint32_t (&x_at)[C::TM][C::XL], int lo, int n, const unsigned char* ring, int l16, int g) {
  constexpr int TM = C::TM, TN = C::TN, D = C::D, LOADS = C::LOADS;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
  const uint32_t ring_addr = (uint32_t)(uintptr_t)(lds_byte_ptr)ring;
  auto issue = [&](int step) {
    const size_t k = (size_t)(lo + 32 * step);
    const uint32_t at = ring_addr + (uint32_t)(step % D) * C::STAGE;
#pragma unroll
    for (int j = 0; j < TN; ++j) load_to_lds_16(wb[j] + 2 * k, w_at[j], at + j * 1024);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int u = 0; u < C::XL; ++u)
        load_to_lds_16(xb + (C::F32 ? 4 : 2) * k, x_at[i][u], at + (TN + C::XL * i + u) * 1024);
  };
  const uint32_t w_off = (uint32_t)(l16 * 64 + ((g ^ swz_rows16<4>(l16)) << 4));
  const uint32_t x_swz = (uint32_t)swz_rows16<8>(l16);
  auto multiply = [&](int step) {
    const unsigned char* at = ring + (step % D) * C::STAGE;
    u32x4_t wf[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) wf[j] = *reinterpret_cast<const u32x4_t*>(at + j * 1024 + w_off);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const unsigned char* xt = at + (TN + C::XL * i) * 1024;
      if constexpr (C::F32) {
        const float4_t a = *reinterpret_cast<const float4_t*>(xt + l16 * 128 + (((2 * g) ^ x_swz) << 4));
        const float4_t b = *reinterpret_cast<const float4_t*>(xt + l16 * 128 + (((2 * g + 1) ^ x_swz) << 4));
        uint4 hi, lw;
        split_bf16x2(a[0], a[1], hi.x, lw.x);
        split_bf16x2(a[2], a[3], hi.y, lw.y);
        split_bf16x2(b[0], b[1], hi.z, lw.z);
        split_bf16x2(b[2], b[3], hi.w, lw.w);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[j]), __builtin_bit_cast(bf16x8_t, hi), acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[j]), __builtin_bit_cast(bf16x8_t, lw), acc[i][j], 0, 0, 0);
        }
      } else {
        const u32x4_t xf = *reinterpret_cast<const u32x4_t*>(xt + w_off);
#pragma unroll
        for (int j = 0; j < TN; ++j)
          if constexpr (C::TYPE == kRingF16)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, wf[j]), __builtin_bit_cast(f16x8_t, xf), acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[j]), __builtin_bit_cast(bf16x8_t, xf), acc[i][j], 0, 0, 0);
      }
    }
  };
#pragma unroll
  for (int s = 0; s < D - 1; ++s)
    if (s < n) issue(s);
  int s = 0;
  for (; s + D - 1 < n; ++s) {  // steps below s + D - 1 have been asked for
    wait_loads_but<LOADS * (D - 2)>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the step before has been read
    issue(s + D - 1);
    multiply(s);
  }
  each_down<D - 2>([&](auto left) {  // all have; so many behind this one
    constexpr int kLeft = decltype(left)::value;
    if (kLeft >= n) return;
    wait_loads_but<LOADS * kLeft>();
    multiply(s++);
  });
}
// Byte offset of the 16 bytes a lane brings in, of rows of K elements (they land at position `lane` of the KB; the swizzle spreads
// the reads over the banks): bf16, row lane / 4 of 16; fp32, row lane / 8 of the half u.
__device__ __forceinline__ uint32_t piece16(int lane, int row, int K) { return 2 * (uint32_t)row * (uint32_t)K + 16 * (uint32_t)((lane & 3) ^ swz_rows16<4>(lane >> 2)); }
__device__ __forceinline__ uint32_t piece32(int lane, int u, int row, int K) {
  return 4 * (uint32_t)row * (uint32_t)K + 16 * (uint32_t)((lane & 7) ^ swz_rows16<8>(8 * u + (lane >> 3)));
}

// The wavefronts' shares of a workgroup's tiles, summed: out(tile, outputs 2p and 2p + 1, p, row of the tile).
template <class C, class Out>
__device__ __forceinline__ void sum_tiles(const float4_t (&acc)[C::TM][C::TN], unsigned char* lds, int tid, int wv, int l16, int g, Out out) {
  constexpr int kRow = C::kRow;
  typedef float Tile[16 * kRow];
  Tile* s_red = reinterpret_cast<Tile*>(lds);  // [wavefront][CH]
  const int p = tid & 7, t = (tid >> 3) & 15;  // consecutive lanes: consecutive outputs of a row
#pragma unroll
  for (int rnd = 0; rnd < C::kTiles / C::CH; ++rnd) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C::CH; ++c) {
      const int at = rnd * C::CH + c;
#pragma unroll
      for (int v = 0; v < 4; ++v) s_red[wv * C::CH + c][(4 * g + v) * kRow + l16] = acc[at / C::TN][at % C::TN][v];
    }
    __syncthreads();
    for (int c = tid >> 7; c < C::CH; c += C::NT / 128) {
      float2 o = make_float2(0.f, 0.f);
#pragma unroll
      for (int w = 0; w < C::NW; ++w) {
        o.x += s_red[w * C::CH + c][2 * p * kRow + t];
        o.y += s_red[w * C::CH + c][2 * p * kRow + t + kRow];
      }
      out(rnd * C::CH + c, o, p, t);
    }
  }
}

// The K steps of wavefront wv: first one, how many.
template <int NW>
__device__ __forceinline__ int2 steps_of(int K, int wv) {
  const int all = K / 32, per = (all + NW - 1) / NW, lo = wv * per;
  return make_int2(lo, lo >= all ? 0 : (lo + per < all ? per : all - lo));
}

// Workgroup w runs on XCD w % 8: the row blocks of one block of outputs are numbered to follow one another on one XCD, so that its
// L2 reads the weights once.  (x: block of outputs, y: of rows; of nx x ny)
__device__ __forceinline__ int2 ring_job(unsigned w, unsigned ny) { return make_int2((int)((w >> 3) / ny * 8 + (w & 7)), (int)((w >> 3) % ny)); }
inline unsigned ring_grid(unsigned nx, unsigned ny) { return (nx + 7) / 8 * 8 * ny; }

}  // namespace

}  // namespace mtla
