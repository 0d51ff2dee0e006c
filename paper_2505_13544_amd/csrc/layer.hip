// The layer around the decode path, for one new token per sequence (bf16 storage, gfx950):
//   layer_front_kernel   x -> q = x W_Q (Eq. (query)), q^R = RoPE(x W_QR), c = x W_r (Eq. (low-rank); its
//                        layer normalisation is done by the step's append, where a whole row meets in
//                        one workgroup), k^R = RoPE(x W_KR) (Section "Decoupled Rotary Position
//                        Embedding in MTLA"); q, q^R and c leave in fp32 (they are rounded where they are
//                        used), k^R in bf16
//                        (Section "Decoupled Rotary Position Embedding in MTLA")
//   layer_out_kernel     y = concat_h(o_h) W_O (Eq. (softmax))
// Weights are output-major, [out_features, d_in], so that the contracted index is innermost for both
// operands of `D[n, token] = sum_k W[n, k] x[token, k]` (v_mfma_f32_16x16x32_bf16: W rows are the A
// operand, token rows the B operand); the products are those of gemm_ring.h.
#include "gemm_ring.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

// Where 16 outputs of the projections belong: tiles in the order q, q^R, k^R, c.
struct FrontTile {
  const uint16_t* W;  // rows of the product it is part of
  int n0, kind;       // first output in that product; 0 q, 1 q^R, 2 k^R, 3 c
};
__device__ __forceinline__ FrontTile front_tile(const LayerFrontArgs& a, int tile) {
  const int nq = a.n_heads * a.d_head, nqr = a.n_heads * a.d_rope;
  int n0 = 16 * tile;
  if (n0 < nq) return FrontTile{reinterpret_cast<const uint16_t*>(a.w_q), n0, 0};
  n0 -= nq;
  if (n0 < nqr) return FrontTile{reinterpret_cast<const uint16_t*>(a.w_qr), n0, 1};
  n0 -= nqr;
  if (n0 < a.d_rope) return FrontTile{reinterpret_cast<const uint16_t*>(a.w_kr), n0, 2};
  return FrontTile{reinterpret_cast<const uint16_t*>(a.w_r), n0 - a.d_rope, 3};
}

// Jobs (ring_job): ceil(tiles / TN) x ceil(batch / (16 TM)), tiles = (n_h d_h + n_h d_R + d_R + r) / 16.
template <class C>
__global__ __launch_bounds__(C::NT) void layer_front_kernel(LayerFrontArgs a) {
  constexpr int TM = C::TM, TN = C::TN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), l16 = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int2 job = ring_job(blockIdx.x, (unsigned)(a.batch + 16 * TM - 1) / (16 * TM));
  const int tok0 = 16 * TM * job.y, K = a.d_model;
  const int tiles = (a.n_heads * (a.d_head + a.d_rope) + a.d_rope + a.r) / 16, tile0 = TN * job.x;
  if (tile0 >= tiles) return;
  const unsigned char* wb[TN];
  uint32_t w_at[TN], x_at[TM][1];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const FrontTile f = front_tile(a, tile0 + j < tiles ? tile0 + j : tiles - 1);
    wb[j] = reinterpret_cast<const unsigned char*>(f.W + (size_t)f.n0 * K);
    w_at[j] = piece16(lane, lane >> 2, K);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {  // tokens past the batch: clamped, never stored
    const int t = 16 * i + (lane >> 2), last = a.batch - 1 - tok0;
    x_at[i][0] = piece16(lane, t < last ? t : last, K);
  }
  const unsigned char* xb = reinterpret_cast<const unsigned char*>(a.x) + 2 * (size_t)tok0 * K;
  const int2 st = steps_of<C::NW>(K, wv);
  float4_t acc[TM][TN];
  contract<C>(acc, wb, w_at, xb, x_at, 32 * st.x, st.y, lds + wv * (C::D * C::STAGE), l16, g);
  sum_tiles<C>(acc, lds, tid, wv, l16, g, [&](int at, float2 o, int p, int t) {
    const int tok = tok0 + 16 * (at / TN) + t, tile = tile0 + at % TN;
    if (tok >= a.batch || tile >= tiles) return;
    const FrontTile f = front_tile(a, tile);
    const int n = f.n0 + 2 * p;
    if (f.kind == 1 || f.kind == 2)  // rotated at the 0-based position of the token this step appends
      o = rope_turn(o, rope_angle(a.seq_len[tok], a.rope_freq[(n % a.d_rope) / 2]));
    if (f.kind == 2)  // the key goes into the cache: storage type
      *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(a.kr) + (size_t)tok * a.d_rope + n) = pack_bf16x2(o.x, o.y);
    else if (f.kind == 0)
      *reinterpret_cast<float2*>(a.q + (size_t)tok * (a.n_heads * a.d_head) + n) = o;
    else if (f.kind == 1)
      *reinterpret_cast<float2*>(a.q_rope + (size_t)tok * (a.n_heads * a.d_rope) + n) = o;
    else  // c = x W_r, before its normalisation (which the step's append does, where the whole row meets)
      *reinterpret_cast<float2*>(a.c + (size_t)tok * a.r + n) = o;
  });
}

// y[token, n] = sum_k o[token, k] W_O[n, k]; o is fp32 and enters as bf16 hi + lo planes, so that only the weights' own
// rounding is left.  Jobs: ceil(d_model / (16 TN)) x ceil(batch / (16 TM)).
template <class C>
__global__ __launch_bounds__(C::NT) void layer_out_kernel(LayerOutArgs a) {
  constexpr int TM = C::TM, TN = C::TN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), l16 = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int2 job = ring_job(blockIdx.x, (unsigned)(a.batch + 16 * TM - 1) / (16 * TM));
  const int tok0 = 16 * TM * job.y, n0 = 16 * TN * job.x, K = a.k;
  if (n0 >= a.d_model) return;
  const unsigned char* wb[TN];
  uint32_t w_at[TN], o_at[TM][2];
#pragma unroll
  for (int j = 0; j < TN; ++j) {  // (d_model is a multiple of 32)
    const int n = n0 + 16 * j < a.d_model ? n0 + 16 * j : a.d_model - 16;
    wb[j] = reinterpret_cast<const unsigned char*>(a.w_o) + 2 * (size_t)n * K;
    w_at[j] = piece16(lane, lane >> 2, K);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = 16 * i + 8 * u + (lane >> 3), last = a.batch - 1 - tok0;
      o_at[i][u] = piece32(lane, u, t < last ? t : last, K);
    }
  const unsigned char* ob = reinterpret_cast<const unsigned char*>(a.o) + 4 * (size_t)tok0 * K;
  const int2 st = steps_of<C::NW>(K, wv);
  float4_t acc[TM][TN];
  contract<C>(acc, wb, w_at, ob, o_at, 32 * st.x, st.y, lds + wv * (C::D * C::STAGE), l16, g);
  sum_tiles<C>(acc, lds, tid, wv, l16, g, [&](int at, float2 y, int p, int t) {
    const int tok = tok0 + 16 * (at / TN) + t, n = n0 + 16 * (at % TN) + 2 * p;
    if (tok < a.batch && n < a.d_model)  // d_model is even
      *reinterpret_cast<float2*>(a.y + (size_t)tok * a.d_model + n) = y;
  });
}

// The state a continuing prefill starts from, in front of an append of its own.
__global__ __launch_bounds__(kBlock) void save_state_kernel(SaveStateArgs a) {
  const size_t idx = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (idx < (size_t)a.batch) a.pos0[idx] = a.seq_len[idx];
  if (idx < (size_t)a.batch * a.r) a.tail_prev[idx] = a.tail_c[idx];
}

}  // namespace

hipError_t launch_save_state(const SaveStateArgs& a, hipStream_t st) {
  const size_t n = (size_t)a.batch * a.r;
  hipLaunchKernelGGL(save_state_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

bool layer_supported(const LayerFrontArgs& a) {
  return a.d_model % 32 == 0 && a.d_model >= 32 && a.d_model <= 16384 && a.d_head % 16 == 0 && a.d_rope % 16 == 0 &&
         a.d_rope <= 64 && a.r % 16 == 0 && a.batch <= 16 * 65535;
}

template <class C>
hipError_t layer_front_as(const LayerFrontArgs& a, hipStream_t st) {
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&layer_front_kernel<C>, C::BYTES, lds_allowed);
  if (e != hipSuccess) return e;
  const int tiles = (a.n_heads * (a.d_head + a.d_rope) + a.d_rope + a.r) / 16;
  hipLaunchKernelGGL(layer_front_kernel<C>, dim3(ring_grid((tiles + C::TN - 1) / C::TN, (a.batch + 16 * C::TM - 1) / (16 * C::TM))), dim3(C::NT), C::BYTES, st, a);
  return hipGetLastError();
}

template <class C>
hipError_t layer_out_as(const LayerOutArgs& a, hipStream_t st) {
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&layer_out_kernel<C>, C::BYTES, lds_allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(layer_out_kernel<C>, dim3(ring_grid((a.d_model / 16 + C::TN - 1) / C::TN, (a.batch + 16 * C::TM - 1) / (16 * C::TM))), dim3(C::NT), C::BYTES, st, a);
  return hipGetLastError();
}

// A workgroup's tokens and outputs: a 16 x 16 tile each as long as that leaves no more of them than the chip holds at once; beyond, a larger
// tile fetches less (a unit is at the rate of its loads) and has fewer sums to meet.  us a launch, weights in turn out of three sets:
//   projections  B = 16, d_model 2048 (228 tiles)   1 x 1 tiles 4.9, 2 x 2 6.2      output  B = 32, 2048 (256)   1 x 1 4.4, 1 x 2 5.2
//                B = 32, 2048 (456)     1 x 1 6.7, 2 x 1 5.7, 2 x 2 7.0                     B = 256, 512 (512)   1 x 1 3.3, 1 x 2 3.0
//                B = 100, 1024 (798)    1 x 1 5.2, 2 x 2 4.6, 4 x 4 10                      B = 64, 4096 (1024)  1 x 2 16, 2 x 2 13, 2 x 4 16
//                B = 64, 4096 (1680)    2 x 2 20, 4 x 4 24                                  B = 256, 2048 (2048) 2 x 2 12.2, 2 x 4 10.1, 4 x 4 15.5
//                B = 256, 2048 (3648)   2 x 2 17.7, 4 x 4 15.7                              B = 189, 4096 (3072) 2 x 4 32, 4 x 4 26.9
// (Operands straight into the registers, 1 x 1 tiles: 6.2, 9.8, 9.3, 51.6, 54.5; 8.0, 5.1, 43.9, 44.2, 125.6.)
hipError_t launch_layer_front(const LayerFrontArgs& a, hipStream_t st) {
  const int token_tiles = (a.batch + 15) / 16;
  const long long tiles = (long long)(a.n_heads * (a.d_head + a.d_rope) + a.d_rope + a.r) / 16 * token_tiles;
  if (token_tiles == 1 || tiles <= 400) return layer_front_as<RingTile<1, 1, 4, 4, kRingBf16>>(a, st);
  if (tiles <= 600) return layer_front_as<RingTile<2, 1, 4, 4, kRingBf16>>(a, st);
  if (tiles <= 2000) return layer_front_as<RingTile<2, 2, 4, 4, kRingBf16>>(a, st);
  return layer_front_as<RingTile<4, 4, 4, 3, kRingBf16>>(a, st);
}

hipError_t launch_layer_out(const LayerOutArgs& a, hipStream_t st) {
  const int token_tiles = (a.batch + 15) / 16;
  const long long tiles = (long long)((a.d_model + 15) / 16) * token_tiles;
  if (tiles <= 300) return layer_out_as<RingTile<1, 1, 8, 3, kRingF32>>(a, st);
  if (token_tiles == 1 || tiles <= 600) return layer_out_as<RingTile<1, 2, 8, 3, kRingF32>>(a, st);
  if (tiles <= 1200) return layer_out_as<RingTile<2, 2, 8, 3, kRingF32>>(a, st);
  if (tiles <= 2600) return layer_out_as<RingTile<2, 4, 4, 3, kRingF32>>(a, st);
  return layer_out_as<RingTile<4, 4, 4, 3, kRingF32>>(a, st);
}

}  // namespace mtla
