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
// operand, token rows the B operand).  At decode batch sizes these are weight-streaming kernels: a
// workgroup owns 16 outputs for 16 tokens, its four wavefronts a quarter of the contraction each, operands straight
// from memory into the operand layout (the token rows come out of L2 for every workgroup after the first); the four
// sums meet in LDS.  With one wavefront per tile walking the whole contraction, front and output took 4.0 and 4.3 us
// at d_model = 512, batch 11, of which it spent half waiting for its own requests: now 3.7 and 3.6.
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

// A wavefront's share of one 16 x 16 tile: its quarter of the K steps (K % 32 == 0), D[n0 + 4g + v, tok0 + l16] for v = 0..3.
// Rows past the ends are clamped (their results are never stored).  The operands of kBatch K steps are requested together,
// so that a contraction of 1024 costs one round trip to memory.
constexpr int kBatch = 8;
struct Steps {
  int lo, hi;  // in elements
};
__device__ __forceinline__ Steps steps_of(int K, int wv) {
  const int per = 32 * ((K / 32 + 3) / 4), lo = wv * per;
  return Steps{lo, lo + per < K ? lo + per : K};
}
__device__ __forceinline__ float4_t linear_tile(const uint16_t* W, int n_out, const uint16_t* x, int n_tok, int K,
                                                int n0, int tok0, int l16, int g, const Steps& st) {
  const int n = n0 + l16 < n_out ? n0 + l16 : n_out - 1, t = tok0 + l16 < n_tok ? tok0 + l16 : n_tok - 1;
  const uint16_t* wp = W + (size_t)n * K + 8 * g;
  const uint16_t* xp = x + (size_t)t * K + 8 * g;
  float4_t acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = st.lo; k0 < st.hi; k0 += 32 * kBatch) {
    uint4 wf[kBatch], xf[kBatch];
#pragma unroll
    for (int half = 0; half < 2; ++half)
      if (k0 + 16 * kBatch * half < st.hi)
#pragma unroll
        for (int i = kBatch / 2 * half; i < kBatch / 2 * (half + 1); ++i) {
          const int k = k0 + 32 * i < st.hi ? k0 + 32 * i : k0;  // past the end: a harmless reload
          wf[i] = *reinterpret_cast<const uint4*>(wp + k);
          xf[i] = *reinterpret_cast<const uint4*>(xp + k);
        }
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
      if (k0 + 32 * i < st.hi)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[i]), __builtin_bit_cast(bf16x8_t, xf[i]),
                                                      acc, 0, 0, 0);
  }
  return acc;
}

// The four wavefronts' shares of a tile, summed; threads below 128 get outputs 2p, 2p + 1 (p = tid / 16) of token tid % 16.
constexpr int kRow = 17;  // floats per output row: a column of four rows apart lies in other banks
__device__ __forceinline__ float2 tile_sum(const float4_t& d, float (*s_red)[16 * kRow], int tid, int wv, int l16, int g) {
#pragma unroll
  for (int v = 0; v < 4; ++v) s_red[wv][(4 * g + v) * kRow + l16] = d[v];
  __syncthreads();
  float2 o = make_float2(0.f, 0.f);
  if (tid < 128) {
    const int at = 2 * (tid >> 4) * kRow + (tid & 15);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      o.x += s_red[w][at];
      o.y += s_red[w][at + kRow];
    }
  }
  return o;
}

// grid = (tiles, ceil(batch / 16)), tiles = (n_h d_h + n_h d_R + d_R + r) / 16 in the order q, q^R, k^R, c.
__global__ __launch_bounds__(kBlock) void layer_front_kernel(LayerFrontArgs a) {
  __shared__ float s_red[4][16 * kRow];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), l16 = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tok0 = 16 * blockIdx.y, K = a.d_model;
  const int tok = tok0 + (tid & 15), n2 = 2 * (tid >> 4);  // what the thread stores: outputs n2, n2 + 1 of the tile
  const bool mine = tid < 128 && tok < a.batch;
  const uint16_t* x = reinterpret_cast<const uint16_t*>(a.x);
  const Steps st = steps_of(K, wv);
  const int nq = a.n_heads * a.d_head, nqr = a.n_heads * a.d_rope;
  int n0 = 16 * blockIdx.x;
  if (n0 < nq) {  // ---- q
    const float2 o = tile_sum(linear_tile(reinterpret_cast<const uint16_t*>(a.w_q), nq, x, a.batch, K, n0, tok0, l16, g, st),
                              s_red, tid, wv, l16, g);
    if (mine) *reinterpret_cast<float2*>(a.q + (size_t)tok * nq + n0 + n2) = o;
    return;
  }
  n0 -= nq;
  if (n0 < nqr + a.d_rope) {  // ---- q^R (per head) and k^R (one shared head): rotated at the token's position
    const bool is_key = n0 >= nqr;
    if (is_key) n0 -= nqr;
    const int n_out = is_key ? a.d_rope : nqr;
    const int pos = mine ? a.seq_len[tok] : 0;  // 0-based position of the token this step appends
    const float2 cs = rope_angle(pos, a.rope_freq[((n0 + n2) % a.d_rope) / 2]);
    float2 o = tile_sum(linear_tile(reinterpret_cast<const uint16_t*>(is_key ? a.w_kr : a.w_qr), n_out, x, a.batch, K, n0, tok0,
                                    l16, g, st), s_red, tid, wv, l16, g);
    if (mine) {
      o = rope_turn(o, cs);
      if (is_key)  // the key goes into the cache: storage type
        *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(a.kr) + (size_t)tok * n_out + n0 + n2) = pack_bf16x2(o.x, o.y);
      else
        *reinterpret_cast<float2*>(a.q_rope + (size_t)tok * n_out + n0 + n2) = o;
    }
    return;
  }
  // ---- c = x W_r, before its normalisation (which the step's append does, where the whole row meets)
  n0 -= nqr + a.d_rope;
  const float2 o = tile_sum(linear_tile(reinterpret_cast<const uint16_t*>(a.w_r), a.r, x, a.batch, K, n0, tok0, l16, g, st), s_red,
                            tid, wv, l16, g);
  if (mine) *reinterpret_cast<float2*>(a.c + (size_t)tok * a.r + n0 + n2) = o;
}

// y[token, n] = sum_k o[token, k] W_O[n, k]; o is fp32 and enters as bf16 hi + lo planes (two matrix
// instructions per step), so that only the weights' own rounding is left.  grid = (ceil(d_model / 16), ceil(batch / 16)).
__global__ __launch_bounds__(kBlock) void layer_out_kernel(LayerOutArgs a) {
  __shared__ float s_red[4][16 * kRow];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), l16 = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tok0 = 16 * blockIdx.y, n0 = 16 * blockIdx.x, K = a.k;
  const int n = n0 + l16 < a.d_model ? n0 + l16 : a.d_model - 1;
  const int t = tok0 + l16 < a.batch ? tok0 + l16 : a.batch - 1;
  const uint16_t* wp = reinterpret_cast<const uint16_t*>(a.w_o) + (size_t)n * K + 8 * g;
  const float* op = a.o + (size_t)t * K + 8 * g;
  const Steps st = steps_of(K, wv);
  float4_t acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = st.lo; k0 < st.hi; k0 += 32 * kBatch) {  // three 16-byte loads per step
    uint4 wf[kBatch];
    float4_t o0[kBatch], o1[kBatch];
#pragma unroll
    for (int half = 0; half < 2; ++half)
      if (k0 + 16 * kBatch * half < st.hi)
#pragma unroll
        for (int i = kBatch / 2 * half; i < kBatch / 2 * (half + 1); ++i) {
          const int k = k0 + 32 * i < st.hi ? k0 + 32 * i : k0;
          wf[i] = *reinterpret_cast<const uint4*>(wp + k);
          o0[i] = *reinterpret_cast<const float4_t*>(op + k);
          o1[i] = *reinterpret_cast<const float4_t*>(op + k + 4);
        }
#pragma unroll
    for (int i = 0; i < kBatch; ++i)
      if (k0 + 32 * i < st.hi) {
        uint4 hi, lo;
        split_bf16x2(o0[i][0], o0[i][1], hi.x, lo.x);
        split_bf16x2(o0[i][2], o0[i][3], hi.y, lo.y);
        split_bf16x2(o1[i][0], o1[i][1], hi.z, lo.z);
        split_bf16x2(o1[i][2], o1[i][3], hi.w, lo.w);
        const bf16x8_t w8 = __builtin_bit_cast(bf16x8_t, wf[i]);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w8, __builtin_bit_cast(bf16x8_t, hi), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w8, __builtin_bit_cast(bf16x8_t, lo), acc, 0, 0, 0);
      }
  }
  const float2 y = tile_sum(acc, s_red, tid, wv, l16, g);
  const int tok = tok0 + (tid & 15), n2 = n0 + 2 * (tid >> 4);
  if (tid < 128 && tok < a.batch && n2 < a.d_model)  // d_model is even
    *reinterpret_cast<float2*>(a.y + (size_t)tok * a.d_model + n2) = y;
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

hipError_t launch_layer_front(const LayerFrontArgs& a, hipStream_t st) {
  const int tiles = (a.n_heads * (a.d_head + a.d_rope) + a.d_rope + a.r) / 16;
  hipLaunchKernelGGL(layer_front_kernel, dim3(tiles, (a.batch + 15) / 16), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_layer_out(const LayerOutArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(layer_out_kernel, dim3((a.d_model + 15) / 16, (a.batch + 15) / 16), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

}  // namespace mtla
