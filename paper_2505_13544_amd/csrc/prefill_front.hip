// What comes before the matrix products of a prefill (bf16 storage but for the append alone), in one launch: the append of the new tokens
// (merge weights and cache), the rows the key / value product reads (slot states of the past and partial states
// C_hat'[m] of the new rows, as fp16), the RoPE keys as fp16, and the weights as fp16.
//
//   append_bulk_kernel      mtla_cache_append of many tokens (the append alone); append_bulk_f32_kernel the same in fp32 storage
//   prefill_front_kernel    the above; MODE 0: the merge weights are given and nothing is appended (part of
//                           mtla_prefill_attn and mtla_prefill_chunk_attn), 1: with the append, 2: with the append,
//                           from unrounded latents that are layer-normalised first (whole-layer prefill)
//
// A new row's partial state is what the append of its slot holds after the row (the update rule after
// Eq. (infer-linear)), so one pass over the latents yields both.  Appending, converting and staging in seven launches took
// 46 us of the 227 us of six pieces of up to 510 rows (r = 512, 16 heads x 128) behind up to 3001 tokens, most of
// it launches that wait for one another; as one launch 13.
#include <type_traits>

#include "bounds.h"
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
__device__ __forceinline__ uint16_t bf16_bits_to_f16_bits(uint16_t v) {
  return __builtin_bit_cast(uint16_t, static_cast<_Float16>(__uint_as_float(uint32_t(v) << 16)));
}
constexpr int kMaxHyper = 64;  // rows of the hyper-network
constexpr int kChunk = 32;  // tokens whose latents are in LDS at a time
constexpr int kChunkSlots = 16, kTurns = 2;  // threads side by side merge 16 slots at a time; a chunk touches at most 32 (17 from a stride of 2)

// One row of latents in LDS: bf16 as they come, or fp32 after their normalisation (LN).  The pitch is an odd multiple of
// 16 bytes, so that 16-byte reads of 16 rows spread over all banks.
template <int R, bool LN>
struct AppendShared {
  static constexpr int kPitch = R * (LN ? 4 : 2) + 16;
  unsigned char row[kChunk][kPitch];
  float z[kChunk][4];  // hyper-network logits of the chunk's tokens, a share per wavefront
  float w[4][kChunk];  // merge weights, a copy per wavefront
  float bias[2][kMaxHyper];               // of the hyper-network; zeros, for all wavefronts but one
  uint16_t g[kChunk][kMaxHyper + 8];      // the tokens' rows of hyp_G
  u32x4_t kr[kTurns][kChunkSlots][16];    // the slots' new RoPE keys, 16 bytes a thread
  __device__ __forceinline__ void values(int u, int e, float (&o)[8]) const {
    if constexpr (LN) {
      const float4_t lo = *reinterpret_cast<const float4_t*>(row[u] + 4 * e), hi = *reinterpret_cast<const float4_t*>(row[u] + 4 * e + 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        o[i] = lo[i];
        o[4 + i] = hi[i];
      }
    } else {
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(row[u] + 2 * e);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t w = v[i];
        o[2 * i] = __uint_as_float(w << 16);
        o[2 * i + 1] = __uint_as_float(w & 0xffff0000u);
      }
    }
  }
};

// A wavefront's part of hyp_A, as matrix operands: k = k0 + 32 i .. + 31 of rows y0 + 16 t .. + 15; zeros where there are none.
template <int R, bool LN>
struct HyperRows {
  // A quarter of k for all rows saves the wavefronts three quarters of the reads (and, unrounded, of the splitting) of a chunk's
  // latents and costs them four sums instead of one.  Narrow rounded latents are cheaper read by all, 16 rows a wavefront: append of 16
  // x 2080 tokens, s = 2, by quarters / by rows: r = 64 8.7 / 7.9 us, 128 9.2 / 8.4, 256 11.4 / 11.0, 512 19.3 / 19.4; the layer over them, r = 256: 160.7 / 162.2.
  static constexpr bool kByRow = R == 64 || (!LN && R <= 256);
  static constexpr int KW = kByRow ? R / 32 : R / 128, YT = kByRow ? 1 : kMaxHyper / 16;
  static __device__ __forceinline__ int y0(int wv) { return kByRow ? 16 * wv : 0; }
  static __device__ __forceinline__ int k0(int wv) { return kByRow ? 0 : 32 * KW * wv; }
  u32x4_t f[YT][KW];
  uint32_t bias = 0;  // bf16, element threadIdx.x
  __device__ __forceinline__ void load(const AppendArgs& a) {
    if (a.w_override) return;
    const int tid = threadIdx.x, l16 = tid & 15, g = (tid & (kWave - 1)) >> 4, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (a.hyp_a && tid < a.d_hyper) bias = reinterpret_cast<const uint16_t*>(a.hyp_a)[tid];
    const uint16_t* A = reinterpret_cast<const uint16_t*>(a.hyp_A) + (size_t)(y0(wv) + l16) * R + k0(wv) + 8 * g;
#pragma unroll
    for (int t = 0; t < YT; ++t)
#pragma unroll
      for (int i = 0; i < KW; ++i) {
        f[t][i] = u32x4_t{0u, 0u, 0u, 0u};
        if (y0(wv) + 16 * t < a.d_hyper) f[t][i] = *reinterpret_cast<const u32x4_t*>(A + (size_t)16 * t * R + 32 * i);
      }
  }
};

// Positions [pos_lo, pos_hi) of sequence b, which begin with a slot or with the call; called by every thread of the
// workgroup (barriers inside).  The latents go through LDS once, 32 tokens at a time, and serve two things:
//   weights  Linear(c) of 16 tokens at a time is a small dense contraction D[y, token] = sum_n hyp_A[y, n] c[token, n];
//            a wavefront takes a quarter of n for all rows y, or 16 rows and all n (their weights stay in its registers for all
//            tokens), dots its share with the slot's row of hyp_G, and the four shares meet in LDS
//   merge    16 threads per slot fold w_n c_n over the slot's tokens in order, in fp32, from the tail shadow when
//            the slot already held tokens; every partial sum is a row of C_hat' (STAGE), the last one the cache row,
//            rounded once
// `tail_out` takes the last slot's fp32 value.
// A workgroup is one round trip to memory and then works out of LDS, while the next chunk's latents travel (LN: its registers are
// full of the fp32 ones); with the rows read straight into the operand layout by each wavefront, and again for the merge,
// 8 x 4096 tokens at r = 512 took 42 us (50 MB); with a workgroup per 16 slots and rows of hyp_A a wavefront, which has every wavefront
// read (and, unrounded, split) all latents of the chunk, 25.5 us, now 21.6; five prompts of up to 1531 tokens, s = 3, one chunk a
// workgroup, 12.9 and 8.9; the whole layer's front launch over 8 x 4096 tokens 51.5 and 44.  What is left is latency: the
// lengths 2.4 us, the weights and latents 2 to 5, then logits, weights and merge 1.3 + 0.5 + 1.3 a chunk.
template <int R, bool LN, bool STAGE>
__device__ __forceinline__ void append_range(const AppendArgs& a, const PrefillFrontArgs* fa, int b, int p0, int n, long long pos_lo,
                                             long long pos_hi, float* tail_out, const HyperRows<R, LN>& hr, AppendShared<R, LN>& sh) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4, q = tid & 15, j = tid >> 4;
  const int s = a.stride, dR = a.d_rope, dy = a.d_hyper;
  const int t0 = int(pos_lo - p0), cnt = int(pos_hi - pos_lo);  // tokens t0 .. t0 + cnt - 1 of the call
  const size_t tok0 = (size_t)b * a.n_new_max + t0;
  constexpr int NP = R >= 128 ? R / 128 : 1;                   // a thread merges pieces q, q + 16, .. of 8 elements
  using Hyper = HyperRows<R, LN>;
  constexpr int KW = Hyper::KW, YT = Hyper::YT;
  const int y0 = Hyper::y0(wv), k0 = Hyper::k0(wv);
  const bool hyper = !a.w_override;
  int past = 0;  // rows of cprime in front of the new ones
  if constexpr (STAGE) past = slots_inside(p0, s, fa->cs.past_pitch);

  const int slot0 = int(pos_lo / s);
  float acc[NP][8];  // of slots slot0 + j, + 16, ..
#pragma unroll
  for (int i = 0; i < NP; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[i][e] = 0.f;
  if (j == 0 && 8 * q < R && (long long)slot0 * s < p0) {  // the slot already holds earlier tokens
#pragma unroll
    for (int i = 0; i < NP; ++i) load8(a.tail_c + (size_t)b * R + 8 * (q + 16 * i), acc[i]);
  }

  // What a chunk takes from memory, on its way to LDS while the one before is folded: latents, 16 threads per token and two tokens per
  // thread; rows of hyp_G, 8 threads per token; the thread's slots' new keys (a slot keeps the key of the newest token folded into it).
  // Nothing else is loaded in the loop: waiting for it would be waiting for these.
  u32x4_t cv[LN ? 1 : 2][LN ? 1 : NP], krv[kTurns];
  uint2 gv[2] = {make_uint2(0u, 0u), make_uint2(0u, 0u)};
  float given = 0.f;  // merge weight of token lane % 32
  auto request = [&](int c0) {
    const int nc = cnt - c0 < kChunk ? cnt - c0 : kChunk;
    if constexpr (!LN) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int u = 16 * h + j < nc ? 16 * h + j : nc - 1;
        const uint16_t* row = reinterpret_cast<const uint16_t*>(a.c_new) + (tok0 + c0 + u) * R;
#pragma unroll
        for (int i = 0; i < NP; ++i) cv[h][i] = *reinterpret_cast<const u32x4_t*>(row + (8 * q < R ? 8 * (q + 16 * i) : 0));
      }
    }
    const int u_w = lane & (kChunk - 1);
    if (a.w_override) given = a.w_override[tok0 + c0 + (u_w < nc ? u_w : nc - 1)];
    const long long first = pos_lo + c0, end = first + nc;
    if (hyper && 8 * (tid & 7) < dy) {
      const int u = tid >> 3 < nc ? tid >> 3 : nc - 1;
      const uint16_t* G = reinterpret_cast<const uint16_t*>(a.hyp_G) + (size_t)((first + u) / s) * dy + 8 * (tid & 7);
      gv[0] = *reinterpret_cast<const uint2*>(G);
      gv[1] = *reinterpret_cast<const uint2*>(G + 4);
    }
    const int slot_c = int(first / s), slot_t = slot_c + ((j - (slot_c - slot0)) & (kChunkSlots - 1));
#pragma unroll
    for (int t = 0; t < kTurns; ++t) {
      const long long sf = (long long)(slot_t + kChunkSlots * t) * s, hi = sf + s < pos_hi ? sf + s : pos_hi;
      if (q < dR / 8 && sf < end && hi <= end)
        krv[t] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.kr_new) +
                                                   ((size_t)b * a.n_new_max + (size_t)(hi - 1 - p0)) * dR + 8 * q);
    }
  };
  request(0);
  if (tid < 2 * kMaxHyper) sh.bias[tid / kMaxHyper][tid % kMaxHyper] = __uint_as_float(hr.bias << 16);  // (0 from 64 on: dy <= 64)
  for (int c0 = 0; c0 < cnt; c0 += kChunk) {
    const int nc = cnt - c0 < kChunk ? cnt - c0 : kChunk;
    if (c0) __syncthreads();
    if constexpr (LN) {
      constexpr int N4 = R / 64;
      float4_t v[2][N4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int u = 16 * h + j < nc ? 16 * h + j : nc - 1;
        const float* row = reinterpret_cast<const float*>(a.c_new) + (tok0 + c0 + u) * R;
#pragma unroll
        for (int i = 0; i < N4; ++i) v[h][i] = *reinterpret_cast<const float4_t*>(row + 4 * (q + 16 * i));
      }
      const bf16* gamma = reinterpret_cast<const bf16*>(a.ln_gamma);
      const bf16* beta = reinterpret_cast<const bf16*>(a.ln_beta);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < N4; ++i) sum += (v[h][i][0] + v[h][i][1]) + (v[h][i][2] + v[h][i][3]);
        sum = group_reduce<16>(sum, LaneSum());
        const float mean = sum / (float)R;
        float sq = 0.f;
#pragma unroll
        for (int i = 0; i < N4; ++i) {
          v[h][i] -= mean;
          sq += (v[h][i][0] * v[h][i][0] + v[h][i][1] * v[h][i][1]) + (v[h][i][2] * v[h][i][2] + v[h][i][3] * v[h][i][3]);
        }
        sq = group_reduce<16>(sq, LaneSum());
        const float rstd = rsqrtf(sq / (float)R + a.ln_eps);
#pragma unroll
        for (int i = 0; i < N4; ++i) {
          const int e = 4 * (q + 16 * i);
          float4_t o = v[h][i] * rstd;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (gamma) o[k] *= to_f32(gamma[e + k]);
            if (beta) o[k] += to_f32(beta[e + k]);
          }
          *reinterpret_cast<float4_t*>(sh.row[16 * h + j] + 4 * e) = o;
        }
      }
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < NP; ++i)
          if (8 * q < R) *reinterpret_cast<u32x4_t*>(sh.row[16 * h + j] + 16 * (q + 16 * i)) = cv[h][i];
    }
    *reinterpret_cast<uint2*>(&sh.g[tid >> 3][8 * (tid & 7)]) = gv[0];
    *reinterpret_cast<uint2*>(&sh.g[tid >> 3][8 * (tid & 7) + 4]) = gv[1];
#pragma unroll
    for (int t = 0; t < kTurns; ++t) sh.kr[t][j][q] = krv[t];
    float wt = given;
    if (c0 + kChunk < cnt) request(c0 + kChunk);
    __syncthreads();

    // ---- logits of the merge weights
    if (hyper) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // (a branch between the halves costs a long append 1 % and saves a call of up to 16 tokens a sequence 0.1 to 0.4 us of 8: r = 512,
        // 3 sequences of 16 tokens 9.45, now 9.05)
        if constexpr (!STAGE) {
          if (16 * h >= nc) break;
        }
        float4_t d[YT];
#pragma unroll
        for (int t = 0; t < YT; ++t) d[t] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KW; ++i) {
          const int e = k0 + 32 * i + 8 * g;
          u32x4_t hi, lo;
          if constexpr (LN) {  // unrounded latents: hi + lo bf16 planes, two matrix instructions per step
            float v[8];
            sh.values(16 * h + l16, e, v);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              uint32_t a0, a1;
              split_bf16x2(v[2 * k], v[2 * k + 1], a0, a1);
              hi[k] = a0;
              lo[k] = a1;
            }
          } else {
            hi = *reinterpret_cast<const u32x4_t*>(sh.row[16 * h + l16] + 2 * e);
          }
#pragma unroll
          for (int t = 0; t < YT; ++t)
            d[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, hr.f[t][i]), __builtin_bit_cast(bf16x8_t, hi), d[t], 0, 0, 0);
          if constexpr (LN) {
#pragma unroll
            for (int t = 0; t < YT; ++t)
              d[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, hr.f[t][i]), __builtin_bit_cast(bf16x8_t, lo), d[t], 0, 0, 0);
          }
        }
        // the lane holds its share of Linear(c)[y0 + 16 t + 4 g + v] of its token
        float z = 0.f;
#pragma unroll
        for (int t = 0; t < YT; ++t) {
          d[t] += *reinterpret_cast<const float4_t*>(sh.bias[Hyper::kByRow || wv == 0 ? 0 : 1] + y0 + 16 * t + 4 * g);
          const uint2 w = *reinterpret_cast<const uint2*>(&sh.g[16 * h + l16][y0 + 16 * t + 4 * g]);
          const float part = (d[t][0] * __uint_as_float(w.x << 16) + d[t][1] * __uint_as_float(w.x & 0xffff0000u)) +
                             (d[t][2] * __uint_as_float(w.y << 16) + d[t][3] * __uint_as_float(w.y & 0xffff0000u));
          z += y0 + 16 * t < dy ? part : 0.f;  // (rows that there are not: of an infinite latent their products are not numbers)
        }
        z = quarter_reduce(z, LaneSum());
        if (g == 0) sh.z[16 * h + l16][wv] = z;
      }
    }
    __syncthreads();
    const int u_w = lane & (kChunk - 1);
    if (hyper) {
      const float4_t z = *reinterpret_cast<const float4_t*>(sh.z[u_w]);
      wt = 1.f / (1.f + expf(-((z[0] + z[1]) + (z[2] + z[3]))));
    }
    sh.w[wv][u_w] = wt;
    __builtin_amdgcn_wave_barrier();  // (the wavefront's own copy)
    if (tid < nc && (a.w_out || a.slot_out)) {
      if (a.w_out) a.w_out[tok0 + c0 + tid] = wt;
      if (a.slot_out) a.slot_out[tok0 + c0 + tid] = int((pos_lo + c0 + tid) / s);
    }

    // ---- temporal merge of the slots' tokens in this chunk
    const long long first = pos_lo + c0, end = first + nc;
    const int slot_c = int(first / s), slot_t = slot_c + ((j - (slot_c - slot0)) & (kChunkSlots - 1));
#pragma unroll
    for (int t = 0; t < kTurns; ++t) {
      const int slot = slot_t + kChunkSlots * t;
      const long long sf = (long long)slot * s, hi = sf + s < pos_hi ? sf + s : pos_hi;
      if (sf >= end) break;
      if (sf >= first && (t || c0)) {  // begins here (the first chunk's: above)
#pragma unroll
        for (int i = 0; i < NP; ++i)
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[i][e] = 0.f;
      }
      const int u_lo = sf > first ? int(sf - first) : 0, u_hi = hi < end ? int(hi - first) : nc;
      for (int u = u_lo; 8 * q < R && u < u_hi; ++u) {
        const float w = sh.w[wv][u];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          float v[8];
          sh.values(u, 8 * (q + 16 * i), v);
          u32x4_t o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            acc[i][2 * e] += w * v[2 * e];
            acc[i][2 * e + 1] += w * v[2 * e + 1];
            o[e] = pack_f16x2(acc[i][2 * e], acc[i][2 * e + 1]);
          }
          if constexpr (STAGE) {
            const ChunkStageArgs& cs = fa->cs;
            *reinterpret_cast<u32x4_t*>(reinterpret_cast<uint16_t*>(cs.cprime) +
                                        ((size_t)b * (cs.past_pitch + cs.T) + past + (size_t)(t0 + c0 + u)) * R + 8 * (q + 16 * i)) = o;
          }
        }
      }
      if (hi > end) break;  // goes on in the next chunk
      const size_t crow = cache_row(a.pages, b, slot, a.max_slots);
      if (8 * q < R) {
        uint16_t* out = reinterpret_cast<uint16_t*>(a.cache_c) + crow * R;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          const int e = 8 * (q + 16 * i);
          *reinterpret_cast<u32x4_t*>(out + e) = u32x4_t{pack_bf16x2(acc[i][0], acc[i][1]), pack_bf16x2(acc[i][2], acc[i][3]),
                                                         pack_bf16x2(acc[i][4], acc[i][5]), pack_bf16x2(acc[i][6], acc[i][7])};
          if (hi == (long long)p0 + n) {  // last slot touched: remains the sequence's tail
            float* to = tail_out + (size_t)b * R + e;
            *reinterpret_cast<float4_t*>(to) = float4_t{acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
            *reinterpret_cast<float4_t*>(to + 4) = float4_t{acc[i][4], acc[i][5], acc[i][6], acc[i][7]};
          }
        }
      }
      if (q < dR / 8) *reinterpret_cast<u32x4_t*>(reinterpret_cast<uint16_t*>(a.cache_kr) + crow * dR + 8 * q) = sh.kr[t][j][q];
    }
  }
}

// Which positions workgroup x of sequence b appends: those of slots `slots` x .. of the ones the call touches, through
// range(p0, n, first slot, first position, behind the last one).  The tail shadow of a sequence is read by the first
// slot (when that slot already held tokens) and written by the last one.  With a staging launch (pos0_out: takes the length
// before the call) the new one goes to tail_next and is put in place by the attention launch.  An append alone has no later
// launch: when the shadow is read, workgroup 0 takes the last slot as well, in a second pass behind a barrier, so the read
// precedes the write.
// `first` requests what does not depend on the lengths; it travels with them.
template <class First, class Range>
__device__ __forceinline__ void append_share(const AppendArgs& a, int slots, int32_t* pos0_out, int x, int b, First first, Range range) {
  const int s = a.stride, p0 = load_uniform_i32(a.seq_len, b);
  int n = a.n_new ? load_uniform_i32(a.n_new, b) : a.n_new_max;
  first();
  n = n < 0 ? 0 : (n > a.n_new_max ? a.n_new_max : n);
  if (pos0_out && x == 0 && threadIdx.x == 0) pos0_out[b] = p0;  // for the launches behind this one
  if (n == 0) return;
  if (const int refused = append_status(p0, n, s, a.max_slots)) {
    if (x == 0 && threadIdx.x == 0) *a.status = refused;
    return;
  }
  const long long end = (long long)p0 + n;
  const int first_slot = p0 / s, last_slot = int((end - 1) / s);
  const bool last_apart = !pos0_out && p0 % s != 0 && last_slot - first_slot >= slots;  // last slot outside workgroup 0's group
  const long long slot0 = first_slot + (long long)slots * x;
  const long long lim = last_apart ? (long long)last_slot * s : end;  // the group's share ends here
  const long long pos_lo = slot0 * s > p0 ? slot0 * s : p0;
  const long long pos_hi = (slot0 + slots) * s < lim ? (slot0 + slots) * s : lim;
  if (pos_lo < pos_hi) range(p0, n, pos_lo, pos_hi);
  if (x == 0 && last_apart) {
    __syncthreads();
    range(p0, n, (long long)last_slot * s, end);
  }
}

template <int R, bool LN, bool STAGE>
__device__ __forceinline__ void append_block(const AppendArgs& a, const PrefillFrontArgs* fa, int slots, int x, int b,
                                             AppendShared<R, LN>& sh) {
  float* tail_out = STAGE ? fa->tail_next : a.tail_c;
  HyperRows<R, LN> hr;
  append_share(a, slots, STAGE ? fa->pos0_out : nullptr, x, b, [&]() { hr.load(a); }, [&](int p0, int n, long long pos_lo, long long pos_hi) {
    append_range<R, LN, STAGE>(a, fa, b, p0, n, pos_lo, pos_hi, tail_out, hr, sh);
  });
}

template <int R>
__global__ __launch_bounds__(kBlock, 2) void append_bulk_kernel(AppendArgs a, int slots) {
  __shared__ __attribute__((aligned(16))) AppendShared<R, false> sh;
  append_block<R, false, false>(a, nullptr, slots, blockIdx.y, blockIdx.x, sh);
}

// The same append in fp32 storage, on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: lane 16 k + i holds A[i, k] and
// B[k, i]; a lane's 16 bytes are its elements for four instructions).  32 threads merge a slot, eight at most per workgroup;
// 16 tokens at a time through LDS.  Bound by latency: the hyper-network's rows and the first tokens are one trip to memory,
// then 16 tokens are r / 4 dependent matrix instructions a wavefront (2048 cycles at r = 256).  With a workgroup per slot that
// read the hyper-network (64 KB) again for every token, three sequences of up to 777 tokens took 14.8 us, r = 256, s = 2.
constexpr int kSlotsF32 = 8, kChunkF32 = 16;  // the most slots of a workgroup, tokens at a time
template <int R>
struct AppendSharedF32 {
  float row[kChunkF32][R + 4];
  float z[4][kChunkF32];
};
// N operands of a wavefront, each 16 rows x 64 bytes brought in by lane / 4 and lane % 4, into the operand layout (row lane % 16, 16 bytes
// lane / 16) through the wavefront's quarter of `bytes` of LDS.  Loaded straight into it, where neighbouring lanes are 16 rows, each keeps the
// address path of the unit for 66 cycles (three sequences of up to 777 tokens, r = 256: append and parallel form 50.1, now 49.2 us; the
// rounded latents' kernels, whose weights travel beside the lengths, gain nothing).
template <int N, class V>
__device__ __forceinline__ void turn_pieces(V* f, unsigned char* lds, size_t bytes) {
  const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g = lane >> 4;
  const int fit = (int)(bytes / 4096);  // at a time (a constant)
  unsigned char* part = lds + wv * (fit * 1024);
  unsigned char* to = part + (lane >> 2) * 64 + (((lane & 3) ^ swz_rows16<4>(lane >> 2)) << 4);
  const unsigned char* from = part + l16 * 64 + ((g ^ swz_rows16<4>(l16)) << 4);
#pragma unroll
  for (int i0 = 0; i0 < N; i0 += fit) {
#pragma unroll
    for (int i = i0; i < (i0 + fit < N ? i0 + fit : N); ++i) *reinterpret_cast<V*>(to + 1024 * (i - i0)) = f[i];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = i0; i < (i0 + fit < N ? i0 + fit : N); ++i) f[i] = *reinterpret_cast<const V*>(from + 1024 * (i - i0));
    __builtin_amdgcn_wave_barrier();
  }
}

template <int R>
__device__ __forceinline__ void append_range_f32(const AppendArgs& a, int b, int p0, int n, int slot_base, long long pos_lo,
                                                 long long pos_hi, AppendSharedF32<R>& sh) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4, q = tid & 31, j = tid >> 5;
  const int s = a.stride, dR = a.d_rope, dy = a.d_hyper;
  const int t0 = int(pos_lo - p0), cnt = int(pos_hi - pos_lo);  // tokens t0 .. t0 + cnt - 1 of the call
  const size_t tok0 = (size_t)b * a.n_new_max + t0;
  constexpr int KK = R / 16, NP = R >= 128 ? R / 128 : 1;       // a thread merges pieces q, q + 32, .. of 4 elements
  constexpr int NL = kChunkF32 * R / 4 / kBlock;                // 16-byte pieces of a chunk that a thread brings
  const bool hyper = !a.w_override && 16 * wv < dy;

  // ---- requests that need nothing but the position
  float4_t af[KK], bias = {0.f, 0.f, 0.f, 0.f};
  if (hyper) {
    const float* A = reinterpret_cast<const float*>(a.hyp_A) + (size_t)(16 * wv + (lane >> 2)) * R + 4 * (lane & 3);  // (turned below)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) af[kk] = *reinterpret_cast<const float4_t*>(A + 16 * kk);
    if (a.hyp_a) {
#pragma unroll
      for (int v = 0; v < 4; ++v) bias[v] = reinterpret_cast<const float*>(a.hyp_a)[16 * wv + 4 * g + v];
    }
  }
  const int slot = slot_base + j;
  const long long sf = (long long)slot * s;
  const long long lo = sf > pos_lo ? sf : pos_lo, hi = sf + s < pos_hi ? sf + s : pos_hi;
  const bool mine = lo < hi && 4 * q < R;  // the slot is touched by this range
  float4_t acc[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) acc[i] = float4_t{0.f, 0.f, 0.f, 0.f};
  if (mine && sf < p0) {  // the slot already holds earlier tokens
#pragma unroll
    for (int i = 0; i < NP; ++i) acc[i] = *reinterpret_cast<const float4_t*>(a.tail_c + (size_t)b * R + 4 * (q + 32 * i));
  }

  for (int c0 = 0; c0 < cnt; c0 += kChunkF32) {
    const int nc = cnt - c0 < kChunkF32 ? cnt - c0 : kChunkF32;
    if (c0) __syncthreads();
    float4_t gv = {0.f, 0.f, 0.f, 0.f};
    if (hyper) {
      const int u = l16 < nc ? l16 : nc - 1;
      gv = *reinterpret_cast<const float4_t*>(reinterpret_cast<const float*>(a.hyp_G) + (size_t)((pos_lo + c0 + u) / s) * dy + 16 * wv + 4 * g);
    }
    float4_t v[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int p = tid + i * kBlock, u = p / (R / 4), e = 4 * (p % (R / 4));
      v[i] = *reinterpret_cast<const float4_t*>(reinterpret_cast<const float*>(a.c_new) + (tok0 + c0 + (u < nc ? u : nc - 1)) * R + e);
    }
    if (c0 == 0 && !a.w_override) {
      if (hyper) turn_pieces<KK>(af, reinterpret_cast<unsigned char*>(sh.row), sizeof(sh.row));
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int p = tid + i * kBlock;
      *reinterpret_cast<float4_t*>(&sh.row[p / (R / 4)][4 * (p % (R / 4))]) = v[i];
    }
    __syncthreads();

    // ---- logits of the merge weights
    if (hyper) {
      float4_t d0 = {0.f, 0.f, 0.f, 0.f}, d1 = d0;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const float4_t c = *reinterpret_cast<const float4_t*>(&sh.row[l16][16 * kk + 4 * g]);
        d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(af[kk][0], c[0], d0, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(af[kk][1], c[1], d1, 0, 0, 0);
        d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(af[kk][2], c[2], d0, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(af[kk][3], c[3], d1, 0, 0, 0);
      }
      // the lane holds Linear(c)[16 wv + 4 g + v] of its token
      float z = 0.f;
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) z += (d0[v4] + d1[v4] + bias[v4]) * gv[v4];
      z = quarter_reduce(z, LaneSum());
      if (g == 0) sh.z[wv][l16] = z;
    }
    __syncthreads();
    auto weight = [&](int u) {
      if (a.w_override) return a.w_override[tok0 + c0 + u];
      float z = 0.f;
      for (int y = 0; 16 * y < dy; ++y) z += sh.z[y][u];
      return 1.f / (1.f + expf(-z));
    };
    if (tid < nc && (a.w_out || a.slot_out)) {
      if (a.w_out) a.w_out[tok0 + c0 + tid] = weight(tid);
      if (a.slot_out) a.slot_out[tok0 + c0 + tid] = int((pos_lo + c0 + tid) / s);
    }

    // ---- temporal merge of the slot's tokens in this chunk
    if (mine) {
      const long long u_lo = lo - pos_lo - c0 > 0 ? lo - pos_lo - c0 : 0, u_hi = hi - pos_lo - c0 < nc ? hi - pos_lo - c0 : nc;
      for (int u = (int)u_lo; u < (int)u_hi; ++u) {
        const float w = weight(u);
#pragma unroll
        for (int i = 0; i < NP; ++i) acc[i] += w * *reinterpret_cast<const float4_t*>(&sh.row[u][4 * (q + 32 * i)]);
      }
    }
  }

  if (lo < hi) {
    const size_t crow = cache_row(a.pages, b, slot, a.max_slots);
    if (4 * q < R) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int e = 4 * (q + 32 * i);
        *reinterpret_cast<float4_t*>(reinterpret_cast<float*>(a.cache_c) + crow * R + e) = acc[i];
        if (hi == (long long)p0 + n) *reinterpret_cast<float4_t*>(a.tail_c + (size_t)b * R + e) = acc[i];  // the sequence's tail
      }
    }
    // RoPE key: the slot keeps the key of the newest token folded into it
    if (q < dR / 4) {
      const float* kr_src = reinterpret_cast<const float*>(a.kr_new) + ((size_t)b * a.n_new_max + (size_t)(hi - 1 - p0)) * dR;
      *reinterpret_cast<float4_t*>(reinterpret_cast<float*>(a.cache_kr) + crow * dR + 4 * q) = *reinterpret_cast<const float4_t*>(kr_src + 4 * q);
    }
  }
}

template <int R>
__global__ __launch_bounds__(kBlock) void append_bulk_f32_kernel(AppendArgs a, int slots) {
  __shared__ __attribute__((aligned(16))) AppendSharedF32<R> sh;
  append_share(a, slots, nullptr, blockIdx.x, blockIdx.y, []() {}, [&](int p0, int n, long long pos_lo, long long pos_hi) {
    append_range_f32<R>(a, blockIdx.y, p0, n, int(pos_lo / a.stride), pos_lo, pos_hi, sh);
  });
}

// Tokens before the new rows, forced into what the arrays hold (the declared past is at most the capacity).
__device__ __forceinline__ int start_of(const ChunkStageArgs& a, int b) {
  if (!a.pos0) return 0;  // whole sequences
  const int p0 = a.pos0[b], inside = start_inside(p0, a.stride, a.past_pitch);
  if (inside != p0) *a.status = 1;  // MTLA_ERR_INVALID_ARG
  return inside;
}

// 16-byte pieces: slot states and RoPE keys of the past (rows k < pos0 / s of a sequence's part of cprime and kr16), and
// the new rows' RoPE keys behind them.  (A sequence's rows are together at the front of its part, so that the key / value
// product meets few tiles that are only partly in use.)  Rows that hold nothing are left alone: nothing reads them.
__device__ __forceinline__ void stage_piece(const ChunkStageArgs& a, size_t idx) {
  const int r8 = a.r / 8, d8 = a.d_rope / 8, past = a.past_pitch, Tp = past + a.T;
  const size_t n1 = (size_t)a.batch * past * (r8 + d8), n3 = (size_t)a.batch * a.T * d8;
  uint16_t* cp = reinterpret_cast<uint16_t*>(a.cprime);
  uint16_t* kr16 = reinterpret_cast<uint16_t*>(a.kr16);
  if (idx < n1) {
    const int piece = int(idx % (r8 + d8)), k = int(idx / (r8 + d8) % past), b = int(idx / ((size_t)(r8 + d8) * past));
    if (k >= start_of(a, b) / a.stride) return;
    int sb = b;  // the sequence whose rows hold slot k: b itself, or the owner of a prompt it shares
    if (a.prefix_owner && k < a.prefix_slots[b]) {
      const int o = a.prefix_owner[b];
      sb = o < 0 ? 0 : (o < a.prefix_rows ? o : a.prefix_rows - 1);
    }
    const size_t src = cache_row(a.pages, sb, k, a.max_slots), dst = (size_t)b * Tp + k;
    const uint16_t* from = piece < r8 ? reinterpret_cast<const uint16_t*>(a.cache_c) + src * a.r + 8 * piece
                                      : reinterpret_cast<const uint16_t*>(a.cache_kr) + src * a.d_rope + 8 * (piece - r8);
    uint16_t* to = piece < r8 ? cp + dst * a.r + 8 * piece : kr16 + dst * a.d_rope + 8 * (piece - r8);
    *reinterpret_cast<u32x4_t*>(to) = bf16x8_to_f16x8(*reinterpret_cast<const u32x4_t*>(from));
    return;
  }
  idx -= n1;
  if (idx >= n3) return;
  const int pd = int(idx % d8), m = int(idx / d8 % a.T), b = int(idx / ((size_t)d8 * a.T));
  if (a.n_new && m >= a.n_new[b]) return;
  *reinterpret_cast<u32x4_t*>(kr16 + ((size_t)b * Tp + start_of(a, b) / a.stride + m) * a.d_rope + 8 * pd) = bf16x8_to_f16x8(
      *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.kr) + ((size_t)b * a.T + m) * a.d_rope + 8 * pd));
}

// Partial states from given merge weights, 8 elements per thread: run jl holds the new tokens of slot pos0 / s + jl; the
// first run continues the slot in progress from tail_prev when pos0 % s != 0.
__device__ __forceinline__ void stage_run(const ChunkStageArgs& a, size_t idx) {
  const int r8 = a.r / 8, s = a.stride, T = a.T, Tp = a.past_pitch + T;
  const int n_runs = (T + s - 1) / s + 1;
  if (idx >= (size_t)a.batch * n_runs * r8) return;
  const int piece = int(idx % r8), jl = int(idx / r8 % n_runs), b = int(idx / ((size_t)r8 * n_runs));
  const int p0 = start_of(a, b), ph = p0 % s, past = p0 / s;
  int n = jl * s - ph;
  int n_end = n + s < T ? n + s : T;
  float run[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (jl == 0 && ph > 0) load8(a.tail_prev + (size_t)b * a.r + 8 * piece, run);
  if (n < 0) n = 0;
  const int len = a.n_new ? a.n_new[b] : T;
  n_end = n_end < len ? n_end : len;
  for (; n < n_end; ++n) {
    const size_t row = (size_t)b * T + n;
    float cv[8];
    load8(reinterpret_cast<const bf16*>(a.c) + row * a.r + 8 * piece, cv);
    const float w = a.w[row];
    u32x4_t o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      run[2 * i] += w * cv[2 * i];
      run[2 * i + 1] += w * cv[2 * i + 1];
      o[i] = pack_f16x2(run[2 * i], run[2 * i + 1]);
    }
    *reinterpret_cast<u32x4_t*>(reinterpret_cast<uint16_t*>(a.cprime) + ((size_t)b * Tp + past + n) * a.r + 8 * piece) = o;
  }
}

// Weights as fp16.  W_K^(h) [r][d_h] is turned on the way (64 x 32 tiles through LDS, both sides in 16-byte pieces: read
// an element at a time down its columns it took 10.8 us for 16 heads x 128, r = 512); W_V^(h) and W_O keep their layout.
constexpr int kConvPieces = 4;  // 16-byte pieces per thread of the plain conversions
__device__ __forceinline__ void convert_block(const PrefillFrontArgs& a, unsigned blk, uint16_t (*tile)[72]) {
  const int tid = threadIdx.x, r = a.cs.r, dh = a.d_head;
  const unsigned per_head = (unsigned)(r / 64) * (unsigned)(dh / 32), n_turn = (unsigned)a.n_heads * per_head;
  if (blk < n_turn) {
    const int h = int(blk / per_head), n0 = 64 * int(blk % per_head / (unsigned)(dh / 32)), d0 = 32 * int(blk % (unsigned)(dh / 32));
    const int n = tid >> 2, d8 = 8 * (tid & 3);
    const u32x4_t v = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.w_uk) + ((size_t)h * r + n0 + n) * dh + d0 + d8);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w = v[i];
      tile[d8 + 2 * i][n] = bf16_bits_to_f16_bits((uint16_t)(w & 0xffffu));
      tile[d8 + 2 * i + 1][n] = bf16_bits_to_f16_bits((uint16_t)(w >> 16));
    }
    __syncthreads();
    const int d = tid >> 3, n8 = 8 * (tid & 7);
    *reinterpret_cast<u32x4_t*>(reinterpret_cast<uint16_t*>(a.w_kT) + ((size_t)h * dh + d0 + d) * r + n0 + n8) =
        *reinterpret_cast<const u32x4_t*>(&tile[d][n8]);
    return;
  }
  const size_t n_v = (size_t)a.n_heads * dh * r / 8, n_o = a.n_wo / 8;
  const size_t first = (size_t)(blk - n_turn) * kBlock * kConvPieces + tid;
#pragma unroll
  for (int i = 0; i < kConvPieces; ++i) {
    const size_t p = first + (size_t)i * kBlock;
    if (p < n_v)
      reinterpret_cast<u32x4_t*>(a.w_v16)[p] = bf16x8_to_f16x8(reinterpret_cast<const u32x4_t*>(a.w_uv)[p]);
    else if (p < n_v + n_o)
      reinterpret_cast<u32x4_t*>(a.w_o16)[p - n_v] = bf16x8_to_f16x8(reinterpret_cast<const u32x4_t*>(a.w_o)[p - n_v]);
  }
}

template <int R, int MODE>
__global__ __launch_bounds__(kBlock, 2) void prefill_front_kernel(PrefillFrontArgs a) {
  struct None {};
  __shared__ __attribute__((aligned(16))) union {
    std::conditional_t<MODE == 0, None, AppendShared<R, MODE == 2>> append;
    uint16_t tile[32][72];
  } sh;
  unsigned blk = blockIdx.x;
  if (blk < a.n_main) {  // the new rows
    if constexpr (MODE == 0) stage_run(a.cs, (size_t)blk * kBlock + threadIdx.x);
    else append_block<R, MODE == 2, true>(a.ap, &a, a.group_slots, blk / (unsigned)a.cs.batch, blk % (unsigned)a.cs.batch, sh.append);
    return;
  }
  blk -= a.n_main;
  if (blk < a.n_conv) {
    convert_block(a, blk, sh.tile);
    return;
  }
  stage_piece(a.cs, (size_t)(blk - a.n_conv) * kBlock + threadIdx.x);
}

// slots a call can touch per sequence: a partly filled first slot plus the rest
int touched_slots(const AppendArgs& a) { return (a.n_new_max + a.stride - 2) / a.stride + 1; }

// Slots of a workgroup (bf16): a chunk of tokens, or as many chunks as leave the chip one round of the workgroups that fit on its
// units (by their registers: four at r = 64 and 128, three at 256, two at 512), the next chunk's latents on their way: each
// fetches the weights of the hyper-network, at r = 512 twice a chunk's latents, and waits for the lengths.  us with one / two / three
// chunks a workgroup, s = 2, over 8 x 4096 tokens, 1024 chunks, and 16 x 2080, 1040: r = 64 7.3 / 7.9 / 10.7 and 7.9 / 8.0 / 10.8, 128 7.8 / 8.3
// and 9.6 / 8.4, 256 11.3 / 10.5 / 12.5 and 12.7 / 11.0 / 12.7, 512 19.2 / 17.2 / 19.4 and 21.6 / 19.3 / 19.4; 12 x 2048, 768 chunks: 256 9.1 / 10.0, 512
// 15.6 / 15.6; 32 x 2048, 2048 chunks: 64 10.8 / 10.4, 256 18.8 / 18.0 / 17.0, 512 31.8 / 28.6 / 29.2, four 25.7.
// With a stride of 1 half a chunk where that leaves half a round free, us with half a chunk / a chunk: r = 128, one of 627 7.4 / 7.9; r = 64, 77 of
// 37 7.5 / 8.0; r = 256, 3 of 100 7.6 / 8.2; r = 512, 16 of 100 9.1 / 10.2 (its turns of 16 slots follow one another).
int group_slots(const AppendArgs& a) {
  const size_t round = 256 * (a.r <= 128 ? 4 : (a.r == 256 ? 3 : 2));
  int one = a.stride < kChunk ? kChunk / a.stride : 1;
  if (one > kChunkSlots && (size_t)((touched_slots(a) + kChunkSlots - 1) / kChunkSlots) * a.batch <= round / 2) one = kChunkSlots;
  const size_t groups = (size_t)(((a.n_new_max + a.stride - 1) / a.stride + one - 1) / one) * a.batch;
  return one * (int)((groups + round - 1) / round);
}

// fp32: 16 tokens' slots, twice that of launches with more than two such workgroups a unit.  A workgroup's chunks follow one another, and
// with eight slots whatever the stride a long one's are many.  us of 1 / 2 / 4 / 8 slots: r = 256, 3 sequences of 700 to 777 tokens, s = 2
// 21.2 / 14.9 / 12.3 / 10.1, s = 4 15.5 / 12.5 / 10.4 / 13.3; 16 of 1000, s = 4 53.7 / 31.9 / 20.5 / 18.5, s = 8 32.5 / 20.9 / 19.8 / 24.6, s = 16 23.4 / 24.4 /
// 34.3 / 60.3; weights given, 8 of 259, s = 16 8.9 / 10.6 / 14.8 / 23.1.  A sequence's last slot apart from workgroup 0's is a second pass of
// its own (append_share): two chunks that one workgroup can take stay together (7 sequences of 22 tokens, s = 4 12.9, apart 14.9).
int group_slots_f32(const AppendArgs& a) {
  if (touched_slots(a) <= kSlotsF32 && a.n_new_max <= 2 * kChunkF32) return kSlotsF32;
  const int one = a.stride < kChunkF32 ? kChunkF32 / a.stride : 1;
  const size_t groups = (size_t)((touched_slots(a) + one - 1) / one) * a.batch;
  const int n = one > 1 && groups > 512 ? 2 * one : one;
  return n < kSlotsF32 ? n : kSlotsF32;
}

template <int MODE>
hipError_t launch_front_mode(const PrefillFrontArgs& a, const dim3& grid, hipStream_t st) {
  switch (a.cs.r) {
    case 64: hipLaunchKernelGGL((prefill_front_kernel<64, MODE>), grid, dim3(kBlock), 0, st, a); break;
    case 128: hipLaunchKernelGGL((prefill_front_kernel<128, MODE>), grid, dim3(kBlock), 0, st, a); break;
    case 256: hipLaunchKernelGGL((prefill_front_kernel<256, MODE>), grid, dim3(kBlock), 0, st, a); break;
    case 512: hipLaunchKernelGGL((prefill_front_kernel<512, MODE>), grid, dim3(kBlock), 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

bool append_bulk_supported(const AppendArgs& a, int dtype) {
  // fp32: rows of the hyper-network and the tail shadow are read 16 bytes at a time, which the calls do not ask of their addresses
  const auto odd = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; };
  if (dtype == 0 && (odd(a.hyp_A) || odd(a.hyp_G) || odd(a.tail_c))) return false;
  return a.tail_c && a.stride <= 16 && a.d_hyper % 16 == 0 && a.d_hyper <= 64 &&
         (a.r == 64 || a.r == 128 || a.r == 256 || a.r == 512) && a.d_rope % 8 == 0 && a.d_rope <= 128;
}

hipError_t launch_append_bulk(const AppendArgs& a, int dtype, hipStream_t st) {
  const bool f32 = dtype == 0;
  const int slots = f32 ? group_slots_f32(a) : group_slots(a);
  const unsigned groups = (unsigned)((touched_slots(a) + slots - 1) / slots);  // bf16: the sequences' last ones, which may be empty, start last
#define MTLA_CASE(RR)                                                                             \
  if (a.r == RR) {                                                                                \
    if (f32) hipLaunchKernelGGL(append_bulk_f32_kernel<RR>, dim3(groups, a.batch), dim3(kBlock), 0, st, a, slots); \
    else hipLaunchKernelGGL(append_bulk_kernel<RR>, dim3(a.batch, groups), dim3(kBlock), 0, st, a, slots);         \
    return hipGetLastError();                                                                     \
  }
  MTLA_CASE(64) MTLA_CASE(128) MTLA_CASE(256) MTLA_CASE(512)
#undef MTLA_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_prefill_front(const PrefillFrontArgs& args, int mode, hipStream_t st) {
  PrefillFrontArgs a = args;
  const ChunkStageArgs& cs = a.cs;
  const size_t r8 = cs.r / 8, d8 = cs.d_rope / 8;
  if (mode != 0) {
    a.group_slots = group_slots(a.ap);
    a.groups = (unsigned)((touched_slots(a.ap) + a.group_slots - 1) / a.group_slots);
  }
  const size_t n_runs = (cs.T + cs.stride - 1) / cs.stride + 1;
  const size_t main = mode == 0 ? ((size_t)cs.batch * n_runs * r8 + kBlock - 1) / kBlock : (size_t)a.groups * cs.batch;
  const size_t plain = ((size_t)a.n_heads * a.d_head * r8 + a.n_wo / 8 + kBlock * kConvPieces - 1) / (kBlock * kConvPieces);
  const size_t conv = (size_t)a.n_heads * (cs.r / 64) * (a.d_head / 32) + plain;
  const size_t pieces = (size_t)cs.batch * cs.past_pitch * (r8 + d8) + (size_t)cs.batch * cs.T * d8;
  const size_t total = main + conv + (pieces + kBlock - 1) / kBlock;
  if (total >= (size_t)1 << 31) return hipErrorInvalidValue;
  a.n_main = (unsigned)main;
  a.n_conv = (unsigned)conv;
  const dim3 grid((unsigned)total);
  return mode == 0 ? launch_front_mode<0>(a, grid, st) : (mode == 1 ? launch_front_mode<1>(a, grid, st) : launch_front_mode<2>(a, grid, st));
}

}  // namespace mtla
