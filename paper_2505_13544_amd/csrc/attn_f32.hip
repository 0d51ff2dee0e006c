// fp32 storage on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 inputs, fp32 products and sums).
//
//   attn_decode_f32_kernel   one query per sequence against its cache slots, static schedule    (Eq. (with-rope))
//   kv_f32_kernel            keys and values of all rows, k = C_hat' W_K^(h), v = C_hat' W_V^(h)  (before Eq. (obsorb))
//   prefill_f32_kernel       the parallel form under the stride-aware mask over those keys and values
//
// Operand layout of the instruction: lane = 16 k + i holds A[i, k] and B[k, i], and D[4 k + v, i] in its four results.
// Which four elements of the contraction one instruction takes is free, as long as A and B agree: a lane loads 16
// bytes (elements 16 c + 4 k .. + 3 of its row) and instruction j of the four that follow takes element j of every lane.
#include "bounds.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = kBlock / kWave;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
// over the four lanes that hold one column of a 16 x 16 result
__device__ __forceinline__ float col_max(float v) {
  return quarter_reduce(v, LaneMax());
}
__device__ __forceinline__ float col_sum(float v) {
  return quarter_reduce(v, LaneSum());
}

// ---------------------------------------------------------------------------
// Decode: workgroup = (chunk of slots, sequence, 16 heads); a wavefront takes every fourth 16-slot tile of the chunk.
// S^T[slot, head] = tile . Q^T, and the weights leave that product exactly as the second one wants them
// (lane = head, four consecutive slots): O^T[n, head] += C_hat^T[n, slot] P^T[slot, head], the transposed tile
// read again from the cache in 64-byte pieces (the first product has just brought it into L1).
// Bound by latency at the sizes fp32 is used for (one sequence of 128 slots, 4 heads x 64, r = 64: 49 KB): every
// load of a tile is requested before the first product, which makes a tile one round trip.  The vector-ALU kernel
// it replaces walked a chunk slot by slot with a cross-lane sum per head and slot: 20.6 us at that size, now 3.9.
// ---------------------------------------------------------------------------
template <int R, int DR>
__global__ __launch_bounds__(kBlock) void attn_decode_f32_kernel(AttnArgs a) {
  constexpr int E = R + DR, KC = R / 16, KE = E / 16;
  constexpr int PC = R < 128 ? R : 128;  // columns merged at a time
  __shared__ float s_o[kWaves][16][PC + 4];
  __shared__ float s_m[kWaves][16], s_l[kWaves][16];
  const int split = blockIdx.x, row = blockIdx.y, h0 = blockIdx.z * 16;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6, l16 = lane & 15, g = lane >> 4;
  const int len = a.seq_len[row];
  const int head = h0 + l16 < a.n_heads ? h0 + l16 : a.n_heads - 1;  // a head past the end: computed, not stored
  const float* qp = reinterpret_cast<const float*>(a.qcat) + ((size_t)row * a.n_heads + head) * E + 4 * g;
  f32x4 qf[KE];
#pragma unroll
  for (int c = 0; c < KE; ++c) qf[c] = ld4(qp + 16 * c);
  const float* lat = reinterpret_cast<const float*>(a.lat) + (size_t)row * a.max_slots * R;
  const float* key = reinterpret_cast<const float*>(a.key) + (size_t)row * a.max_slots * DR;
  const int k0 = split * a.chunk;
  const int live = live_slots(len, a.stride, a.max_slots);
  const int k1 = live < k0 + a.chunk ? live : k0 + a.chunk;
  if (k0 >= k1) return;

  float m = -INFINITY, l = 0.f;
  f32x4 acc[KC];
#pragma unroll
  for (int t = 0; t < KC; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int s0 = k0 + 16 * wv; s0 < k1; s0 += 16 * kWaves) {
    const int slot = s0 + l16 < k1 ? s0 + l16 : k1 - 1;
    const float* cr = lat + (size_t)slot * R + 4 * g;
    const float* kr = key + (size_t)slot * DR + 4 * g;
    f32x4 kf[KE];
#pragma unroll
    for (int c = 0; c < KC; ++c) kf[c] = ld4(cr + 16 * c);
#pragma unroll
    for (int c = KC; c < KE; ++c) kf[c] = ld4(kr + 16 * (c - KC));
    const float* vr[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int sv = s0 + 4 * g + v < k1 ? s0 + 4 * g + v : k1 - 1;  // its weight is zero when it is past the end
      vr[v] = lat + (size_t)sv * R + l16;
    }
    float vf[KC][4];
    if constexpr (R <= 256) {
#pragma unroll
      for (int t = 0; t < KC; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) vf[t][v] = vr[v][16 * t];
    }
    f32x4 s_a = {0.f, 0.f, 0.f, 0.f}, s_b = s_a;
#pragma unroll
    for (int c = 0; c < KE; ++c) {
      s_a = mfma4(kf[c][0], qf[c][0], s_a);
      s_b = mfma4(kf[c][1], qf[c][1], s_b);
      s_a = mfma4(kf[c][2], qf[c][2], s_a);
      s_b = mfma4(kf[c][3], qf[c][3], s_b);
    }
    float p[4];
    float mt = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p[v] = s0 + 4 * g + v < k1 ? s_a[v] + s_b[v] : -INFINITY;
      mt = fmaxf(mt, p[v]);
    }
    const float mn = fmaxf(m, col_max(mt));  // finite: a tile holds at least one live slot
    const float alpha = __builtin_amdgcn_exp2f(m - mn);
    l *= alpha;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p[v] = __builtin_amdgcn_exp2f(p[v] - mn);
      l += p[v];
    }
    m = mn;
#pragma unroll
    for (int t = 0; t < KC; ++t) {
      acc[t] *= alpha;
      if constexpr (R > 256) {
#pragma unroll
        for (int v = 0; v < 4; ++v) vf[t][v] = vr[v][16 * t];
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[t] = mfma4(vf[t][v], p[v], acc[t]);
    }
  }
  l = col_sum(l);

  // ---- one partial out of the four wavefronts' states
  if (g == 0) {
    s_m[wv][l16] = m;
    s_l[wv][l16] = l;
  }
  __syncthreads();
  float ms = s_m[0][l16];  // the first wavefront always has a tile
#pragma unroll
  for (int w = 1; w < kWaves; ++w) ms = fmaxf(ms, s_m[w][l16]);
  const float f = __builtin_amdgcn_exp2f(m - ms);  // 0 for a wavefront without a tile
  const size_t piece = ((size_t)row * a.n_splits + split) * a.n_heads + h0;
  if (tid < 16 && h0 + tid < a.n_heads) {
    float ls = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) ls += s_l[w][tid] * __builtin_amdgcn_exp2f(s_m[w][tid] - ms);
    *reinterpret_cast<float2*>(a.part_ml + (piece + tid) * 2) = make_float2(ms, ls);
  }
  for (int n0 = 0; n0 < R; n0 += PC) {
    if (n0) __syncthreads();
#pragma unroll
    for (int t = 0; t < KC; ++t)
      if (16 * t >= n0 && 16 * t < n0 + PC) *reinterpret_cast<f32x4*>(&s_o[wv][l16][16 * t - n0 + 4 * g]) = acc[t] * f;
    __syncthreads();
    for (int i = tid; i < 16 * PC / 4; i += kBlock) {
      const int hh = i / (PC / 4), n = 4 * (i % (PC / 4));
      if (h0 + hh >= a.n_heads) continue;
      f32x4 o = *reinterpret_cast<f32x4*>(&s_o[0][hh][n]);
#pragma unroll
      for (int w = 1; w < kWaves; ++w) o += *reinterpret_cast<f32x4*>(&s_o[w][hh][n]);
      *reinterpret_cast<f32x4*>(a.part_o + (piece + hh) * R + n0 + n) = o;
    }
  }
}

// ---------------------------------------------------------------------------
// Keys (blockIdx.z = 0) and values (1) of all rows: C[m, h d_h + k] = sum_n C_hat'[m, n] W^(h)[n, k].
// 64 x 64 tile per workgroup, the contraction 32 at a time through LDS (rows of 36 floats: the 16-byte reads of 16
// rows spread over all banks), the next piece requested before this one is multiplied.  D = W . C_hat'^T, so a lane
// holds four consecutive columns of its row.  2331 rows x 512 x 256, both: 1.2 GFLOP in 23 us.
// ---------------------------------------------------------------------------
constexpr int kGT = 64, kGK = 32, kGP = kGK + 4;
__global__ __launch_bounds__(kBlock) void kv_f32_kernel(ExplicitArgs a) {
  __shared__ float sA[kGT][kGP], sW[kGT][kGP];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6, l16 = lane & 15, g = lane >> 4;
  const int M = a.batch * a.T, N = a.n_heads * a.d_head, r = a.r, dh = a.d_head;
  const int n0 = blockIdx.x * kGT, m0 = blockIdx.y * kGT;
  const bool keys = blockIdx.z == 0;
  // pieces a thread brings: two of the rows (16 bytes of the contraction), two of the weight
  const int ar = tid >> 3, ak = 4 * (tid & 7);  // row (and row + 32), place in the contraction
  const float* ap[2];
  const float* wp[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + ar + 32 * i < M ? m0 + ar + 32 * i : M - 1;
    ap[i] = reinterpret_cast<const float*>(a.cprime) + (size_t)m * r + ak;
  }
  const int wk = tid >> 4, wc = 4 * (tid & 15);  // keys: place in the contraction (and + 16), four columns of one head
  if (keys) {                                    // w_uk [h][n][k]: the columns are contiguous
    const int c = n0 + wc < N ? n0 + wc : 0;
    const float* w = reinterpret_cast<const float*>(a.w_uk) + (size_t)(c / dh) * r * dh + c % dh;
    wp[0] = w + (size_t)wk * dh;
    wp[1] = w + (size_t)(wk + 16) * dh;
  } else {                                       // w_uv [h][k][n]: the contraction is contiguous
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = n0 + ar + 32 * i < N ? n0 + ar + 32 * i : 0;
      wp[i] = reinterpret_cast<const float*>(a.w_uv) + (size_t)c * r + ak;
    }
  }
  const size_t wstep = keys ? (size_t)kGK * dh : kGK;
  f32x4 ra[2], rw[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    ra[i] = ld4(ap[i]);
    rw[i] = ld4(wp[i]);
  }
  f32x4 acc[2][2];  // [columns][rows] of the wavefront's 32 x 32 quarter
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int cw = 32 * (wv & 1), rw0 = 32 * (wv >> 1);
  for (int k = 0; k < r; k += kGK) {
    if (k) __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      *reinterpret_cast<f32x4*>(&sA[ar + 32 * i][ak]) = ra[i];
      if (keys) {
#pragma unroll
        for (int j = 0; j < 4; ++j) sW[wc + j][wk + 16 * i] = rw[i][j];
      } else {
        *reinterpret_cast<f32x4*>(&sW[ar + 32 * i][ak]) = rw[i];
      }
    }
    __syncthreads();
    if (k + kGK < r) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        ra[i] = ld4(ap[i] + k + kGK);
        rw[i] = ld4(wp[i] + wstep * (size_t)(k / kGK + 1));
      }
    }
#pragma unroll
    for (int c = 0; c < kGK / 16; ++c) {
      f32x4 fw[2], fa[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fw[i] = ld4(&sW[cw + 16 * i + l16][16 * c + 4 * g]);
        fa[i] = ld4(&sA[rw0 + 16 * i + l16][16 * c + 4 * g]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < 2; ++q) acc[i][q] = mfma4(fw[i][j], fa[q][j], acc[i][q]);
    }
  }
  float* out = reinterpret_cast<float*>(keys ? a.kx : a.vx);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int m = m0 + rw0 + 16 * q + l16;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int n = n0 + cw + 16 * i + 4 * g;
      if (m < M && n < N) *reinterpret_cast<f32x4*>(out + (size_t)m * N + n) = acc[i][q];
    }
  }
}

// ---------------------------------------------------------------------------
// Parallel form: workgroup = 16 RT query rows of one (head, sequence); its four wavefronts take the 16-column tiles in
// turn (so that a short sequence still gives every wavefront work) and are merged at the end.  Columns: the chunk-final
// rows below the block, then the block's own rows under the mask (row c is open to row q iff c == q, or c < q and c
// closes its chunk).  DV value columns per workgroup: d_head for `out`, slices of the partial states for the
// latent-space output.  Bound by the fp32 matrix rate (256 flop per clock and unit) plus the latency of a tile.
// Three sequences of up to 777 tokens, 8 heads x 64: 30 us; the vector-ALU kernel over absorbed queries took 353 us
// (and 45 + 67 us for the absorption and the value projection, which this form does not have).
// ---------------------------------------------------------------------------
template <int DH, int DR, int DV, int RT>
__global__ __launch_bounds__(kBlock) void prefill_f32_kernel(ExplicitArgs a) {
  constexpr int KE = (DH + DR) / 16, KC = DH / 16, NV = DV / 16, MB = 16 * RT;
  __shared__ float s_o[kWaves][MB][DV + 4];
  __shared__ float s_m[kWaves][MB], s_l[kWaves][MB];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6, l16 = lane & 15, g = lane >> 4;
  const int b = blockIdx.z, h = (int)blockIdx.y % a.n_heads, slice = (int)blockIdx.y / a.n_heads;
  const int m0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * MB;  // the blocks with most columns first
  const bool latent = a.n_slices > 0;
  const int width = latent ? a.r : DH;                         // columns of an output row of this head
  float* out = a.out + (((size_t)b * a.T) * a.n_heads + h) * width + slice * DV;
  const size_t out_pitch = (size_t)a.n_heads * width;
  int len = a.seq_len ? a.seq_len[b] : a.T;
  len = len < a.T ? len : a.T;
  if (m0 >= len) {  // padding
    for (int i = tid; i < MB * DV / 4; i += kBlock) {
      const int q = i / (DV / 4), n = 4 * (i % (DV / 4));
      if (m0 + q < a.T) *reinterpret_cast<f32x4*>(out + (size_t)(m0 + q) * out_pitch + n) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    return;
  }
  const size_t kpitch = (size_t)a.n_heads * DH;
  const float* kx = reinterpret_cast<const float*>(a.kx) + (size_t)b * a.T * kpitch + h * DH;
  const float* kr = reinterpret_cast<const float*>(a.kr) + (size_t)b * a.T * DR;
  const size_t vpitch = latent ? (size_t)a.r : kpitch;
  const float* vx = latent ? reinterpret_cast<const float*>(a.cprime) + (size_t)b * a.T * a.r + slice * DV
                           : reinterpret_cast<const float*>(a.vx) + (size_t)b * a.T * kpitch + h * DH;
  // queries of the block's rows, scaled to the log2 domain
  f32x4 qf[RT][KE];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const int m = m0 + 16 * t + l16 < len ? m0 + 16 * t + l16 : len - 1;
    const size_t qr = ((size_t)b * a.T + m) * a.n_heads + h;
    const float* q = reinterpret_cast<const float*>(a.q) + qr * DH + 4 * g;
    const float* qrope = reinterpret_cast<const float*>(a.q_rope) + qr * DR + 4 * g;
#pragma unroll
    for (int c = 0; c < KC; ++c) qf[t][c] = ld4(q + 16 * c);
#pragma unroll
    for (int c = KC; c < KE; ++c) qf[t][c] = ld4(qrope + 16 * (c - KC));
#pragma unroll
    for (int c = 0; c < KE; ++c) qf[t][c] *= a.scale_log2;
  }
  float m[RT], l[RT];
  f32x4 acc[RT][NV];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    m[t] = -INFINITY;
    l[t] = 0.f;
#pragma unroll
    for (int n = 0; n < NV; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int s = a.stride, n_sh = m0 / s, sh_tiles = (n_sh + 15) / 16;
  for (int tile = wv; tile < sh_tiles + RT; tile += kWaves) {
    const bool shared = tile < sh_tiles;
    const int c0 = shared ? 16 * tile : 16 * (tile - sh_tiles);  // first column of the tile: chunk index, or row of the block
    auto src = [&](int i) {                                      // row that column c0 + i of the tile stands for
      const int c = c0 + i;
      if (shared) return (c < n_sh ? c : n_sh - 1) * s + s - 1;
      return m0 + c < len ? m0 + c : len - 1;
    };
    const int krow = src(l16);
    const float* kp = kx + (size_t)krow * kpitch + 4 * g;
    const float* krp = kr + (size_t)krow * DR + 4 * g;
    f32x4 kf[KE];
#pragma unroll
    for (int c = 0; c < KC; ++c) kf[c] = ld4(kp + 16 * c);
#pragma unroll
    for (int c = KC; c < KE; ++c) kf[c] = ld4(krp + 16 * (c - KC));
    float vf[NV][4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float* vp = vx + (size_t)src(4 * g + v) * vpitch + l16;
#pragma unroll
      for (int n = 0; n < NV; ++n) vf[n][v] = vp[16 * n];
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      if (!shared && c0 > 16 * t + 15) continue;  // wholly above the rows
      f32x4 s_a = {0.f, 0.f, 0.f, 0.f}, s_b = s_a;
#pragma unroll
      for (int c = 0; c < KE; ++c) {
        s_a = mfma4(kf[c][0], qf[t][c][0], s_a);
        s_b = mfma4(kf[c][1], qf[t][c][1], s_b);
        s_a = mfma4(kf[c][2], qf[t][c][2], s_a);
        s_b = mfma4(kf[c][3], qf[t][c][3], s_b);
      }
      float p[4];
      float mt = -INFINITY;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = c0 + 4 * g + v, q = 16 * t + l16;
        const bool open = shared ? c < n_sh : (c == q || (c < q && (m0 + c + 1) % s == 0));
        p[v] = open ? s_a[v] + s_b[v] : -INFINITY;
        mt = fmaxf(mt, p[v]);
      }
      const float mn = fmaxf(m[t], col_max(mt));
      const float ref = mn == -INFINITY ? 0.f : mn;  // no open column so far
      const float alpha = __builtin_amdgcn_exp2f(m[t] - ref);
      l[t] *= alpha;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p[v] = __builtin_amdgcn_exp2f(p[v] - ref);
        l[t] += p[v];
      }
      m[t] = mn;
#pragma unroll
      for (int n = 0; n < NV; ++n) {
        acc[t][n] *= alpha;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[t][n] = mfma4(vf[n][v], p[v], acc[t][n]);
      }
    }
  }
  // ---- merge the wavefronts
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const float lt = col_sum(l[t]);
    if (g == 0) {
      s_m[wv][16 * t + l16] = m[t];
      s_l[wv][16 * t + l16] = lt;
    }
#pragma unroll
    for (int n = 0; n < NV; ++n) *reinterpret_cast<f32x4*>(&s_o[wv][16 * t + l16][16 * n + 4 * g]) = acc[t][n];
  }
  __syncthreads();
  for (int i = tid; i < MB * DV / 4; i += kBlock) {
    const int q = i / (DV / 4), n = 4 * (i % (DV / 4));
    if (m0 + q >= a.T) continue;
    float ms = s_m[0][q];  // a row's own column is always open, so the maximum over the wavefronts is finite
#pragma unroll
    for (int w = 1; w < kWaves; ++w) ms = fmaxf(ms, s_m[w][q]);
    float ls = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = __builtin_amdgcn_exp2f(s_m[w][q] - ms);
      ls += f * s_l[w][q];
      o += *reinterpret_cast<f32x4*>(&s_o[w][q][n]) * f;
    }
    o *= 1.f / ls;
    if (m0 + q >= len) o = f32x4{0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<f32x4*>(out + (size_t)(m0 + q) * out_pitch + n) = o;
  }
}

template <int DH, int DR, int DV, int RT>
void launch_prefill_rows(const ExplicitArgs& a, int slices, hipStream_t st, const EventPair& ev) {
  const dim3 grid((a.T + 16 * RT - 1) / (16 * RT), a.n_heads * slices, a.batch);
  launch_timed(prefill_f32_kernel<DH, DR, DV, RT>, grid, dim3(kBlock), 0, st, ev, a);
}

}  // namespace

hipError_t launch_attn_decode_f32(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
  const dim3 grid(a.n_splits, a.batch, (a.n_heads + 15) / 16);
#define MTLA_CASE(RR, DD)                                                                     \
  if (a.r == RR && a.d_rope == DD) {                                                          \
    launch_timed(attn_decode_f32_kernel<RR, DD>, grid, dim3(kBlock), 0, st, ev, a);            \
    return hipGetLastError();                                                                 \
  }
  MTLA_CASE(64, 32)
  MTLA_CASE(64, 64)
  MTLA_CASE(128, 32)
  MTLA_CASE(128, 64)
  MTLA_CASE(256, 32)
  MTLA_CASE(256, 64)
  MTLA_CASE(512, 32)
  MTLA_CASE(512, 64)
#undef MTLA_CASE
  return hipErrorInvalidValue;
}

bool prefill_f32_supported(const ExplicitArgs& a) {
  return (a.d_head == 32 || a.d_head == 64 || a.d_head == 128) && (a.d_rope == 32 || a.d_rope == 64) && a.r % 64 == 0 &&
         a.batch <= 65535 && (size_t)a.batch * a.T <= 65535u;  // the rows of the key / value product are a grid dimension
}

hipError_t launch_prefill_f32(const ExplicitArgs& args, hipStream_t st, const EventPair& ev) {
  ExplicitArgs a = args;
  a.n_slices = 0;
  const dim3 grid((a.n_heads * a.d_head + kGT - 1) / kGT, (a.batch * a.T + kGT - 1) / kGT, 2);
  hipLaunchKernelGGL(kv_f32_kernel, grid, dim3(kBlock), 0, st, a);
#define MTLA_CASE(HH, DD, RT)                                                                        \
  if (a.d_head == HH && a.d_rope == DD) {                                                            \
    launch_prefill_rows<HH, DD, HH, RT>(a, 1, st, ev);                                               \
    if (args.out_latent) {                                                                           \
      a.out = args.out_latent;                                                                       \
      a.n_slices = a.r / 64;                                                                         \
      launch_prefill_rows<HH, DD, 64, RT>(a, a.n_slices, st, EventPair());                           \
    }                                                                                                \
    return hipGetLastError();                                                                        \
  }
  MTLA_CASE(32, 32, 2)
  MTLA_CASE(32, 64, 2)
  MTLA_CASE(64, 32, 2)
  MTLA_CASE(64, 64, 2)
  MTLA_CASE(128, 32, 1)
  MTLA_CASE(128, 64, 1)
#undef MTLA_CASE
  return hipErrorInvalidValue;
}

}  // namespace mtla
