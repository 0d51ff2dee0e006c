// fp32 storage on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 inputs, fp32 products and sums).
//
//   attn_decode_f32_kernel   one query per sequence against its cache slots, static schedule    (Eq. (with-rope))
//   kv_f32_kernel            keys and values of all rows, k = C_hat' W_K^(h), v = C_hat' W_V^(h)  (before Eq. (obsorb))
//   prefill_f32_kernel       the parallel form under the stride-aware mask over those keys and values
//
// Operand layout of the instruction: lane = 16 k + i holds A[i, k] and B[k, i], and D[4 k + v, i] in its four results.
// Which four elements of the contraction one instruction takes is free, as long as A and B agree: a lane loads 16
// bytes (elements 16 c + 4 k .. + 3 of its row) and instruction j of the four that follow takes element j of every lane.
#include <type_traits>

#include "bounds.h"
#include "lds_stream.h"
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
// Keys (the first half of blockIdx.x) and values of all rows: C[m, h d_h + k] = sum_n C_hat'[m, n] W^(h)[n, k].
// 32 rows x 64 columns per workgroup, the contraction 32 at a time through two LDS buffers and one barrier a stage; two
// stages are on their way from memory.  D = W . C_hat'^T, so a lane holds four consecutive columns of its row.  W_V^(h) has
// the contraction innermost and is read 16 bytes a lane (rows of 36 floats: 16 rows spread over all banks).  W_K^(h) has it
// outermost: it stays as it is in LDS ([n][64 columns], rows of 68) and a lane picks its four elements with 4-byte reads,
// 16 lanes side by side; turned on the way in, its 4-byte writes met 8 to a bank.
// Bound by the fp32 matrix rate (256 flop per clock and unit) behind the first stages' trip to memory (5 us of it, all
// workgroups at once): 1920 rows x 512 x 256, both, 1 GFLOP, 23.2 us with 64 x 64 tiles over all rows; 15.7 us now.  What counts
// is that all units do the same: the row blocks of all sequences come first, padding last, and kKvPad keeps a fifth workgroup
// off a unit that another one lacks (18 us without it).  Sequences without padding, or short ones, are one sequence to it (launch_prefill_f32).
// ---------------------------------------------------------------------------
constexpr int kGT = 64, kGK = 32, kGP = kGK + 4, kGN = kGT + 4, kKvRows = 32;
constexpr size_t kKvPad = 12 << 10;  // LDS that a workgroup of the keys and values takes beyond its 27 KB: four per unit
__global__ __launch_bounds__(kBlock) void kv_f32_kernel(ExplicitArgs a) {
  constexpr int ROWS = kKvRows, RT = ROWS / 32;                  // 16-row tiles per wavefront, and row pieces per thread
  constexpr int W_FLOATS = kGT * kGP > kGK * kGN ? kGT * kGP : kGK * kGN;
  __shared__ __attribute__((aligned(16))) float sA[2][ROWS][kGP], sW[2][W_FLOATS];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6, l16 = lane & 15, g = lane >> 4;
  const int N = a.n_heads * a.d_head, r = a.r, dh = a.d_head;
  const int cols = (int)gridDim.x / 2, b = blockIdx.y, m0 = blockIdx.z * ROWS;
  const bool keys = (int)blockIdx.x < cols;
  const int n0 = ((int)blockIdx.x - (keys ? 0 : cols)) * kGT;
  // pieces a thread brings: RT of the rows (16 bytes of the contraction), two of the weight
  const int ar = tid >> 3, ak = 4 * (tid & 7);  // row (and row + 32), place in the contraction
  const float* ap[RT];
  const float* wp[2];
  int w_at[2];                                   // their places in sW
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int m = m0 + ar + 32 * i < a.T ? m0 + ar + 32 * i : a.T - 1;
    ap[i] = reinterpret_cast<const float*>(a.cprime) + ((size_t)b * a.T + m) * r + ak;
  }
  if (keys) {                                    // w_uk [h][n][k]: four columns of one head at one place of the contraction (and + 16)
    const int wk = tid >> 4, wc = 4 * (tid & 15);
    const int c = n0 + wc < N ? n0 + wc : 0;
    const float* w = reinterpret_cast<const float*>(a.w_uk) + (size_t)(c / dh) * r * dh + c % dh;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      wp[i] = w + (size_t)(wk + 16 * i) * dh;
      w_at[i] = (wk + 16 * i) * kGN + wc;
    }
  } else {                                       // w_uv [h][k][n]
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = n0 + ar + 32 * i < N ? n0 + ar + 32 * i : 0;
      wp[i] = reinterpret_cast<const float*>(a.w_uv) + (size_t)c * r + ak;
      w_at[i] = (ar + 32 * i) * kGP + ak;
    }
  }
  const size_t wstep = keys ? (size_t)kGK * dh : kGK;
  f32x4 ra[2][RT], rw[2][2];                     // two stages on their way (four: no faster)
  auto request = [&](int buf, int stage) {
#pragma unroll
    for (int i = 0; i < RT; ++i) ra[buf][i] = ld4(ap[i] + kGK * stage);
#pragma unroll
    for (int i = 0; i < 2; ++i) rw[buf][i] = ld4(wp[i] + wstep * (size_t)stage);
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int i = 0; i < RT; ++i) *reinterpret_cast<f32x4*>(&sA[buf][ar + 32 * i][ak]) = ra[buf][i];
#pragma unroll
    for (int i = 0; i < 2; ++i) *reinterpret_cast<f32x4*>(&sW[buf][w_at[i]]) = rw[buf][i];
  };
  const int stages = r / kGK;  // (r is a multiple of 64: an even number)
  request(0, 0);
  request(1, 1);
  if (a.seq_len && m0 >= a.seq_len[b]) return;  // padding only: nothing reads its keys and values
  f32x4 acc[2][RT];  // [columns][rows] of the wavefront's 32 x 16 RT quarter
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < RT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int cw = 32 * (wv & 1), rw0 = 16 * RT * (wv >> 1);
  put(0);
  __syncthreads();
  auto walk = [&](auto KEYS) {
    auto step = [&](int buf, int k) {
      // the operands of the stage, then the next one into the other buffer, then the products
      f32x4 fw[kGK / 16][2], fa[kGK / 16][RT];
#pragma unroll
      for (int c = 0; c < kGK / 16; ++c) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if constexpr (KEYS) {
#pragma unroll
            for (int j = 0; j < 4; ++j) fw[c][i][j] = sW[buf][(16 * c + 4 * g + j) * kGN + cw + 16 * i + l16];
          } else {
            fw[c][i] = ld4(&sW[buf][(cw + 16 * i + l16) * kGP + 16 * c + 4 * g]);
          }
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) fa[c][i] = ld4(&sA[buf][rw0 + 16 * i + l16][16 * c + 4 * g]);
      }
      if (k + 1 < stages) put(buf ^ 1);
      request(buf, k + 2 < stages ? k + 2 : stages - 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < kGK / 16; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < RT; ++q) acc[i][q] = mfma4(fw[c][i][j], fa[c][q][j], acc[i][q]);
      __syncthreads();
    };
    for (int k = 0; k < stages; k += 2) {
      step(0, k);
      step(1, k + 1);
    }
  };
  if (keys) walk(std::true_type());
  else walk(std::false_type());
  float* out = reinterpret_cast<float*>(keys ? a.kx : a.vx);
#pragma unroll
  for (int q = 0; q < RT; ++q) {
    const int m = m0 + rw0 + 16 * q + l16;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int n = n0 + cw + 16 * i + 4 * g;
      if (m < a.T && n < N) *reinterpret_cast<f32x4*>(out + ((size_t)b * a.T + m) * N + n) = acc[i][q];
    }
  }
}

// ---------------------------------------------------------------------------
// Parallel form: workgroup = RT blocks of 16 query rows of one (head, sequence); its four wavefronts take the 16-column
// tiles in turn (so that a short sequence still gives every wavefront work) and are merged at the end.  Columns: the
// chunk-final rows below a block, then the block's own rows under the mask (row c is open to row q iff c == q, or c < q and c
// closes its chunk).  DV value columns per workgroup: d_head for `out`, slices of the partial states for the
// latent-space output.  Bound by the fp32 matrix rate (256 flop per clock and unit) plus the latency of the first tile.
// With RT = 2 the blocks are one from either end of the sequence: the columns of the light one are among those of the heavy
// one, so they share the tiles, and all workgroups of a sequence do the same work.  (32 rows in one piece gave some units the two
// heaviest workgroups of the launch, 1.8 times the mean.)  AHEAD: a wavefront's next tile is on its way while one is multiplied.  Heads of
// 128, one block a workgroup, have no registers for that with two workgroups a unit: there the next tile's keys are asked for when this one's
// have been multiplied, the values in front of the keys' product.  us of the call, 8 heads, r = 256, s = 2, ahead with one workgroup a unit / so: 8
// prompts of 512 tokens 128 / 107, 12 of 777 333 / 272, 10 of 128 (640 workgroups) 42.1 / 39.6; 4 heads, 3 of 700 (528) 52.0 / 52.8, with s = 1
// 60.9 / 69.8; 8 heads, one of 700 (352) 36.9 / 41.2: kAheadMost.  (Beyond it one prompt of 4096 alone is slower so, 343 / 355.)
// TURNED (RT = 2): queries and tiles come in as whole rows, 16 bytes a lane, and change lanes in the wavefront's part of LDS: loaded straight into
// the operands' layout (16 rows for neighbours; the values 4 bytes a lane) a tile keeps the address path of the unit for some 650 cycles
// beside its 1280 of products, four wavefronts side by side.  us of the append and the parallel form, 8 heads x 64, r = 256: 3 prompts of 500 to 777 tokens
// 49.6 -> 46.2, 2 of up to 900 with the latent output 92.2 -> 82.7; 4 heads, r = 64, 4 of 1024 40.5 -> 37.8.  A launch of at most a workgroup a unit loads as before
// where it has more than 300 columns or hardly any (20 rows, 4 heads 29.8 / 30.3), and so do heads of 128: the
// turns lengthen the chain of a wavefront that has its SIMD for itself (4 heads, 3 of 700, s = 1 70.3 / 75.5; 4 heads x 64, r = 64, s = 1, one of 2000 (252 workgroups)
// 66.9 / 73.1, of 1000 45.6 / 48.5, of 500 36.2 / 37.2, but of 200 30.1 / 29.9, and 3 of 777 (300) 57.2 / 54.1; 8 heads x 128, 200 of 16 70.0 / 73.9; one
// of 4096 365 / 339 though).
// Three sequences of up to 777 tokens, 8 heads x 64: the vector-ALU kernel over absorbed queries took 353 us
// (and 45 + 67 us for the absorption and the value projection, which this form does not have).
// ---------------------------------------------------------------------------
// 16 rows of COLS floats on their way: load i of a lane is piece 64 i + lane of them, 16 bytes each.
template <int COLS>
struct RowsF32 {
  static constexpr int N = COLS / 16, PPR = COLS / 4, RS = kWave / PPR;  // loads, pieces a row, rows a load
  f32x4 f[N];
  // row i is the one min(i, last) steps behind `first`
  __device__ __forceinline__ void request(int lane, const float* first, size_t step, int last) {
    const int row0 = lane / PPR, col = 4 * (lane % PPR);
    if (last >= 15) {
      const float* p = first + (size_t)(uint32_t)row0 * step + col;
#pragma unroll
      for (int i = 0; i < N; ++i) f[i] = ld4(p + (size_t)(RS * i) * step);
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) f[i] = ld4(first + (size_t)(uint32_t)(row0 + RS * i < last ? row0 + RS * i : last) * step + col);
    }
  }
  // In LDS piece j of row i sits at j ^ swz_rows16(i).  A load's rows and a lane's pieces differ in bits of their own, so that either's places
  // are one exclusive or from the first.
  __device__ __forceinline__ void put(int lane, unsigned char* to) const {
    const int row0 = lane / PPR, at = row0 * (COLS * 4) + 16 * ((lane % PPR) ^ swz_rows16<PPR>(row0));
#pragma unroll
    for (int i = 0; i < N; ++i) *reinterpret_cast<f32x4*>(to + (at ^ (16 * swz_rows16<PPR>(RS * i))) + RS * i * (COLS * 4)) = f[i];
  }
  static __device__ __forceinline__ f32x4 operand(const unsigned char* from, int lane, int c) {  // columns 16 c + 4 (lane / 16) .. + 3 of row lane % 16
    const int row = lane & 15, at = row * (COLS * 4) + 16 * ((lane >> 4) ^ swz_rows16<PPR>(row));
    return *reinterpret_cast<const f32x4*>(from + (at ^ (64 * c)));
  }
  __device__ __forceinline__ void put_plain(int lane, float (*to)[COLS + 4]) const {
#pragma unroll
    for (int i = 0; i < N; ++i) *reinterpret_cast<f32x4*>(&to[lane / PPR + RS * i][4 * (lane % PPR)]) = f[i];
  }
};

constexpr size_t kAheadMost = 576;  // workgroups of a launch over heads of 128
template <int DH, int DR, int DV, int RT, bool AHEAD, bool TURNED>
__global__ __launch_bounds__(kBlock, AHEAD && RT == 1 ? 1 : 2) void prefill_f32_kernel(ExplicitArgs a) {
  constexpr int KE = (DH + DR) / 16, KC = DH / 16, NV = DV / 16;
  // the wavefronts' values (rows of DV + 4, so that 4-byte reads of four rows spread over the banks), in the end their sums; their keys
  __shared__ __attribute__((aligned(16))) float s_o[kWaves][16][DV + 4];
  __shared__ __attribute__((aligned(16))) float s_k[TURNED ? kWaves : 1][TURNED ? 16 * (DH + DR) : 4];
  __shared__ float s_m[kWaves][16 * RT], s_l[kWaves][16 * RT];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), l16 = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // (a tile is the same for all lanes: its branches and addresses are scalar)
  const int b = blockIdx.y, h = (int)blockIdx.x % a.n_heads, slice = (int)blockIdx.x / a.n_heads, x = blockIdx.z;
  const bool latent = a.n_slices > 0;
  const int width = latent ? a.r : DH;                         // columns of an output row of this head
  float* out = a.out + (((size_t)b * a.T) * a.n_heads + h) * width + slice * DV;
  const size_t out_pitch = (size_t)a.n_heads * width;
  int len = a.seq_len ? a.seq_len[b] : a.T;
  len = len < a.T ? len : a.T;
  const int n_all = (a.T + 15) / 16, n_blocks = len > 0 ? (len + 15) / 16 : 0;
  for (int blk = n_blocks + x; blk < n_all; blk += gridDim.z) {  // blocks of padding
    for (int i = tid; i < 16 * DV / 4; i += kBlock) {
      const int m = 16 * blk + i / (DV / 4), n = 4 * (i % (DV / 4));
      if (m < a.T) *reinterpret_cast<f32x4*>(out + (size_t)m * out_pitch + n) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  if (RT * x >= n_blocks) return;
  // first rows of the blocks, from the sequence's end and from its front (the one in the middle stands alone: -1)
  int m0[RT];
  m0[0] = 16 * (n_blocks - 1 - x);
  if constexpr (RT > 1) m0[1] = 2 * x + 1 < n_blocks ? 16 * x : -1;
  const size_t kpitch = (size_t)a.n_heads * DH;
  const float* kx = reinterpret_cast<const float*>(a.kx) + (size_t)b * a.T * kpitch + h * DH;
  const float* kr = reinterpret_cast<const float*>(a.kr) + (size_t)b * a.T * DR;
  const size_t vpitch = latent ? (size_t)a.r : kpitch;
  const float* vx = latent ? reinterpret_cast<const float*>(a.cprime) + (size_t)b * a.T * a.r + slice * DV
                           : reinterpret_cast<const float*>(a.vx) + (size_t)b * a.T * kpitch + h * DH;
  f32x4 qf[RT][KE];
  if constexpr (!TURNED) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int m_lane = (m0[t] < 0 ? 0 : m0[t]) + l16, m = m_lane < len ? m_lane : len - 1;
      const size_t qr = ((size_t)b * a.T + m) * a.n_heads + h;
      const float* q = reinterpret_cast<const float*>(a.q) + qr * DH + 4 * g;
      const float* qrope = reinterpret_cast<const float*>(a.q_rope) + qr * DR + 4 * g;
#pragma unroll
      for (int c = 0; c < KC; ++c) qf[t][c] = ld4(q + 16 * c);
#pragma unroll
      for (int c = KC; c < KE; ++c) qf[t][c] = ld4(qrope + 16 * (c - KC));
    }
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
  const int s = a.stride, n_sh = m0[0] / s, sh_tiles = (n_sh + 15) / 16;
  // tiles 0 .. sh_tiles - 1: the chunk-final rows below the first block; behind them every block's own rows
  const int tiles = sh_tiles + (RT > 1 && m0[RT - 1] < 0 ? RT - 1 : RT);
  auto src = [&](int tile, int i) {  // row that column i of a tile stands for
    if (tile < sh_tiles) {
      const int c = 16 * tile + i;
      return (c < n_sh ? c : n_sh - 1) * s + s - 1;
    }
    const int own = (tile == sh_tiles ? m0[0] : m0[RT - 1]) + i;
    return own < len ? own : len - 1;
  };
  struct Tile {
    f32x4 k[KE];
    float v[NV][4];
  };
  auto request_k = [&](Tile& t, int tile) {
    const int krow = src(tile, l16);
    const float* kp = kx + (size_t)krow * kpitch + 4 * g;
    const float* krp = kr + (size_t)krow * DR + 4 * g;
#pragma unroll
    for (int c = 0; c < KC; ++c) t.k[c] = ld4(kp + 16 * c);
#pragma unroll
    for (int c = KC; c < KE; ++c) t.k[c] = ld4(krp + 16 * (c - KC));
  };
  auto request_v = [&](Tile& t, int tile) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float* vp = vx + (size_t)src(tile, 4 * g + v) * vpitch + l16;
#pragma unroll
      for (int n = 0; n < NV; ++n) t.v[n][v] = vp[16 * n];
    }
  };
  auto multiply = [&](Tile& tl, int tile, auto&& behind_keys) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int own = sh_tiles + t, open_sh = m0[t] < 0 ? 0 : m0[t] / s;  // the block's own tile; its open chunks
      if (tile != own && (tile >= sh_tiles || 16 * tile >= open_sh)) continue;
      f32x4 s_a = {0.f, 0.f, 0.f, 0.f}, s_b = s_a;
#pragma unroll
      for (int c = 0; c < KE; ++c) {
        s_a = mfma4(tl.k[c][0], qf[t][c][0], s_a);
        s_b = mfma4(tl.k[c][1], qf[t][c][1], s_b);
        s_a = mfma4(tl.k[c][2], qf[t][c][2], s_a);
        s_b = mfma4(tl.k[c][3], qf[t][c][3], s_b);
      }
      behind_keys();
      float p[4];
      if (tile != own) {
#pragma unroll
        for (int v = 0; v < 4; ++v) p[v] = 16 * tile + 4 * g + v < open_sh ? s_a[v] + s_b[v] : -INFINITY;
        if (t > 0 && 16 * tile + 16 > open_sh) {  // the heavy block's columns: of an infinite value a weight of zero makes no number
#pragma unroll
          for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int n = 0; n < NV; ++n) tl.v[n][v] = 16 * tile + 4 * g + v < open_sh ? tl.v[n][v] : 0.f;
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int c = 4 * g + v;
          const bool open = (c == l16) | ((c < l16) & ((m0[t] + c + 1) % s == 0));
          p[v] = open ? s_a[v] + s_b[v] : -INFINITY;
        }
      }
      const float mt = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]));
      const float mn = fmaxf(m[t], col_max(mt));
      const float ref = mn == -INFINITY ? 0.f : mn;  // (every logit so far overflowed)
      const float alpha = __builtin_amdgcn_exp2f(m[t] - ref);
      l[t] *= alpha;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p[v] = __builtin_amdgcn_exp2f(p[v] - ref);
        l[t] += p[v];
      }
      m[t] = mn;
#pragma unroll
      for (int n = 0; n < NV; ++n) acc[t][n] *= alpha;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int n = 0; n < NV; ++n) acc[t][n] = mfma4(tl.v[n][v], p[v], acc[t][n]);
    }
  };
  // (a request past the last tile repeats the last one)
  auto to_log2 = [&]() {  // behind the first request
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int c = 0; c < KE; ++c) qf[t][c] *= a.scale_log2;
  };
  if constexpr (TURNED) {
    unsigned char* lds_k = reinterpret_cast<unsigned char*>(s_k[wv]);
    unsigned char* lds_r = lds_k + 16 * DH * 4;
    float (*lds_v)[DV + 4] = s_o[wv];
    RowsF32<DH> next_k;
    RowsF32<DR> next_r;
    RowsF32<DV> next_v;
    auto request = [&](int tile) {
      const bool shared = tile < sh_tiles;
      const int first = shared ? src(tile, 0) : (tile == sh_tiles ? m0[0] : m0[RT - 1]), step = shared ? s : 1;
      const int last = shared ? n_sh - 1 - 16 * tile : len - 1 - first;
      next_k.request(lane, kx + (size_t)first * kpitch, step * kpitch, last);
      next_r.request(lane, kr + (size_t)first * DR, (size_t)step * DR, last);
      next_v.request(lane, vx + (size_t)first * vpitch, step * vpitch, last);
    };
    auto operand = [&](int c) { return c < KC ? RowsF32<DH>::operand(lds_k, lane, c) : RowsF32<DR>::operand(lds_r, lane, c - KC); };
    if (wv < tiles) {
      RowsF32<DH> q[RT];
      RowsF32<DR> q_rope[RT];
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int first = m0[t] < 0 ? 0 : m0[t];
        const size_t row = ((size_t)b * a.T + first) * a.n_heads + h;
        q[t].request(lane, reinterpret_cast<const float*>(a.q) + row * DH, kpitch, len - 1 - first);
        q_rope[t].request(lane, reinterpret_cast<const float*>(a.q_rope) + row * DR, (size_t)a.n_heads * DR, len - 1 - first);
      }
      request(wv);
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        q[t].put(lane, lds_k);
        q_rope[t].put(lane, lds_r);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < KE; ++c) qf[t][c] = operand(c);
        __builtin_amdgcn_wave_barrier();
      }
      to_log2();
      for (int tile = wv; tile < tiles; tile += kWaves) {
        Tile tl;
        next_k.put(lane, lds_k);
        next_r.put(lane, lds_r);
        next_v.put_plain(lane, lds_v);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < KE; ++c) tl.k[c] = operand(c);
#pragma unroll
        for (int n = 0; n < NV; ++n)
#pragma unroll
          for (int v = 0; v < 4; ++v) tl.v[n][v] = lds_v[4 * g + v][16 * n + l16];
        __builtin_amdgcn_wave_barrier();
        if (tile + kWaves < tiles) request(tile + kWaves);
        multiply(tl, tile, []() {});
      }
    }
  } else if constexpr (AHEAD) {
    auto request = [&](Tile& t, int tile) {
      request_k(t, tile);
      request_v(t, tile);
    };
    auto nothing = [&]() {};
    if (wv < tiles) {
      Tile ta, tb;
      request(ta, wv);
      to_log2();
      for (int tile = wv;;) {
        const int second = tile + kWaves, third = tile + 2 * kWaves;
        request(tb, second < tiles ? second : tiles - 1);
        multiply(ta, tile, nothing);
        if (second >= tiles) break;
        request(ta, third < tiles ? third : tiles - 1);
        multiply(tb, second, nothing);
        if (third >= tiles) break;
        tile = third;
      }
    }
  } else {
    static_assert(RT == 1, "one block: its keys are multiplied once a tile");
    if (wv < tiles) {
      Tile tl;
      request_k(tl, wv);
      to_log2();
      for (int tile = wv; tile < tiles; tile += kWaves) {
        request_v(tl, tile);
        __builtin_amdgcn_sched_barrier(0);
        multiply(tl, tile, [&]() {
          __builtin_amdgcn_sched_barrier(0);
          request_k(tl, tile + kWaves < tiles ? tile + kWaves : tiles - 1);
          __builtin_amdgcn_sched_barrier(0);
        });
      }
    }
  }
  // ---- merge the wavefronts, 16 rows at a time
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    const float lt = col_sum(l[t]);
    if (g == 0) {
      s_m[wv][16 * t + l16] = m[t];
      s_l[wv][16 * t + l16] = lt;
    }
  }
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    if (m0[t] < 0) break;
    if (t) __syncthreads();
#pragma unroll
    for (int n = 0; n < NV; ++n) *reinterpret_cast<f32x4*>(&s_o[wv][l16][16 * n + 4 * g]) = acc[t][n];
    __syncthreads();
    for (int i = tid; i < 16 * DV / 4; i += kBlock) {
      const int qt = i / (DV / 4), q = 16 * t + qt, n = 4 * (i % (DV / 4));
      if (m0[t] + qt >= a.T) continue;
      float ms = s_m[0][q];  // a row's own column is always open, so the maximum over the wavefronts is finite
#pragma unroll
      for (int w = 1; w < kWaves; ++w) ms = fmaxf(ms, s_m[w][q]);
      float ls = 0.f;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const float f = __builtin_amdgcn_exp2f(s_m[w][q] - ms);
        ls += f * s_l[w][q];
        o += *reinterpret_cast<f32x4*>(&s_o[w][qt][n]) * f;
      }
      o *= 1.f / ls;
      if (m0[t] + qt >= len) o = f32x4{0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f32x4*>(out + (size_t)(m0[t] + qt) * out_pitch + n) = o;
    }
  }
}

template <int DH, int DR, int DV, int RT>
void launch_prefill_rows(const ExplicitArgs& a, int slices, hipStream_t st, const EventPair& ev) {
  const unsigned blocks = (a.T + 15) / 16;
  const dim3 grid(a.n_heads * slices, a.batch, (blocks + RT - 1) / RT);
  const size_t n = (size_t)grid.x * grid.y * grid.z;
  if constexpr (RT > 1) {
    if (n <= 256 && (a.T <= 32 || a.T > (long long)300 * a.stride)) launch_timed(prefill_f32_kernel<DH, DR, DV, RT, true, false>, grid, dim3(kBlock), 0, st, ev, a);
    else launch_timed(prefill_f32_kernel<DH, DR, DV, RT, true, true>, grid, dim3(kBlock), 0, st, ev, a);
  } else {
    if (n <= kAheadMost) launch_timed(prefill_f32_kernel<DH, DR, DV, RT, true, false>, grid, dim3(kBlock), 0, st, ev, a);
    else launch_timed(prefill_f32_kernel<DH, DR, DV, RT, false, false>, grid, dim3(kBlock), 0, st, ev, a);
  }
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
         a.batch <= 65535 && (size_t)a.batch * a.T <= 65535u;  // (the call refuses more rows of fp32 storage, as the interface states)
}

hipError_t launch_prefill_f32(const ExplicitArgs& args, hipStream_t st, const EventPair& ev) {
  ExplicitArgs a = args;
  a.n_slices = 0;
  // Rows of the product: blocks of their own for every sequence skip its padding and waste half a block at its end.  us of the call, 8
  // heads x 64, r = 256, a block's own / all rows as one: 600 sequences of 5 tokens 130 / 59, 90 of 33 54 / 41, 90 of up to 33 40 / 38, 60 of
  // up to 50 38.5 / 38.5, 46 of up to 64 33.8 / 36.4, 3 of 500 to 777 39.7 / 42.0.
  ExplicitArgs kv = a;
  if ((!a.seq_len || a.T <= 56) && (size_t)a.batch * a.T <= (size_t)65535 * kKvRows) {
    kv.T = a.batch * a.T;
    kv.batch = 1;
    kv.seq_len = nullptr;
  }
  // Of a ragged launch about half of the blocks are padding: kKvPad where the others are a round of four a unit.  Without / with it: 3
  // sequences of 500 to 777 tokens (1200 workgroups) 41.6 / 39.7, 15 of up to 200 (1680) 34.1 / 32.6, 30 of up to 100 (1920) 32.9 / 33.8, 4 of 100 to
  // 1024 (2048) 66.5 / 68.5.
  const dim3 kv_grid(2 * ((a.n_heads * a.d_head + kGT - 1) / kGT), kv.batch, (kv.T + kKvRows - 1) / kKvRows);
  const size_t pad = kv.seq_len && (size_t)kv_grid.x * kv_grid.y * kv_grid.z <= 1792 ? kKvPad : 0;
  hipLaunchKernelGGL(kv_f32_kernel, kv_grid, dim3(kBlock), pad, st, kv);
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
