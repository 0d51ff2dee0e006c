// Decode over few short sequences (gfx950): attention, normalisation and the value up-projection of one (sequence, head) in
// one workgroup, so that a step is two launches instead of three.
//
// A decode step at small batch is a chain of latencies: behind the front launch the split attention and the combine of its
// partials took 4.8 to 5.3 and 4.4 to 6.0 us, most of it the launch, the first loads and the last stores of each.  Where a
// sequence's slots are few enough for one workgroup to walk, nothing has to be combined: the workgroup ends with the head's
// latent output in LDS and multiplies it by its W_V^(h), requested when the kernel began.  A sequence's rows are then read
// once per head instead of once, and W_V^(h) once per sequence: the launcher's limits are where that costs what the launch
// saves.
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kWaves = kBlock / kWave;
constexpr int kStep = 16 * kWaves;  // slots of a step

// ---------------------------------------------------------------------------
// bf16 storage.  64 slots a step: a wavefront brings 16 rows, memory -> LDS in whole rows and up to two steps ahead, forms
// their logits, and then multiplies all 64 by a quarter of the latent columns (as attn_split_kernel does for 16
// heads).  With one head the sixteen columns of a matrix operand are free: the even ones hold the hi plane and the odd ones the
// lo plane of the query, of the weights (which one plane would round to 8 bits) and of the latent output before W_V^(h), each
// at the price of one.
// Rows straight into the operand layout, 64 bytes of each of 16 rows a request, took 1.1 us a step at r = 256, the
// workgroup's other work half of that.
// SH, PG: shared prefixes and paged storage, as in attn_mfma.hip.
// ---------------------------------------------------------------------------
template <int R, int DR>
struct WholeLds {
  static constexpr int rows = kStep * R * 2, step = rows + kStep * DR * 2;  // [latent rows][RoPE keys] of a step
  static constexpr int NB = R >= 512 ? 2 : 3;                               // steps
  static constexpr int weights = NB * step, stats = weights + kWaves * kWave * 8, bytes = stats + 2 * kWaves * 4;
  static_assert(bytes <= 160 * 1024 && R * 4 <= step, "LDS of one compute unit; the latent output takes a step's place");
};

template <int R, int DR, int DH, bool SH, bool PG>
__global__ __launch_bounds__(kBlock, R >= 512 ? 1 : 2) void attn_whole_kernel(WholeArgs w) {
  using L = WholeLds<R, DR>;
  constexpr int KC = R / 32, KT = (R + DR) / 32, MW = R / 16 / kWaves, NT = DH / 64, NB = L::NB;
  constexpr int PC = R / 8, RC = DR / 8;  // 16-byte pieces of a row
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  uint2* sP = reinterpret_cast<uint2*>(smem + L::weights);  // [wavefront][lane]: weights of slots 4g .. 4g + 3
  float* sM = reinterpret_cast<float*>(smem + L::stats);    // [wavefront]
  float* sL = sM + kWaves;
  float* sO = reinterpret_cast<float*>(smem);               // [R], behind the last step

  const AttnArgs& a = w.at;
  const int b = blockIdx.x, h = blockIdx.y;  // an XCD takes the heads of a few sequences and reads their rows once
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const uint16_t* lat = reinterpret_cast<const uint16_t*>(a.lat) + (PG ? 0 : (size_t)b * a.max_slots * R);
  const uint16_t* key = reinterpret_cast<const uint16_t*>(a.key) + (PG ? 0 : (size_t)b * a.max_slots * DR);
  const int32_t* pt = PG ? a.pages.table + (size_t)b * a.pages.max_pages : nullptr;
  SharedPrefix sp{0, 0, 0};
  if constexpr (SH) {
    int owner = a.prefix_owner[b], n = a.prefix_slots[b];
    owner = owner < 0 ? 0 : (owner < a.prefix_rows ? owner : a.prefix_rows - 1);
    sp.n = n < 0 ? 0 : (n < a.max_slots ? n : a.max_slots);
    sp.dlat = (long long)(owner - b) * a.max_slots * R;
    sp.dkey = (long long)(owner - b) * a.max_slots * DR;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_ptr)smem;
  // The wavefront's 16 rows of step t (slots past `last`: a readable duplicate) on their way into place t % NB: KT loads.
  // Piece j of row i sits at j ^ swizzle(i).
  auto issue = [&](int t, int last) {
    const int base = kStep * t + 16 * wv;
    const uint32_t to = lds0 + (uint32_t)(t % NB) * (uint32_t)L::step;
    size_t page = 0;
    if constexpr (PG) {
      const int s0 = base < last ? base : last;  // a page holds whole 16-slot tiles
      int pg = load_uniform_i32(pt, s0 >> a.pages.shift);
      pg = pg < 0 ? 0 : (pg < a.pages.n_pages ? pg : a.pages.n_pages - 1);
      page = (size_t)pg << a.pages.shift;
    }
    auto one = [&](int i, int place, const uint16_t* array, long long shared, int width, uint32_t at) {
      const int slot = base + i < last ? base + i : last;
      const size_t row = PG ? page + (size_t)(slot & ((1 << a.pages.shift) - 1)) : (size_t)slot;
      const uint16_t* src = array + row * width + 8 * place;
      if constexpr (SH) {
        if (slot < sp.n) src += shared;
      }
      load_to_lds_16(src, at);
    };
#pragma unroll
    for (int c = 0; c < R / 32; ++c) {
      const int at = 64 * c + lane, i = at / PC;
      one(i, (at % PC) ^ swz_rows16<PC>(i), lat, sp.dlat, R, to + (uint32_t)(16 * wv * R * 2 + 1024 * c));
    }
#pragma unroll
    for (int c = 0; c < DR / 32; ++c) {
      const int at = 64 * c + lane, i = at / RC;
      one(i, (at % RC) ^ swz_rows16<RC>(i), key, sp.dkey, DR, to + (uint32_t)(L::rows + 16 * wv * DR * 2 + 1024 * c));
    }
  };
  // first rows, length (a scalar load), query and W_V^(h) are requested together
  issue(0, a.max_slots - 1);
  const int len = load_uniform_i32(a.seq_len, b);  // nothing writes it while the kernel runs
  u32x4_t q[KT];
  {
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.qcat) + ((size_t)b * a.n_heads + h) * (R + DR) + 8 * g +
                         ((l16 & 1) ? a.q_plane : 0);
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) q[kk] = *reinterpret_cast<const u32x4_t*>(qp + 32 * kk);
  }
  u32x4_t wf[NT][KC];
  {
    const uint16_t* wp = reinterpret_cast<const uint16_t*>(w.w_uv) + ((size_t)h * DH + wv * (DH / kWaves) + l16) * R + 8 * g;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) wf[i][kk] = *reinterpret_cast<const u32x4_t*>(wp + 16 * i * R + 32 * kk);
  }
  const int live = (len + a.stride - 1) / a.stride, n_steps = (live + kStep - 1) / kStep;
  const size_t oh = (size_t)b * a.n_heads + h;
  wait_loads_but<NT * KC>();  // the first rows and the query: W_V^(h) may still travel
#pragma unroll
  for (int kk = 0; kk < KT; ++kk) asm volatile("" : "+v"(q[kk]));  // (and the compiler waits here, not behind the next step's loads)
  if (n_steps > 1) issue(1, live - 1);

  float m_ref = -INFINITY, l_run = 0.f;  // m_ref: the same in all wavefronts; l_run: this lane's slots only
  float4_t acc[MW];
#pragma unroll
  for (int mt = 0; mt < MW; ++mt) acc[mt] = float4_t{0.f, 0.f, 0.f, 0.f};

  for (int t = 0; t < n_steps; ++t) {
    unsigned char* rows = smem + (t % NB) * L::step;
    if (t > 0) {
      if (NB > 2 && t + 1 < n_steps) wait_loads_but<KT>();  // the step behind it may travel on
      else wait_loads_but<0>();
    } else if (live < kStep) {
      // rows of the first step that no slot stands for may never have been written: zeros, or 0 x NaN would reach the sums
#pragma unroll
      for (int c = 0; c < R / 32; ++c) {
        const int at = 64 * c + lane;
        if (16 * wv + at / PC >= live) *reinterpret_cast<u32x4_t*>(rows + 16 * wv * R * 2 + 16 * at) = u32x4_t{0u, 0u, 0u, 0u};
      }
    }
    const int base = kStep * t + 16 * wv;
    const unsigned char* xr = rows + (16 * wv + l16) * R * 2;
    const unsigned char* kr = rows + L::rows + (16 * wv + l16) * DR * 2;
    float4_t se = {0.f, 0.f, 0.f, 0.f}, so = se;
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) {
      const u32x4_t x = kk < KC ? *reinterpret_cast<const u32x4_t*>(xr + (((4 * kk + g) ^ swz_rows16<PC>(l16)) << 4))
                                : *reinterpret_cast<const u32x4_t*>(kr + (((4 * (kk - KC) + g) ^ swz_rows16<RC>(l16)) << 4));
      float4_t& s = (kk & 1) ? so : se;
      s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, q[kk]), s, 0, 0, 0);
    }
    float sv[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float s = se[v] + so[v];
      sv[v] = base + 4 * g + v < live ? s + row_permuted<0xb1>(s) : -INFINITY;  // the planes' columns are neighbours
    }
    const float mloc = quarter_reduce(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), LaneMax());
    if (lane == 0) sM[wv] = mloc;
    __syncthreads();  // the maxima are there, everyone's rows too, and nobody still reads those of the step before
    if (t + NB - 1 < n_steps && t + NB - 1 > 1) issue(t + NB - 1, live - 1);
    const float top = fmaxf(fmaxf(sM[0], sM[1]), fmaxf(sM[2], sM[3]));
    constexpr float kRebase = 40.f;
    if (top - m_ref > kRebase) {  // uniform; true at the first step (m_ref = -inf)
      const float alpha = __builtin_amdgcn_exp2f(m_ref - top);
      m_ref = top;
      l_run *= alpha;
#pragma unroll
      for (int mt = 0; mt < MW; ++mt) acc[mt] *= alpha;
    }
    float pw[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) pw[v] = __builtin_amdgcn_exp2f(sv[v] - m_ref);
    uint32_t hi01, lo01, hi23, lo23;  // hi plane in the even columns, lo plane in the odd ones
    split_bf16x2(pw[0], pw[1], hi01, lo01);
    split_bf16x2(pw[2], pw[3], hi23, lo23);
    sP[wv * kWave + lane] = (l16 & 1) ? make_uint2(lo01, lo23) : make_uint2(hi01, hi23);
    l_run += (pw[0] + pw[1]) + (pw[2] + pw[3]);
    if (t + 1 == n_steps) {  // last step: the wavefront's share of the normaliser
      const float l = quarter_reduce(l_run, LaneSum());
      if (lane == 0) sL[wv] = l;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the weights are written (loads of rows need not have landed here)
    barrier_only();
    const int vrow = 4 * g + (l16 >> 2);  // row of the lane's transposing reads in a 16-slot tile
#pragma unroll
    for (int k = 0; k < kWaves / 2; ++k) {
      const uint2 u0 = sP[(2 * k) * kWave + lane], u1 = sP[(2 * k + 1) * kWave + lane];
      const bf16x8_t pb = __builtin_bit_cast(bf16x8_t, u32x4_t{u0.x, u0.y, u1.x, u1.y});
      const unsigned char* vr = rows + (32 * k + vrow) * R * 2 + 8 * (l16 & 1);
#pragma unroll
      for (int mt = 0; mt < MW; ++mt) {
        const unsigned char* src = vr + ((((wv * (R / kWaves) + 16 * mt) / 8 + ((l16 & 3) >> 1)) ^ swz_rows16<PC>(vrow)) << 4);
        const short4_t c0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)src);
        const short4_t c1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(src + 16 * R * 2));
        const uint2 a0 = __builtin_bit_cast(uint2, c0), a1 = __builtin_bit_cast(uint2, c1);
        acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, u32x4_t{a0.x, a0.y, a1.x, a1.y}), pb,
                                                          acc[mt], 0, 0, 0);
      }
    }
  }
  __syncthreads();  // the rows have been read: sO takes their place

  const float l = live > 0 ? (sL[0] + sL[1]) + (sL[2] + sL[3]) : 0.f;
  const float inv = live > 0 ? 1.f / l : 0.f;  // a sequence without a slot gives zeros
#pragma unroll
  for (int mt = 0; mt < MW; ++mt) {
    float4_t o;  // columns 16 mt + 4g .. + 3 of the wavefront's quarter: the planes' columns are neighbours
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = (acc[mt][v] + row_permuted<0xb1>(acc[mt][v])) * inv;
    if (l16 == 0) {
      const int n = wv * (R / kWaves) + 16 * mt + 4 * g;
      *reinterpret_cast<float4_t*>(sO + n) = o;
      if (w.out_latent) *reinterpret_cast<float4_t*>(w.out_latent + oh * R + n) = o;
    }
  }
  if (w.lse && tid == 0) w.lse[oh] = live > 0 ? (m_ref + log2f(l)) * 0.6931471805599453f : -INFINITY;
  __syncthreads();
  float4_t o[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) o[i] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < KC; ++kk) {
    const float4_t lo4 = *reinterpret_cast<const float4_t*>(sO + 32 * kk + 8 * g), hi4 = *reinterpret_cast<const float4_t*>(sO + 32 * kk + 8 * g + 4);
    u32x4_t p;  // hi plane in the even columns, what it leaves of the value in the odd ones
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e0 = i < 2 ? lo4[2 * i] : hi4[2 * i - 4], e1 = i < 2 ? lo4[2 * i + 1] : hi4[2 * i - 3];
      uint32_t hi, lo;
      split_bf16x2(e0, e1, hi, lo);
      p[i] = (l16 & 1) ? lo : hi;
    }
#pragma unroll
    for (int i = 0; i < NT; ++i)
      o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[i][kk]), __builtin_bit_cast(bf16x8_t, p), o[i], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < NT; ++i) {
#pragma unroll
    for (int v = 0; v < 4; ++v) o[i][v] += row_permuted<0xb1>(o[i][v]);
    if (l16 == 0) *reinterpret_cast<float4_t*>(w.out + oh * DH + wv * (DH / kWaves) + 16 * i + 4 * g) = o[i];
  }
}

// ---------------------------------------------------------------------------
// fp32 storage, on the vector ALU: with one head the matrix instruction would work on sixteen copies of a column.  Eight lanes
// share a slot, each with every eighth 16-byte piece of its row (a request is 128 bytes of each of eight rows): the piece
// serves the logit and, weighted, the lane's sum of the latent columns, so a row is read once and never leaves its registers.
// 64 slots a step, two in every lane group.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float row_rotated(float v) {  // inside 16 lanes
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + CTRL, 0xf, 0xf, true));
}

template <int R, int DR>
__global__ __launch_bounds__(kBlock, 1) void attn_whole_f32_kernel(WholeArgs w) {
  constexpr int E = R + DR, KC = R / 32, KE = E / 32;
  __shared__ __attribute__((aligned(16))) float sO[kWaves][R];
  __shared__ float sM[kWaves], sL[kWaves];
  const AttnArgs& a = w.at;
  const int b = blockIdx.x, h = blockIdx.y;  // an XCD takes the heads of a few sequences and reads their rows once
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int sl = lane >> 3, q8 = lane & 7;
  const float* lat = reinterpret_cast<const float*>(a.lat) + (size_t)b * a.max_slots * R + 4 * q8;
  const float* key = reinterpret_cast<const float*>(a.key) + (size_t)b * a.max_slots * DR + 4 * q8;
  const int len = a.seq_len[b];
  float4_t x[2][KE], q[KE], wf[2][KC];
  auto load_rows = [&](int s0, int last) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int slot = s0 + 16 * wv + 8 * u + sl < last ? s0 + 16 * wv + 8 * u + sl : last;
#pragma unroll
      for (int c = 0; c < KE; ++c)
        x[u][c] = *reinterpret_cast<const float4_t*>(c < KC ? lat + (size_t)slot * R + 32 * c : key + (size_t)slot * DR + 32 * (c - KC));
    }
  };
  load_rows(0, a.max_slots - 1);
  const float* qp = reinterpret_cast<const float*>(a.qcat) + ((size_t)b * a.n_heads + h) * E + 4 * q8;
#pragma unroll
  for (int c = 0; c < KE; ++c) q[c] = *reinterpret_cast<const float4_t*>(qp + 32 * c);
  // W_V^(h): eight lanes share an output column, 64 columns at a time
  const float* wp = reinterpret_cast<const float*>(w.w_uv) + ((size_t)h * w.d_head + (tid >> 3)) * R + 4 * q8;
  auto load_w = [&]() {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int c = 0; c < KC; ++c) wf[u][c] = *reinterpret_cast<const float4_t*>(wp + (size_t)32 * u * R + 32 * c);
  };
  load_w();
  const int live = (len + a.stride - 1) / a.stride;

  float m = -INFINITY, l = 0.f;
  float4_t acc[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) acc[c] = float4_t{0.f, 0.f, 0.f, 0.f};
  auto step = [&](int s0) {
    float s[2];
    bool ok[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float4_t d4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < KE; ++c) d4 += x[u][c] * q[c];
      ok[u] = s0 + 16 * wv + 8 * u + sl < live;
      const float dot = group_reduce<8>((d4[0] + d4[1]) + (d4[2] + d4[3]), LaneSum());
      s[u] = ok[u] ? dot : -INFINITY;
    }
    const float mn = fmaxf(m, wave_max(fmaxf(s[0], s[1])));
    const float ref = mn == -INFINITY ? 0.f : mn;  // no live slot so far
    const float alpha = __builtin_amdgcn_exp2f(m - ref);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int c = 0; c < KC; ++c) acc[c] *= alpha;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float p = __builtin_amdgcn_exp2f(s[u] - ref);
      l += p;
#pragma unroll
      for (int c = 0; c < KC; ++c)  // (a slot past the end may hold anything: its row is dropped, not weighted)
        acc[c] += ok[u] ? x[u][c] * p : float4_t{0.f, 0.f, 0.f, 0.f};
    }
  };
  if (live > 0) {
    step(0);
    for (int s0 = kStep; s0 < live; s0 += kStep) {
      load_rows(s0, live - 1);
      step(s0);
    }
  }
  // over the wavefront's eight lane groups
  auto over_slots = [&](float v) {
    v += row_rotated<8>(v);
    return quarter_reduce(v, LaneSum());
  };
  l = over_slots(l);
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    float4_t t;
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = over_slots(acc[c][i]);
    if (lane < 8) *reinterpret_cast<float4_t*>(&sO[wv][32 * c + 4 * q8]) = t;
  }
  if (lane == 0) {
    sM[wv] = m;
    sL[wv] = l;
  }
  __syncthreads();
  const size_t oh = (size_t)b * a.n_heads + h;
  const float ms = fmaxf(fmaxf(sM[0], sM[1]), fmaxf(sM[2], sM[3]));
  float f[kWaves], ls = 0.f;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    f[i] = live > 0 ? __builtin_amdgcn_exp2f(sM[i] - ms) : 0.f;  // 0 for a wavefront without a slot
    ls += f[i] * sL[i];
  }
  const float inv = live > 0 ? 1.f / ls : 0.f;
  if (w.lse && tid == 0) w.lse[oh] = live > 0 ? (ms + log2f(ls)) * 0.6931471805599453f : -INFINITY;
  float4_t o[KC];  // the normalised latent output, this lane's pieces
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    o[c] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kWaves; ++i) o[c] += f[i] * *reinterpret_cast<const float4_t*>(&sO[i][32 * c + 4 * q8]);
    o[c] *= inv;
    if (w.out_latent && tid < 8) *reinterpret_cast<float4_t*>(w.out_latent + oh * R + 32 * c + 4 * q8) = o[c];
  }
  for (int d0 = 0; d0 < w.d_head; d0 += 64) {
    if (d0) {
      wp += (size_t)64 * R;
      load_w();
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float4_t d4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < KC; ++c) d4 += wf[u][c] * o[c];
      const float v = group_reduce<8>((d4[0] + d4[1]) + (d4[2] + d4[3]), LaneSum());
      if (q8 == 0) w.out[oh * w.d_head + d0 + 32 * u + (tid >> 3)] = v;
    }
  }
}

template <int R, int DR, int DH, bool SH, bool PG>
hipError_t launch_whole(const WholeArgs& w, hipStream_t st, const EventPair& ev) {
  constexpr size_t smem = WholeLds<R, DR>::bytes;
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&attn_whole_kernel<R, DR, DH, SH, PG>, smem, lds_allowed);
  if (e != hipSuccess) return e;
  launch_timed(attn_whole_kernel<R, DR, DH, SH, PG>, dim3(w.at.batch, w.at.n_heads), dim3(kBlock), smem, st, ev, w);
  return hipGetLastError();
}

template <int R, int DR, int DH>
hipError_t launch_form(const WholeArgs& w, hipStream_t st, const EventPair& ev) {
  if (w.at.pages.table) return w.at.prefix_owner ? hipErrorInvalidValue : launch_whole<R, DR, DH, false, true>(w, st, ev);
  return w.at.prefix_owner ? launch_whole<R, DR, DH, true, false>(w, st, ev) : launch_whole<R, DR, DH, false, false>(w, st, ev);
}

}  // namespace

bool attn_whole_supported(const WholeArgs& w, int dtype) {
  const AttnArgs& a = w.at;
  const auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (!w.out || !w.w_uv || a.T != 0 || a.n_persistent > 0 || !al16(w.out) || !al16(w.out_latent) || !al16(w.w_uv)) return false;
  // Where one workgroup per (sequence, head) is the faster form, in slots a sequence may hold.  A step of 64 slots costs it 0.5 us
  // (r = 64, fp32) to 2.0 (r = 512), what it saves are 3 to 6 us.  us a decode step, three launches / two:
  //   fp32, 8 heads x 64, r = 256, 8 sequences: 64 slots 15.9 / 9.4, 512 18.2 / 17.0, 640 18.8 / 19.3
  //   fp32, 4 heads x 64, r = 64, 1 sequence: 128 slots 10.2 / 7.1, 768 12.2 / 11.2, 1024 12.7 / 12.8
  //   bf16, 8 heads x 64, r = 256, 16 sequences: 64 slots 12.9 / 8.9, 256 13.1 / 11.9, 384 13.2 / 13.8
  //   bf16, 16 heads x 128, r = 512, 8 sequences: 64 slots 20.8 / 14.2, 256 21.5 / 20.6, 320 21.6 / 22.7
  // From 256 workgroups on a unit gets a second one, at once only at r = 128 (64 sequences of 8 heads: 64 slots 11.2 / 8.7, 256 11.7 /
  // 11.6) and in fp32; at r = 256 and 512 it waits for the first (15.5 / 15.7 at 64 slots, worse above).
  const size_t jobs = (size_t)a.n_heads * a.batch;
  if (dtype == 0)  // fp32
    return (a.r == 64 || a.r == 128 || a.r == 256) && (a.d_rope == 32 || a.d_rope == 64) && w.d_head % 64 == 0 && jobs <= 512 &&
           a.max_slots <= (a.r == 256 ? 512 : 768);
  const int most = a.r == 128 ? (jobs <= 256 ? 320 : 256) : 256;
  return (a.r == 128 || a.r == 256 || a.r == 512) && ((w.d_head == 64 && a.d_rope == 32) || (w.d_head == 128 && a.d_rope == 64)) &&
         jobs <= (a.r == 128 ? 512 : 256) && a.max_slots <= most;
}

hipError_t launch_attn_whole(const WholeArgs& w, int dtype, hipStream_t st, const EventPair& ev) {
  const AttnArgs& a = w.at;
  if (dtype == 0) {
#define MTLA_CASE(RR, DD)                                                                                          \
  if (a.r == RR && a.d_rope == DD) {                                                                               \
    launch_timed(attn_whole_f32_kernel<RR, DD>, dim3(a.batch, a.n_heads), dim3(kBlock), 0, st, ev, w);              \
    return hipGetLastError();                                                                                      \
  }
    MTLA_CASE(64, 32)
    MTLA_CASE(64, 64)
    MTLA_CASE(128, 32)
    MTLA_CASE(128, 64)
    MTLA_CASE(256, 32)
    MTLA_CASE(256, 64)
#undef MTLA_CASE
    return hipErrorInvalidValue;
  }
#define MTLA_CASE(RR, DD, HH) \
  if (a.r == RR && a.d_rope == DD && w.d_head == HH) return launch_form<RR, DD, HH>(w, st, ev);
  MTLA_CASE(128, 32, 64)
  MTLA_CASE(256, 32, 64)
  MTLA_CASE(512, 32, 64)
  MTLA_CASE(128, 64, 128)
  MTLA_CASE(256, 64, 128)
  MTLA_CASE(512, 64, 128)
#undef MTLA_CASE
  return hipErrorInvalidValue;
}

}  // namespace mtla
