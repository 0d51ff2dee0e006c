// Decode over short sequences (gfx950): attention, normalisation and the value up-projection of a sequence and a few of its
// heads in one workgroup, so that a step is two launches instead of three.
//
// Such a step is a chain of latencies: behind the front launch the split attention and the combine of its partials took
// 4.8 to 5.3 and 4.4 to 6.0 us at small batch, most of it the launch, the first loads and the last stores of each.  Where a
// workgroup can walk all of a sequence's slots in the time that saves, nothing has to be combined: it ends with its heads'
// latent outputs in LDS and multiplies them by W_V^(h).  A sequence's rows are then read once per workgroup instead of once, and
// W_V^(h) once per sequence: the limits below are where that costs what the launch saves.
#include <type_traits>

#include "append_step.h"
#include "bounds.h"
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------
// bf16 storage.  Every wavefront walks 16-slot tiles of its own (tile t belongs to wavefront t mod NW) with a softmax state of
// its own; the states meet once, behind the last tile.  No barrier stands in the walk.  Tiles come memory -> LDS in whole
// rows, one ahead of the one being multiplied (rows straight into the operand layout, 64 bytes of each of 16 rows a
// request, took twice as long), and the logits' layout [slot, column] is the K = 16 operand of the product with the latent
// rows as it stands.  One wavefront per SIMD issues a vector instruction every four cycles, so what is left of a tile is kept off
// the vector ALU: a load's address is a base for the wavefront and one clamped offset, an LDS address a register and
// a constant (the two places of a wavefront's tiles are two copies of the walk's body).
// A head takes two of the sixteen columns of a matrix operand: the even ones hold the hi plane and the odd ones the lo plane of
// the query, of the weights (which one plane would round to 8 bits) and of the latent output before W_V^(h), each at the
// price of one.  So HPW heads, up to eight, cost the walk what one does: a workgroup takes one where the workgroups
// find a compute unit each, and more where they would not.
// SH, PG: shared prefixes and paged storage, as in attn_mfma.hip.
// ---------------------------------------------------------------------------
constexpr int kWaves = kBlock / kWave;

template <int R, int DR, int HPW, int NW>
struct WholeGeom {
  static constexpr int tile = 16 * (R + DR) * 2;  // [latent rows][RoPE keys]
  static constexpr int query = (2 * HPW * (R + DR) * 2 + 1023) / 1024 * 1024;  // [plane][head][R + DR], whole requests
  static constexpr bool query_lds = R < 512;  // (its tiles fill the LDS)
  static constexpr int area = 2 * tile + (query_lds ? query : 0);  // a wavefront's two tiles, its copy of the query
  static constexpr int bytes = NW * area;
  // behind the walk an area holds its wavefront's sums, two planes a head, and (m, l); the first one also the planes of the result
  static constexpr int ml = 2 * HPW * R * 4, planes = ml + 64, plane = R * 2 + 64;
  static_assert(bytes <= 160 * 1024 && planes + 2 * HPW * plane <= 2 * tile && planes % 16 == 0 && 8 * HPW <= 64, "LDS of one compute unit");
  // register budget: 256 and fewer stay clear of copies to and from the accumulation registers
  static constexpr int per_simd = NW / 4 * (4 * NW * tile <= 160 * 1024 ? 2 : 1);
};

template <int R, int DR, int DH, int HPW, int NW, bool SH, bool PG>
__global__ __launch_bounds__(NW * kWave, (WholeGeom<R, DR, HPW, NW>::per_simd)) void attn_whole_kernel(WholeArgs w) {
  using G = WholeGeom<R, DR, HPW, NW>;
  constexpr int KC = R / 32, KT = (R + DR) / 32, MT = R / 16, OT = DH / 16, NT = OT < NW ? 1 : OT / NW;  // NT: output tiles of a wavefront, per head
  constexpr int PC = R / 8, RC = DR / 8;  // 16-byte pieces of a row
  static_assert(HPW <= 8, "two columns a head");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const AttnArgs& a = w.at;
  const int b = blockIdx.x, h0 = blockIdx.y * HPW;  // an XCD takes the heads of a few sequences and reads their rows once
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
  unsigned char* area = smem + wv * G::area;
  const uint32_t area0 = (uint32_t)(uintptr_t)(lds_byte_ptr)smem + (uint32_t)(wv * G::area);
  auto tile_base = [&](int k) { return 16 * (wv + NW * k); };
  // Byte offsets of the lane's 16-byte pieces in a tile of consecutive rows; piece j of row i sits at j ^ swizzle(i).
  uint32_t at_lat[R / 32], at_key[DR / 32];
#pragma unroll
  for (int c = 0; c < R / 32; ++c) {
    const int at = 64 * c + lane, i = at / PC;
    at_lat[c] = (uint32_t)(i * R * 2 + (((at % PC) ^ swz_rows16<PC>(i)) << 4));
  }
#pragma unroll
  for (int c = 0; c < DR / 32; ++c) {
    const int at = 64 * c + lane, i = at / RC;
    at_key[c] = (uint32_t)(i * DR * 2 + (((at % RC) ^ swz_rows16<RC>(i)) << 4));
  }
  // The wavefront's tile k on its way into place P: KT loads.  Slots past `last` become copies of that row's end: readable,
  // and their weights are zero.
  auto issue = [&](int k, int last, auto place) {
    constexpr int P = decltype(place)::value;
    const int base = tile_base(k);
    const uint32_t to = area0 + (uint32_t)(P * G::tile), to_key = to + (uint32_t)(16 * R * 2);
    if constexpr (SH) {
      auto one = [&](uint32_t off, const uint16_t* array, long long shared, int width, uint32_t at) {
        const int i = (int)off / (2 * width), slot = base + i < last ? base + i : last;
        load_to_lds_16(array + (size_t)slot * width + ((int)off - i * 2 * width) / 2 + (slot < sp.n ? shared : 0), at);
      };
#pragma unroll
      for (int c = 0; c < R / 32; ++c) one(at_lat[c], lat, sp.dlat, R, to + 1024u * c);
#pragma unroll
      for (int c = 0; c < DR / 32; ++c) one(at_key[c], key, sp.dkey, DR, to_key + 1024u * c);
    } else {
      const int s0 = base < last ? base : last;  // (only behind the last tile's)
      size_t row = (size_t)s0;
      if constexpr (PG) {  // a page holds whole 16-slot tiles
        int pg = load_uniform_i32(pt, s0 >> a.pages.shift);
        pg = pg < 0 ? 0 : (pg < a.pages.n_pages ? pg : a.pages.n_pages - 1);
        row = ((size_t)pg << a.pages.shift) + (size_t)(s0 & ((1 << a.pages.shift) - 1));
      }
      const uint32_t rows = (uint32_t)(last - s0 + 1);  // that may be read from there on
      const uint32_t end_lat = rows * (R * 2) - 16, end_key = rows * (DR * 2) - 16;
#pragma unroll
      for (int c = 0; c < R / 32; ++c) load_to_lds_16(lat + row * R, at_lat[c] < end_lat ? at_lat[c] : end_lat, to + 1024u * c);
#pragma unroll
      for (int c = 0; c < DR / 32; ++c) load_to_lds_16(key + row * DR, at_key[c] < end_key ? at_key[c] : end_key, to_key + 1024u * c);
    }
  };
  // Length (a scalar load), first rows and query are requested together, then the second rows and, where there are registers for
  // it during the walk, W_V^(h) (second rows behind W_V^(h): 16 sequences of 8 heads x 64, r = 256, 384 slots 11.1 -> 11.5 us a step).
  constexpr bool kEarly = 4 * (KT + MT + NT * KC) <= (G::per_simd > 1 ? 180 : 250);
  constexpr bool kNext = G::query_lds && kEarly;
  const auto place0 = std::integral_constant<int, 0>{};
  const auto place1 = std::integral_constant<int, 1>{};
  int len;  // nothing writes it while the kernel runs
  if constexpr (kNext) len = load_uniform_i32(a.seq_len, b);
  if (tile_base(0) < a.max_slots) issue(0, a.max_slots - 1, place0);
  if constexpr (!kNext) len = load_uniform_i32(a.seq_len, b);
  // Sixteen columns' fragments straight from memory are a full request for every 128 bytes of a head's query, as slow as the rows;
  // a copy in LDS is a request or two.
  u32x4_t q[KT];
  unsigned char* own_q = area + 2 * G::tile;
  if constexpr (G::query_lds) {
    constexpr int QP = HPW * (R + DR) / 8;  // 16-byte pieces of a plane
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.qcat) + ((size_t)b * a.n_heads + h0) * (R + DR);
    const int most = (a.n_heads - h0 < HPW ? a.n_heads - h0 : HPW) * ((R + DR) / 8) - 1;  // heads there are none of: copies
#pragma unroll
    for (int c = 0; c < G::query / 1024; ++c) {
      const int at = 64 * c + lane, i = at < QP ? at : at - QP;
      load_to_lds_16(qp + (at < QP ? 0 : a.q_plane) + 8 * (i < most ? i : most), area0 + (uint32_t)(2 * G::tile) + 1024u * c);
    }
  } else {
    const int h = h0 + (l16 >> 1) % HPW;
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.qcat) +
                         ((size_t)b * a.n_heads + (h < a.n_heads ? h : a.n_heads - 1)) * (R + DR) + 8 * g + ((l16 & 1) ? a.q_plane : 0);
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) q[kk] = *reinterpret_cast<const u32x4_t*>(qp + 32 * kk);
  }
  // W_V^(h) of this many heads is in registers or on its way: the first one's from the top, the others' from where the walk's sums
  // leave theirs.  Head after head through the same registers, the kernel ended in a trip to memory for each: us a step, before and
  // now, 8 heads x 64, r = 256, 250 slots: 64 sequences (two heads a workgroup) 11.5 / 10.8, 128 (four) 14.9 / 13.5; 8 heads x 128, r = 256,
  // 64 sequences 12.6 / 11.1.  (r = 512, whose registers are full of sums: one, 18.0 against 18.25 with two.)
  constexpr int HA0 = (G::per_simd > 1 ? 144 : 0) / (4 * NT * KC), HA = HA0 < 1 ? 1 : (HA0 < HPW ? HA0 : HPW);
  u32x4_t wf[HA][NT][KC];
  const int d0 = 16 * NT * wv;  // the wavefront's output columns
  // It comes with four neighbouring lanes to 64 bytes of a row and changes lanes behind the walk, in the last of the wavefront's area: in
  // the operand's layout, sixteen rows to sixteen lanes, a load is 66 cycles of the unit's address path, which the walk's rows wait for, this
  // one 24.  Where the walk fills that path or W_V^(h) is 64 KB; elsewhere the change costs more (us a step, operand's layout / changed: r = 256,
  // 8 heads x 64, 16 sequences of 528 slots, eight wavefronts 11.59 / 11.44; 16 x 128, 8 of 400, 12.47 / 12.02, 16 of 300 11.44 / 11.14; but 8 x 64 on four
  // wavefronts, 350 slots, 10.75 / 10.91, two heads a workgroup 10.46 / 10.94, r = 128 9.15 / 9.38, r = 512 17.8 / 18.1).
  constexpr bool kTurn = R == 256 && HPW == 1 && (NW == 8 || DH == 128);
  static_assert(!kTurn || G::planes + 2 * HPW * G::plane + KC * 1024 <= 2 * G::tile, "behind the sums and planes");
  const int w_row = kTurn ? lane >> 2 : l16, w_piece = kTurn ? lane & 3 : g;
  auto turn_w = [&](int hp) {
    if constexpr (kTurn) {
      int ln = lane;
      asm volatile("" : "+v"(ln));
      unsigned char* at = area + 2 * G::tile - KC * 1024;
#pragma unroll
      for (int i = 0; i < NT; ++i) {
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) *reinterpret_cast<u32x4_t*>(at + 1024 * kk + (ln >> 2) * 64 + (((ln & 3) ^ swz_rows16<4>(ln >> 2)) << 4)) = wf[hp % HA][i][kk];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) wf[hp % HA][i][kk] = *reinterpret_cast<const u32x4_t*>(at + 1024 * kk + (ln & 15) * 64 + (((ln >> 4) ^ swz_rows16<4>(ln & 15)) << 4));
        __builtin_amdgcn_wave_barrier();
      }
    }
  };
  auto load_w = [&](int hp) {
    const int h = h0 + hp;
    const uint16_t* wp = reinterpret_cast<const uint16_t*>(w.w_uv) + ((size_t)(h < a.n_heads ? h : a.n_heads - 1) * DH + d0 + w_row) * R + 8 * w_piece;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) wf[hp % HA][i][kk] = *reinterpret_cast<const u32x4_t*>(wp + 16 * i * R + 32 * kk);
  };
  const bool multiplies = OT >= NW || wv < OT;  // (a wavefront too many has no output columns)
  if (!kNext && kEarly && multiplies) load_w(0);
  const int live = live_slots(len, a.stride, a.max_slots), tiles = (live + 15) / 16;
  const int mine = tiles > wv ? (tiles - wv + NW - 1) / NW : 0;
  constexpr int W = kEarly ? NT * KC : 0;
  auto wait_but_w = [&](auto others) {  // and W_V^(h)
    if (multiplies) wait_loads_but<decltype(others)::value + W>();
    else wait_loads_but<decltype(others)::value>();
  };
  const auto none = std::integral_constant<int, 0>{};
  const auto one_tile = std::integral_constant<int, KT>{};
  if (kNext && mine > 1) issue(1, live - 1, place1);
  // Loads come back in the order they were asked for, 64 bytes a clock and unit.  With eight wavefronts the first head's W_V^(h) goes
  // out behind the third tile, if the wavefront has one (16 sequences of 8 heads x 64, r = 256, 512 slots 12.1, now 11.54 us a step;
  // 128 sequences, r = 128, 512 slots 12.1 and 11.1).  With four, one on a SIMD, it is too late there (r = 256, 350 slots 10.7 and 11.0).
  const bool late = kNext && NW == 8 && mine > 2;
  if (kNext && multiplies && !late) load_w(0);
  if (late) wait_loads_but<KT>();
  else if (kNext && mine > 1) wait_but_w(one_tile);
  else wait_but_w(none);
  if constexpr (G::query_lds) {
    const unsigned char* qp = own_q + ((l16 & 1) * HPW + (l16 >> 1) % HPW) * (R + DR) * 2 + 16 * g;
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) q[kk] = *reinterpret_cast<const u32x4_t*>(qp + 64 * kk);
  } else {
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) asm volatile("" : "+v"(q[kk]));  // (the compiler waits here, not behind the next tile's loads)
  }
  if (!kNext && mine > 1) issue(1, live - 1, place1);

  float m_ref = -INFINITY, l_run = 0.f;  // of the column's head; l_run: this lane's slots only
  float4_t acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) acc[mt] = float4_t{0.f, 0.f, 0.f, 0.f};

  const int vrow = 4 * g + (l16 >> 2);  // row of the lane's transposing reads
  auto step = [&](int k, auto place) {
    unsigned char* rows = area + decltype(place)::value * G::tile;
    const int base = tile_base(k);
    if (kNext && (k == 1 || (k == 2 && late))) {  // W_V^(h) and the tile behind it may travel on
      if (k + 1 < mine) wait_but_w(one_tile);
      else wait_but_w(none);
    } else if (k > 0) {
      if (k + 1 < mine) wait_loads_but<KT>();
      else wait_loads_but<0>();
    } else if (live < base + 16) {
      // rows of the first tile that no slot stands for may never have been written: zeros, or 0 x NaN would reach the sums
#pragma unroll
      for (int c = 0; c < R / 32; ++c) {
        const int at = 64 * c + lane;
        if (base + at / PC >= live) *reinterpret_cast<u32x4_t*>(rows + 16 * at) = u32x4_t{0u, 0u, 0u, 0u};
      }
    }
    float4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
    const unsigned char* xr = rows + l16 * R * 2;
    const unsigned char* kr = rows + 16 * R * 2 + l16 * DR * 2;
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) {
      const u32x4_t x = kk < KC ? *reinterpret_cast<const u32x4_t*>(xr + (((4 * kk + g) ^ swz_rows16<PC>(l16)) << 4))
                                : *reinterpret_cast<const u32x4_t*>(kr + (((4 * (kk - KC) + g) ^ swz_rows16<RC>(l16)) << 4));
      float4_t& s = (kk & 1) ? s1 : s0;
      s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x), __builtin_bit_cast(bf16x8_t, q[kk]), s, 0, 0, 0);
    }
    float sv[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float t = s0[v] + s1[v];
      // The planes' columns are neighbours.  At r = 512, whose sums are in the accumulation registers, a branch: as selects the walk lost, us a
      // step, select / branch: 12 heads x 128, 4 sequences of 345 slots 18.2 / 17.5, behind a shared prefix 20.8 / 18.8; 20 heads x 64, 4 of 336
      // 17.2 / 16.4 and 19.8 / 18.1; 16 heads x 128, 16 of 384 22.6 / 22.6.
      if constexpr (R == 512) {
        sv[v] = base + 4 * g + v < live ? t + row_permuted<0xb1>(t) : -INFINITY;
      } else {
        const float both = t + row_permuted<0xb1>(t);
        sv[v] = 4 * g + v < live - base ? both : -INFINITY;
      }
    }
    const float top = quarter_reduce(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])), LaneMax());
    constexpr float kRebase = 40.f;
    if (__any(top - m_ref > kRebase)) {  // true at the first tile (m_ref = -inf)
      // Selects, and nothing to scale at the first tile: as branches of the lanes these (and, below r = 512, the mask above) were part of every tile's
      // chain (r = 256, 8 heads x 64, 350 slots 11.05, now 10.74 us a step; r = 128, 600 slots 9.99 and 9.62).
      const bool moves = top - m_ref > kRebase;
      if (k > 0) {
        const float alpha = moves ? __builtin_amdgcn_exp2f(m_ref - top) : 1.f;
        l_run *= alpha;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] *= alpha;
      }
      m_ref = moves ? top : m_ref;
    }
    float pw[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) pw[v] = __builtin_amdgcn_exp2f(sv[v] - m_ref);
    l_run += (pw[0] + pw[1]) + (pw[2] + pw[3]);
    uint32_t hi01, lo01, hi23, lo23;  // hi plane in the even columns, lo plane in the odd ones
    split_bf16x2(pw[0], pw[1], hi01, lo01);
    split_bf16x2(pw[2], pw[3], hi23, lo23);
    const short4_t p = __builtin_bit_cast(short4_t, (l16 & 1) ? make_uint2(lo01, lo23) : make_uint2(hi01, hi23));
    const unsigned char* vr = rows + vrow * R * 2 + 8 * (l16 & 1);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const short4_t c = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_short4_ptr)(vr + (((2 * mt + ((l16 & 3) >> 1)) ^ swz_rows16<PC>(vrow)) << 4)));
      acc[mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(c, p, acc[mt], 0, 0, 0);
    }
    if (k + 2 < mine) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the tile has been read: its place takes the one after the next
      issue(k + 2, live - 1, place);
      if (late && k == 0 && multiplies) load_w(0);
    }
  };
  for (int k = 0; k < mine; k += 2) {
    step(k, place0);
    if (k + 1 < mine) step(k + 1, place1);
  }

  // ---- the wavefronts' states side by side, each in its area
  if (!kEarly && multiplies) load_w(0);
  const float l_own = quarter_reduce(l_run, LaneSum());
  if (l16 < 2 * HPW) {  // columns 16 mt + 4g .. + 3 of head l16 / 2, from one plane of the weights
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) *reinterpret_cast<float4_t*>(area + l16 * R * 4 + 4 * (16 * mt + 4 * g)) = acc[mt];
    if (g == 0 && !(l16 & 1)) *reinterpret_cast<float2*>(area + G::ml + 4 * l16) = make_float2(m_ref, l_own);
  }
  if (multiplies) {
#pragma unroll
    for (int hp = 1; hp < HA; ++hp) load_w(hp);
    if (kEarly) turn_w(0);  // (landed during the walk)
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < (HPW * R / 2 + (NW * kWave) - 1) / (NW * kWave); ++u) {  // two columns a thread
    const int at = tid + (NW * kWave) * u, hp = at / (R / 2), col = 2 * (at % (R / 2));
    if (hp >= HPW) break;
    const size_t oh = (size_t)b * a.n_heads + h0 + hp;
    float2 ml[NW];
    float ms = -INFINITY, l = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      ml[i] = *reinterpret_cast<const float2*>(smem + i * G::area + G::ml + 8 * hp);
      ms = fmaxf(ms, ml[i].x);
    }
    float2 o = make_float2(0.f, 0.f);
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const float f = live > 0 ? __builtin_amdgcn_exp2f(ml[i].x - ms) : 0.f;  // 0 for a wavefront without a tile
      const float2 x = *reinterpret_cast<const float2*>(smem + i * G::area + (2 * hp) * R * 4 + 4 * col);
      const float2 y = *reinterpret_cast<const float2*>(smem + i * G::area + (2 * hp + 1) * R * 4 + 4 * col);
      l += f * ml[i].y;
      o.x += f * (x.x + y.x);
      o.y += f * (x.y + y.y);
    }
    const float inv = live > 0 ? 1.f / l : 0.f;  // a sequence without a slot gives zeros
    o.x *= inv;
    o.y *= inv;
    if (h0 + hp < a.n_heads) {
      if (w.out_latent) *reinterpret_cast<float2*>(w.out_latent + oh * R + col) = o;
      if (w.lse && col == 0) w.lse[oh] = live > 0 ? (ms + log2f(l)) * 0.6931471805599453f : -INFINITY;
    }
    uint32_t hi, lo;
    split_bf16x2(o.x, o.y, hi, lo);
    *reinterpret_cast<uint32_t*>(smem + G::planes + 2 * hp * G::plane + 2 * col) = hi;
    *reinterpret_cast<uint32_t*>(smem + G::planes + (2 * hp + 1) * G::plane + 2 * col) = lo;
  }
  __syncthreads();
  if (!multiplies) return;
#pragma unroll
  for (int hp = 0; hp < HPW; ++hp) {
    float4_t o[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) o[i] = float4_t{0.f, 0.f, 0.f, 0.f};
    if (!kEarly || hp > 0) turn_w(hp);
    const unsigned char* pl = smem + G::planes + (2 * hp + (l16 & 1)) * G::plane + 16 * g;
#pragma unroll
    for (int kk = 0; kk < KC; ++kk) {
      const bf16x8_t p = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(pl + 64 * kk));
#pragma unroll
      for (int i = 0; i < NT; ++i) o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[hp % HA][i][kk]), p, o[i], 0, 0, 0);
    }
    if (hp + HA < HPW) load_w(hp + HA);
    if (h0 + hp >= a.n_heads) break;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
#pragma unroll
      for (int v = 0; v < 4; ++v) o[i][v] += row_permuted<0xb1>(o[i][v]);
      if (l16 == 0) *reinterpret_cast<float4_t*>(w.out + ((size_t)b * a.n_heads + h0 + hp) * DH + d0 + 16 * i + 4 * g) = o[i];
    }
  }
}

// ---------------------------------------------------------------------------
// fp32 storage, on the vector ALU: with one head the matrix instruction would work on sixteen copies of a column.  Eight lanes
// share a slot, each with every eighth 16-byte piece of its row (a request is 128 bytes of each of eight rows): the piece
// serves the logit and, weighted, the lane's sum of the latent columns, so a row is read once and never leaves its registers.
// 64 slots a step, two in every lane group.
// ---------------------------------------------------------------------------
constexpr int kStep = 16 * kWaves;  // slots of a step

// DH > 0: the whole step as one launch (heads of that width).  Every workgroup of a sequence forms the token's slot and its own head's
// query for itself, with the sums in the order of append_step_block and absorb_f32_block; nobody waits for anybody: the sequence's
// workgroups count themselves when they have read its state, and the last one writes it.
template <int R, int DR, int DH>
struct StepSharedF32 {
  float query[R + DR];         // the absorbed query
  float row[R + DR];           // the token's slot after it
  float append[256 + 12 + R];  // AppendStep's
  float q[DH];
  int32_t arrival;
};
struct NoShared {};

template <int R, int DR, int DH>
__global__ __launch_bounds__(kBlock, 1) void attn_whole_f32_kernel(std::conditional_t<DH == 0, WholeArgs, WholeStepArgs> w) {
  constexpr int E = R + DR, KC = R / 32, KE = E / 32;
  __shared__ __attribute__((aligned(16))) float sO[kWaves][R];
  __shared__ float sM[kWaves], sL[kWaves];
  const AttnArgs& a = w.at;
  const int b = blockIdx.x, h = blockIdx.y;  // an XCD takes the heads of a few sequences and reads their rows once
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int sl = lane >> 3, q8 = lane & 7;
  const float* lat = reinterpret_cast<const float*>(a.lat) + (size_t)b * a.max_slots * R + 4 * q8;
  const float* key = reinterpret_cast<const float*>(a.key) + (size_t)b * a.max_slots * DR + 4 * q8;
  __shared__ __attribute__((aligned(16))) std::conditional_t<DH == 0, NoShared, StepSharedF32<R, DR, DH == 0 ? 64 : DH>> sh;
  int len;
  if constexpr (DH == 0) len = a.seq_len[b];  // a scalar load, ahead of the rows: behind a vector one a step of two launches took 0.3 us more
  else len = *const_cast<const volatile int32_t*>(a.seq_len + b);  // read once: the step's last workgroup writes it
  int slot = -1;                                                  // that the step's token goes into, if it takes one
  float4_t x[2][KE], q[KE], wf[2][KC];
  AppendStep<float, R / 32> st;  // (DH > 0)
  constexpr int QN = DH == 0 ? 1 : R / 64, QK = DH == 0 ? 1 : DH / 16;
  float4_t wk[QN][QK], qs = {0.f, 0.f, 0.f, 0.f};
  float qr = 0.f;
  int arrival = 0;
  const int q4 = tid & 3;
  if constexpr (DH != 0) {  // four lanes share a column of the absorbed query, 64 columns at a time
    st.request(w.ap, b, tid);
#pragma unroll
    for (int u = 0; u < QN; ++u)
#pragma unroll
      for (int i = 0; i < QK; ++i)
        wk[u][i] = *reinterpret_cast<const float4_t*>(reinterpret_cast<const float*>(w.w_uk) + ((size_t)h * R + 64 * u + (tid >> 2)) * DH + 16 * i + 4 * q4);
    const size_t bh = (size_t)b * a.n_heads + h;
    if (tid < DH / 4) qs = *reinterpret_cast<const float4_t*>(reinterpret_cast<const float*>(w.q) + bh * DH + 4 * tid);
    if (tid < DR) qr = reinterpret_cast<const float*>(w.q_rope)[bh * DR + tid];
  }
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
  if constexpr (DH == 0) {
    const float* qp = reinterpret_cast<const float*>(a.qcat) + ((size_t)b * a.n_heads + h) * E + 4 * q8;
#pragma unroll
    for (int c = 0; c < KE; ++c) q[c] = *reinterpret_cast<const float4_t*>(qp + 32 * c);
  }
  // W_V^(h): eight lanes share an output column, 64 columns at a time
  const float* wp = reinterpret_cast<const float*>(w.w_uv) + ((size_t)h * w.d_head + (tid >> 3)) * R + 4 * q8;
  auto load_w = [&]() {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int c = 0; c < KC; ++c) wf[u][c] = *reinterpret_cast<const float4_t*>(wp + (size_t)32 * u * R + 32 * c);
  };
  // Loads come back in the order they were asked for, 64 bytes a clock: W_V^(h), needed last, is asked for behind the slot's row of G
  // (r = 128, 4 sequences of 600 slots 12.36, now 12.13 us a step), where it is 64 KB behind the merge weight (r = 256, 8 sequences
  // of 32 slots 9.42, now 9.32; at r = 64 the later place costs 0.1 us, the earlier one gains 0.03).
  constexpr bool kLate = R >= 256;
  if constexpr (DH == 0) load_w();
  if constexpr (DH != 0) {
    st.request_slot(w.ap, tid, len);
    if (!kLate) load_w();
    if (tid < DH / 4) *reinterpret_cast<float4_t*>(&sh.q[4 * tid]) = qs;
    if (tid < DR) sh.query[R + tid] = qr * w.scale_log2;
    const float wt = st.weight(w.ap, b, tid, sh.append);  // (barriers inside: sh.q is there behind it)
#pragma unroll
    for (int u = 0; u < QN; ++u) {  // as absorb_f32_block forms it
      float dot = 0.f;
#pragma unroll
      for (int i = 0; i < QK; ++i) {
        const float4_t y = *reinterpret_cast<const float4_t*>(&sh.q[16 * i + 4 * q4]);
        dot += wk[u][i][0] * y[0] + wk[u][i][1] * y[1] + wk[u][i][2] * y[2] + wk[u][i][3] * y[3];
      }
      dot = group_reduce<4>(dot, LaneSum());
      if (q4 == 0) sh.query[64 * u + (tid >> 2)] = dot * w.scale_log2;
    }
    if (append_status(len, 1, a.stride, a.max_slots) == 0) {
      slot = len / a.stride;
      const bool continuing = len != slot * a.stride;
#pragma unroll
      for (int i = 0; i < kMaxRPerThread; ++i) {
        const int e = tid + i * kBlock;
        if (e < R) sh.row[e] = (continuing ? st.told[i] : 0.f) + wt * st.cel[i];
      }
      if (tid < DR / 8) st.krv.store(&sh.row[R + 8 * tid]);
    }
    len += slot >= 0 ? 1 : 0;
    if (kLate) load_w();
    __syncthreads();
    // Behind here the workgroup reads no more of what the step changes (a row of the slot that is on its way is dropped).
    if (tid == kBlock - kWave) arrival = __hip_atomic_fetch_add(w.arrived + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int c = 0; c < KE; ++c) q[c] = *reinterpret_cast<const float4_t*>(&sh.query[4 * q8 + 32 * c]);
  }
  const int live = live_slots(len, a.stride, a.max_slots);
  // the last row that memory holds: not yet the token's slot, whose row comes out of LDS
  const int last = DH != 0 && slot > 0 ? slot - 1 : (live > 0 ? live - 1 : 0);

  float m = -INFINITY, l = 0.f;
  float4_t acc[KC];
#pragma unroll
  for (int c = 0; c < KC; ++c) acc[c] = float4_t{0.f, 0.f, 0.f, 0.f};
  auto step = [&](int s0) {
    float s[2];
    bool ok[2];
    if constexpr (DH != 0) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (s0 + 16 * wv + 8 * u + sl == slot) {
#pragma unroll
          for (int c = 0; c < KE; ++c) x[u][c] = *reinterpret_cast<const float4_t*>(&sh.row[4 * q8 + 32 * c]);
        }
    }
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
      load_rows(s0, last);
      step(s0);
    }
  }
  if constexpr (DH != 0) {
    if (tid == kBlock - kWave) sh.arrival = arrival;
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
  if constexpr (DH != 0) {
    if (sh.arrival == (int)gridDim.y - 1) {
      const AppendArgs& ap = w.ap;
      if (slot >= 0) {
        const size_t crow = (size_t)b * a.max_slots + slot;
        for (int e = tid; e < R; e += kBlock) {
          reinterpret_cast<float*>(ap.cache_c)[crow * R + e] = sh.row[e];
          if (ap.tail_c) ap.tail_c[(size_t)b * R + e] = sh.row[e];
        }
        if (tid < DR) reinterpret_cast<float*>(ap.cache_kr)[crow * DR + tid] = sh.row[R + tid];
        if (tid == 0) ap.seq_len[b] = len;
      } else if (tid == 0) {
        *ap.status = append_status(len, 1, a.stride, a.max_slots);
      }
      if (tid == 0) __hip_atomic_store(w.arrived + b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
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

template <int R, int DR, int DH, int HPW, int NW, bool SH, bool PG>
hipError_t launch_whole(const WholeArgs& w, hipStream_t st, const EventPair& ev) {
  constexpr size_t smem = WholeGeom<R, DR, HPW, NW>::bytes;
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&attn_whole_kernel<R, DR, DH, HPW, NW, SH, PG>, smem, lds_allowed);
  if (e != hipSuccess) return e;
  launch_timed(attn_whole_kernel<R, DR, DH, HPW, NW, SH, PG>, dim3(w.at.batch, (w.at.n_heads + HPW - 1) / HPW), dim3(NW * kWave),
               smem, st, ev, w);
  return hipGetLastError();
}

template <int R, int DR, int DH, int HPW, int NW>
hipError_t launch_form(const WholeArgs& w, hipStream_t st, const EventPair& ev) {
  if (w.at.pages.table) return w.at.prefix_owner ? hipErrorInvalidValue : launch_whole<R, DR, DH, HPW, NW, false, true>(w, st, ev);
  return w.at.prefix_owner ? launch_whole<R, DR, DH, HPW, NW, true, false>(w, st, ev) : launch_whole<R, DR, DH, HPW, NW, false, false>(w, st, ev);
}

template <int R, int DR, int DH, int NW>
hipError_t launch_heads(const WholeArgs& w, hipStream_t st, const EventPair& ev) {
  const size_t jobs = (size_t)w.at.n_heads * w.at.batch;
  return jobs <= 256   ? launch_form<R, DR, DH, 1, NW>(w, st, ev)
         : jobs <= 512 ? launch_form<R, DR, DH, 2, NW>(w, st, ev)
                       : launch_form<R, DR, DH, 4, NW>(w, st, ev);
}

}  // namespace

bool attn_whole_supported(const WholeArgs& w, int dtype) {
  const AttnArgs& a = w.at;
  const auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (!w.out || !w.w_uv || a.T != 0 || !al16(w.out) || !al16(w.out_latent) || !al16(w.w_uv)) return false;
  // Where this is the faster form, in (sequence, head) pairs and in slots a sequence may hold: a workgroup walks a whole sequence,
  // so the limits leave room for batches in which most are far shorter than the longest.  us a decode step, three
  // launches / two:
  //   fp32, 8 heads x 64, r = 256, 8 sequences: 64 slots 15.9 / 9.4, 512 18.2 / 17.0, 640 18.8 / 19.3
  //   fp32, 4 heads x 64, r = 64, 1 sequence: 128 slots 10.2 / 7.1, 768 12.2 / 11.2, 1024 12.7 / 12.8
  //   bf16, 8 heads x 64, r = 128, 16 sequences: 64 slots 11.1 / 7.0, 640 12.5 / 10.0; 128: 64 slots 11.2 / 9.1, 640 18.7 / 13.4;
  //     240 (480 workgroups of four heads): 64 slots 12.4 / 11.3, 256 19.0 / 14.1, 384 21.1 / 19.9; 16 heads, 240 sequences: 64 slots
  //     13.6 / 16.6
  //   bf16, 8 heads x 64, r = 256, 16 sequences: 64 slots 12.6 / 8.0, 256 13.1 / 10.0, 528 13.4 / 12.3, 640 13.4 / 13.1; 64: 64 slots
  //     13.1 / 9.5, 576 18.5 / 14.8; 128: 64 slots 13.8 / 12.4, 576 22.9 / 18.9; 20 heads, 64 sequences: 64 slots 16.1 / 16.2
  //   bf16, 8 heads x 128, r = 256, 16 sequences: 64 slots 13.8 / 8.5, 512 14.4 / 13.5; 64: 64 slots 14.5 / 11.3, 384 19.3 / 15.3; 128: 64
  //     slots 15.4 / 17
  //   bf16, 16 heads x 128, r = 512, 16 sequences: 64 slots 20.9 / 12.9, 384 23.0 / 20.0, 640 24.1 / 25.6; 32: 256 25.1 / 22.4; 48: 25.9 / 30.8
  const size_t jobs = (size_t)a.n_heads * a.batch;
  if (dtype == 0)  // fp32
    return (a.r == 64 || a.r == 128 || a.r == 256) && (a.d_rope == 32 || a.d_rope == 64) && w.d_head % 64 == 0 && jobs <= 512 &&
           a.max_slots <= (a.r == 256 ? 512 : 768);
  // (head shapes that are built; 64 with 64 and 128 with 32 are not, and have not been measured)
  const bool narrow = w.d_head == 64 && a.d_rope == 32, wide = w.d_head == 128 && a.d_rope == 64;
  if (!narrow && !wide) return false;
  if (a.r == 128 && jobs > 1024) return narrow && jobs <= 2048 && a.max_slots <= 320;  // (two workgroups a unit)
  if (a.r == 128) return a.max_slots <= (jobs <= 256 ? 768 : 640);
  if (a.r == 256 && narrow) return jobs <= 1024 && a.max_slots <= (jobs <= 256 ? 640 : 576);
  if (a.r == 256) return jobs <= 512 && a.max_slots <= (jobs > 256 ? 384 : 512);
  return a.r == 512 && jobs <= 512 && a.max_slots <= (jobs > 256 ? 256 : 384);
}

hipError_t launch_attn_whole(const WholeArgs& w, int dtype, hipStream_t st, const EventPair& ev) {
  const AttnArgs& a = w.at;
  if (dtype == 0) {
#define MTLA_CASE(RR, DD)                                                                                          \
  if (a.r == RR && a.d_rope == DD) {                                                                               \
    launch_timed(attn_whole_f32_kernel<RR, DD, 0>, dim3(a.batch, a.n_heads), dim3(kBlock), 0, st, ev, w);           \
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
  // Long: eight wavefronts, two per SIMD, hide more of a tile's chain than their meeting costs (16 sequences of 8 heads, us a step
  // with four / eight: r = 128: 128 slots 7.7 / 8.3, 512 10.5 / 10.0; r = 256: 384 slots 11.1 / 11.5, 528 12.9 / 12.3, where several
  // heads' queries leave no room for them; not built for 128-wide heads at r = 256)
  if (a.r == 128 && a.max_slots > 320) {
    if (a.d_rope == 32 && w.d_head == 64) return launch_heads<128, 32, 64, 8>(w, st, ev);
    if (a.d_rope == 64 && w.d_head == 128) return launch_heads<128, 64, 128, 8>(w, st, ev);
  }
  if (a.r == 256 && a.d_rope == 32 && w.d_head == 64 && a.max_slots > 448 && (size_t)a.n_heads * a.batch <= 256)
    return launch_form<256, 32, 64, 1, 8>(w, st, ev);
#define MTLA_CASE(RR, DD, HH) \
  if (a.r == RR && a.d_rope == DD && w.d_head == HH) return launch_heads<RR, DD, HH, 4>(w, st, ev);
  MTLA_CASE(128, 32, 64)
  MTLA_CASE(256, 32, 64)
  MTLA_CASE(512, 32, 64)
  MTLA_CASE(128, 64, 128)
  MTLA_CASE(256, 64, 128)
  MTLA_CASE(512, 64, 128)
#undef MTLA_CASE
  return hipErrorInvalidValue;
}

bool attn_step_supported(const WholeStepArgs& w, int dtype) {
  // fp32 storage.  Every workgroup reads the hyper-network and its head's W_K for itself, and a sequence's meet at its counter: one
  // launch loses where they are many, more so of many heads and wide weights.  us a replayed step of 24 / 200 slots, two launches -> one:
  //   4 heads x 64, r = 64, 8 sequences 6.6 -> 5.7 / 7.8 -> 6.9, 48: 6.7 -> 6.2 / 8.1 -> 7.5, 64: 6.8 -> 7.1 / 8.2 -> 8.6
  //   8 heads x 64, r = 256, 16: 9.3 -> 9.3 / 12.6 -> 12.2, 24: 9.3 -> 10.1 / 12.7 -> 13.2; r = 128, 24: 7.6 -> 7.8 / 9.5 -> 9.6
  //   32 heads x 64, r = 64, 3: 6.7 -> 6.5 / 8.0 -> 7.7, 4: 6.6 -> 6.7 / 8.0 -> 8.0, 8: 6.8 -> 8.2 / 8.1 -> 9.5
  //   32 heads x 128, r = 128, 2: 7.9 -> 7.9 / 9.5 -> 9.7, 3: 7.9 -> 8.3 / 9.5 -> 10.1
  //   8 heads x 128, r = 256, 1: 9.7 -> 10.3 / 12.8 -> 13.6; 32 heads, 8: 13.4 -> 17.9 / 16.9 -> 21.1 (not taken, not built)
  // As eager calls, where the host's part of two launches is what counts, one gains more (the first line 9.1 -> 6.4 / 9.0 -> 7.6).  In
  // bf16, 32 KB of the hyper-network and of W_K a workgroup, it was built and gains nothing: 16 sequences of 8 heads x 64, r = 256:
  // 150 slots 9.2 / 10.0, 528 12.2 / 12.6; r = 128: 20 slots 7.0 / 6.7, 200 8.3 / 8.6.
  const AttnArgs& a = w.at;
  const AppendArgs& ap = w.ap;
  const int weight = a.r * w.d_head;  // elements of a head's W_K
  const size_t most = a.n_heads <= 4 ? 192 : (a.n_heads <= 8 ? 128 : (weight <= 8192 ? 96 : 64));
  return dtype == 0 && attn_whole_supported(w, dtype) && (w.d_head == 64 || w.d_head == 128) && weight <= 16384 &&
         (size_t)a.n_heads * a.batch <= most && a.batch <= kStepArrivals && ap.tail_c && !ap.w_override && !ap.n_new && !ap.w_out && !ap.slot_out;
}

hipError_t launch_attn_step(const WholeStepArgs& w, hipStream_t st, const EventPair& ev) {
  const AttnArgs& a = w.at;
#define MTLA_CASE(RR, DD, HH)                                                                                      \
  if (a.r == RR && a.d_rope == DD && w.d_head == HH) {                                                             \
    launch_timed(attn_whole_f32_kernel<RR, DD, HH>, dim3(a.batch, a.n_heads), dim3(kBlock), 0, st, ev, w);          \
    return hipGetLastError();                                                                                      \
  }
  MTLA_CASE(64, 32, 64)
  MTLA_CASE(64, 64, 64)
  MTLA_CASE(128, 32, 64)
  MTLA_CASE(128, 64, 64)
  MTLA_CASE(256, 32, 64)
  MTLA_CASE(256, 64, 64)
  MTLA_CASE(64, 32, 128)
  MTLA_CASE(64, 64, 128)
  MTLA_CASE(128, 32, 128)
  MTLA_CASE(128, 64, 128)
#undef MTLA_CASE
  return hipErrorInvalidValue;
}

}  // namespace mtla
