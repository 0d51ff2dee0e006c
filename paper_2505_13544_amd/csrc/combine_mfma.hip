// Split combine + value up-projection on the matrix cores (bf16 storage, gfx950).
//
// Eq. (with-rope), last two steps: the partial (m, l, o~) triples of a row are merged with
// weights 2^(m_p - m*), divided by the merged normaliser, and every head's latent output is
// taken through its own W_V^(h):  out[row, h, :] = o~[row, h, :] W_V^(h).
// Heads do not share W_V^(h), rows do, so the up-projection is a dense contraction once 16 rows
// of one head are put side by side:
//     out^T[d, row] = W_V^(h)[d, :] . o~[row, :]^T          (M = d_h, N = 16 rows, K = r)
// A workgroup owns one head and a run of 16-row tiles.  Its W_V^(h) is brought into LDS at the top, by loads that take
// whole rows of it (straight into the A-operand layout of v_mfma_f32_16x16x32_bf16 a request touches 64 bytes of each of 16
// rows: 128 KB took 4 us that way, beside which everything else of the kernel waited), each wavefront the share of the d_h
// rows that it multiplies.  Per tile, 16 threads per row merge the row's partials (all
// requests of up to PB pieces go out together, before the normaliser is known), write the
// normalised latent row where the caller wants it, and park it in LDS as two bf16 planes
// (hi + lo, an almost-fp32 value) that the wavefronts read back as the B operand.
// At r = 512, d_h = 128: 256 sequences, 16 heads 9.4 us, now 8.8; 1000 sequences 29.3, now 24.5; 8 sequences of 33 pieces,
// 32 heads 9.1, now 7.0.  There the 128 KB leave a unit one workgroup: with eight wavefronts, two a SIMD, to cover each other's waits, and fewer
// products one behind the other, a step of 256 sequences of 512 to 4096 slots' tokens, 16 heads, took 85.3 us, now 84.1; 200 of 300, 33.8, now 32.7; 8 heads,
// 128 of 2000, 43.3, now 42.2; 8 of 32768, s = 4, 32 heads, 37.1, now 36.2.
#include "bounds.h"
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

constexpr int kTileRows = 16;

struct Pieces {
  int first, count;
};

// Balanced schedule: workgroup i emitted piece i + row for its share of the row, whose work units are
// [p0, p1) of `total`.
__device__ __forceinline__ Pieces pieces_balanced(const CombineArgs& a, int row, int rows, int p0, int p1, int total) {
  Pieces p{0, 0};
  if (row >= rows || p1 == p0) return p;
  const int share = (total + a.n_persistent - 1) / a.n_persistent;
  const int first = (p0 + a.run_cost) / share, last = (p1 - 1) / share;  // the row's tiles follow its fixed units
  p.first = first + row;
  p.count = last - first + 1;
  return p;
}

// Which partials belong to `row` (see the two attention schedules): none for a row without a
// live column.
__device__ __forceinline__ Pieces pieces_of_row(const CombineArgs& a, int row, int rows, int total) {
  Pieces p{0, 0};
  if (a.n_persistent > 0) {  // balanced: workgroup i emitted piece i + row for its share of the row
    // the row's two counts are requested together, before anything is decided; `total` (the last entry
    // of the list) was read once when the kernel started: one round trip per row, not three
    const int rc = row < rows ? row : rows - 1;
    const int p0 = a.tile_prefix[rc], p1 = a.tile_prefix[rc + 1];
    return pieces_balanced(a, row, rows, p0, p1, total);
  } else {
    if (row >= rows) return p;  // static: chunk c of row b is piece b * n_splits + c
    int live;
    if (a.T == 0) {
      live = live_slots(a.seq_len[row], a.stride, a.max_slots);
    } else {
      const int b = row / a.T, m = row - b * a.T;
      const int len = a.seq_len ? a.seq_len[b] : a.T;
      live = m < len ? m / a.stride + 1 : 0;
    }
    p.first = row * a.n_splits;
    p.count = (live + a.chunk - 1) / a.chunk;
  }
  return p;
}

// grid = (runs of row tiles, n_heads)
// RPT = rows a workgroup really fills of each 16-row tile.  16 is the dense case; 4 is for small
// batches (decode), where the merge of the partials is the long part and wants more workgroups:
// a row is then merged by a whole wavefront and the tile's other columns are copies nobody stores.
// PF16 = the partials are normalised IEEE-half rows (o_p / l_p) from the column-split decode kernel:
// a piece then weighs l_p 2^(m_p - m*) instead of 2^(m_p - m*).
// PS = few rows, their pieces split over the wavefronts (at r = 128 and 64 over halves and quarters of them: a lane takes four
// columns): one row per workgroup (RPT = 1), the weighted sums added through LDS.  One round of requests instead of one per PB pieces, and four times the
// workgroups, each wavefront with its share of the partials to bring in and to add up.
// HF = the head is the fast grid index: the workgroups that share an XCD (and its L2) then share the
// W_V^(h) of a few heads instead of each XCD fetching all of them.
// NW = wavefronts: eight where the weights leave a unit one workgroup (four rows a workgroup are merged by a wavefront each).
template <int R, int DH, int RPT, bool PS>
struct CombineLds {  // [W_V^(h)][hi and lo planes of the rows][piece split: the other groups' sums]
  static constexpr int NW = R == 512 && DH == 128 && (PS || RPT == 16) ? 8 : 4, threads = NW * kWave;
  static constexpr int TPR = !PS ? threads / RPT : (R / 4 < kWave ? R / 4 : kWave), groups = PS ? threads / TPR : 1;  // threads merging one row
  static constexpr int planes = DH * R * 2, red = planes + 2 * RPT * R * 2, bytes = red + (groups - 1) * R * 4;
  static_assert(bytes <= 160 * 1024, "LDS of one compute unit");
};

template <int R, int DH, int RPT, bool PF16, bool PS = false, bool HF = PS>
__global__ __launch_bounds__((CombineLds<R, DH, RPT, PS>::threads)) void combine_mfma_kernel(CombineArgs a, int tiles_per_wg) {
  static_assert(!PS || RPT == 1, "piece split: one row per workgroup");
  using L = CombineLds<R, DH, RPT, PS>;
  constexpr int KK = R / 32;         // K steps
  constexpr int DW = DH / L::NW, NT = DW / 16;  // output dims of a wavefront, 16-row tiles
  constexpr int TPR = L::TPR;        // threads merging one row (piece split: a group of NG)
  constexpr int NG = L::groups;
  constexpr int CJ = R / (4 * TPR);  // float4 pieces of a latent row per thread
  static_assert(CJ >= 1, "a thread merges at least one float4 of its row");
  constexpr int PC = R / 8;          // 16-byte pieces of a row
  // partials requested together per thread: what 128 registers hold, at most 16 (12 with the pieces split: 48 a row; in the
  // dense case, whose rows have a few, 4 or 8: requests beyond a row's pieces are reloads, but not free)
  constexpr int kFit = 128 / (CJ * (PF16 ? 2 : 4)), kMost = PS ? 48 / L::NW : (RPT < kTileRows ? 16 : (R >= 512 ? 4 : 8));
  constexpr int PB = kFit < kMost ? kFit : kMost;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  // rows in LDS: piece p of row i at place p ^ swz(i), so that 16 rows' reads of one piece spread over the banks
  uint16_t* sA = reinterpret_cast<uint16_t*>(smem + L::planes);  // [plane][RPT][R]
  float* sRed = reinterpret_cast<float*>(smem + L::red);         // [NG - 1][R]

  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int h = HF ? blockIdx.x : blockIdx.y;
  const int rows = a.T ? a.batch * a.T : a.batch;
  const int n_tiles = (rows + RPT - 1) / RPT;
  const int t0 = (HF ? blockIdx.y : blockIdx.x) * tiles_per_wg;
  const int t1 = t0 + tiles_per_wg < n_tiles ? t0 + tiles_per_wg : n_tiles;

  // balanced schedule, first tile: a row's counts and the list's total go out together and before the
  // weights (loads return in order, and one count asked for after the other would be a round trip each)
  const int tid0 = threadIdx.x;
  int ps_p0 = 0, ps_p1 = 0, ps_total = 0;
  if ((PS || HF) && a.n_persistent > 0) {
    const int row0 = PS ? t0 : RPT * t0 + tid0 / TPR;
    const int rc = row0 < rows ? row0 : rows - 1;
    ps_p0 = a.tile_prefix[rc];
    ps_p1 = a.tile_prefix[rc + 1];
    ps_total = a.tile_prefix[a.batch];
  }

  // this wavefront's d_h / 4 rows of W_V^(h), 1 KB per request
  if (a.out) {
    typedef const __attribute__((address_space(1))) void* global_ptr;
    typedef __attribute__((address_space(3))) void* lds_ptr;
    constexpr int kBytes = DW * R * 2;
    const int uw = __builtin_amdgcn_readfirstlane(wv);
    const uint16_t* wsrc = reinterpret_cast<const uint16_t*>(a.w_uv) + ((size_t)h * DH + uw * DW) * R;
#pragma unroll
    for (int i = 0; i < kBytes / 1024; ++i) {
      const int at = 64 * i + lane, row = at / PC;
      __builtin_amdgcn_global_load_lds((global_ptr)(wsrc + row * R + 8 * ((at % PC) ^ swz_rows16<PC>(row))),
                                       (lds_ptr)(smem + uw * kBytes + 1024 * i), 16, 0, 0);
    }
  }

  const int total_tiles = (PS || HF) ? ps_total : (a.n_persistent > 0 ? a.tile_prefix[a.batch] : 0);
  const int rr = PS ? 0 : tid / TPR, sub = tid % TPR;  // merge phase: TPR threads per row
  const int grp = PS ? tid / TPR : 0;                  // ... or, of one row, NG groups of as many
  for (int t = t0; t < t1; ++t) {
    const int row = RPT * t + rr;
    // static schedule: piece ids row*n_splits + 0 .. n_splits-1 are readable whatever the row's
    // length turns out to be, so the requests below do not wait for it
    const bool fixed_ids = a.n_persistent == 0;
    const Pieces pc = ((PS || HF) && a.n_persistent > 0 && t == t0) ? pieces_balanced(a, row, rows, ps_p0, ps_p1, ps_total)
                                                                     : pieces_of_row(a, row, rows, total_tiles);
    const int row_c = row < rows ? row : rows - 1;
    const size_t pb = (size_t)(fixed_ids ? row_c * a.n_splits : pc.first) * a.n_heads + h;  // + p * n_heads
    const int p_last = fixed_ids ? a.n_splits - 1 : (pc.count > 0 ? pc.count - 1 : 0);
    // piece split: a group's share of the row's pieces where the count came first, else (requests do not wait for the count) every
    // NG-th from its own number on
    const int pq = (pc.count + NG - 1) / NG, pw0 = fixed_ids ? grp : grp * pq, ps = fixed_ids ? NG : 1;
    const int cnt = !PS ? pc.count : (fixed_ids ? (pc.count - grp + NG - 1) / NG : (pc.count - pw0 < pq ? pc.count - pw0 : pq));

    // ---- first PB pieces: requested before anything is known about m* (any piece id that can
    // come out of pieces_of_row is readable workspace)
    float2 mp[PB];  // (m_p, l_p)
    typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
    float4_t v[PF16 ? 1 : PB][PF16 ? 1 : CJ];   // fp32 partials as loaded
    u32x2_t vh[PF16 ? PB : 1][PF16 ? CJ : 1];   // half partials stay packed until they are used
    auto request = [&](int p0) {
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        const int p = PS ? pw0 + ps * (p0 + i) : p0 + i;
        const size_t pi = pb + (size_t)(p < p_last ? p : p_last) * a.n_heads;
        mp[i] = *reinterpret_cast<const float2*>(a.part_ml + pi * 2);
#pragma unroll
        for (int j = 0; j < CJ; ++j) {
          if (PF16)
            vh[PF16 ? i : 0][PF16 ? j : 0] = *reinterpret_cast<const u32x2_t*>(
                reinterpret_cast<const uint16_t*>(a.part_o) + pi * R + 4 * sub + 4 * TPR * j);
          else
            v[PF16 ? 0 : i][PF16 ? 0 : j] = *reinterpret_cast<const float4_t*>(a.part_o + pi * R + 4 * sub + 4 * TPR * j);
        }
      }
    };
    request(0);

    // ---- m* = max_p m_p,  l* = sum_p l_p 2^(m_p - m*): piece p is looked at by thread p mod TPR
    float2 ml0 = *reinterpret_cast<const float2*>(a.part_ml + (pb + (size_t)(sub < p_last ? sub : p_last) * a.n_heads) * 2);
    if (sub >= pc.count) ml0 = make_float2(-INFINITY, 0.f);
    float mloc = ml0.x;
    for (int p = sub + TPR; p < pc.count; p += TPR) mloc = fmaxf(mloc, a.part_ml[(pb + (size_t)p * a.n_heads) * 2]);
    const float mstar = group_reduce<TPR>(mloc, LaneMax());
    float lloc = sub < pc.count ? __builtin_amdgcn_exp2f(ml0.x - mstar) * ml0.y : 0.f;
    for (int p = sub + TPR; p < pc.count; p += TPR) {
      const float2 ml = *reinterpret_cast<const float2*>(a.part_ml + (pb + (size_t)p * a.n_heads) * 2);
      lloc += __builtin_amdgcn_exp2f(ml.x - mstar) * ml.y;
    }
    const float lstar = group_reduce<TPR>(lloc, LaneSum());

    // ---- o~ = sum_p 2^(m_p - m*) o_p / l*
    float4_t acc[CJ];
#pragma unroll
    for (int j = 0; j < CJ; ++j) acc[j] = float4_t{0.f, 0.f, 0.f, 0.f};
    for (int p0 = 0; p0 < cnt; p0 += PB) {
      if (p0 > 0) request(p0);
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        if (p0 + i < cnt) {  // a piece beyond the row's own may hold anything: never touched
          const float f = __builtin_amdgcn_exp2f(mp[i].x - mstar) * (PF16 ? mp[i].y : 1.f);
#pragma unroll
          for (int j = 0; j < CJ; ++j) {
            if (PF16) {
              const u32x2_t hv = vh[PF16 ? i : 0][PF16 ? j : 0];
              acc[j] += f * float4_t{f16_lo_to_f32(hv[0]), f16_hi_to_f32(hv[0]), f16_lo_to_f32(hv[1]), f16_hi_to_f32(hv[1])};
            } else {
              acc[j] += f * v[PF16 ? 0 : i][PF16 ? 0 : j];
            }
          }
        }
      }
    }
    if constexpr (PS) {  // group 0 adds the other sums to its own
      if (grp > 0) {
#pragma unroll
        for (int j = 0; j < CJ; ++j) *reinterpret_cast<float4_t*>(sRed + (grp - 1) * R + 4 * sub + 4 * TPR * j) = acc[j];
      }
      __syncthreads();
      if (grp == 0) {
#pragma unroll
        for (int w = 0; w < NG - 1; ++w)
#pragma unroll
          for (int j = 0; j < CJ; ++j) acc[j] += *reinterpret_cast<const float4_t*>(sRed + w * R + 4 * sub + 4 * TPR * j);
      }
    }
    const float inv = pc.count > 0 ? 1.f / lstar : 0.f;  // a row with no live column gives zeros
#pragma unroll
    for (int j = 0; j < CJ; ++j) acc[j] *= inv;
    if (row < rows && (!PS || grp == 0)) {
      const size_t oh = (size_t)row * a.n_heads + h;
      if (a.out_latent) {
#pragma unroll
        for (int j = 0; j < CJ; ++j)
          *reinterpret_cast<float4_t*>(a.out_latent + oh * R + 4 * sub + 4 * TPR * j) = acc[j];
      }
      if (a.lse && sub == 0) a.lse[oh] = pc.count > 0 ? (mstar + log2f(lstar)) * 0.6931471805599453f : -INFINITY;
    }
    if (!a.out) continue;

    // ---- park the row as hi + lo bf16 planes
    if (!PS || grp == 0) {
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        const uint32_t h01 = pack_bf16x2(acc[j][0], acc[j][1]), h23 = pack_bf16x2(acc[j][2], acc[j][3]);
        const uint32_t l01 = pack_bf16x2(acc[j][0] - __uint_as_float(h01 << 16), acc[j][1] - __uint_as_float(h01 & 0xffff0000u));
        const uint32_t l23 = pack_bf16x2(acc[j][2] - __uint_as_float(h23 << 16), acc[j][3] - __uint_as_float(h23 & 0xffff0000u));
        const int e = 4 * sub + 4 * TPR * j;
        uint16_t* dst = sA + rr * R + 8 * ((e >> 3) ^ swz_rows16<PC>(rr)) + (e & 7);
        *reinterpret_cast<uint2*>(dst) = make_uint2(h01, h23);
        *reinterpret_cast<uint2*>(dst + RPT * R) = make_uint2(l01, l23);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the weights have landed
    __syncthreads();

    // ---- out^T[d, row] for this wavefront's output dims
    float4_t o[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) o[nt] = float4_t{0.f, 0.f, 0.f, 0.f};
    const uint16_t* wrow = reinterpret_cast<const uint16_t*>(smem) + (wv * DW + l16) * R;  // (16 rows on, the same swizzle)
    if constexpr (RPT <= 8) {  // the hi planes in columns 0 to 7, the lo planes in the others: one product, half the reads
      const int rb = l16 % RPT;
      const uint16_t* brow = sA + rb * R + (l16 >> 3) * RPT * R;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8_t b = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(brow + 8 * ((4 * kk + g) ^ swz_rows16<PC>(rb))));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x8_t wa = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(wrow + 16 * nt * R + 8 * ((4 * kk + g) ^ swz_rows16<PC>(l16))));
          o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, b, o[nt], 0, 0, 0);
        }
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[nt][v] += row_rotated<8>(o[nt][v]);
    } else {
      const uint16_t* brow = sA + l16 * R;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const int at = 8 * ((4 * kk + g) ^ swz_rows16<PC>(l16));
        const bf16x8_t bh = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(brow + at));
        const bf16x8_t bl = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(brow + RPT * R + at));
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x8_t wa = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(wrow + 16 * nt * R + at));
          o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, bh, o[nt], 0, 0, 0);
          o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, bl, o[nt], 0, 0, 0);
        }
      }
    }
    // lane holds row l16 of the tile, output dims wv * DW + 16nt + 4g .. +3
    const int orow = RPT * t + l16;
    if (l16 < RPT && orow < rows) {
      float* dst = a.out + ((size_t)orow * a.n_heads + h) * DH + wv * DW + 4 * g;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<float4_t*>(dst + 16 * nt) = o[nt];
    }
    __syncthreads();  // the planes are rewritten by the next tile
  }
}

template <int R, int DH, int RPT, bool PF16, bool PS = false, bool HF = PS>
hipError_t launch_one(const CombineArgs& a, const dim3& grid, int tiles_per_wg, hipStream_t st) {
  constexpr int smem = CombineLds<R, DH, RPT, PS>::bytes;
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&combine_mfma_kernel<R, DH, RPT, PF16, PS, HF>, smem, lds_allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((combine_mfma_kernel<R, DH, RPT, PF16, PS, HF>), grid, dim3(CombineLds<R, DH, RPT, PS>::threads), smem, st, a, tiles_per_wg);
  return hipGetLastError();
}

template <int R, int DH, bool PF16>
hipError_t launch_rdh_pf(const CombineArgs& a, hipStream_t st) {
  const int rows = a.T ? a.batch * a.T : a.batch;
  // a handful of rows of eight or more pieces each (balanced: at most n_persistent + rows pieces exist): one row per
  // workgroup, its pieces split over the wavefronts
  if (PF16 && a.n_persistent > 0 && rows <= 16 && a.n_persistent + rows >= 8 * rows)
    return launch_one<R, DH, 1, PF16, true>(a, dim3(a.n_heads, rows), 1, st);
  // a small decode step, at most one (row, head) per compute unit, where a row is long (r = 512) or its pieces are more
  // than one round of requests: likewise.  With four rows per workgroup 4 sequences of 32 pieces, 16 heads, r = 512 took
  // 10.5 us on 16 workgroups, in this form 7.8, with the weights through LDS 6.0.  (16 sequences of 10 pieces, 8 heads, r = 256: 4.4 us either way; beyond a
  // row and head per unit every row's own copy of W_V^(h) costs more than the merge gains.)  Narrow latents have sixteen rows a
  // workgroup else: us a step, 8 heads x 64, r = 128: 1 sequence of 16 pieces 11.1 / 10.7, 1 of 96 28.3 / 21.1, 4 of 141 30.0 / 17.0; 16 heads, 16
  // of 24 16.9 / 13.0; r = 64: 1 of 63 16.2 / 10.9, but 4 of 16 10.4 / 10.6.
  if (!PF16 && a.n_persistent == 0 && a.T == 0 && rows * a.n_heads <= 256 && (R == 512 || a.n_splits > (R == 128 ? 8 : 16)))
    return launch_one<R, DH, 1, PF16, true>(a, dim3(a.n_heads, rows), 1, st);
  if constexpr (R >= 256) {
    if (rows <= 64)  // small batch: four rows per workgroup, one wavefront merging each
      return launch_one<R, DH, 4, PF16>(a, dim3((rows + 3) / 4, a.n_heads), 1, st);
  }
  const int n_tiles = (rows + kTileRows - 1) / kTileRows;
  // long runs amortise the W_V^(h) fetch; short ones keep every compute unit busy
  long long tpw = (long long)n_tiles * a.n_heads / 2048;
  tpw = tpw < 1 ? 1 : (tpw > 8 ? 8 : tpw);
  const dim3 grid((n_tiles + (int)tpw - 1) / (int)tpw, a.n_heads);
  if constexpr (PF16) {
    // decode over many rows, balanced schedule (a few half-size partials per row): heads as the fast grid index
    if (tpw == 1 && a.T == 0 && a.n_persistent > 0)
      return launch_one<R, DH, kTileRows, true, false, true>(a, dim3(a.n_heads, grid.x), 1, st);
  }
  return launch_one<R, DH, kTileRows, PF16>(a, grid, (int)tpw, st);
}

template <int R, int DH>
hipError_t launch_rdh(const CombineArgs& a, hipStream_t st) {
  return a.part_f16 ? launch_rdh_pf<R, DH, true>(a, st) : launch_rdh_pf<R, DH, false>(a, st);
}

}  // namespace

bool combine_mfma_supported(const CombineArgs& a) {
  const bool dims = (a.r == 64 || a.r == 128 || a.r == 256 || a.r == 512) && (a.d_head == 64 || a.d_head == 128);
  const auto al16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  return dims && al16(a.out) && al16(a.out_latent) && al16(a.w_uv) && a.n_heads <= 65535;
}

hipError_t launch_combine_mfma(const CombineArgs& a, hipStream_t st) {
#define MTLA_CASE(RR, DD) \
  if (a.r == RR && a.d_head == DD) return launch_rdh<RR, DD>(a, st);
  MTLA_CASE(64, 64)
  MTLA_CASE(64, 128)
  MTLA_CASE(128, 64)
  MTLA_CASE(128, 128)
  MTLA_CASE(256, 64)
  MTLA_CASE(256, 128)
  MTLA_CASE(512, 64)
  MTLA_CASE(512, 128)
#undef MTLA_CASE
  return hipErrorInvalidValue;
}

}  // namespace mtla
