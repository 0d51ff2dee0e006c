// Parallel form with the latent-space output as well (bf16 storage, fp16 inside, gfx950): out = softmax . V and
// out_latent = softmax . C_hat' from one set of weights.
//
// Beside the d_h values per column of the plain form (attn_explicit_kernel, whose notes on layouts, columns and
// references hold here too) every column brings r latent ones, the same for all heads.  The logits are formed once: a
// workgroup owns 128 query rows, its eight wavefronts form the weights of 16 rows each, hand them to one another through LDS
// (as the B operand of the value product, 1 KB per 16 rows and tile), and multiply 64 rows by a quarter of the
// d_h + r value columns each.  The weights of tile t + 1 are formed between the barrier that makes those of tile t
// visible and the next one, so the matrix instructions of one tile cover the arithmetic of the other.
// With a pass of the plain kernel for every d_h of the r columns (the logits formed r / d_h + 1 times: 3200 flop per pair
// instead of 1664 at r = 512, d_h = 128) 5 ragged prompts of up to 1531 rows, 16 heads, took 211 us; in one pass 122, then 110 with
// the rows leaving by whole lines, the queries, own keys and own values coming by 64 bytes of a row and more, all in flight at once, and
// the blocks ordered as the plain form's, and now 99 with the rows leaving past the caches
// (the outputs alone, 313 MB, are 66 at the rate of a large copy).
#include <type_traits>

#include "attn_blocks.h"
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

template <int DH, int DR, int R>
struct LatentGeom {
  static constexpr int BN = 32, BM = 128, NW = 8;
  static constexpr int VC = DH / 8, RC = DR / 8, CC = R / 8;                                      // 16-byte pieces per row
  static constexpr int K_BYTES = BN * DH * 2, R_BYTES = BN * DR * 2, C_BYTES = BN * R * 2;
  static constexpr int KT = K_BYTES + R_BYTES, VT = K_BYTES + C_BYTES;                            // one tile's keys, values
  static constexpr int KBUF = 3, VBUF = 2;
  static constexpr int P_BYTES = BM * BN * 2;                                                     // one tile's weights
  static constexpr int K_OFF = 0, V_OFF = KBUF * KT, P_OFF = V_OFF + VBUF * VT, BYTES = P_OFF + 2 * P_BYTES;
  static constexpr int NCK = K_BYTES / 1024, NCR = R_BYTES / 1024, NCC = C_BYTES / 1024;          // wavefront loads per region
  static constexpr int NLC = NCC / NW > 0 ? NCC / NW : 1;                                         // per wavefront
  static constexpr int NV = DH / 64, NC = R / 64;                                                 // 16-column value tiles per wavefront
  static_assert(NCK <= NW && NCR <= NW, "one load per wavefront");
};

template <int DH, int DR, int R, bool STREAM>
__global__ __launch_bounds__(512, 1) void attn_latent_kernel(ExplicitArgs a) {
  using G = LatentGeom<DH, DR, R>;
  constexpr int BN = G::BN, BM = G::BM, NT = 64 * G::NW, KD = DH / 32, KQ = (DH + DR) / 32;
  constexpr int VC = G::VC, RC = G::RC, CC = G::CC, NV = G::NV, NC = G::NC;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[G::BYTES];
  __shared__ float s_alpha[2][BM];  // a tile's change of a row's reference
  __shared__ __attribute__((aligned(16))) int s_flag[2][G::NW];  // whether it has any
  __shared__ float s_inv[BM];

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int jc = wv & 3, ir = wv >> 2;  // quarter of the value columns, half of the rows
  const int T = a.T, s = a.stride, nh = a.n_heads;
  // (sequence, head) pairs dealt to the XCDs, their blocks on one of them, those with most columns first
  const int n_blocks = (T + BM - 1) / BM;
  const AttnBlock mine = attn_block(blockIdx.x, nh * a.batch, n_blocks, a.group);
  const int m0 = mine.block * BM, hb = mine.pair;
  if (hb >= nh * a.batch) return;
  const int h = hb % nh, b = hb / nh;
  const int len = a.seq_len ? (a.seq_len[b] < T ? a.seq_len[b] : T) : T;
  float* out = a.out + ((size_t)b * T * nh + h) * DH;
  float* latent = a.out_latent + ((size_t)b * T * nh + h) * R;
  if (m0 >= len) {  // padding rows only
    const int rows = T - m0 < BM ? T - m0 : BM;
    constexpr int N4 = (DH + R) / 4;
    for (int i = tid; i < rows * N4; i += NT) {
      const size_t row = (size_t)(m0 + i / N4);
      const int c = 4 * (i % N4);
      *reinterpret_cast<float4_t*>(c < DH ? out + row * nh * DH + c : latent + row * nh * R + (c - DH)) = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    return;
  }
  const uint16_t* kx = reinterpret_cast<const uint16_t*>(a.kx) + ((size_t)b * T * nh + h) * DH;
  const uint16_t* vx = reinterpret_cast<const uint16_t*>(a.vx) + ((size_t)b * T * nh + h) * DH;
  const uint16_t* cx = reinterpret_cast<const uint16_t*>(a.cprime) + (size_t)b * T * R;
  const uint16_t* kr16 = reinterpret_cast<const uint16_t*>(a.kr16) + (size_t)b * T * DR;
  const uint32_t kv_stride = (uint32_t)(nh * DH);

  const int m_last = (m0 + BM < len ? m0 + BM : len) - 1;
  const int n_cols = m_last / s, n_tiles = (n_cols + BN - 1) / BN;

  // ---- what this wavefront brings in of every tile: 1 KB pieces of each region.  Regions with fewer of them than
  // wavefronts are brought by some twice, so that every wavefront has the same number of loads in flight.
  const int pk = 64 * (wv % G::NCK) + lane, pr = 64 * (wv % G::NCR) + lane, pc = 64 * (wv % G::NCC) + lane;
  const int row_k = pk / VC, row_r = pr / RC, row_c = pc / CC;
  constexpr int C_ROWS = 64 * G::NW / CC;  // rows between a wavefront's pieces of the latent region (a multiple of 8)
  const uint32_t src_k = 8 * ((pk % VC) ^ swz_rows16<VC>(row_k)), src_v = 8 * ((pk % VC) ^ swz_tr<VC>(row_k));
  const uint32_t src_r = 8 * ((pr % RC) ^ swz_rows16<RC>(row_r)), src_c = 8 * ((pc % CC) ^ swz_tr<CC>(row_c));
  const uint32_t off_k = 2 * ((uint32_t)(row_k * s) * kv_stride + src_k), off_v = 2 * ((uint32_t)(row_k * s) * kv_stride + src_v);
  const uint32_t off_r = 2 * ((uint32_t)(row_r * s) * DR + src_r), off_c = 2 * ((uint32_t)(row_c * s) * R + src_c);
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_byte_ptr)lds;
  const int full = n_cols / BN;            // tiles whose rows are all there, s apart
  auto src_row = [&](int c) -> uint32_t {  // source row of column c (columns past the last one: a readable duplicate)
    c = c < n_cols ? c : n_cols - 1;
    return (uint32_t)(c * s + s - 1);
  };
  // The lane's place, out of sight of the compiler: what only a partial last tile needs is then formed there instead of
  // being kept in registers across the loop (160 of the 256 hold the sums).
  auto here = [&](int x) {
    asm volatile("" : "+v"(x));
    return x;
  };
  auto issue_keys = [&](int t) {  // two loads
    const uint32_t buf = lds_addr + G::K_OFF + (uint32_t)(t % G::KBUF) * (uint32_t)G::KT;
    const uint32_t dk = buf + (uint32_t)(wv % G::NCK) * 1024u, dr = buf + G::K_BYTES + (uint32_t)(wv % G::NCR) * 1024u;
    if (t < full) {
      const size_t row0 = (size_t)(BN * t) * s + s - 1;
      load_to_lds_16(kx + row0 * kv_stride, off_k, dk);
      load_to_lds_16(kr16 + row0 * DR, off_r, dr);
    } else {
      const int xk = here(pk), xr = here(pr);
      load_to_lds_16(kx + (size_t)src_row(BN * t + xk / VC) * kv_stride + 8 * ((xk % VC) ^ swz_rows16<VC>(xk / VC)), dk);
      load_to_lds_16(kr16 + (size_t)src_row(BN * t + xr / RC) * DR + 8 * ((xr % RC) ^ swz_rows16<RC>(xr / RC)), dr);
    }
  };
  auto issue_value = [&](int t, int i) {  // load i of 1 + NLC
    const uint32_t buf = lds_addr + G::V_OFF + (uint32_t)(t & 1) * (uint32_t)G::VT;
    if (i == 0) {
      const uint32_t dv = buf + (uint32_t)(wv % G::NCK) * 1024u;
      if (t < full) {
        load_to_lds_16(vx + ((size_t)(BN * t) * s + s - 1) * kv_stride, off_v, dv);
      } else {
        const int x = here(pk);
        load_to_lds_16(vx + (size_t)src_row(BN * t + x / VC) * kv_stride + 8 * ((x % VC) ^ swz_tr<VC>(x / VC)), dv);
      }
    } else {
      const uint32_t dc = buf + G::K_BYTES + (uint32_t)(wv % G::NCC + G::NW * (i - 1)) * 1024u;
      if (t < full) {
        load_to_lds_16(cx + ((size_t)(BN * t + C_ROWS * (i - 1)) * s + s - 1) * R, off_c, dc);
      } else {
        const int x = here(pc);
        load_to_lds_16(cx + (size_t)src_row(BN * t + x / CC + C_ROWS * (i - 1)) * R + 8 * ((x % CC) ^ swz_tr<CC>(x / CC)), dc);
      }
    }
  };
  if (n_tiles > 0) {
    issue_keys(0);
    for (int i = 0; i <= G::NLC; ++i) issue_value(0, i);
    if (n_tiles > 1) issue_keys(1);
    if (n_tiles > 2) issue_keys(2);
  }

  // ---- queries of the wavefront's 16 rows (its share of the weights), and the row's own column: reference, weight 1
  u32x4_t qf[KQ];
  float neg_ref;  // minus the row's reference
  float l_run;
  const int m_own = m0 + 16 * wv + l16, m_clamp = m_own < len ? m_own : len - 1;
  const int bound = m_clamp / s;                              // columns open to the lane's row
  // The values of the wavefront's 64 rows, a quarter of the columns, all asked for at once: piece `at` of them is 16 bytes of row
  // at / (two pieces a tile).
  u32x4_t own_v[2 * NV], own_c[2 * NC];
  auto load_own = [&](auto& own, const uint16_t* from, uint32_t stride, int ln) {
    constexpr int N = sizeof(own) / 32;  // tiles of 16 columns
#pragma unroll
    for (int i = 0; i < 2 * N; ++i) {
      const int at = 64 * i + ln, m = m0 + 64 * ir + at / (2 * N);
      own[i] = *reinterpret_cast<const u32x4_t*>(from + (size_t)(m < len ? m : len - 1) * stride + 16 * N * jc + 8 * (at % (2 * N)));
    }
  };
  // Read from memory by 64 bytes of 4 rows to 16 neighbouring lanes (the operand's layout, 16 rows, is 66 cycles of the unit's address path a
  // load, 12 loads a wavefront, this one 24).  In this layout the row's own logit is formed as well; the queries then change lanes in the
  // wavefront's place among the weights.
  {
    const int ln = here(lane), m_load = m0 + 16 * wv + (ln >> 2);
    const int m_from = m_load < len ? m_load : len - 1;
    const size_t row = ((size_t)b * T + m_from) * nh + h;
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + row * DH + 8 * (ln & 3);
    const uint16_t* qrp = reinterpret_cast<const uint16_t*>(a.q_rope) + row * DR + 8 * (ln & 3);
    const uint16_t* kp = kx + (size_t)m_from * kv_stride + 8 * (ln & 3);
    const uint16_t* krp = kr16 + (size_t)m_from * DR + 8 * (ln & 3);
    u32x4_t kd[KQ];
#pragma unroll
    for (int kk = 0; kk < KQ; ++kk) {
      qf[kk] = kk < KD ? *reinterpret_cast<const u32x4_t*>(qp + 32 * kk) : *reinterpret_cast<const u32x4_t*>(qrp + 32 * (kk - KD));
      kd[kk] = kk < KD ? *reinterpret_cast<const u32x4_t*>(kp + 32 * kk) : *reinterpret_cast<const u32x4_t*>(krp + 32 * (kk - KD));
    }
    load_own(own_v, vx, kv_stride, ln);
    load_own(own_c, cx, R, ln);
    asm volatile("" ::: "memory");
    float e = 0.f;
#pragma unroll
    for (int kk = 0; kk < KQ; ++kk) {
      qf[kk] = bf16x8_to_f16x8(qf[kk], a.scale_log2);  // logits in units of log2
      e = dot8(kd[kk], qf[kk], e);
    }
    e += __shfl_xor(e, 1);
    e += __shfl_xor(e, 2);
    neg_ref = -__shfl(e, 4 * (ln & 15));
    l_run = g == 0 ? 1.f : 0.f;
    unsigned char* turn = lds + G::P_OFF + wv * 1024;
#pragma unroll
    for (int kk = 0; kk < KQ; kk += 2) {
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (kk + k < KQ) *reinterpret_cast<u32x4_t*>(turn + k * G::P_BYTES + (ln >> 2) * 64 + (((ln & 3) ^ swz_rows16<4>(ln >> 2)) << 4)) = qf[kk + k];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int k = 0; k < 2; ++k)
        if (kk + k < KQ) qf[kk + k] = *reinterpret_cast<const u32x4_t*>(turn + k * G::P_BYTES + (ln & 15) * 64 + (((ln >> 4) ^ swz_rows16<4>(ln & 15)) << 4));
      __builtin_amdgcn_wave_barrier();
    }
  }
  const int all_below = (m0 + 16 * wv) / s, none_from = (m0 + 16 * wv + 15) / s;  // of the rows whose weights it forms
  const int none_rows = (m0 + 64 * ir + 63) / s;                                  // of the rows it sums

  // where this lane reads: key rows 16 sb + l16 (piece 4 kk + g), value rows 4g + l16/4 (+16)
  const uint32_t k_row_off = (uint32_t)(l16 * VC * 16), k_swz = (uint32_t)(swz_rows16<VC>(l16) ^ g) << 4;
  const uint32_t r_row_off = (uint32_t)(l16 * RC * 16), r_swz = (uint32_t)(swz_rows16<RC>(l16) ^ g) << 4;
  const int v_row = 4 * g + (l16 >> 2);
  const uint32_t v_off = (uint32_t)(v_row * VC * 16 + 8 * (l16 & 1)), v_swz = (uint32_t)(swz_tr<VC>(v_row) ^ ((l16 & 3) >> 1)) << 4;
  const uint32_t c_off = (uint32_t)(v_row * CC * 16 + 8 * (l16 & 1)), c_swz = (uint32_t)(swz_tr<CC>(v_row) ^ ((l16 & 3) >> 1)) << 4;

  // The weights of tile t for the wavefront's 16 rows into LDS, as the B operand of the value product.
  auto form_weights = [&](int t) {
    unsigned char* dst = lds + G::P_OFF + (t & 1) * G::P_BYTES + wv * 1024 + lane * 16;
    u32x4_t pb = {0u, 0u, 0u, 0u};
    int flag = 0;
    if (BN * t < none_from) {
      const unsigned char* kb = lds + G::K_OFF + (t % G::KBUF) * G::KT + k_row_off;
      const unsigned char* rb = lds + G::K_OFF + (t % G::KBUF) * G::KT + G::K_BYTES + r_row_off;
      const uint32_t ks = (uint32_t)here((int)k_swz), rs = (uint32_t)here((int)r_swz);
      float4_t sacc[2];
      sacc[0] = sacc[1] = float4_t{neg_ref, neg_ref, neg_ref, neg_ref};
      constexpr int KG = KQ % 3 == 0 ? 3 : 2;  // steps whose keys are read together
#pragma unroll
      for (int k0 = 0; k0 < KQ; k0 += KG) {
        u32x4_t kf[KG][2];
#pragma unroll
        for (int k = 0; k < KG; ++k)
#pragma unroll
          for (int sb = 0; sb < 2; ++sb) {
            const int kk = k0 + k;
            if (kk < KQ)
              kf[k][sb] = kk < KD ? *reinterpret_cast<const u32x4_t*>(kb + sb * (16 * VC * 16) + ((uint32_t)(64 * kk) ^ ks))
                                  : *reinterpret_cast<const u32x4_t*>(rb + sb * (16 * RC * 16) + ((uint32_t)(64 * (kk - KD)) ^ rs));
          }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < KG; ++k)
#pragma unroll
          for (int sb = 0; sb < 2; ++sb)
            if (k0 + k < KQ)
              sacc[sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, kf[k][sb]),
                                                                __builtin_bit_cast(f16x8_t, qf[k0 + k]), sacc[sb], 0, 0, 0);
      }
      if (BN * t + BN > all_below) {
        const int d = bound - (BN * t + 4 * g);
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
          for (int v = 0; v < 4; ++v) sacc[sb][v] = 16 * sb + v < d ? sacc[sb][v] : -INFINITY;
      }
      constexpr float kRebase = 12.f;
      int top = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float x = sacc[i >> 2][i & 3];
        top = max(top, __float_as_int(x));
      }
      if (__any(top > __float_as_int(kRebase))) {  // the rows' sums are scaled by whoever holds them, before they take this tile
        float up = -INFINITY;
#pragma unroll
        for (int i = 0; i < 8; ++i) up = fmaxf(up, sacc[i >> 2][i & 3]);
        up = quarter_reduce(up, LaneMax());
        float alpha = 1.f;
        if (up > kRebase) {
          alpha = __builtin_amdgcn_exp2f(-up);
          neg_ref -= up;
          l_run *= alpha;
          sacc[0] -= up;
          sacc[1] -= up;
        }
        if (g == 0) s_alpha[t & 1][16 * wv + l16] = alpha;
        flag = 1;
      }
      const f16x2_t ones = {(_Float16)1.f, (_Float16)1.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4_t& x = sacc[i >> 1];
        const uint32_t two = pack_f16x2(__builtin_amdgcn_exp2f(x[2 * (i & 1)]), __builtin_amdgcn_exp2f(x[2 * (i & 1) + 1]));
        pb[i] = two;
        l_run = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2_t, two), ones, l_run, false);
      }
    }
    *reinterpret_cast<u32x4_t*>(dst) = pb;
    if (lane == 0) s_flag[t & 1][wv] = flag;
  };

  // ---- sums of the wavefront's 64 rows and quarter of the columns, from the rows' own values.  They change lanes in the wavefront's part
  // of the second tile's place, 16 rows at a time: read from memory in the sums' layout (8 bytes of each of 16 rows per load) a
  // block spent 29000 cycles here, brought to LDS by the block, half the rows after the other, 13000.
  float4_t acc[4][NV + NC];
  unsigned char* own_place = lds + G::V_OFF + G::VT + wv * (512 * (NV + NC));
  static_assert(G::NW * 512 * (NV + NC) <= G::VT, "16 rows of every wavefront");
  auto take_own = [&](auto& own, int rt, int first, unsigned char* place) {
    constexpr int N = sizeof(own) / 32, PPR = 2 * N;
    const int ln = here(lane);
    if constexpr (N == 1) {
      const int row = (ln >> 1) & 15;  // a load holds two row tiles
      if ((ln >> 5) == (rt & 1)) *reinterpret_cast<u32x4_t*>(place + row * 32 + (((ln & 1) ^ swz_rows16<2>(row)) << 4)) = own[rt >> 1];
    } else {
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        const int at = 64 * i + ln, row = at / PPR;
        *reinterpret_cast<u32x4_t*>(place + row * (16 * PPR) + (((at % PPR) ^ swz_rows16<PPR>(row)) << 4)) = own[rt * (N / 2) + i];
      }
    }
    __builtin_amdgcn_wave_barrier();
    const int row = ln & 15;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint2 v = *reinterpret_cast<const uint2*>(place + row * (16 * PPR) + (((2 * i + (ln >> 5)) ^ swz_rows16<PPR>(row)) << 4) + 8 * ((ln >> 4) & 1));
      acc[rt][first + i] = float4_t{f16_lo_to_f32(v.x), f16_hi_to_f32(v.x), f16_lo_to_f32(v.y), f16_hi_to_f32(v.y)};
    }
    __builtin_amdgcn_wave_barrier();
  };
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    take_own(own_v, rt, 0, own_place);
    take_own(own_c, rt, NV, own_place + 512 * NV);
  }
  wait_loads_but<0>();
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the own values' place has been read (it is filled behind the next barrier)
  barrier_only();
  if (n_tiles > 0) form_weights(0);
  for (int t = 0; t < n_tiles; ++t) {
    // values of tile t and keys of tile t + 1 have landed (keys of t + 2 may be under way), weights of tile t are written
    if (t + 2 < n_tiles) wait_loads_but<2>();
    else wait_loads_but<0>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier_only();
    // What the step brings in (values of t + 1, keys of t + 3) is asked for piece by piece between the products: all at once,
    // the wavefronts stood at the full queue of the memory path for 600 to 900 of a step's 3750 cycles.
    constexpr int STEPS = (NV + NC + 1) / 2;
    auto issue_part = [&](int k) {  // part k of STEPS
#pragma unroll
      for (int i = 0; i <= G::NLC; ++i)
        if (i * STEPS / (G::NLC + 1) == k && t + 1 < n_tiles) issue_value(t + 1, i);
      if (k == STEPS - 1 && t + 3 < n_tiles) issue_keys(t + 3);
    };

    const int4 flags = *reinterpret_cast<const int4*>(&s_flag[t & 1][4 * ir]);
    if (__builtin_amdgcn_readfirstlane(flags.x | flags.y | flags.z | flags.w)) {
      const int f4[4] = {flags.x, flags.y, flags.z, flags.w};
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) {
        if (!f4[rt]) continue;
        const float alpha = s_alpha[t & 1][64 * ir + 16 * rt + l16];
#pragma unroll
        for (int i = 0; i < NV + NC; ++i) acc[rt][i] *= alpha;
      }
    }
    // The two wavefronts of a SIMD (the two halves of the rows) take the two parts of the step in opposite order, so that the
    // matrix instructions of one meet the arithmetic and the reads of the other.
    if (ir == 0 && t + 1 < n_tiles) form_weights(t + 1);
    if (BN * t < none_rows) {  // some row of this half is open to the tile
      // ---- O^T[d, row] += V^T[d, col] P^T[col, row]: the reads of two value tiles ahead of the products of the two before
      const unsigned char* pb_at = lds + G::P_OFF + (t & 1) * G::P_BYTES + ir * 4096 + lane * 16;
      const unsigned char* vb = lds + G::V_OFF + (t & 1) * G::VT + v_off;
      const unsigned char* cb = lds + G::V_OFF + (t & 1) * G::VT + G::K_BYTES + c_off;
      const uint32_t vs = (uint32_t)here((int)v_swz), cs = (uint32_t)here((int)c_swz);
      auto read_v = [&](int i) -> u32x4_t {
        const unsigned char* p = i < NV ? vb + ((uint32_t)(32 * (NV * jc + i)) ^ vs) : cb + ((uint32_t)(32 * (NC * jc + i - NV)) ^ cs);
        const short4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)p);
        const short4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(p + 256 * (i < NV ? VC : CC)));
        const uint2 u0 = __builtin_bit_cast(uint2, v0), u1 = __builtin_bit_cast(uint2, v1);
        return u32x4_t{u0.x, u0.y, u1.x, u1.y};
      };
      u32x4_t pb[4], vf[2][2];
      vf[0][0] = read_v(0);
      vf[0][1] = read_v(1);
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) pb[rt] = *reinterpret_cast<const u32x4_t*>(pb_at + rt * 1024);
#pragma unroll
      for (int i = 0; i < NV + NC; i += 2) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
          if (i + 2 + k < NV + NC) vf[(i / 2 + 1) & 1][k] = read_v(i + 2 + k);
        issue_part(i / 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 2; ++k)
          if (i + k < NV + NC)
#pragma unroll
            for (int rt = 0; rt < 4; ++rt)
              acc[rt][i + k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, vf[(i / 2) & 1][k]),
                                                                      __builtin_bit_cast(f16x8_t, pb[rt]), acc[rt][i + k], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int k = 0; k < STEPS; ++k) issue_part(k);
    }
    if (ir == 1 && t + 1 < n_tiles) form_weights(t + 1);
  }

  // ---- normalise and store: lane holds row l16 of row tile rt, output columns 16 i + 4g .. +3.  The rows leave through LDS, up to whole
  // lines at a time (as they stand, a store is 64 bytes of 16 rows, 67 cycles of the address path, 320 of them a block), and past the caches where the
  // launcher says so: 320 KB a block and unit otherwise take the place of the tiles that the blocks beside it read, and are written back in bursts.
  {
    const float l = quarter_reduce(l_run, LaneSum());
    if (g == 0) s_inv[16 * wv + l16] = m_own < len ? 1.f / l : 0.f;
  }
  __syncthreads();
  const int ln = here(lane);
  unsigned char* leave = lds + wv * (1024 * (NV + NC));
  static_assert(8 * 1024 * (NV + NC) <= G::BYTES, "the rows fit");
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    const int mt0 = m0 + 64 * ir + 16 * rt;
    if (mt0 >= T) break;
    const bool live = mt0 + (ln & 15) < len;  // padding rows are zeros, whatever their inputs held
    const float inv = s_inv[64 * ir + 16 * rt + (ln & 15)];
    auto leave_rows = [&](auto n_tag, int first, unsigned char* area, unsigned char* to, size_t to_row) {  // N tiles of 16 columns from `first` on
      constexpr int N = decltype(n_tag)::value, PPR = 4 * N, SW = PPR < 16 ? PPR - 1 : 15;  // piece j of row i sits at j ^ (i & SW)
#pragma unroll
      for (int i = 0; i < N; ++i)
        *reinterpret_cast<float4_t*>(area + (ln & 15) * (16 * PPR) + (((4 * i + (ln >> 4)) ^ (ln & SW)) << 4)) =
            live ? acc[rt][first + i] * inv : float4_t{0.f, 0.f, 0.f, 0.f};
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int at = 64 * i + ln, row = at / PPR, c = at % PPR;
        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(area + row * (16 * PPR) + ((c ^ (row & SW)) << 4));
        if (mt0 + row < T) {
          u32x4_t* at_row = reinterpret_cast<u32x4_t*>(to + row * to_row + 16 * c);
          if constexpr (STREAM) __builtin_nontemporal_store(v, at_row);
          else *at_row = v;
        }
      }
      __builtin_amdgcn_wave_barrier();
    };
    leave_rows(std::integral_constant<int, NV>(), 0, leave, reinterpret_cast<unsigned char*>(out + (size_t)mt0 * nh * DH + 16 * NV * jc), (size_t)nh * DH * 4);
    leave_rows(std::integral_constant<int, NC>(), NV, leave + 1024 * NV, reinterpret_cast<unsigned char*>(latent + (size_t)mt0 * nh * R + 16 * NC * jc), (size_t)nh * R * 4);
  }
}

template <int DH, int DR>
hipError_t launch_r(const ExplicitArgs& a, hipStream_t st, const EventPair& ev) {
  static_assert(kAttnRows == LatentGeom<DH, DR, 64>::BM, "rows of a block");
  const int pairs = a.n_heads * a.batch;
  ExplicitArgs x = a;
  x.group = attn_group(pairs, DH, false);
  // Outputs past the caches, but for those of medium size: with them whoever reads the outputs next would wait for what the call gains.  us alone and with an
  // elementwise pass over both outputs behind it, ordinary / past the caches: 16 heads x 128, r = 512, one of 409 (16 MB) 56.4 / 53.8 and 63.7 / 61.9, one of 1228 (48 MB) 82.7 / 80.3
  // and 98.4 / 100.3, 4 of 409 (64 MB) 63.6 / 62.3 and 83.6 / 85.5, 4 of 614 (96 MB) 85.2 / 83.4 and 120.8 / 116.5, 4 of 1920 (300 MB) 253.6 / 219.4 and 363.9 / 333.4; 12 x 128,
  // r = 256, 4 of 910 (64 MB) 77.1 / 74.2 and 97.6 / 98.5, 4 of 1820 (128 MB) 139.4 / 134.2 and 191.2 / 186.1; 8 x 64, 4 of 819 (32 MB) 54.9 / 52.2 and 65.4 / 64.9, 4 of 1228
  // (48 MB) 64.2 / 62.5 and 79.5 / 80.4.
  const size_t out_bytes = (size_t)a.batch * a.T * a.n_heads * (DH + a.r) * 4;
  const bool stream = out_bytes <= (size_t)32 << 20 || out_bytes > (size_t)80 << 20;
  const dim3 grid((unsigned)((a.T + kAttnRows - 1) / kAttnRows) * (unsigned)(attn_pairs(pairs) * kXcds)), block(512);
#define MTLA_CASE(RR)                                                                    \
  if (a.r == RR) {                                                                       \
    if (stream) launch_timed(attn_latent_kernel<DH, DR, RR, true>, grid, block, 0, st, ev, x); \
    else launch_timed(attn_latent_kernel<DH, DR, RR, false>, grid, block, 0, st, ev, x); \
    return hipGetLastError();                                                            \
  }
  MTLA_CASE(64)
  MTLA_CASE(128)
  MTLA_CASE(256)
  MTLA_CASE(512)
#undef MTLA_CASE
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_attn_latent(const ExplicitArgs& a, hipStream_t st, const EventPair& ev) {
  if (a.d_head == 64 && a.d_rope == 32) return launch_r<64, 32>(a, st, ev);
  if (a.d_head == 64 && a.d_rope == 64) return launch_r<64, 64>(a, st, ev);
  if (a.d_head == 128 && a.d_rope == 32) return launch_r<128, 32>(a, st, ev);
  if (a.d_head == 128 && a.d_rope == 64) return launch_r<128, 64>(a, st, ev);
  return hipErrorInvalidValue;
}

}  // namespace mtla
