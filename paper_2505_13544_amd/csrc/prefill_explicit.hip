// Parallel (prefill / training-forward) form with explicit per-head keys and values (bf16 storage,
// fp16 inside, gfx950).
//
// Eq. (with-rope) before absorption: k_n^(h) = C_hat'[n] W_K^(h), v_n^(h) = C_hat'[n] W_V^(h), and
// for query row m of head h
//     e_n = ( <q_m^(h), k_n^(h)> + <q_m^R(h), k_n^R> ) / sqrt(d_h),   o_m^(h) = softmax(e) V^(h)
// over the columns the stride-aware causal mask leaves open to m: the final states of the chunks
// that ended before m (rows j*s + s-1, j < m/s) and the row's own running state (row m).  With many
// query rows per head this is the cheaper form (2 (d_h + d_R) + 2 d_h flop per open (row, column)
// pair instead of 2 (r + d_R) + 2 r), it needs neither the absorbed query operand nor the latent
// partials, and every matrix instruction works on 16 real query rows.  The absorbed form remains
// for decode (one row per head).  The latent-space output, where it is asked for, comes from the same weights
// (prefill_latent.hip).
//
// Everything between the bf16 inputs and the fp32 output is IEEE half: the partial states, the
// keys, the values and the softmax weights each carry 11 significant bits instead of bf16's 8 (the
// intermediate roundings of this form would otherwise use up the whole 2e-2 budget), and all of
// them are of order 1, far inside the half range.  bf16 inputs (RoPE keys, weights) convert exactly
// apart from values below 6e-5; the queries are multiplied by log2(e) / sqrt(d_h) before their one
// rounding to half.
//
// Two kernels behind the front launch (prefill_front.hip: partial states, RoPE keys and weights as fp16):
//   gemm_nt_kernel        K = C_hat' W_K, V = C_hat' W_V for all T rows: a plain MFMA GEMM, its tile sized
//                         to the rows there are, operands streamed from memory straight into LDS (also the
//                         projections of the whole-layer prefill, with rotation / scaling on the way out)
//   attn_explicit_kernel  one workgroup per block of 128 rows of a (head, sequence), in the order of attn_blocks.h; keys, RoPE keys and values of 32 columns at a
//                         time stream from memory straight into LDS and are shared by the four wavefronts
//                         (32 query rows each, queries in registers)
#include <cmath>
#include <type_traits>

#include "attn_blocks.h"
#include "bounds.h"
#include "gemm_tiles.h"
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

// C[row][n] = sum_k A[row][k] W[n][k]   (A [M][K], W [N][K], C [M][N]; A and W both fp16 or both bf16,
// K % 32 == 0, N % 8 == 0), fp32 accumulation, one of three ways out (GemmSegment::epi):
//   0  C fp16 = scale * acc                       (keys, values, queries)
//   1  C fp16 = scale * RoPE(acc), 2 the same as bf16 without the scale (RoPE queries, the shared RoPE key: row
//      b*T + t is turned at pos0[b] + t; 64 x 64 tiles form the cosines and sines they need, the larger ones read a table, rope_cs[row][k])
//   3  C fp32 = acc
// A launch takes up to four products that share A ("segments", each with its own weights, columns and way out): a short
// prompt's projections are one launch instead of four.
// BM x BN tile; K is walked 32 at a time through NBUF LDS stages.  A wavefront owns a WM x WN part: W rows are the A
// operand, A rows the B operand, so a lane ends up with four consecutive n of one row (two RoPE pairs).
// Rows that hold nothing (GemmRows: padding of ragged sequences, slots of the past that a sequence does not have) are
// left out: the row blocks are those of the sequences' rows in use, one after the other, so what is left over at the
// end of the launch returns at once.  Where the caller wants zeros in such rows the blocks are the matrix's own.
//
// Tiles: short prompts' products go to gemm_ring.hip, large ones to the streams of gemm_wide.hip; between them 64 x 64 to 128 x 128 here (1000 rows x 1024
// columns, K = 512: 4.9 us in 64 x 64 tiles; 2000 x 2048: 9 us in 128 x 128), and 256 x 256 (eight wavefronts, one workgroup per CU)
// where a contraction that is no multiple of 64 keeps a large one out of the streams.
template <int BM, int BN>
struct GemmGeom {
  static constexpr int NWV = BM * BN >= 65536 ? 8 : 4, NT = 64 * NWV, BK = 32;
  static constexpr int WCOLS = BN >= 128 ? BN / 64 : 2, WN = BN / WCOLS, WROWS = NWV / WCOLS, WM = BM / WROWS;
  static constexpr int W_BYTES = BN * BK * 2, A_BYTES = BM * BK * 2, STAGE = W_BYTES + A_BYTES;
  // A small tile's stage is a chain of waits and reads for a few products: two are done behind one barrier, with constant
  // waits.  64 x 64, K = 512 and 2048, a tile a unit or less: 5.8 and 15.6 us, now 4.8 and 10.5.  More buffers take a third
  // workgroup from the unit and gain nothing between other kernels, where the operands come from beyond the L2.
  static constexpr int SPB = BM >= 256 ? 1 : 2;  // stages per barrier
  static constexpr int NBUF = BM >= 256 ? 3 : (BM == 128 ? 4 : 6), PF = NBUF - SPB;
  static constexpr int NLW = W_BYTES / 1024 / NWV, NLA = A_BYTES / 1024 / NWV, LOADS = NLW + NLA;  // loads per wavefront and stage
  static constexpr int PER_CU = BM == 256 && BN == 256 ? 1 : 2;
  // Tiles of 64 rows form their angles while their first operands are on the way: a row is a lane, a frequency a wavefront's.  A
  // launch that writes a table first is 3 us of a prompt's; the layer over 1000 tokens 46.0, now 44.4 us.  (Where the larger tiles pay there are thousands of rows: each would be turned once per column block, and the table's
  // launch is 6 us of 1280.)
  static constexpr bool OWN_ANGLES = gemm_own_angles(BM, BN);
  static_assert(PF >= SPB && 2 * LOADS * SPB <= 63 && NLW >= 1 && NLA >= 1, "buffers, wait counts");
};

template <bool BF16, int BM, int BN>
__global__ __launch_bounds__((GemmGeom<BM, BN>::NT), (GemmGeom<BM, BN>::PER_CU)) void gemm_nt_kernel(GemmArgs a) {
  typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
  using G = GemmGeom<BM, BN>;
  constexpr int BK = G::BK, NBUF = G::NBUF, PF = G::PF, NWV = G::NWV, NT = G::NT, WN = G::WN, WM = G::WM;
  constexpr int W_BYTES = G::W_BYTES, STAGE = G::STAGE, NLW = G::NLW, NLA = G::NLA, LOADS = G::LOADS;
  constexpr int JM = WM / 16, IN = WN / 16;
  constexpr bool kAngles = BF16 && G::OWN_ANGLES;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NBUF * STAGE];

  const int M = a.M, K = a.K;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  // Job order: groups of four column blocks of the weights (1 MB at K = 512 and 128 columns, stays in
  // L2) slowest, then the row blocks of A, then the jobs of one row block inside the group.  Row blocks are dealt to the
  // eight XCDs in turn (workgroup w runs on XCD w % 8), so the workgroups that read the same rows of A run on one XCD
  // and rows that hold nothing (ragged sequences) fall on all of them.
  const unsigned gx = (unsigned)a.col_blocks, gy = a.row_blocks, w = blockIdx.x;
  const unsigned nx = a.xcds, ry = (gy + nx - 1) / nx, job = w / nx;  // row blocks per XCD
  // groups of four column blocks, then one group with the blocks that are left
  const unsigned full_jobs = (gx / 4u) * 4u * ry;
  const bool in_full = job < full_jobs;
  const unsigned gsz = in_full ? 4u : gx % 4u, per_group = gsz * ry;
  const unsigned first = in_full ? (job / per_group) * 4u : (gx / 4u) * 4u;
  const unsigned rem = in_full ? job % per_group : job - full_jobs;
  const int ib = (int)(rem / gsz * nx + w % nx);  // row block
  int rb = ib * BM, row_end = M;
  bool work = rb < M;
  double freq[kAngles ? 32 / NWV : 1];  // asked for here: behind the first operands each would be a wait of its own
  int start = 0;                        // of the block's sequence, where the rows are told apart
  if constexpr (kAngles) {
#pragma unroll
    for (int i = 0; i < 32 / NWV; ++i) {
      freq[i] = a.rope_freq[wv + NWV * i];
      asm volatile("" : "+s"(freq[i]));
    }
  }
  if (a.rows.n_new || a.rows.pos0) {
    work = false;
    const GemmRows& q = a.rows;
    const int Tp = q.past + q.T, n_seq = M / Tp;
    auto used_rows = [&](int b) {
      return (q.pos0 ? slots_inside(q.pos0[b], q.stride, q.past) : 0) + (q.n_new ? new_rows(q.n_new[b], q.T) : q.T);
    };
    if (q.zeros) {  // the block as it is; without rows of its own it only writes zeros
      for (int b = rb / Tp; b < n_seq && b * Tp < rb + BM && !work; ++b) {
        const int used = used_rows(b);
        work = rb < b * Tp + used && used > 0;
      }
      if (rb >= M) return;
    } else {        // block ib of those that the sequences use, each sequence's from its first row on
      int before = 0;
      for (int b0 = 0; b0 < n_seq && !work; b0 += kWave) {
        const int used = b0 + lane < n_seq ? used_rows(b0 + lane) : 0;
        const int from = kAngles && a.rope_pos0 && b0 + lane < n_seq ? a.rope_pos0[b0 + lane] : 0;
        const int n = (used + BM - 1) / BM;
        const int upto = wave_scan(n);  // blocks of sequences b0 .. b0 + lane
        const unsigned long long here = __ballot(ib - before < upto);
        if (here) {
          const int at = __builtin_ctzll(here);
          rb = (b0 + at) * Tp + (ib - before - (__shfl(upto, at, kWave) - __shfl(n, at, kWave))) * BM;
          row_end = (b0 + at) * Tp + __shfl(used, at, kWave);
          start = __shfl(from, at, kWave);
          work = true;
        }
        before += __shfl(upto, kWave - 1, kWave);
      }
      if (!work) return;
      rb = __builtin_amdgcn_readfirstlane(rb);
      row_end = __builtin_amdgcn_readfirstlane(row_end);
    }
  } else if (!work) {
    return;
  }
  // the segment the column block belongs to
  int cb = (int)(first + rem % gsz), z = 0;
  while (z + 1 < a.n_seg && cb >= (a.seg[z].N + BN - 1) / BN) {
    cb -= (a.seg[z].N + BN - 1) / BN;
    ++z;
  }
  const GemmSegment sg = a.seg[z];
  const int nb = cb * BN, N = sg.N, epi = sg.epi;
  const uint16_t* A = reinterpret_cast<const uint16_t*>(a.A);
  const uint16_t* W = reinterpret_cast<const uint16_t*>(sg.W);
  const int wn = WN * (wv % G::WCOLS), wm = WM * (wv / G::WCOLS);

  // what this thread brings in of every stage: 1 KB chunk c of a region = rows 16 c .. 16 c + 15 (4
  // pieces of 8 k each); wavefront wv fills chunks wv, wv + NWV, ..
  const int prow = lane >> 2;
  const uint32_t psrc = 8 * ((lane & 3) ^ swz_rows16<4>(prow));
  const uint16_t* wsrc[NLW];
  const uint16_t* asrc[NLA];
#pragma unroll
  for (int i = 0; i < NLW; ++i) {
    const int row = nb + 16 * (wv + NWV * i) + prow;
    wsrc[i] = W + (size_t)(row < N ? row : N - 1) * K + psrc;
  }
#pragma unroll
  for (int i = 0; i < NLA; ++i) {
    const int row = rb + 16 * (wv + NWV * i) + prow;
    asrc[i] = A + (size_t)(row < row_end ? row : row_end - 1) * K + psrc;
  }
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_byte_ptr)lds;
  auto issue = [&](int st) {  // stage st: k = 32 st ..
    const uint32_t buf = lds_addr + (uint32_t)((st % NBUF) * STAGE);
#pragma unroll
    for (int i = 0; i < NLW; ++i) load_to_lds_16(wsrc[i] + BK * st, buf + (uint32_t)((wv + NWV * i) * 1024));
#pragma unroll
    for (int i = 0; i < NLA; ++i) load_to_lds_16(asrc[i] + BK * st, buf + W_BYTES + (uint32_t)((wv + NWV * i) * 1024));
  };
  // where this lane reads: rows 16 i + l16 of a quarter, logical piece g
  const uint32_t frag_off = (uint32_t)(l16 * 64 + ((g ^ swz_rows16<4>(l16)) << 4));

  float4_t acc[JM][IN];  // [token tile][n tile]
#pragma unroll
  for (int j = 0; j < JM; ++j)
#pragma unroll
    for (int i = 0; i < IN; ++i) acc[j][i] = float4_t{0.f, 0.f, 0.f, 0.f};

  const int n_stages = work ? K / BK : 0;
#pragma unroll
  for (int st = 0; st < PF; ++st)
    if (st < n_stages) issue(st);
  float2 turn[kAngles ? 32 / NWV : 1];  // lane: row; the wavefronts take the frequencies in turn
#pragma unroll
  for (float2& t : turn) t = make_float2(1.f, 0.f);
  if constexpr (kAngles) {
    if (work && (epi == 1 || epi == 2) && !a.rope_ready) {
      const int T = a.rows.T, row = rb + lane;
      int pos = start + row % T;
      if (!a.rows.n_new && !a.rows.pos0 && a.rope_pos0) {  // rows of several sequences (scalar loads: none that waits for the operands)
        for (int b = rb / T; b * T < rb + BM && b * T < M; ++b) {
          start = load_uniform_i32(a.rope_pos0, b);
          if (row >= b * T) pos = start + row - b * T;
        }
      }
#pragma unroll
      for (int i = 0; i < 32 / NWV; ++i)
        if (wv + NWV * i < a.d_rope / 2) turn[i] = rope_angle(pos, freq[i]);
    }
  }
  constexpr int SPB = G::SPB;
  auto multiply = [&](int st) {
    const unsigned char* wb = lds + (st % NBUF) * STAGE + wn * 64 + frag_off;
    const unsigned char* ab = lds + (st % NBUF) * STAGE + W_BYTES + wm * 64 + frag_off;
    u32x4_t wf[IN], af[JM];
#pragma unroll
    for (int i = 0; i < IN; ++i) wf[i] = *reinterpret_cast<const u32x4_t*>(wb + i * 1024);
#pragma unroll
    for (int j = 0; j < JM; ++j) af[j] = *reinterpret_cast<const u32x4_t*>(ab + j * 1024);
#pragma unroll
    for (int j = 0; j < JM; ++j)
#pragma unroll
      for (int i = 0; i < IN; ++i) {
        if constexpr (BF16)
          acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[i]),
                                                              __builtin_bit_cast(bf16x8_t, af[j]), acc[j][i], 0, 0, 0);
        else
          acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, wf[i]),
                                                             __builtin_bit_cast(f16x8_t, af[j]), acc[j][i], 0, 0, 0);
      }
  };
  int st = 0;
  for (; st + PF <= n_stages; st += SPB) {  // stages below st + PF have been asked for
    wait_loads_but<LOADS * (PF - SPB)>();
    barrier_only();
#pragma unroll
    for (int i = 0; i < SPB; ++i)
      if (st + PF + i < n_stages) issue(st + PF + i);  // into the buffers the stages before were read from
#pragma unroll
    for (int i = 0; i < SPB; ++i) multiply(st + i);
  }
  for (; st < n_stages; st += SPB) {        // all have
    const int left = n_stages - st;
    if (left >= 3 * SPB) wait_loads_but<LOADS * 2 * SPB>();
    else if (left >= 2 * SPB) wait_loads_but<LOADS * SPB>();
    else wait_loads_but<0>();
    barrier_only();
#pragma unroll
    for (int i = 0; i < SPB; ++i)
      if (st + i < n_stages) multiply(st + i);
  }

  // ---- the tile leaves through LDS, RP rows at a time (as many as the stage buffers hold), so that
  // memory sees whole row segments of 128 bytes or more
  unsigned char* Cb = reinterpret_cast<unsigned char*>(sg.C);
  const float sc = sg.scale;
  barrier_only();  // every wavefront is done with the last stage
  constexpr int kAnglesAt = BM * (4 * BN + 16);  // behind the rows on their way out: [two pairs of a head][row]
  static_assert(!kAngles || kAnglesAt + 16 * 16 * BM <= NBUF * STAGE, "the angles fit in the stage buffers");
  const bool own_angles = kAngles && (epi == 1 || epi == 2) && !a.rope_ready;
  if constexpr (kAngles) {
    if (own_angles) {
#pragma unroll
      for (int i = 0; i < 32 / NWV; ++i) {
        const int k = wv + NWV * i;
        if (k < a.d_rope / 2) *reinterpret_cast<float2*>(lds + kAnglesAt + ((k >> 1) * BM + lane) * 16 + 8 * (k & 1)) = turn[i];
      }
      __syncthreads();
    }
  }
  auto way_out = [&](auto kind) {
    constexpr int EPI = decltype(kind)::value;
    constexpr int ES = EPI == 3 ? 4 : 2;                       // bytes per output element
    constexpr int CS = ES * BN + 16;                           // LDS row pitch
    constexpr int RP = BM >= 256 && NBUF * STAGE / CS >= 256 ? 256 : (BM >= 128 && NBUF * STAGE / CS >= 128 ? 128 : 64);
    static_assert(RP * CS <= NBUF * STAGE && RP <= BM, "the rows of a pass fit in the stage buffers");
    constexpr int PPR = BN * ES / 16;                          // 16-byte pieces per row
    static_assert(RP * PPR % NT == 0, "whole rounds of stores");
#pragma unroll
    for (int pass = 0; pass < BM / RP; ++pass) {
#pragma unroll
      for (int j = 0; j < JM; ++j) {
        const int row = wm + 16 * j;                           // wavefront-uniform
        if (row / RP != pass) continue;
        unsigned char* lrow = lds + (row - RP * pass + l16) * CS;
        const int grow = rb + row + l16 < row_end ? rb + row + l16 : row_end - 1;
#pragma unroll
        for (int i = 0; i < IN; ++i) {
          const int col = wn + 16 * i + 4 * g;
          float4_t o = acc[j][i];
          if constexpr (EPI == 1 || EPI == 2) {  // rotation: the lane's columns are two pairs of one head
            const int jn = (nb + col) % a.d_rope;              // element inside the head, a multiple of 4
            float4_t cs;                                       // (cos, sin) of both
            if (own_angles) cs = *reinterpret_cast<const float4_t*>(lds + kAnglesAt + (jn / 4 * BM + row + l16) * 16);
            else cs = *reinterpret_cast<const float4_t*>(a.rope_cs + (size_t)grow * (a.d_rope / 2) + jn / 2);
            o = float4_t{o[0] * cs[0] - o[1] * cs[1], o[0] * cs[1] + o[1] * cs[0], o[2] * cs[2] - o[3] * cs[3], o[2] * cs[3] + o[3] * cs[2]};
          }
          if constexpr (EPI == 3) *reinterpret_cast<float4_t*>(lrow + 4 * col) = o;
          else if constexpr (EPI == 2) *reinterpret_cast<uint2*>(lrow + 2 * col) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
          else *reinterpret_cast<uint2*>(lrow + 2 * col) = make_uint2(pack_f16x2(sc * o[0], sc * o[1]), pack_f16x2(sc * o[2], sc * o[3]));
        }
        if constexpr (EPI == 1 || EPI == 2) __builtin_amdgcn_sched_barrier(0);  // one row's table entries in registers at a time
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RP * PPR / NT; ++i) {
        const int p_ = tid + NT * i, row = p_ / PPR, c = p_ % PPR;
        const int grow = rb + RP * pass + row, gcol = nb + c * (16 / ES);
        if (grow < row_end && gcol < N)  // N is a multiple of 8
          *reinterpret_cast<u32x4_t*>(Cb + ((size_t)grow * N + gcol) * ES) = *reinterpret_cast<const u32x4_t*>(lds + row * CS + 16 * c);
      }
      if (pass + 1 < BM / RP) __syncthreads();
    }
  };
  if (epi == 3) way_out(std::integral_constant<int, 3>());
  else if (BF16 && epi == 1) way_out(std::integral_constant<int, 1>());
  else if (BF16 && epi == 2) way_out(std::integral_constant<int, 2>());
  else way_out(std::integral_constant<int, 0>());
}

// ---- attention over explicit keys and values -------------------------------------------------
//
// A tile is 32 columns: their keys [32][d_h] (swz_rows16), RoPE keys [32][d_R] (swz_rows16) and
// values [32][d_h] (swz_tr), fp16; one pair of tiles is fetched while the pair before is multiplied (four LDS buffers).
template <int DH, int DR>
struct TileGeom {
  static constexpr int BN = 32, VC = DH / 8, RC = DR / 8;  // 16-byte pieces per key / value row, per RoPE key row
  static constexpr int K_BYTES = BN * DH * 2, R_BYTES = BN * DR * 2;
  static constexpr int K_OFF = 0, R_OFF = K_BYTES, V_OFF = K_BYTES + R_BYTES, BYTES = 2 * K_BYTES + R_BYTES;
  static constexpr int NCK = BN * VC / 64, NCR = BN * RC / 64;  // wavefront loads (1 KB) per region
  static_assert(BYTES % 1024 == 0 && K_BYTES % 1024 == 0 && R_BYTES % 1024 == 0, "1 KB per wavefront load");
};

// The open columns of row m are the final states of the slots that closed before it, j < (p0 + m) / s -- the same
// columns for all heads' rows of a block up to where they end -- and the row's own running state.  That own
// column is not a tile column: it starts the row off (reference = its logit, weight 1, output = its value), formed
// from the row's own key and value in the layouts the queries and the output already have.  So a block of 128 rows walks
// ((p0 + m0 + 127) / s) / 32 tiles and only the last few have a mask; with the block's own rows as masked tiles, one by
// one, it was 128 / 32 - (128 / s) / 32 tiles more (two of the 36 a block walks on average at 4096 rows and s = 2).
//
// NW wavefronts of 32 query rows each per workgroup (RT = 2 tiles of 16; of 16 where attn_rows takes half a block).  NW = 4 is what the
// launcher uses: two workgroups per CU, whose
// wavefronts drift apart so that one multiplies while the other does softmax arithmetic.  What bounds it is the chain
// of a pair of tiles (operand reads, 80 matrix instructions, the arithmetic of the weights) with two wavefronts per SIMD
// to overlap, and what lies around the tile loop: matrix pipes busy 45 % (at 750 thousand cycles, the same at any
// clock from 1.7 to 2.2 GHz, as power allows), 2 % bank conflicts.  8 sequences x 4096 rows, 16 heads x 128, s = 2 (0.344 TFLOP): 460
// us with the own rows as masked tiles and one tile per step, 414 with two blocks a workgroup and operands' loads in the operand's layout (820 thousand
// cycles), now 391 (879 TFLOP/s).
// CONT: the sequences continue from a cache (a.pos0, a.past_pitch); whole sequences are compiled without it.
// LAYER: the whole-layer prefill's operands (queries already fp16 and scaled, output as fp16 for W_O).
template <int DH, int DR, int NW, bool CONT, bool LAYER, int RT>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void attn_explicit_kernel(ExplicitArgs a) {
  using G = TileGeom<DH, DR>;
  constexpr int KD = DH / 32, KQ = (DH + DR) / 32, MT = DH / 16;
  constexpr int NT = 64 * NW, BM = 16 * RT * NW, BN = G::BN, VC = G::VC, RC = G::RC;
  constexpr int NBUF = 4;                 // tiles in LDS: two pairs
  constexpr int NIK = G::NCK / NW;  // loads per wavefront and region of keys or values
  constexpr int IROWS = 64 * NW / VC;     // rows between a wavefront's chunks of a region
  constexpr int kOwn = 2 * G::BYTES / NW; // a wavefront's part of a pair of buffers
  static_assert(1024 * (KQ + KD) <= kOwn, "sixteen rows' queries and values fit");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NBUF * G::BYTES];

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int T = a.T, s = a.stride, nh = a.n_heads;
  const int n_blocks = (T + BM - 1) / BM;
  const AttnBlock job = attn_block(blockIdx.x, nh * a.batch, n_blocks, a.group);
  const int hb = __builtin_amdgcn_readfirstlane(job.pair);
  if (hb >= nh * a.batch) return;
  const int h = hb % nh, b = hb / nh;
  const int len = a.seq_len ? (a.seq_len[b] < T ? a.seq_len[b] : T) : T;
  // A continuing sequence has p0 tokens behind it: the final states of its first p0 / s slots are the
  // first rows of its part of the key / value arrays (one per slot), its new rows follow.
  const int Tp = (CONT ? a.past_pitch : 0) + T;
  const int p0 = CONT ? __builtin_amdgcn_readfirstlane(start_inside(a.pos0[b], s, a.past_pitch)) : 0;
  const int j0 = p0 / s, past = j0;
  if (CONT && a.advance && job.block == 0 && h == 0) {
    const int old = a.pos0[b];
    if (len > 0 && append_status(old, len, s, a.max_slots) == 0) {  // as the append took it
      if (tid == 0) a.advance[b] = old + len;
      for (int e = tid; e < a.r; e += NT) a.tail_c[(size_t)b * a.r + e] = a.tail_next[(size_t)b * a.r + e];
    }
  }
  const size_t out_stride = (size_t)nh * DH;  // elements per output row
  float* out = a.out + ((size_t)b * T * nh + h) * DH;
  const uint16_t* kx = reinterpret_cast<const uint16_t*>(a.kx) + ((size_t)b * Tp * nh + h) * DH;
  const uint16_t* vx = reinterpret_cast<const uint16_t*>(a.vx) + ((size_t)b * Tp * nh + h) * DH;
  const uint16_t* kr16 = reinterpret_cast<const uint16_t*>(a.kr16) + (size_t)b * Tp * DR;
  const uint32_t kv_stride = (uint32_t)(nh * DH);

  // ---- what this thread brings in of every tile.  Wavefront wv fills the 1 KB chunks wv, wv + NW, ..
  // of a region; lane i of it the chunk's piece i: row and (swizzled) source piece, the same for
  // all of the wavefront's chunks (they lie a multiple of 16 rows apart).
  const int pk = 64 * wv + lane;
  const int row_k = pk / VC;
  const uint32_t src_k = 8 * ((pk % VC) ^ swz_rows16<VC>(row_k));  // element offset inside the source row
  const uint32_t src_v = 8 * ((pk % VC) ^ swz_tr<VC>(row_k));
  static_assert(NIK == 1 || IROWS % 16 == 0, "same swizzle for all chunks of a wavefront");
  static_assert(G::NCR <= NW, "one RoPE key chunk per wavefront at most");
  static_assert(G::NCK % NW == 0, "whole rounds of key and value chunks");
  // RoPE keys: fewer chunks than wavefronts at d_R = 32, where two wavefronts bring the same one, so that every wavefront
  // has the same 2 NIK + 1 loads in flight
  const int wr = wv % G::NCR, row_r = (64 * wr + lane) / RC;
  const uint32_t src_r = 8 * (((64 * wr + lane) % RC) ^ swz_rows16<RC>(row_r));
  // ---- where this lane reads: key rows 16 sb + l16 (piece 4 kk + g), value rows 4g + l16/4 (+16)
  const uint32_t k_row_off = (uint32_t)(l16 * VC * 16), k_swz = (uint32_t)(swz_rows16<VC>(l16) ^ g) << 4;
  const uint32_t r_row_off = (uint32_t)(l16 * RC * 16), r_swz = (uint32_t)(swz_rows16<RC>(l16) ^ g) << 4;
  const int v_row = 4 * g + (l16 >> 2);
  const uint32_t v_row_off = (uint32_t)(v_row * VC * 16 + 8 * (l16 & 1));
  const uint32_t v_swz = (uint32_t)(swz_tr<VC>(v_row) ^ ((l16 & 3) >> 1)) << 4;

  const int m0 = __builtin_amdgcn_readfirstlane(job.block) * BM;
  if (m0 >= len) {  // padding rows only
    const int rows = T - m0 < BM ? T - m0 : BM;
    for (int i = tid; i < rows * (DH / 4); i += NT) {
      const size_t row = (size_t)(m0 + i / (DH / 4));
      if constexpr (LAYER)
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.out16) + (((size_t)b * T + row) * nh + h) * DH + 4 * (i % (DH / 4))) =
            make_uint2(0u, 0u);
      else
        *reinterpret_cast<float4_t*>(out + row * out_stride + 4 * (i % (DH / 4))) = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    return;
  }
  // ---- the columns: slots j < (p0 + last row) / s (a slot of the past: row j; one closed inside the chunk: the
  // chunk's row j*s + s-1 - p0)
  const int m_last = (m0 + BM < len ? m0 + BM : len) - 1;
  const int n_cols = (p0 + m_last) / s, n_tiles = (n_cols + BN - 1) / BN;
  // source row of column c (columns past the last one: a readable duplicate)
  auto src_row = [&](int c) -> uint32_t {
    c = c < n_cols ? c : n_cols - 1;
    return (uint32_t)(c < j0 ? c : past + c * s + s - 1 - p0);
  };
  // this wavefront's part of tile t on its way into buffer t % NBUF: 2 NIK + 1 loads.  Tiles are asked for in order; while
  // their rows are at one distance (`rs`: 1 among the slots of the past, s among the chunk-final rows) the next
  // tile's addresses are the last one's plus a constant: uniform bases and lane offsets that stand.
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_byte_ptr)lds;
  int run_end = 0;              // tiles below it follow the bases as they are
  uint64_t base_k[NIK], base_v[NIK];              // (addresses)
  uint32_t at_r = 0;                              // of the RoPE keys' array (its bytes stay below 2^32)
  uint32_t step_k = 0, step_r = 0;                // bytes from a tile to the next (values as keys)
  uint32_t off_k = 0, off_v = 0, off_r = 0;       // bytes from a tile's first source row to the lane's piece
  auto start_run = [&](int t) {  // tile t begins a run of tiles whose rows are at one distance, or is one of its own
    const int c0 = BN * t;
    const bool in_past = CONT && c0 < j0;
    const int lim = in_past ? (j0 < n_cols ? j0 : n_cols) : n_cols;  // columns of this kind
    run_end = lim / BN;
    if (run_end <= t) return;
    const int rs = in_past ? 1 : s;
    const uint32_t row0 = in_past ? (uint32_t)c0 : (uint32_t)(past + c0 * s + s - 1 - p0);
    off_k = 2 * ((uint32_t)(row_k * rs) * kv_stride + src_k);
    off_v = 2 * ((uint32_t)(row_k * rs) * kv_stride + src_v);
    off_r = 2 * ((uint32_t)(row_r * rs) * DR + src_r);
#pragma unroll
    for (int i = 0; i < NIK; ++i) {
      base_k[i] = (uint64_t)(uintptr_t)kx + 2 * (uint64_t)(row0 + (uint32_t)(i * IROWS * rs)) * kv_stride;
      base_v[i] = (uint64_t)(uintptr_t)vx + 2 * (uint64_t)(row0 + (uint32_t)(i * IROWS * rs)) * kv_stride;
    }
    at_r = 2 * row0 * DR;
    step_k = 2 * (uint32_t)(BN * rs) * kv_stride;
    step_r = 2 * (uint32_t)(BN * rs) * DR;
  };
  auto issue = [&](int t) {
    const uint32_t buf = lds_addr + (uint32_t)(t % NBUF) * (uint32_t)G::BYTES;
    if (t >= run_end) start_run(t);
    if (t < run_end) {
#pragma unroll
      for (int i = 0; i < NIK; ++i) {
        const uint32_t chunk = (uint32_t)((wv + NW * i) * 1024);
        load_to_lds_16(reinterpret_cast<const void*>(base_k[i]), off_k, buf + G::K_OFF + chunk);
        load_to_lds_16(reinterpret_cast<const void*>(base_v[i]), off_v, buf + G::V_OFF + chunk);
        base_k[i] += step_k;
        base_v[i] += step_k;
      }
      load_to_lds_16(reinterpret_cast<const unsigned char*>(kr16) + at_r, off_r, buf + G::R_OFF + (uint32_t)(wr * 1024));
      at_r += step_r;
      return;
    }
#pragma unroll
    for (int i = 0; i < NIK; ++i) {
      const uint32_t srow = src_row(BN * t + row_k + i * IROWS);
      const uint32_t chunk = (uint32_t)((wv + NW * i) * 1024);
      load_to_lds_16(kx + srow * kv_stride + src_k, buf + G::K_OFF + chunk);
      load_to_lds_16(vx + srow * kv_stride + src_v, buf + G::V_OFF + chunk);
    }
    load_to_lds_16(kr16 + src_row(BN * t + row_r) * DR + src_r, buf + G::R_OFF + (uint32_t)(wr * 1024));
  };

  // the first tiles travel while the rows are set up
#pragma unroll
  for (int t = 0; t < 2; ++t)
    if (n_tiles > 0) issue(t);

  // ---- queries of this wavefront's 32 rows: B operand, lane = row l16 of row tile rt; the row's own column.
  // They come in with four neighbouring lanes to 64 bytes of a row and change places through the wavefront's part of the buffers
  // that the second pair of tiles will take: in the operand layout neighbouring lanes are 16 rows, which a unit's address path takes one
  // lane a cycle (66 cycles a load, 10 thousand a block; now 2.5).  Stores likewise, see below.
  u32x4_t qf[RT][KQ];
  float4_t neg_ref[RT];        // - reference of the row's weights, where the logits' sums start
  float l_run[RT];
  float4_t acc[RT][MT];
  int bound[RT];               // columns open to the lane's rows
  {
    int ln = lane;
    asm volatile("" : "+v"(ln));              // (what depends on it is formed here, not kept in registers over the tile loop)
    const int qr = ln >> 2, qc = ln & 3;      // row and 16 bytes of the 64 that a load brings of it
    u32x4_t qd[RT][KQ], kd[RT][KQ], vd[RT][KD];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int m = m0 + 16 * RT * wv + 16 * rt + qr, mr = m < len ? m : len - 1;
      const size_t row = (size_t)b * T + mr;
      const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + (row * nh + h) * DH + 8 * qc;
      const uint16_t* qrp = reinterpret_cast<const uint16_t*>(a.q_rope) + (row * nh + h) * DR + 8 * qc;
      const uint32_t own = (uint32_t)(past + mr);
      const uint16_t* kp = kx + own * kv_stride + 8 * qc;
      const uint16_t* krp = kr16 + own * DR + 8 * qc;
      const uint16_t* vp = vx + own * kv_stride + 8 * qc;
#pragma unroll
      for (int kk = 0; kk < KQ; ++kk) {
        qd[rt][kk] = kk < KD ? *reinterpret_cast<const u32x4_t*>(qp + 32 * kk) : *reinterpret_cast<const u32x4_t*>(qrp + 32 * (kk - KD));
        kd[rt][kk] = kk < KD ? *reinterpret_cast<const u32x4_t*>(kp + 32 * kk) : *reinterpret_cast<const u32x4_t*>(krp + 32 * (kk - KD));
      }
#pragma unroll
      for (int kk = 0; kk < KD; ++kk) vd[rt][kk] = *reinterpret_cast<const u32x4_t*>(vp + 32 * kk);
    }
    unsigned char* own_lds = lds + 2 * G::BYTES + wv * kOwn;  // [query pieces | value pieces][row][64 bytes]
    unsigned char* to = own_lds + qr * 64 + ((qc ^ swz_rows16<4>(qr)) << 4);
    const unsigned char* from = own_lds + l16 * 64;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      __builtin_amdgcn_sched_barrier(0);
      const int m = m0 + 16 * RT * wv + 16 * rt + l16;
      bound[rt] = (p0 + (m < len ? m : len - 1)) / s;
      float e = 0.f;
#pragma unroll
      for (int kk = 0; kk < KQ; ++kk) {
        // logits come out in units of log2: log2(e) / sqrt(d_h) folded in
        if (!LAYER) qd[rt][kk] = bf16x8_to_f16x8(qd[rt][kk], a.scale_log2);
        e = dot8(kd[rt][kk], qd[rt][kk], e);
        *reinterpret_cast<u32x4_t*>(to + 1024 * kk) = qd[rt][kk];
      }
#pragma unroll
      for (int kk = 0; kk < KD; ++kk) *reinterpret_cast<u32x4_t*>(to + 1024 * (KQ + kk)) = vd[rt][kk];
      __builtin_amdgcn_wave_barrier();
      e = group_reduce<4>(e, LaneSum());
      e = __int_as_float(__builtin_amdgcn_ds_bpermute(16 * l16, __float_as_int(e)));  // of row l16: lane 4 l16
      neg_ref[rt] = float4_t{-e, -e, -e, -e};
      l_run[rt] = g == 0 ? 1.f : 0.f;  // the four lanes of a row sum their own columns' weights
#pragma unroll
      for (int kk = 0; kk < KQ; ++kk) qf[rt][kk] = *reinterpret_cast<const u32x4_t*>(from + 1024 * kk + ((g ^ swz_rows16<4>(l16)) << 4));
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {  // dims 16 mt + 4g ..
        const uint2 v = *reinterpret_cast<const uint2*>(from + 1024 * (KQ + (mt >> 1)) + (((2 * (mt & 1) + (g >> 1)) ^ swz_rows16<4>(l16)) << 4) + 8 * (g & 1));
        acc[rt][mt] = float4_t{f16_lo_to_f32(v.x), f16_hi_to_f32(v.x), f16_lo_to_f32(v.y), f16_hi_to_f32(v.y)};
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read before the barrier behind which those buffers are filled
  }
  // columns open to all of the wavefront's rows, and to any of them
  const int all_below = (p0 + m0 + 16 * RT * wv) / s;
  const int none_from = (p0 + m0 + 16 * RT * wv + 16 * RT - 1) / s;

  // Two tiles per step: while one pair is multiplied the other is on its way (four buffers), one wait and one barrier for
  // both, and the matrix products of one tile beside the softmax arithmetic of the other.
  for (int t = 0; t < n_tiles; t += 2) {
    wait_loads_but<0>();                  // the pair has landed: this wavefront's part, then everyone's
    barrier_only();
    if (t + 2 < n_tiles) {                // into the buffers the pair before was read from: every wavefront is past that
      issue(t + 2);
      issue(t + 3);
    }
    if (BN * t >= none_from) continue;    // above all of this wavefront's rows

    const uint32_t buf = (uint32_t)(t & 2) * (uint32_t)G::BYTES;  // byte offset of the pair in `lds`
    const unsigned char* kb = lds + buf + G::K_OFF + k_row_off;
    const unsigned char* rb = lds + buf + G::R_OFF + r_row_off;
    const unsigned char* vb = lds + buf + G::V_OFF + v_row_off;
    auto read_k = [&](int u, int kk, int sb) -> u32x4_t {  // tile t + u: [k | k^R] rows 16 sb + l16, elements 32 kk + 8g ..
      return kk < KD ? *reinterpret_cast<const u32x4_t*>(kb + u * G::BYTES + sb * (16 * VC * 16) + ((uint32_t)(64 * kk) ^ k_swz))
                     : *reinterpret_cast<const u32x4_t*>(rb + u * G::BYTES + sb * (16 * RC * 16) + ((uint32_t)(64 * (kk - KD)) ^ r_swz));
    };
    auto read_v = [&](int u, int mt) -> u32x4_t {  // V^T rows 16 mt + l16 (dims), columns 8g .. (K index of the PV product)
      const unsigned char* p = vb + u * G::BYTES + ((uint32_t)(32 * mt) ^ v_swz);
      const short4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)p);
      const short4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(p + 16 * VC * 16));
      const uint2 u0 = __builtin_bit_cast(uint2, v0), u1 = __builtin_bit_cast(uint2, v1);
      return u32x4_t{u0.x, u0.y, u1.x, u1.y};
    };

    // ---- S^T[col, row] - reference = [k | k^R][col, :] . [q | q^R][row, :]: the reads of one group of K
    // steps are in flight while the group before is multiplied
    float4_t sacc[2][RT][2];  // [tile][row tile][16 columns]
    constexpr int KG = 2, NG = 2 * KQ / KG;  // K steps per group, groups of both tiles
    static_assert(KQ % KG == 0 || KQ % 2 == 1, "groups");
    u32x4_t kf[2][KG][2];
    auto read_group = [&](int i) {
#pragma unroll
      for (int j = 0; j < KG; ++j)
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
          const int x = i * KG + j;
          kf[i & 1][j][sb] = read_k(x / KQ, x % KQ, sb);
        }
    };
    __builtin_amdgcn_s_setprio(1);  // the stretch of matrix instructions ahead of the other wavefront's arithmetic (1 - 2 %)
    read_group(0);
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      if (i + 1 < NG) read_group(i + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < KG; ++j)
#pragma unroll
        for (int sb = 0; sb < 2; ++sb)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            const int x = i * KG + j, u = x / KQ, kk = x % KQ;
            sacc[u][rt][sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, kf[i & 1][j][sb]),
                                                                     __builtin_bit_cast(f16x8_t, qf[rt][kk]),
                                                                     kk == 0 ? neg_ref[rt] : sacc[u][rt][sb], 0, 0, 0);
          }
    }
    constexpr int VPRE = MT / 2;
    u32x4_t vf[MT];  // values of the tile whose product comes next
#pragma unroll
    for (int mt = 0; mt < VPRE; ++mt) vf[mt] = read_v(0, mt);
    __builtin_amdgcn_sched_barrier(0);

    __builtin_amdgcn_s_setprio(0);
    // ---- softmax weights: lane holds row l16 of row tile rt and columns 16 sb + 4g + v
    if (BN * t + 2 * BN > all_below) {  // wavefront-uniform: the last tiles only
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const int d = bound[rt] - (BN * (t + u) + 4 * g);
#pragma unroll
          for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int v = 0; v < 4; ++v) sacc[u][rt][sb][v] = 16 * sb + v < d ? sacc[u][rt][sb][v] : -INFINITY;
        }
    }
    // fixed reference per row (its own column's logit, re-based only when a tile tops it by more than 2^kRebase): no
    // accumulator rescaling and no cross-lane traffic per tile.  Weights more than 2^-24 below the reference
    // vanish in fp16; they are that much smaller than weights already summed.
    constexpr float kRebase = 12.f;  // fp16 weights: 2^(s - reference) stays far below 65504
    // Does any logit top it?  On the bit patterns: as integers the positive floats are in order and above all negative
    // ones, and an integer maximum takes three operands without first quieting each.
    int top = 0;
#pragma unroll
    for (int i = 0; i < 16 * RT; ++i) {
      const float x = sacc[i / (8 * RT)][(i >> 3) % RT][(i >> 2) & 1][i & 3];
      top = max(top, __float_as_int(x));
    }
    if (__any(top > __float_as_int(kRebase))) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        float up = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) up = fmaxf(up, sacc[i >> 3][rt][(i >> 2) & 1][i & 3]);
        up = quarter_reduce(up, LaneMax());
        if (up > kRebase) {
          const float alpha = __builtin_amdgcn_exp2f(-up);
          neg_ref[rt] -= up;
          l_run[rt] *= alpha;
#pragma unroll
          for (int i = 0; i < 4; ++i) sacc[i >> 1][rt][i & 1] -= up;
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[rt][mt] *= alpha;
        }
      }
    }
    const f16x2_t ones = {(_Float16)1.f, (_Float16)1.f};
    auto weights = [&](int u, int rt) -> u32x4_t {  // B operand of the K = 32 PV product
      // K index 8g + e of the tile: e < 4 -> column 4g + e of its first 16, else of its second 16
      u32x4_t pb;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4_t& x = sacc[u][rt][i >> 1];
        const uint32_t two = pack_f16x2(__builtin_amdgcn_exp2f(x[2 * (i & 1)]), __builtin_amdgcn_exp2f(x[2 * (i & 1) + 1]));
        pb[i] = two;
        l_run[rt] = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2_t, two), ones, l_run[rt], false);  // the weights as they are used
      }
      return pb;
    };
    auto product = [&](int mt, const u32x4_t& v, const u32x4_t (&pb)[RT]) {  // O^T[d, row] += V^T[d, col] P^T[col, row]
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        acc[rt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, v), __builtin_bit_cast(f16x8_t, pb[rt]),
                                                             acc[rt][mt], 0, 0, 0);
    };
    u32x4_t pb0[RT], pb1[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) pb0[rt] = weights(0, rt);
#pragma unroll
    for (int mt = VPRE; mt < MT; ++mt) vf[mt] = read_v(0, mt);
    // the weights of the second tile beside the first tile's product
    pb1[0] = weights(1, 0);
#pragma unroll
    for (int mt = 0; mt < VPRE; ++mt) product(mt, vf[mt], pb0);
#pragma unroll
    for (int mt = 0; mt < VPRE; ++mt) vf[mt] = read_v(1, mt);
    if constexpr (RT == 2) pb1[1] = weights(1, 1);
#pragma unroll
    for (int mt = VPRE; mt < MT; ++mt) product(mt, vf[mt], pb0);
#pragma unroll
    for (int mt = VPRE; mt < MT; ++mt) vf[mt] = read_v(1, mt);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) product(mt, vf[mt], pb1);
  }

  // ---- normalise and store: lane holds row l16 of row tile rt, output dims 16 mt + 4g .. +3.  The rows leave through LDS, whole
  // lines at a time (as they stand, a store is 64 bytes of 16 rows, 67 cycles of the address path), in the wavefront's part of the pair
  // of buffers that the last step did not read: every wavefront is past the step before it.
  int ln = lane;
  asm volatile("" : "+v"(ln));
  unsigned char* leave = lds + (n_tiles > 0 ? (~(n_tiles - 1) & 2) : 0) * G::BYTES + wv * kOwn;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    constexpr int ES = LAYER ? 2 : 4, RB = DH * ES, PPR = RB / 16;  // bytes of a row, 16-byte pieces; piece j of row i sits at j ^ (i % 16), in RB
    static_assert(16 * RB <= kOwn && PPR >= 8, "the rows fit");
    const float l = quarter_reduce(l_run[rt], LaneSum());
    const int mt0 = m0 + 16 * RT * wv + 16 * rt;
    const bool live = mt0 + (ln & 15) < len;  // rows past the sequence's length are zeros, whatever their inputs held
    const float inv = live ? 1.f / l : 0.f;
    constexpr int SW = PPR < 16 ? PPR - 1 : 15;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const float4_t o = live ? acc[rt][mt] * inv : float4_t{0.f, 0.f, 0.f, 0.f};
      if constexpr (LAYER)
        *reinterpret_cast<uint2*>(leave + (ln & 15) * RB + (((2 * mt + ((ln >> 5) & 1)) ^ (ln & SW)) << 4) + 8 * ((ln >> 4) & 1)) = make_uint2(pack_f16x2(o[0], o[1]), pack_f16x2(o[2], o[3]));
      else
        *reinterpret_cast<float4_t*>(leave + (ln & 15) * RB + (((4 * mt + (ln >> 4)) ^ (ln & SW)) << 4)) = o;
    }
    __builtin_amdgcn_wave_barrier();
    unsigned char* out_rows = LAYER ? reinterpret_cast<unsigned char*>(a.out16) + (((size_t)b * T + mt0) * nh + h) * RB
                                    : reinterpret_cast<unsigned char*>(out) + (size_t)mt0 * out_stride * 4;
#pragma unroll
    for (int i = 0; i < 16 * PPR / 64; ++i) {
      const int at = 64 * i + ln, row = at / PPR, c = at % PPR;
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(leave + row * RB + ((c ^ (row & SW)) << 4));
      unsigned char* to = out_rows + (size_t)row * out_stride * ES + 16 * c;
      if (mt0 + row < T) {
        if (!LAYER && a.stream_out) {  // (as a store of its own kind: the compiler makes one of two that differ in a hint)
          const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(out_rows, 0, 16 * (int)out_stride * ES, 0x00027000);
          __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)(to - out_rows), 0, 2 /* nt */);
        } else {
          *reinterpret_cast<u32x4_t*>(to) = v;
        }
      }
    }
  }
}

template <int DH, int DR>
hipError_t launch_attn_explicit(const ExplicitArgs& a, hipStream_t st, const EventPair& ev) {
  constexpr int NW = 4;
  static_assert(32 * NW == kAttnRows, "rows of a block");
  const int pairs = a.n_heads * a.batch, rows = attn_rows(a.T, pairs, DH, a.past_pitch);
  const int n_blocks = (a.T + rows - 1) / rows;
  ExplicitArgs x = a;
  x.group = attn_group(pairs, DH, attn_at_once(rows, pairs, n_blocks, DH, a.past_pitch));
  // Outputs past the caches where what reads them next would hardly find them there.  us a pass, ordinary / past the caches, alone and with an elementwise
  // pass over them behind it: 8 prompts of 4096, 16 heads x 128 (268 MB) 556 / 548 and 636 / 635, of 2400 (157 MB) 290 / 278 and 344 / 342; 8 of 1000, 12 heads (49 MB)
  // 77.2 / 75.5 and 92.0 / 93.1.
  x.stream_out = !a.out16 && (size_t)a.batch * a.T * a.n_heads * DH * 4 > kStreamOut;
  const dim3 grid((unsigned)n_blocks * (unsigned)(attn_pairs(pairs) * kXcds));
  const size_t more_lds = attn_two_a_unit(rows, pairs, n_blocks, a.T, a.stride, DH, a.past_pitch) ? 20 * 1024 : 0;  // (three of 60 KB do not fit)
  const bool layer = a.q_f16 != 0;  // comes with out16
  if (layer != (a.out16 != nullptr) || (layer && !a.pos0)) return hipErrorInvalidValue;
  auto launch = [&](auto cont, auto lay) {
    constexpr bool C = decltype(cont)::value, L = decltype(lay)::value;
    if (rows == kAttnRows / 2) launch_timed(attn_explicit_kernel<DH, DR, NW, C, L, 1>, grid, dim3(64 * NW), more_lds, st, ev, x);
    else launch_timed(attn_explicit_kernel<DH, DR, NW, C, L, 2>, grid, dim3(64 * NW), more_lds, st, ev, x);
  };
  if (layer) launch(std::true_type(), std::true_type());
  else if (a.pos0) launch(std::true_type(), std::false_type());
  else launch(std::false_type(), std::false_type());
  return hipGetLastError();
}

}  // namespace

bool prefill_explicit_supported(const ExplicitArgs& a) {
  return (a.d_head == 64 || a.d_head == 128) && (a.d_rope == 32 || a.d_rope == 64) && a.r % 64 == 0 && a.r >= 64 &&
         a.r <= 512 && a.n_heads <= 65535 && a.batch <= 65535 &&
         (size_t)((a.T + 127) / 128) * ((size_t)a.n_heads * a.batch + 7) < (size_t)1 << 31 &&  // workgroups of the attention launch
         (!a.out_latent || ((a.r & (a.r - 1)) == 0 && !a.pos0 && !a.q_f16)) &&
         (size_t)(a.past_pitch + a.T) * a.n_heads * a.d_head < (size_t)1 << 31 &&  // 32-bit element offsets inside one sequence
         (size_t)a.batch * (a.past_pitch + a.T) < (size_t)1 << 31;                 // rows of the key / value product
}

bool gemm_nt_supported(const GemmArgs& a) {
  if (a.M < 1 || a.K < 32 || a.K % 32 != 0 || a.n_seg < 1 || a.n_seg > GemmArgs::kSegments) return false;
  size_t blocks = 0;
  for (int i = 0; i < a.n_seg; ++i) {
    const GemmSegment& g = a.seg[i];
    if (g.N < 8 || g.N % 8 != 0 || !(g.epi >= 0 && g.epi <= 3)) return false;
    if ((g.epi == 1 || g.epi == 2) && (!a.in_bf16 || a.d_rope % 4 != 0 || a.d_rope < 4 || a.d_rope > 64 || !a.rope_cs || g.N % a.d_rope != 0)) return false;
    blocks += (size_t)(g.N + 63) / 64;
  }
  if (!gemm_turned_rows_supported(a)) return false;
  if (a.rows.T < 1 || ((a.rows.n_new || a.rows.pos0) && a.M % (a.rows.past + a.rows.T) != 0)) return false;
  const size_t n_seq = a.rows.n_new || a.rows.pos0 ? (size_t)a.M / (a.rows.past + a.rows.T) : 1;
  return blocks * ((size_t)(a.M + 63) / 64 + n_seq + 8) < (size_t)1 << 31;
}

// (cos, sin) of pos * freq[k] for row b*T + t at position pos0[b] + t, k < d_rope / 2
__global__ __launch_bounds__(kBlock) void rope_table_kernel(RopeTableArgs a) {
  const size_t idx = (size_t)blockIdx.x * kBlock + threadIdx.x;
  const int half = a.d_rope / 2;
  if (idx >= a.rows * half) return;
  const size_t row = idx / half;
  const int k = int(idx % half), b = int(row / a.T);
  const int pos = (a.pos0 ? a.pos0[b] : 0) + int(row - (size_t)b * a.T);
  a.table[idx] = rope_angle(pos, a.rope_freq[k]);
}

namespace {

hipError_t launch_rope_table(const GemmArgs& g, hipStream_t st) {
  RopeTableArgs a;
  a.pos0 = g.rope_pos0;
  a.table = g.rope_cs;
  a.rows = (size_t)g.M;
  a.T = g.rows.T;
  a.d_rope = g.d_rope;
  for (int k = 0; k < 32; ++k) a.rope_freq[k] = g.rope_freq[k];
  const size_t n = a.rows * (a.d_rope / 2);
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_gemm(const GemmArgs& args, bool part, hipStream_t st) {
  GemmArgs a = args;
  const GemmPlan plan = gemm_plan(a, part, gemm_wide_supported);
  if (plan.ring) return launch_gemm_ring(a, st);
  const bool turned = gemm_turns(a);
  auto table = [&]() {
    a.rope_ready = 1;
    return launch_rope_table(a, st);
  };
  if (plan.alone >= 0) {
    GemmArgs one, rest;
    gemm_without(a, plan.alone, one, rest);
    hipError_t e = turned && !a.rope_ready ? table() : hipSuccess;  // one for both
    one.rope_ready = rest.rope_ready = a.rope_ready;
    if (e == hipSuccess) e = launch_gemm(rest, true, st);
    return e != hipSuccess ? e : launch_gemm(one, true, st);
  }
  const int pick = plan.pick;
  if (turned && !a.rope_ready && (pick == kWide || !gemm_own_angles(kGemmTiles[pick].bm, kGemmTiles[pick].bn))) {
    const hipError_t e = table();
    if (e != hipSuccess) return e;
  }
  if (pick == kWide) return launch_gemm_wide(a, st);
  const int bm = kGemmTiles[pick].bm;
  a.col_blocks = gemm_col_blocks(a, kGemmTiles[pick].bn);
  unsigned gy = (unsigned)((a.M + bm - 1) / bm);
  if ((a.rows.n_new || a.rows.pos0) && !a.rows.zeros) {  // every sequence starts a block of its own
    const int Tp = a.rows.past + a.rows.T;
    gy = (unsigned)(a.M / Tp) * (unsigned)((Tp + bm - 1) / bm);
  }
  a.row_blocks = gy;
  a.xcds = gy >= 8 ? 8 : 1;
  const dim3 grid((unsigned)a.col_blocks * ((gy + a.xcds - 1) / a.xcds * a.xcds));
#define MTLA_GEMM(I, BM, BN)                                                                                     \
  if (pick == I) {                                                                                               \
    const dim3 block(GemmGeom<BM, BN>::NT);                                                                      \
    if (a.in_bf16) hipLaunchKernelGGL((gemm_nt_kernel<true, BM, BN>), grid, block, 0, st, a);                    \
    else hipLaunchKernelGGL((gemm_nt_kernel<false, BM, BN>), grid, block, 0, st, a);                             \
  }
  MTLA_GEMM(0, 256, 256)
  MTLA_GEMM(1, 256, 128)
  MTLA_GEMM(2, 128, 128)
  MTLA_GEMM(3, 64, 64)
#undef MTLA_GEMM
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_nt(const GemmArgs& a, hipStream_t st) {
  return gemm_nt_supported(a) ? launch_gemm(a, false, st) : hipErrorInvalidValue;
}

// the front launch has filled a.cprime, a.kr16 ([B*(past_pitch + T), ..]), a.w_kT and a.w_v16
hipError_t launch_prefill_explicit(const ExplicitArgs& a, hipStream_t st, const EventPair& ev) {
  GemmArgs ga;  // K = C_hat' W_K, V = C_hat' W_V for all rows that hold something
  ga.A = a.cprime;
  ga.M = a.batch * (a.past_pitch + a.T);
  ga.K = a.r;
  ga.n_seg = 2;
  for (int i = 0; i < 2; ++i) {
    ga.seg[i].W = i ? a.w_v16 : a.w_kT;
    ga.seg[i].C = i ? a.vx : a.kx;
    ga.seg[i].N = a.n_heads * a.d_head;
  }
  ga.rows.pos0 = a.pos0;
  ga.rows.n_new = a.seq_len;
  ga.rows.past = a.past_pitch;
  ga.rows.T = a.T;
  ga.rows.stride = a.stride;
  hipError_t e = launch_gemm_nt(ga, st);
  if (e != hipSuccess) return e;
  auto attend = [&](const ExplicitArgs& x, const EventPair& e) -> hipError_t {
    if (x.d_head == 64 && x.d_rope == 32) return launch_attn_explicit<64, 32>(x, st, e);
    if (x.d_head == 64 && x.d_rope == 64) return launch_attn_explicit<64, 64>(x, st, e);
    if (x.d_head == 128 && x.d_rope == 32) return launch_attn_explicit<128, 32>(x, st, e);
    if (x.d_head == 128 && x.d_rope == 64) return launch_attn_explicit<128, 64>(x, st, e);
    return hipErrorInvalidValue;
  };
  return a.out_latent ? launch_attn_latent(a, st, ev) : attend(a, ev);
}

}  // namespace mtla
