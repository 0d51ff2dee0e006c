// bf16 matrix-core decode attention over the cache slots (gfx950).
//
// Eq. (with-rope), incremental case: all heads of a sequence share each cached
// row (C_hat[k], K_hat^R[k]), so the pass over the cache is two small dense
// contractions per 16-slot tile with the heads as one matrix dimension:
//     S^T[slot, head] = [C_hat | K_hat^R][slot, :] . [q~ | q^R][head, :]      (K = r + d_R)
//     O^T[col,  head] += C_hat^T[col, slot] . P^T[slot, head]                  (K = 16 slots)
// Each wavefront of a workgroup streams its own 16-slot tiles and keeps its own
// online-softmax state; there is no workgroup barrier inside the loop.  Per
// tile and wavefront:
//   * the tile and the query operand are loaded from memory straight into the
//     operand layouts of v_mfma_f32_16x16x32_bf16 (lane = row, 8 consecutive
//     elements of the contraction), so the logits need no staging at all; the
//     query comes as two bf16 planes (hi + lo, an almost-fp32 value), one MFMA
//     chain each, so the only rounding left in the logits is the cache's own;
//   * S^T leaves the matrix core with lane = head column and 4 consecutive slots
//     per lane, which is exactly the B-operand layout of the K=16 bf16 MFMA, so
//     the probabilities never leave registers;
//   * the latent part of the tile is parked in a wavefront-private LDS region
//     and read back transposed (ds_read_b64_tr_b16) as the C_hat^T operand.
// At the end of a piece every wavefront drops its unnormalised state into LDS
// and the whole workgroup sums the copies into one partial (m, l, o[r]) per
// (piece, head).
//
// Where this file is used: the static schedule below is the decode kernel for small batches; for
// large or ragged batches and for the parallel form the column-split kernels take over whenever
// r >= 128, and the balanced and per-row kernels of this file remain for r = 64.
//
// Two schedules share that inner loop:
//   static    grid (chunks, sequences): workgroup (c, b) scans slots
//             [c*chunk, (c+1)*chunk) of sequence b.  For decode at small batch,
//             where a wavefront sees a tile or two and the kernel is all latency:
//             a single wavefront issues at most one instruction every four
//             cycles, so the code is kept short -- one round trip to memory for
//             everything whose address does not depend on the sequence length,
//             hardware bf16 conversion and exp2, a fixed softmax reference per
//             wavefront instead of a running maximum (no accumulator rescaling and no
//             cross-lane traffic on the hot path), and a single-pass merge.  Up to 16
//             heads with short chunks have a kernel of their own (attn_split_kernel), in
//             which the wavefronts share their rows and weights through LDS instead.
//   balanced  one persistent workgroup per compute unit.  The tiles of all
//             sequences form one flat list that is cut into equal ranges, so
//             ragged batches keep every compute unit streaming until the end; a
//             workgroup emits one partial per sequence its range touches.
#include "bounds.h"
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kWaves = kBlock / kWave;
constexpr int kTile = 16;  // slots per wavefront tile

template <int R_, int DR_, int NHT_>
struct MfmaCfg {
  static constexpr int R = R_, DR = DR_, NHT = NHT_;
  static constexpr int E = R + DR;
  static constexpr int HP = 16 * NHT;       // heads padded to whole 16-row tiles
  static constexpr int WPT = kWaves / NHT;  // wavefronts sharing one head tile
  static constexpr int KC = R / 32;         // K steps over the latent part
  static constexpr int KR = DR / 32;        // K steps over the RoPE part
  static constexpr int KT = KC + KR;
  static constexpr int MT = R / 16;         // output column tiles
  static constexpr int TS = R + 16;         // tile row stride: 2R+32 bytes, 8 words mod 64 banks
  static constexpr int OS = R + 4;          // merge row stride (floats)
  static constexpr int QS = E + 8;          // query row stride in LDS (bf16 elements)
  static constexpr int kStep = WPT * kTile; // slots between consecutive tiles of one wavefront
  static constexpr size_t tile_bytes = (size_t)kWaves * kTile * TS * 2;
  static constexpr size_t merge_bytes = (size_t)kWaves * 16 * OS * 4;  // one copy per wavefront
  static constexpr size_t q_bytes = (size_t)2 * HP * QS * 2;  // hi and lo planes
  // loop phase: tile regions (+ the query when it sits in LDS); merge phase reuses the space
  static constexpr size_t body_bytes(bool ql) {
    const size_t loop = tile_bytes + (ql ? q_bytes : 0);
    return loop > merge_bytes ? loop : merge_bytes;
  }
  static constexpr size_t ml_bytes = (size_t)2 * kWaves * 16 * 4;
};

template <class C>
struct TileRegs {
  uint4 xc[C::KC], xr[C::KR];
  __device__ __forceinline__ void select_live(bool keep) {  // dead rows become exact zeros
    const uint32_t m = keep ? 0xffffffffu : 0u;
#pragma unroll
    for (int kk = 0; kk < C::KC; ++kk) xc[kk] = make_uint4(xc[kk].x & m, xc[kk].y & m, xc[kk].z & m, xc[kk].w & m);
#pragma unroll
    for (int kk = 0; kk < C::KR; ++kk) xr[kk] = make_uint4(xr[kk].x & m, xr[kk].y & m, xr[kk].z & m, xr[kk].w & m);
  }
};

// How a wavefront's column index k maps to a row of the latent / key arrays.
//   decode  (stride == 0): column k is cache slot k.
//   prefill (stride == s): column k < nfin is the final state of chunk k, row k*s + s-1 of
//           C_hat'; the last column is the query row's own running state, row `own`
//           (exactly the columns the stride-aware causal mask leaves open).
struct Cols {
  int step;               // columns between consecutive tiles of this wavefront
  int stride, nfin, own;
  __device__ __forceinline__ int row(int k) const {
    return stride == 0 ? k : (k < nfin ? k * stride + stride - 1 : own);
  }
};

// Branch-free fetch of tile columns base + l16 (clamped to `last`): lane (l16, g) takes elements
// 32kk + 8g .. +7 of its row.  A clamped column is a duplicate of a readable one; its logits are
// masked to -inf in the softmax, so it contributes exact zeros.
// PG: paged storage (decode only): lat / key are the pool, and the tile's page comes out of the sequence's
// page-table row with one wavefront-uniform (scalar) load, clamped into the pool.
template <class C, bool SH = false, bool PG = false>
__device__ __forceinline__ void load_tile(TileRegs<C>& t, const uint16_t* lat, const uint16_t* key, int base,
                                          int last, int l16, int g, const Cols& cm,
                                          const SharedPrefix& sp = SharedPrefix{0, 0, 0},
                                          const PageRow& pr = PageRow{nullptr, 0, 0}) {
  const int slot = cm.row(base + l16 < last ? base + l16 : last);
  size_t row = (size_t)slot;
  if constexpr (PG) {
    const int s0 = __builtin_amdgcn_readfirstlane(base < last ? base : last);  // the tile, or the one every lane clamps to
    int pg = load_uniform_i32(pr.pt, s0 >> pr.shift);
    pg = pg < 0 ? 0 : (pg < pr.n_pages ? pg : pr.n_pages - 1);
    row = ((size_t)pg << pr.shift) + (size_t)(slot & ((1 << pr.shift) - 1));
  }
  const uint16_t* cr = lat + row * C::R + 8 * g;
  const uint16_t* kr = key + row * C::DR + 8 * g;
  if constexpr (SH) {  // decode only (cm.row is the identity there)
    if (slot < sp.n) {
      cr += sp.dlat;
      kr += sp.dkey;
    }
  }
#pragma unroll
  for (int kk = 0; kk < C::KC; ++kk) t.xc[kk] = *reinterpret_cast<const uint4*>(cr + 32 * kk);
#pragma unroll
  for (int kk = 0; kk < C::KR; ++kk) t.xr[kk] = *reinterpret_cast<const uint4*>(kr + 32 * kk);
}

// Per-wavefront attention state over the tiles it has seen.
template <class C>
struct WaveState {
  float m_ref, l_run;  // l_run: this lane's slots only, see l_total()
  float4_t acc_o[C::MT];
  __device__ __forceinline__ float l_total() const {  // normaliser of the lane's head
    return quarter_reduce(l_run, LaneSum());
  }
  __device__ __forceinline__ void reset() {
    m_ref = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) acc_o[mt] = float4_t{0.f, 0.f, 0.f, 0.f};
  }
};

// Streams this wavefront's tiles base, base + kStep, ... below k1 through the two contractions.
// tl[0..NS) hold the first NS tiles on entry (register-staged software pipeline).  Every
// iteration runs all NS stages and every stage refills itself unconditionally (row indices are
// clamped, dead tiles are masked): with a fixed number of loads between a tile's request and its
// use, the compiler can wait for exactly that tile and leave the younger requests in flight.  At
// most NS-1 dead tiles are processed at the end.
// QM says where the two query planes live: 0 = both in registers (qv[0..KT) hi, qv[KT..2KT) lo),
// 1 = both in LDS (qrow: hi row, lo row HP*QS further), 2 = hi in registers, lo in LDS (qrow).
constexpr int kQRegs = 0, kQLds = 1, kQMixed = 2;
template <class C, int QM>
struct QRegCount {
  static constexpr int value = QM == kQRegs ? 2 * C::KT : (QM == kQLds ? 1 : C::KT);
};

// Where a wavefront's tile stream continues once its run [base, k1) is used up: the refills of
// the last NS tiles fetch tiles base, base + step, ... of `lat` / `key` (columns clamped to
// `last`) instead of dead duplicates, so the caller finds the first NS tiles of its next run in
// tl[] -- requested a whole tile pass before they are needed.  A caller without a next run points
// it at the current arrays with base > last (every column clamps to a readable row).
struct NextRun {
  const uint16_t* lat;
  const uint16_t* key;
  int base, last;
  PageRow pr = PageRow{nullptr, 0, 0};  // paged storage: the next run's page-table row
};

template <class C, int NS, int QM, bool SH = false, bool PG = false>  // SH: `sp` applies to this run and to the next one (same sequence)
__device__ __forceinline__ void stream_tiles(TileRegs<C> (&tl)[NS], const uint4 (&qv)[QRegCount<C, QM>::value],
                                             const uint16_t* qrow, uint16_t* sTw, const uint16_t* lat,
                                             const uint16_t* key, int base, int k1, int l16, int g,
                                             const Cols& cm, WaveState<C>& ws, const NextRun& nx,
                                             const SharedPrefix& sp = SharedPrefix{0, 0, 0},
                                             const PageRow& pr = PageRow{nullptr, 0, 0}) {
  const int n_iter = (k1 - base + NS * cm.step - 1) / (NS * cm.step);  // <= 0 for an idle wavefront
  for (int it = 0; it < n_iter; ++it) {
    const bool tail = it == n_iter - 1;  // this pass refills from the next run
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      TileRegs<C>& t = tl[st];
      // ---- logits S^T[slot, head] for this tile (log2 units: the query is pre-scaled): one
      // accumulator chain for the hi plane of the query and one for the lo plane; query pieces
      // are fetched from LDS a group at a time so one wait covers a group of matrix instructions
      float4_t s0 = float4_t{0.f, 0.f, 0.f, 0.f}, s1 = float4_t{0.f, 0.f, 0.f, 0.f};
      constexpr int kQGroup = 3;
#pragma unroll
      for (int k0g = 0; k0g < C::KT; k0g += kQGroup) {
        uint4 qh[kQGroup], ql[kQGroup];
#pragma unroll
        for (int j = 0; j < kQGroup; ++j)
          if (k0g + j < C::KT) {
            const int kk = k0g + j;  // latent pieces first, then the RoPE pieces (contiguous in a row)
            qh[j] = QM == kQLds ? *reinterpret_cast<const uint4*>(qrow + 32 * kk) : qv[QM == kQLds ? 0 : kk];
            ql[j] = QM == kQRegs ? qv[QM == kQRegs ? C::KT + kk : 0]
                                 : *reinterpret_cast<const uint4*>(qrow + (QM == kQLds ? C::HP * C::QS : 0) + 32 * kk);
          }
#pragma unroll
        for (int j = 0; j < kQGroup; ++j)
          if (k0g + j < C::KT) {
            const int kk = k0g + j;
            const uint4 x = kk < C::KC ? t.xc[kk < C::KC ? kk : 0] : t.xr[kk < C::KC ? 0 : kk - C::KC];
            s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x),
                                                         __builtin_bit_cast(bf16x8_t, qh[j]), s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x),
                                                         __builtin_bit_cast(bf16x8_t, ql[j]), s1, 0, 0, 0);
          }
      }
      // ---- park the latent rows in this wavefront's LDS region (row = slot, as loaded)
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int kk = 0; kk < C::KC; ++kk)
        *reinterpret_cast<uint4*>(sTw + l16 * C::TS + 32 * kk + 8 * g) = t.xc[kk];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();

      // ---- refill this stage NS tiles ahead while the softmax and PV run
      load_tile<C, SH, PG>(t, tail ? nx.lat : lat, tail ? nx.key : key, tail ? nx.base + st * cm.step : base + NS * cm.step,
                           tail ? nx.last : k1 - 1, l16, g, cm, sp, tail ? nx.pr : pr);

      // ---- softmax weights; lane holds head l16 of its head tile and slots 4g..4g+3
      float sv[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) sv[v] = (base + 4 * g + v < k1) ? s0[v] + s1[v] : -INFINITY;
      // Weights are taken relative to a reference m_ref fixed at the wavefront's first live tile
      // instead of the running maximum: 2^(s - m_ref) has the whole fp32/bf16 exponent range to
      // grow into, so the accumulators are never rescaled on the hot path, and the hot path needs
      // no cross-lane traffic at all: the four lanes that share a head keep their own partial
      // normaliser (summed by l_total() at the end), and the tile maximum is only formed on the
      // two cold paths -- fixing the reference, and re-basing the state when a tile tops the
      // reference by more than 2^kRebase.
      constexpr float kRebase = 40.f;
      const float mloc = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
      if (__any(ws.m_ref == -INFINITY || mloc - ws.m_ref > kRebase)) {
        float mt_ = quarter_reduce(mloc, LaneMax());
        if (ws.m_ref == -INFINITY) {
          ws.m_ref = mt_;  // still -inf if the tile is dead
        } else if (mt_ - ws.m_ref > kRebase) {
          const float alpha = __builtin_amdgcn_exp2f(ws.m_ref - mt_);
          ws.m_ref = mt_;
          ws.l_run *= alpha;
#pragma unroll
          for (int mt = 0; mt < C::MT; ++mt) ws.acc_o[mt] *= alpha;
        }
      }
      const float m_sub = ws.m_ref == -INFINITY ? 0.f : ws.m_ref;  // nothing live yet: p = 2^-inf = 0
      float p[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) p[v] = __builtin_amdgcn_exp2f(sv[v] - m_sub);
      // weights as bf16 (hardware round-to-nearest-even); the normaliser sums the rounded values
      const uint32_t p01 = pack_bf16x2(p[0], p[1]), p23 = pack_bf16x2(p[2], p[3]);
      const short4_t pb = __builtin_bit_cast(short4_t, make_uint2(p01, p23));
      ws.l_run += (__uint_as_float(p01 << 16) + __uint_as_float(p01 & 0xffff0000u)) +
                  (__uint_as_float(p23 << 16) + __uint_as_float(p23 & 0xffff0000u));

      // ---- O^T[col, head] += C_hat^T[col, slot] P^T[slot, head], transposed operand from LDS.
      // Lane i of each 16-lane group points at row 4g + i/4, columns 4(i%4)..+3 of the column
      // tile; the transposing read hands lane i the four rows of column i.
      const uint16_t* trow = sTw + (4 * g + (l16 >> 2)) * C::TS + 4 * (l16 & 3);
#pragma unroll
      for (int mt = 0; mt < C::MT; ++mt) {
        const short4_t ct = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(trow + 16 * mt));
        ws.acc_o[mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ct, pb, ws.acc_o[mt], 0, 0, 0);
      }
      base += cm.step;
    }
  }
}

// Merge: every wavefront publishes (m, l, o) as it stands; the workgroup then sums the WPT copies
// of each head with weights 2^(m_w - m*) and writes the piece's partial.  The caller has made sure
// (barrier) that nobody still uses the LDS body, which sO aliases.
template <class C>
__device__ __forceinline__ void merge_store(const WaveState<C>& ws, float* sO, float* sM, float* sL, float* part_o,
                                            float* part_ml, size_t piece, int n_heads, int tid, int wv, int l16,
                                            int g) {
  const float l_head = ws.l_total();
  if (g == 0) {
    sM[wv * 16 + l16] = ws.m_ref;
    sL[wv * 16 + l16] = l_head;
  }
  {
    float* dst = sO + (size_t)(wv * 16 + l16) * C::OS + 4 * g;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) *reinterpret_cast<float4_t*>(dst + 16 * mt) = ws.acc_o[mt];
  }
  __syncthreads();
  const size_t pbase = piece * n_heads;
  constexpr int R4 = C::R / 4;
  for (int idx = tid; idx < n_heads * R4; idx += kBlock) {
    const int h = idx / R4, c4 = idx - h * R4;
    const int w0 = (h >> 4) * C::WPT, hl = h & 15;
    float mw[C::WPT], mstar = -INFINITY;
#pragma unroll
    for (int w = 0; w < C::WPT; ++w) {
      mw[w] = sM[(w0 + w) * 16 + hl];
      mstar = fmaxf(mstar, mw[w]);
    }
    float4_t o = float4_t{0.f, 0.f, 0.f, 0.f};
    float lstar = 0.f;
#pragma unroll
    for (int w = 0; w < C::WPT; ++w) {
      const float f = __builtin_amdgcn_exp2f(mw[w] - mstar);  // 0 for a wavefront that saw no slot
      o += f * *reinterpret_cast<const float4_t*>(sO + (size_t)((w0 + w) * 16 + hl) * C::OS + 4 * c4);
      lstar += f * sL[(w0 + w) * 16 + hl];
    }
    *reinterpret_cast<float4_t*>(part_o + (pbase + h) * C::R + 4 * c4) = o;
    if (c4 == 0) {
      part_ml[(pbase + h) * 2 + 0] = mstar;
      part_ml[(pbase + h) * 2 + 1] = lstar;
    }
  }
}

// Query operand [q~ | q^R] of sequence b, hi and lo planes: registers (lane = head 16*ht + l16,
// elements 32kk + 8g .. +7) or LDS rows [plane][head].  Padded heads duplicate the last real
// head and are never stored.  For LDS the fetch is split in two: query_request brings every piece
// of the thread into registers (one round trip, may be issued long before the LDS rows are
// free), query_commit stores them.
template <class C, bool QL>
struct QueryRegs {
  static constexpr int chunks = C::E / 8, total = 2 * C::HP * chunks;
  static constexpr int n = QL ? (total + kBlock - 1) / kBlock : 2 * C::KT;
  uint4 r[n];
};

template <class C, bool QL>
__device__ __forceinline__ void query_request(QueryRegs<C, QL>& q, const uint16_t* qbase, size_t plane, int n_heads,
                                              int ht, int tid, int l16, int g) {
  using Q = QueryRegs<C, QL>;
  if (!QL) {
    const int h = 16 * ht + l16 < n_heads ? 16 * ht + l16 : n_heads - 1;
#pragma unroll
    for (int kk = 0; kk < C::KT; ++kk) {
      q.r[QL ? 0 : kk] = *reinterpret_cast<const uint4*>(qbase + (size_t)h * C::E + 8 * g + 32 * kk);
      q.r[QL ? 0 : C::KT + kk] = *reinterpret_cast<const uint4*>(qbase + plane + (size_t)h * C::E + 8 * g + 32 * kk);
    }
  } else {
#pragma unroll
    for (int i = 0; i < Q::n; ++i) {
      const int idx = tid + i * kBlock;
      const int pl = idx / (C::HP * Q::chunks), rem = idx - pl * C::HP * Q::chunks;
      const int hh = rem / Q::chunks, c8 = rem - hh * Q::chunks;
      const int h = hh < n_heads ? hh : n_heads - 1;
      if (idx < Q::total) q.r[i] = *reinterpret_cast<const uint4*>(qbase + pl * plane + (size_t)h * C::E + c8 * 8);
    }
  }
}

template <class C, bool QL>
__device__ __forceinline__ void query_commit(const QueryRegs<C, QL>& q, uint16_t* sQ, int tid) {
  using Q = QueryRegs<C, QL>;
  if (QL) {
#pragma unroll
    for (int i = 0; i < Q::n; ++i) {
      const int idx = tid + i * kBlock;
      const int pl = idx / (C::HP * Q::chunks), rem = idx - pl * C::HP * Q::chunks;
      const int hh = rem / Q::chunks, c8 = rem - hh * Q::chunks;
      if (idx < Q::total) *reinterpret_cast<uint4*>(sQ + (pl * C::HP + hh) * C::QS + c8 * 8) = q.r[i];
    }
  }
}

// ---------------------------------------------------------------------------
// static schedule
// NHT = number of 16-head tiles.  With two head tiles the wavefronts split into two pairs, one
// per head tile, each pair striding over all 16-slot tiles of the chunk (a tile is then fetched
// by one wavefront of each pair; the second fetch is served by the cache hierarchy).  One head
// tile per wavefront keeps the output accumulators (r/16 x 4 registers) resident.
// NS = tiles in flight per wavefront.  QL = the query operand lives in LDS instead of registers:
// with r = 512 the registers are needed for the accumulators and the tiles in flight.
// ---------------------------------------------------------------------------
// SH: the sequence may read its first slots from another sequence's rows (a.prefix_owner, a.prefix_slots).
// PG: paged storage (a.pages): a.lat / a.key are the pool, the sequence's rows are found through its page-table row.
template <int R, int DR, int NHT, int NS, bool QL, bool SH, bool PG>
__global__ __launch_bounds__(kBlock) void attn_mfma_kernel(AttnArgs a) {
  using C = MfmaCfg<R, DR, NHT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* sT = reinterpret_cast<uint16_t*>(smem);
  float* sO = reinterpret_cast<float*>(smem);  // aliases sT (and sQ) after the main loop
  uint16_t* sQ = reinterpret_cast<uint16_t*>(smem + C::tile_bytes);  // QL only
  float* sM = reinterpret_cast<float*>(smem + C::body_bytes(QL));   // [kWaves][16]
  float* sL = sM + kWaves * 16;

  const int split = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int ht = wv / C::WPT, wl = wv - ht * C::WPT;  // head tile of this wavefront, rank inside it
  const int k0 = split * a.chunk;
  const uint16_t* lat = reinterpret_cast<const uint16_t*>(a.lat) + (PG ? 0 : (size_t)b * a.max_slots * R);
  const uint16_t* key = reinterpret_cast<const uint16_t*>(a.key) + (PG ? 0 : (size_t)b * a.max_slots * DR);
  const PageRow pr{PG ? a.pages.table + (size_t)b * a.pages.max_pages : nullptr, a.pages.shift, a.pages.n_pages};

  // Everything whose address does not depend on the sequence length is requested before the
  // length is looked at: the length, the query operand and this wavefront's first NS tiles (any
  // slot below max_slots is readable memory) travel together, one round trip instead of three.
  const int len = a.seq_len[b];
  SharedPrefix sp{0, 0, 0};
  if constexpr (SH) {  // one more round trip before the first tiles; both values clamped, so that every
                       // address stays inside the caches whatever the two arrays hold
    int owner = a.prefix_owner[b], n = a.prefix_slots[b];
    owner = owner < 0 ? 0 : (owner < a.prefix_rows ? owner : a.prefix_rows - 1);
    sp.n = n < 0 ? 0 : (n < a.max_slots ? n : a.max_slots);
    sp.dlat = (long long)(owner - b) * a.max_slots * R;
    sp.dkey = (long long)(owner - b) * a.max_slots * DR;
  }
  TileRegs<C> tl[NS];
  const int base = k0 + wl * kTile;
  const Cols cm{C::kStep, 0, 0, 0};
#pragma unroll
  for (int st = 0; st < NS; ++st) load_tile<C, SH, PG>(tl[st], lat, key, base + st * C::kStep, a.max_slots - 1, l16, g, cm, sp, pr);
  QueryRegs<C, QL> qr;
  query_request<C, QL>(qr, reinterpret_cast<const uint16_t*>(a.qcat) + (size_t)b * a.n_heads * C::E, a.q_plane,
                       a.n_heads, ht, tid, l16, g);
  const int live = live_slots(len, a.stride, a.max_slots);
  const int k1 = live < k0 + a.chunk ? live : k0 + a.chunk;
  if (k0 >= k1) return;
  query_commit<C, QL>(qr, sQ, tid);
  if (QL) __syncthreads();
  const uint4 (&qv)[QL ? 1 : 2 * C::KT] = reinterpret_cast<const uint4 (&)[QL ? 1 : 2 * C::KT]>(qr.r);
#pragma unroll
  for (int st = 0; st < NS; ++st)  // the first tiles may have touched rows that were never written
    tl[st].select_live(base + st * C::kStep + l16 < k1);

  WaveState<C> ws;
  ws.reset();
  stream_tiles<C, NS, QL ? kQLds : kQRegs, SH, PG>(tl, qv, sQ + (16 * ht + l16) * C::QS + 8 * g, sT + wv * kTile * C::TS,
                                                   lat, key, base, k1, l16, g, cm, ws, NextRun{lat, key, k1, k1 - 1, pr}, sp, pr);
  __syncthreads();  // every wavefront is done with its tile region (and the query), which sO aliases
  merge_store<C>(ws, sO, sM, sL, a.part_o, a.part_ml, (size_t)b * a.n_splits + split, a.n_heads, tid, wv, l16, g);
}

// ---------------------------------------------------------------------------
// static schedule, short chunks: one workgroup per (chunk, sequence) takes 64 slots a step.  With one head tile a wavefront forms the
// logits of its own 16 slots, with two those of 32 slots and one head tile; then every wavefront takes the value product of a quarter of
// the latent columns over all 64.  A decode step at small batch is a chain of latencies, not of bytes: with each wavefront taking its
// slots through both contractions the four results had to be merged through LDS, 1.1 us behind 1.2 us of contractions.
// Two barriers a step: one behind the wavefronts' maxima (all weights are taken relative to one reference per head), one behind the weights.
// Rows and query come memory -> LDS, four neighbouring lanes to 64 bytes of a row, and the sums leave through LDS in whole lines: straight to
// and from the operand layouts the address path of the unit takes a load or store one lane a cycle, 66 cycles each, and each wavefront fetched the
// query for itself.  us a step: 31 sequences of 640 slots, 20 heads x 128, r = 512 38.0, now 30.5; 7 of 700, 32 heads (whole layer) 52.3 and 38.0; 16
// of 750, 16 heads, r = 512 24.3 and 20.4; 79 of 195, 16 heads x 64, r = 256 19.3 and 17.6.
// ---------------------------------------------------------------------------
// Chunks of more than one step: where two workgroups a unit still fit (r = 128, and 64 with two head tiles) a step's rows travel while the step before is
// multiplied into a second place (DB), and the query stays in registers.  us a step, rows asked for at the step's top / so, 8 sequences of 1024 slots: r = 128, 8 heads,
// chunks of 128 12.2 / 11.8, of 320 14.6 / 13.6, 32 heads, of 160 14.8 / 13.8.
// r = 64 and one head tile (OPS): three loads of rows and six of the query a wavefront are not worth the way through LDS.  They go straight into the operands' layout,
// the first rows before the length is known, the next step's behind the maxima's barrier, and only the latents are put into LDS for the
// value product.  us a step, through LDS / so: 16 heads, 8 sequences of 1024 in chunks of 320 12.4 / 12.3, 4 heads, 4 in chunks of 64 10.74 / 10.66 (16 heads,
// 32 in chunks of 64 13.0 / 13.3).
template <int R, int DR, int NHT, bool DB>
struct SplitGeom {
  static constexpr int KC = R / 32, KT = (R + DR) / 32, HP = 16 * NHT, MW = R / 16 / kWaves;
  static constexpr int TILE = KT * 1024;                              // 16 slots: [K step][slot][64 bytes], pieces swizzled
  static constexpr int STEP = kWaves * TILE, ROWS = (DB ? 2 : 1) * STEP;
  static constexpr int Q = NHT * 2 * KT * 1024;                       // query: [head tile][plane][K step][head][64 bytes]
  static constexpr int OUT = HP * R * 4;                              // the sums on their way out, in place of the rows
  static constexpr int BODY = ROWS > OUT ? ROWS : OUT;
  static constexpr int WEIGHTS = kWaves * NHT * kWave * 8;
  static constexpr int BYTES = BODY + Q + WEIGHTS + 2 * kWaves * HP * 4;
  static constexpr int PER_CU = 2 * BYTES <= 160 * 1024 ? 2 : 1;
  static_assert(BYTES <= 160 * 1024, "LDS budget of one compute unit");
};

template <int R, int DR, int NHT, bool DB, bool SH, bool PG>
__global__ __launch_bounds__(kBlock, (SplitGeom<R, DR, NHT, DB>::PER_CU)) void attn_split_kernel(AttnArgs a) {
  using G = SplitGeom<R, DR, NHT, DB>;
  constexpr int KC = G::KC, KT = G::KT, E = R + DR, HP = G::HP, MW = G::MW;
  constexpr int GROUPS = kWaves / NHT;  // of wavefronts that share a head tile's slots
  constexpr bool OPS = R == 64 && NHT == 1, QR = DB || OPS;  // operands straight into registers; the query stays in registers
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char* sQ = smem + G::BODY;
  uint2* sP = reinterpret_cast<uint2*>(sQ + G::Q);  // [slot tile][head tile][lane]: weights of slots 4g .. 4g + 3, head l16
  float* sM = reinterpret_cast<float*>(sQ + G::Q + G::WEIGHTS);  // [group][HP]
  float* sL = sM + kWaves * HP;

  const int split = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int k0 = split * a.chunk;
  const uint16_t* lat = reinterpret_cast<const uint16_t*>(a.lat) + (PG ? 0 : (size_t)b * a.max_slots * R);
  const uint16_t* key = reinterpret_cast<const uint16_t*>(a.key) + (PG ? 0 : (size_t)b * a.max_slots * DR);

  const int len = load_uniform_i32(a.seq_len, b);  // nothing writes it while the kernel runs
  SharedPrefix sp{0, 0, 0};
  if constexpr (SH) {
    int owner = a.prefix_owner[b], n = a.prefix_slots[b];
    owner = owner < 0 ? 0 : (owner < a.prefix_rows ? owner : a.prefix_rows - 1);
    sp.n = n < 0 ? 0 : (n < a.max_slots ? n : a.max_slots);
    sp.dlat = (long long)(owner - b) * a.max_slots * R;
    sp.dkey = (long long)(owner - b) * a.max_slots * DR;
  }
  const int in_row = OPS ? l16 : lane >> 2, piece = OPS ? g : (lane & 3) ^ swz_rows16<4>(in_row);  // what a lane brings in: 16 bytes of that row's 64
  u32x4_t own[OPS ? KT : 1];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte_ptr)smem;
  // the wavefront's 16 slots from `base` on, into the step's place; slots past `last` become copies of that one
  auto issue_rows = [&](int base, int last, uint32_t step_at) {
    const uint32_t to = lds0 + step_at + (uint32_t)(wv * G::TILE);
    const int s0 = base < last ? base : last, slot = base + in_row < last ? base + in_row : last;
    if constexpr (SH) {
      const uint16_t* lr = lat + (size_t)slot * R + 8 * piece + (slot < sp.n ? sp.dlat : 0);
      const uint16_t* kr = key + (size_t)slot * DR + 8 * piece + (slot < sp.n ? sp.dkey : 0);
#pragma unroll
      for (int kk = 0; kk < KT; ++kk) {
        const uint16_t* from = kk < KC ? lr + 32 * kk : kr + 32 * (kk - KC);
        if constexpr (OPS) own[kk] = *reinterpret_cast<const u32x4_t*>(from);
        else load_to_lds_16(from, to + 1024u * kk);
      }
    } else {
      size_t row = (size_t)s0;
      if constexpr (PG) {  // a page holds whole 16-slot tiles
        int pg = load_uniform_i32(a.pages.table + (size_t)b * a.pages.max_pages, s0 >> a.pages.shift);
        pg = pg < 0 ? 0 : (pg < a.pages.n_pages ? pg : a.pages.n_pages - 1);
        row = ((size_t)pg << a.pages.shift) + (size_t)(s0 & ((1 << a.pages.shift) - 1));
      }
      const uint32_t i = (uint32_t)(slot - s0), at_lat = i * (R * 2) + 16 * piece, at_key = i * (DR * 2) + 16 * piece;
#pragma unroll
      for (int kk = 0; kk < KT; ++kk) {
        const uint16_t* from = kk < KC ? lat + row * R + 32 * kk : key + row * DR + 32 * (kk - KC);
        if constexpr (OPS) own[kk] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const unsigned char*>(from) + (kk < KC ? at_lat : at_key));
        else load_to_lds_16(from, kk < KC ? at_lat : at_key, to + 1024u * kk);
      }
    }
  };
  u32x4_t qf[QR ? 2 * KT : 1];  // the query, where it is read more than once
  if constexpr (OPS) {
    issue_rows(k0 + wv * kTile, a.max_slots - 1, 0);
    const uint16_t* q = reinterpret_cast<const uint16_t*>(a.qcat) + ((size_t)b * a.n_heads + (l16 < a.n_heads ? l16 : a.n_heads - 1)) * E + 8 * g;
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) {
      qf[kk] = *reinterpret_cast<const u32x4_t*>(q + 32 * kk);
      qf[QR ? KT + kk : 0] = *reinterpret_cast<const u32x4_t*>(q + a.q_plane + 32 * kk);
    }
  } else {
    const uint16_t* q = reinterpret_cast<const uint16_t*>(a.qcat) + (size_t)b * a.n_heads * E;
    uint32_t at_q[NHT];  // heads past the last one: copies of it, never stored
#pragma unroll
    for (int ht = 0; ht < NHT; ++ht) {
      const int h = 16 * ht + in_row < a.n_heads ? 16 * ht + in_row : a.n_heads - 1;
      at_q[ht] = (uint32_t)(h * E * 2 + 16 * piece);
    }
    constexpr int PER = (2 * KT + kWaves - 1) / kWaves;  // a wavefront's share of a head tile's pieces
#pragma unroll
    for (int ht = 0; ht < NHT; ++ht)
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int c = wv + kWaves * i < 2 * KT ? wv + kWaves * i : 2 * KT - 1;  // (a few twice)
        const int plane = c >= KT ? 1 : 0, kk = c - plane * KT;
        load_to_lds_16(q + (plane ? a.q_plane : 0) + 32 * kk, at_q[ht], lds0 + (uint32_t)(G::BODY + (ht * 2 * KT + c) * 1024));
      }
  }
  const int live = live_slots(len, a.stride, a.max_slots);
  const int k1 = live < k0 + a.chunk ? live : k0 + a.chunk;
  if (!OPS && k0 < k1) issue_rows(k0 + wv * kTile, k1 - 1, 0);

  const int hq = NHT == 2 ? wv & 1 : 0, grp = NHT == 2 ? wv >> 1 : wv;  // head tile and slot tiles NHT grp .. of the wavefront's logits
  float m_ref[NHT], l_run = 0.f;  // m_ref: the same in all wavefronts; l_run: this lane's slots only
  float4_t acc[NHT][MW];
#pragma unroll
  for (int ht = 0; ht < NHT; ++ht) {
    m_ref[ht] = -INFINITY;
#pragma unroll
    for (int mt = 0; mt < MW; ++mt) acc[ht][mt] = float4_t{0.f, 0.f, 0.f, 0.f};
  }
  const uint32_t frag = (uint32_t)(l16 * 64 + ((g ^ swz_rows16<4>(l16)) << 4));
  const int vrow = 4 * g + (l16 >> 2);  // row of the lane's transposing reads

  if (!OPS) wait_loads_but<0>();
  if (k0 >= k1) return;  // (nothing of this workgroup is on its way into LDS any more)
  if constexpr (OPS) {  // the first rows were asked for before the length was known: those past it may never have been written
    if (k0 + wv * kTile + l16 >= k1) {
#pragma unroll
      for (int kk = 0; kk < KT; ++kk) own[kk] = u32x4_t{0u, 0u, 0u, 0u};
    }
  }
  const unsigned char* qr = sQ + hq * (2 * KT * 1024) + frag;
  if constexpr (DB) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2 * KT; ++i) qf[i] = *reinterpret_cast<const u32x4_t*>(qr + 1024 * i);
  }
  uint32_t step_at = 0;  // this step's rows in LDS
  for (int s0 = k0; s0 < k1; s0 += kWaves * kTile) {
    if (!DB && !OPS && s0 > k0) {
      __syncthreads();
      issue_rows(s0 + wv * kTile, k1 - 1, 0);
    }
    if (!OPS && s0 > k0) wait_loads_but<0>();
    if (!QR || (NHT > 1 && s0 > k0)) __syncthreads();  // rows and query are there (with one head tile the rows are the wavefront's own)
    // ---- logits S^T[slot, head] (log2 units), one chain per query plane
    float4_t sh[NHT], sl[NHT];
#pragma unroll
    for (int u = 0; u < NHT; ++u) sh[u] = sl[u] = float4_t{0.f, 0.f, 0.f, 0.f};
    const unsigned char* xr = smem + step_at + NHT * grp * G::TILE + frag;
#pragma unroll
    for (int kk = 0; kk < KT; ++kk) {
      const u32x4_t qh = QR ? qf[QR ? kk : 0] : *reinterpret_cast<const u32x4_t*>(qr + 1024 * kk);
      const u32x4_t ql = QR ? qf[QR ? KT + kk : 0] : *reinterpret_cast<const u32x4_t*>(qr + 1024 * (KT + kk));
#pragma unroll
      for (int u = 0; u < NHT; ++u) {
        const bf16x8_t x = __builtin_bit_cast(bf16x8_t, OPS ? own[OPS ? kk : 0] : *reinterpret_cast<const u32x4_t*>(xr + u * G::TILE + 1024 * kk));
        sh[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, __builtin_bit_cast(bf16x8_t, qh), sh[u], 0, 0, 0);
        sl[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, __builtin_bit_cast(bf16x8_t, ql), sl[u], 0, 0, 0);
      }
    }
    float sv[NHT][4], mloc = -INFINITY;
#pragma unroll
    for (int u = 0; u < NHT; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sv[u][v] = (s0 + (NHT * grp + u) * kTile + 4 * g + v < k1) ? sh[u][v] + sl[u][v] : -INFINITY;
        mloc = fmaxf(mloc, sv[u][v]);
      }
    mloc = quarter_reduce(mloc, LaneMax());
    if (g == 0) sM[grp * HP + 16 * hq + l16] = mloc;
    __syncthreads();  // the maxima are there, and nobody reads the rows of the step before
    if constexpr (OPS) {  // the rows' latents to where the value products read them
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) *reinterpret_cast<u32x4_t*>(smem + wv * G::TILE + 1024 * kk + frag) = own[kk];
    }
    if ((DB || OPS) && s0 + kWaves * kTile < k1) issue_rows(s0 + kWaves * kTile + wv * kTile, k1 - 1, (uint32_t)G::STEP - step_at);
    // ---- reference (fixed at the first step, moved when a step tops it by 2^40), weights as bf16
    constexpr float kRebase = 40.f;
#pragma unroll
    for (int ht = 0; ht < NHT; ++ht) {
      float top = sM[16 * ht + l16];
#pragma unroll
      for (int w = 1; w < GROUPS; ++w) top = fmaxf(top, sM[w * HP + 16 * ht + l16]);
      if (__any(top - m_ref[ht] > kRebase)) {  // the same decision in every wavefront; true at the first step (m_ref = -inf)
        if (top - m_ref[ht] > kRebase) {
          const float alpha = __builtin_amdgcn_exp2f(m_ref[ht] - top);
          m_ref[ht] = top;
          if (ht == hq) l_run *= alpha;
#pragma unroll
          for (int mt = 0; mt < MW; ++mt) acc[ht][mt] *= alpha;
        }
      }
    }
    const float ref = NHT == 2 && hq == 1 ? m_ref[NHT - 1] : m_ref[0];
#pragma unroll
    for (int u = 0; u < NHT; ++u) {
      float pw[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) pw[v] = __builtin_amdgcn_exp2f(sv[u][v] - ref);
      const uint32_t p01 = pack_bf16x2(pw[0], pw[1]), p23 = pack_bf16x2(pw[2], pw[3]);
      sP[((NHT * grp + u) * NHT + hq) * kWave + lane] = make_uint2(p01, p23);
      l_run += (__uint_as_float(p01 << 16) + __uint_as_float(p01 & 0xffff0000u)) +
               (__uint_as_float(p23 << 16) + __uint_as_float(p23 & 0xffff0000u));
    }
    if (s0 + kWaves * kTile >= k1) {  // last step: the wavefront's share of the normaliser
      const float l = quarter_reduce(l_run, LaneSum());
      if (g == 0) sL[grp * HP + 16 * hq + l16] = l;
    }
    __syncthreads();
    // ---- O^T[col, head] += C_hat^T[col, slot] P^T[slot, head]: a lane's eight slots of a K step are 4g .. + 3 of two tiles
#pragma unroll
    for (int k = 0; k < kWaves / 2; ++k) {
      if (QR && k > 0 && s0 + 2 * kTile * k >= k1) break;  // (weights of zero)
      bf16x8_t pb[NHT];
#pragma unroll
      for (int ht = 0; ht < NHT; ++ht) {
        const uint2 u0 = sP[((2 * k) * NHT + ht) * kWave + lane], u1 = sP[((2 * k + 1) * NHT + ht) * kWave + lane];
        pb[ht] = __builtin_bit_cast(bf16x8_t, make_uint4(u0.x, u0.y, u1.x, u1.y));
      }
#pragma unroll
      for (int mt = 0; mt < MW; ++mt) {  // latent columns 16 (MW wv + mt) ..: half of a K step's 32
        const int ct = MW * wv + mt;
        const unsigned char* src = smem + step_at + 2 * k * G::TILE + 1024 * (ct >> 1) + vrow * 64 + 8 * (l16 & 1) +
                                   (((2 * (ct & 1) + ((l16 & 3) >> 1)) ^ swz_rows16<4>(vrow)) << 4);
        const short4_t c0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)src);
        const short4_t c1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(src + G::TILE));
        const uint2 a0 = __builtin_bit_cast(uint2, c0), a1 = __builtin_bit_cast(uint2, c1);
        const bf16x8_t ct8 = __builtin_bit_cast(bf16x8_t, make_uint4(a0.x, a0.y, a1.x, a1.y));
#pragma unroll
        for (int ht = 0; ht < NHT; ++ht) acc[ht][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ct8, pb[ht], acc[ht][mt], 0, 0, 0);
      }
    }
    if (DB) step_at = (uint32_t)G::STEP - step_at;
  }

  // ---- the partial of all heads, one run of memory: lane holds head 16 ht + l16, columns 16 mt + 4g .. + 3 of its quarter; piece j (16
  // bytes) of head i sits at j ^ (i % 16).  (Of a quarter of 16 columns a wavefront has one store a head tile: as it stands.)
  const size_t ph = ((size_t)b * a.n_splits + split) * a.n_heads;
  float* po = a.part_o + ph * R;
  if constexpr (MW == 1) {
#pragma unroll
    for (int ht = 0; ht < NHT; ++ht)
      if (16 * ht + l16 < a.n_heads) *reinterpret_cast<float4_t*>(po + (size_t)(16 * ht + l16) * R + 16 * wv + 4 * g) = acc[ht][0];
  } else {
    __syncthreads();  // the rows have been read
#pragma unroll
    for (int ht = 0; ht < NHT; ++ht)
#pragma unroll
      for (int mt = 0; mt < MW; ++mt)
        *reinterpret_cast<float4_t*>(smem + (16 * ht + l16) * (R * 4) + (((4 * (MW * wv + mt) + g) ^ l16) << 4)) = acc[ht][mt];
    __syncthreads();
    for (int at = tid; at < a.n_heads * (R / 4); at += kBlock) {
      const int h = at / (R / 4), j = at % (R / 4);
      *reinterpret_cast<float4_t*>(po + 4 * (size_t)at) = *reinterpret_cast<const float4_t*>(smem + h * (R * 4) + ((j ^ (h & 15)) << 4));
    }
  }
  if (tid < a.n_heads) {
    float l = sL[tid];
#pragma unroll
    for (int w = 1; w < GROUPS; ++w) l += sL[w * HP + tid];
    a.part_ml[(ph + tid) * 2 + 1] = l;
  }
  if (wv == 0 && g == 0) {
#pragma unroll
    for (int ht = 0; ht < NHT; ++ht)
      if (16 * ht + l16 < a.n_heads) a.part_ml[(ph + 16 * ht + l16) * 2] = m_ref[ht];
  }
}

// ---------------------------------------------------------------------------
// balanced schedule: gridDim.x persistent workgroups, one flat list of tiles.
// Sequence b owns tiles [pre[b], pre[b+1]) with pre the running sum of ceil(live_b / 16);
// workgroup i takes tiles [i*S, (i+1)*S), S = ceil(total / gridDim.x), and emits partial
// number i + b for every sequence b its range touches (ids never collide: moving to the next
// workgroup or to the next sequence both advance the id).  Workgroup 0 publishes pre[] so the
// combine kernel can find each sequence's partials.
// ---------------------------------------------------------------------------
template <int R, int DR, int NHT, int NS, bool QL>
__global__ __launch_bounds__(kBlock) void attn_mfma_balanced_kernel(AttnArgs a) {
  using C = MfmaCfg<R, DR, NHT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* sT = reinterpret_cast<uint16_t*>(smem);
  float* sO = reinterpret_cast<float*>(smem);
  uint16_t* sQ = reinterpret_cast<uint16_t*>(smem + C::tile_bytes);
  float* sM = reinterpret_cast<float*>(smem + C::body_bytes(QL));
  float* sL = sM + kWaves * 16;
  int* sPre = reinterpret_cast<int*>(smem + C::body_bytes(QL) + C::ml_bytes);  // [batch + 1]
  int* sLive = sPre + a.batch + 1;                                             // [batch] live slots
  int* sScan = sLive + a.batch;                                                // [kBlock]

  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int ht = wv / C::WPT, wl = wv - ht * C::WPT;
  const int B = a.batch;

  // ---- pre[]: every thread sums a contiguous run of sequences, the run totals are scanned
  const int per = (B + kBlock - 1) / kBlock;
  const int b_lo = tid * per, b_hi = b_lo + per < B ? b_lo + per : B;
  int run = 0;
  for (int bb = b_lo; bb < b_hi; ++bb) run += (live_slots(a.seq_len[bb], a.stride, a.max_slots) + kTile - 1) / kTile;
  sScan[tid] = run;
  __syncthreads();
  for (int off = 1; off < kBlock; off <<= 1) {  // inclusive Hillis-Steele scan over the 256 run totals
    const int v = tid >= off ? sScan[tid - off] : 0;
    __syncthreads();
    sScan[tid] += v;
    __syncthreads();
  }
  {
    int acc = tid ? sScan[tid - 1] : 0;
    for (int bb = b_lo; bb < b_hi; ++bb) {
      const int lv = live_slots(a.seq_len[bb], a.stride, a.max_slots);
      sPre[bb] = acc;
      sLive[bb] = lv;
      acc += (lv + kTile - 1) / kTile;
    }
    if (tid == kBlock - 1) sPre[B] = sScan[kBlock - 1];
  }
  __syncthreads();
  const int total = sPre[B];
  if (blockIdx.x == 0)
    for (int bb = tid; bb <= B; bb += kBlock) a.tile_prefix[bb] = sPre[bb];
  const int share = (total + (int)gridDim.x - 1) / (int)gridDim.x;
  int pos = blockIdx.x * share;
  const int end = pos + share < total ? pos + share : total;
  if (pos >= end) return;

  // ---- first sequence of the range: last b with pre[b] <= pos (sequences without tiles are skipped)
  int b;
  {
    int lo = 0, hi = B;  // invariant: pre[lo] <= pos < pre[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (sPre[mid] <= pos) lo = mid; else hi = mid;
    }
    b = lo;
  }
  uint16_t* sTw = sT + wv * kTile * C::TS;
  const uint16_t* qrow = sQ + (16 * ht + l16) * C::QS + 8 * g;
  const uint16_t* lat_all = reinterpret_cast<const uint16_t*>(a.lat);
  const uint16_t* key_all = reinterpret_cast<const uint16_t*>(a.key);
  const uint16_t* q_all = reinterpret_cast<const uint16_t*>(a.qcat);
  const Cols cm{C::kStep, 0, 0, 0};

  // The workgroup's range is a chain of runs, one per sequence it touches.  The tile stream never
  // drains between them: while a run's last tiles are in the matrix cores the refills already
  // fetch the first tiles of the next run, and the next query is requested before the merge of
  // the finished run, so the only latency a run exposes is the first one's.
  struct Run {
    int b, k0, k1, seg_end;
  };
  auto run_at = [&](int p, int& bb) {  // run starting at flat tile p (p < end); bb: sequence hint
    while (sPre[bb + 1] <= p) ++bb;    // skip sequences that own no tile
    Run r;
    r.b = bb;
    r.seg_end = end < sPre[bb + 1] ? end : sPre[bb + 1];
    const int live = sLive[bb];
    r.k0 = (p - sPre[bb]) * kTile;
    r.k1 = live < (r.seg_end - sPre[bb]) * kTile ? live : (r.seg_end - sPre[bb]) * kTile;
    return r;
  };
  Run cur = run_at(pos, b);
  TileRegs<C> tl[NS];
  QueryRegs<C, QL> qr;
  {
    const uint16_t* lat = lat_all + (size_t)cur.b * a.max_slots * R;
    const uint16_t* key = key_all + (size_t)cur.b * a.max_slots * DR;
#pragma unroll
    for (int st = 0; st < NS; ++st)
      load_tile(tl[st], lat, key, cur.k0 + wl * kTile + st * C::kStep, cur.k1 - 1, l16, g, cm);
    query_request<C, QL>(qr, q_all + (size_t)cur.b * a.n_heads * C::E, a.q_plane, a.n_heads, ht, tid, l16, g);
  }
  while (true) {
    const uint16_t* lat = lat_all + (size_t)cur.b * a.max_slots * R;
    const uint16_t* key = key_all + (size_t)cur.b * a.max_slots * DR;
    const int base = cur.k0 + wl * kTile;
    const bool more = cur.seg_end < end;
    Run nxt = cur;
    NextRun nx{lat, key, cur.k1, cur.k1 - 1};  // no next run: dead refills clamp to a live row
    if (more) {
      nxt = run_at(cur.seg_end, b);
      nx.lat = lat_all + (size_t)nxt.b * a.max_slots * R;
      nx.key = key_all + (size_t)nxt.b * a.max_slots * DR;
      nx.base = nxt.k0 + wl * kTile;
      nx.last = nxt.k1 - 1;
    }
    query_commit<C, QL>(qr, sQ, tid);
    if (QL) __syncthreads();

    WaveState<C> ws;
    ws.reset();
    const uint4 (&qv)[QL ? 1 : 2 * C::KT] = reinterpret_cast<const uint4 (&)[QL ? 1 : 2 * C::KT]>(qr.r);
    stream_tiles<C, NS, QL ? kQLds : kQRegs>(tl, qv, qrow, sTw, lat, key, base, cur.k1, l16, g, cm, ws, nx);
    if (more) {
      if (base >= cur.k1) {  // this wavefront had no tile in the run: nothing was prefetched for it
#pragma unroll
        for (int st = 0; st < NS; ++st) load_tile(tl[st], nx.lat, nx.key, nx.base + st * C::kStep, nx.last, l16, g, cm);
      }
      query_request<C, QL>(qr, q_all + (size_t)nxt.b * a.n_heads * C::E, a.q_plane, a.n_heads, ht, tid, l16, g);
    }
    __syncthreads();  // tile regions and the query are free: sO aliases them
    merge_store<C>(ws, sO, sM, sL, a.part_o, a.part_ml, (size_t)blockIdx.x + cur.b, a.n_heads, tid, wv, l16, g);
    if (!more) break;
    __syncthreads();  // the merge buffer has been read: the next run may overwrite it
    cur = nxt;
  }
}

// ---------------------------------------------------------------------------
// parallel (prefill / training) form: one wavefront per (query row, 16-head tile).
// Row m of a sequence attends the final states of the m/s chunks before its own and its own
// running state C_hat'[m] -- the columns the stride-aware causal mask leaves open -- so the
// wavefront streams columns 0 .. m/s through the same two contractions as the decode pass, with
// the column -> row map of `Cols` standing in for the mask (nothing masked is ever computed).
// The kernel reads C_hat' [B, T, r] and the uncompressed keys [B, T, d_R] and writes one
// unnormalised partial per (row, head), which the combine kernel normalises and up-projects.
// grid = (ceil(T / rows per workgroup), B); the wavefronts of a workgroup take consecutive rows,
// so they walk almost the same columns and share them through the cache hierarchy.
// ---------------------------------------------------------------------------
template <int R, int DR, int NHT, int NS>
__global__ __launch_bounds__(kBlock) void attn_mfma_rows_kernel(AttnArgs a) {
  using C = MfmaCfg<R, DR, NHT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* sT = reinterpret_cast<uint16_t*>(smem);
  uint16_t* sQlo = reinterpret_cast<uint16_t*>(smem + C::tile_bytes);  // [kWaves][16][QS] lo plane

  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int ht = wv % NHT, b = blockIdx.y;
  const int m = blockIdx.x * C::WPT + wv / NHT;  // WPT = rows per workgroup here
  if (m >= a.T) return;
  if (a.seq_len && m >= a.seq_len[b]) return;  // padding row: the combine kernel writes zeros

  const uint16_t* lat = reinterpret_cast<const uint16_t*>(a.lat) + (size_t)b * a.T * R;
  const uint16_t* key = reinterpret_cast<const uint16_t*>(a.key) + (size_t)b * a.T * DR;
  const int n_cols = m / a.stride + 1;
  const Cols cm{kTile, a.stride, n_cols - 1, m};
  TileRegs<C> tl[NS];
#pragma unroll
  for (int st = 0; st < NS; ++st) load_tile(tl[st], lat, key, st * kTile, n_cols - 1, l16, g, cm);

  // query planes of head 16*ht + l16: hi stays in registers, lo goes through this wavefront's
  // LDS rows (each lane reads back exactly the pieces it stored)
  const size_t rowg = (size_t)b * a.T + m;
  const int h = 16 * ht + l16 < a.n_heads ? 16 * ht + l16 : a.n_heads - 1;
  const uint16_t* qsrc = reinterpret_cast<const uint16_t*>(a.qcat) + (rowg * a.n_heads + h) * C::E + 8 * g;
  uint16_t* qlo = sQlo + (wv * 16 + l16) * C::QS + 8 * g;
  uint4 qv[C::KT];
#pragma unroll
  for (int kk = 0; kk < C::KT; ++kk) {
    qv[kk] = *reinterpret_cast<const uint4*>(qsrc + 32 * kk);
    *reinterpret_cast<uint4*>(qlo + 32 * kk) = *reinterpret_cast<const uint4*>(qsrc + a.q_plane + 32 * kk);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();

  WaveState<C> ws;
  ws.reset();
  stream_tiles<C, NS, kQMixed>(tl, qv, qlo, sT + wv * kTile * C::TS, lat, key, 0, n_cols, l16, g, cm, ws,
                              NextRun{lat, key, n_cols, n_cols - 1});

  const float l_head = ws.l_total();
  if (16 * ht + l16 < a.n_heads) {  // lane holds head h, columns 16mt + 4g .. +3 of every column tile
    float* po = a.part_o + (rowg * a.n_heads + h) * R + 4 * g;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt) *reinterpret_cast<float4_t*>(po + 16 * mt) = ws.acc_o[mt];
    if (g == 0) {
      a.part_ml[(rowg * a.n_heads + h) * 2 + 0] = ws.m_ref;
      a.part_ml[(rowg * a.n_heads + h) * 2 + 1] = l_head;
    }
  }
}

template <int R, int DR, int NHT, int NS>
hipError_t launch_rows(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
  using C = MfmaCfg<R, DR, NHT>;
  constexpr size_t smem = C::tile_bytes + (size_t)kWaves * 16 * C::QS * 2;
  static_assert(smem <= 160 * 1024, "LDS budget of one compute unit");
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&attn_mfma_rows_kernel<R, DR, NHT, NS>, smem, lds_allowed);
  if (e != hipSuccess) return e;
  const dim3 grid((a.T + C::WPT - 1) / C::WPT, a.batch);
  launch_timed(attn_mfma_rows_kernel<R, DR, NHT, NS>, grid, dim3(kBlock), smem, st, ev, a);
  return hipGetLastError();
}

template <int R, int DR, int NHT, bool DB, bool SH, bool PG>
hipError_t launch_split_as(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
  constexpr size_t smem = SplitGeom<R, DR, NHT, DB>::BYTES;
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&attn_split_kernel<R, DR, NHT, DB, SH, PG>, smem, lds_allowed);
  if (e != hipSuccess) return e;
  launch_timed(attn_split_kernel<R, DR, NHT, DB, SH, PG>, dim3(a.n_splits, a.batch), dim3(kBlock), smem, st, ev, a);
  return hipGetLastError();
}
template <int R, int DR, int NHT, bool SH, bool PG>
hipError_t launch_split(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
  if constexpr (R == 128 || (R == 64 && NHT == 2)) {
    if (a.chunk > kTile * kWaves) return launch_split_as<R, DR, NHT, true, SH, PG>(a, st, ev);
  }
  return launch_split_as<R, DR, NHT, false, SH, PG>(a, st, ev);
}

template <int R, int DR, int NHT, int NS, bool QL, bool SH, bool PG>
hipError_t launch_static(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
  using C = MfmaCfg<R, DR, NHT>;
  constexpr size_t smem = C::body_bytes(QL) + C::ml_bytes;
  static_assert(smem <= 160 * 1024, "LDS budget of one compute unit");
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&attn_mfma_kernel<R, DR, NHT, NS, QL, SH, PG>, smem, lds_allowed);
  if (e != hipSuccess) return e;
  launch_timed(attn_mfma_kernel<R, DR, NHT, NS, QL, SH, PG>, dim3(a.n_splits, a.batch), dim3(kBlock), smem, st, ev, a);
  return hipGetLastError();
}

template <int R, int DR, int NHT, int NS, bool QL>
hipError_t launch_one(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
  if (a.n_persistent > 0) {
    if constexpr (R == 64) {  // (attn_cols.hip has every other width)
      using C = MfmaCfg<R, DR, NHT>;
      if (a.prefix_owner || a.pages.table) return hipErrorInvalidValue;  // shared prefixes, pages: static schedule or the column-split kernel
      const size_t smem = C::body_bytes(QL) + C::ml_bytes + (size_t)(2 * a.batch + 1 + kBlock) * sizeof(int);
      if (smem > 160 * 1024) return hipErrorInvalidValue;
      static DeviceSet lds_allowed;
      const hipError_t e = allow_lds(&attn_mfma_balanced_kernel<R, DR, NHT, NS, QL>, 160 * 1024, lds_allowed);
      if (e != hipSuccess) return e;
      launch_timed(attn_mfma_balanced_kernel<R, DR, NHT, NS, QL>, dim3(a.n_persistent), dim3(kBlock), smem, st, ev, a);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  if (a.pages.table) return a.prefix_owner ? hipErrorInvalidValue : launch_static<R, DR, NHT, NS, QL, false, true>(a, st, ev);
  return a.prefix_owner ? launch_static<R, DR, NHT, NS, QL, true, false>(a, st, ev)
                        : launch_static<R, DR, NHT, NS, QL, false, false>(a, st, ev);
}

// Pipeline depth: a workgroup that will see only a step or two (decode at small batch) is attn_split_kernel's; long runs keep several tiles in flight
// per wavefront, which is what it takes to cover HBM latency with four wavefronts per compute
// unit.
template <int R, int DR>
hipError_t launch_rd(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
  constexpr int kDeep = R >= 512 ? 2 : 3;  // what the 512-register budget per lane allows
  constexpr bool kDeepQL = R >= 512;
  const int nht = a.n_heads <= 16 ? 1 : 2;
  const int tiles_per_wave = a.chunk / (kTile * (kWaves / nht));
  const bool deep = a.n_persistent > 0 || tiles_per_wave >= 2 * kDeep;
  if (deep) return nht == 1 ? launch_one<R, DR, 1, kDeep, kDeepQL>(a, st, ev) : launch_one<R, DR, 2, kDeep, kDeepQL>(a, st, ev);
  if (a.pages.table) {
    if (a.prefix_owner) return hipErrorInvalidValue;
    return nht == 1 ? launch_split<R, DR, 1, false, true>(a, st, ev) : launch_split<R, DR, 2, false, true>(a, st, ev);
  }
  if (a.prefix_owner) return nht == 1 ? launch_split<R, DR, 1, true, false>(a, st, ev) : launch_split<R, DR, 2, true, false>(a, st, ev);
  return nht == 1 ? launch_split<R, DR, 1, false, false>(a, st, ev) : launch_split<R, DR, 2, false, false>(a, st, ev);
}

template <int R, int DR>
hipError_t launch_case(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
  if (a.T == 0) return launch_rd<R, DR>(a, st, ev);
  if constexpr (R == 64)  // (attn_cols.hip has the parallel form of every other width)
    return a.n_heads <= 16 ? launch_rows<R, DR, 1, 2>(a, st, ev) : launch_rows<R, DR, 2, 2>(a, st, ev);
  return hipErrorInvalidValue;
}

}  // namespace

bool attn_mfma_supported(const AttnArgs& a) {
  return a.n_heads <= 32 && a.batch <= 65535 && (a.r == 64 || a.r == 128 || a.r == 256 || a.r == 512) &&
         (a.d_rope == 32 || a.d_rope == 64);
}

hipError_t launch_attn_mfma(const AttnArgs& a, hipStream_t st, const EventPair& ev) {
#define MTLA_CASE(RR, DD) \
  if (a.r == RR && a.d_rope == DD) return launch_case<RR, DD>(a, st, ev);
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

}  // namespace mtla
