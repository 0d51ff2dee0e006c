// The matrix products of a prefill (GemmArgs: C = A W^T for up to four W, with its rows and ways out) where they are small: short prompts.
// Tiles of 16 x 16 to 32 x 32 outputs, the contraction dealt to the wavefronts (gemm_ring.h).
//
// A short prompt's products are a few 64 x 64 tiles whose K stages follow one another behind a barrier each; as many times more, smaller
// tiles on as many more units, each wavefront a quarter of K without a barrier, take half the time.
#include "bounds.h"
#include "gemm_ring.h"
#include "gemm_tiles.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

// Jobs (ring_job): column blocks of all segments (a segment starts one of its own) x row blocks.  Rows: with lengths or starts each
// sequence's from its first row on, `per_seq` blocks for as many as it may have; without, or where the caller wants zeros in rows that hold
// nothing, the matrix's own.
template <class C>
__global__ __launch_bounds__(C::NT) void gemm_ring_kernel(GemmArgs a, int per_seq) {
  constexpr int TM = C::TM, TN = C::TN, BM = 16 * TM, BN = 16 * TN;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), l16 = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int2 job = ring_job(blockIdx.x, a.row_blocks);
  if (job.x >= a.col_blocks) return;
  const GemmRows& q = a.rows;
  const bool ragged = q.n_new || q.pos0;
  const int K = a.K, Tp = q.past + q.T;
  int rb = BM * job.y, row_end = a.M, b0 = 0;  // b0: the block's sequence, where the blocks are the sequences'
  bool work = true;
  auto used_rows = [&](int b) {
    return (q.pos0 ? slots_inside(load_uniform_i32(q.pos0, b), q.stride, q.past) : 0) + (q.n_new ? new_rows(load_uniform_i32(q.n_new, b), q.T) : q.T);
  };
  if (ragged && q.zeros) {
    work = false;  // without a row of its own the block only writes zeros
    for (int b = rb / Tp; b * Tp < rb + BM && b * Tp < a.M && !work; ++b) work = used_rows(b) > 0 && rb < b * Tp + used_rows(b);
  } else if (ragged) {
    b0 = job.y / per_seq;
    const int first = BM * (job.y - b0 * per_seq), used = used_rows(b0);
    if (first >= used) return;
    rb = b0 * Tp + first;
    row_end = b0 * Tp + used;
  }
  // the segment the column block belongs to
  int cb = job.x, z = 0;
  while (z + 1 < a.n_seg && cb >= (a.seg[z].N + BN - 1) / BN) {
    cb -= (a.seg[z].N + BN - 1) / BN;
    ++z;
  }
  const GemmSegment sg = a.seg[z];
  const int nb = cb * BN, N = sg.N, epi = sg.epi;

  const unsigned char* wb[TN];
  uint32_t w_at[TN], x_at[TM][1];
#pragma unroll
  for (int j = 0; j < TN; ++j) {  // columns past the end: clamped, never stored
    const int n = nb + 16 * j < N ? nb + 16 * j : nb, last = N - 1 - n;
    wb[j] = reinterpret_cast<const unsigned char*>(sg.W) + 2 * (size_t)n * K;
    w_at[j] = piece16(lane, (lane >> 2) < last ? lane >> 2 : last, K);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {  // rows likewise
    const int t = 16 * i + (lane >> 2), last = row_end - 1 - rb;
    x_at[i][0] = piece16(lane, t < last ? t : last, K);
  }
  const unsigned char* xb = reinterpret_cast<const unsigned char*>(a.A) + 2 * (size_t)rb * K;
  int2 st = steps_of<C::NW>(K, wv);
  if (!work) st.y = 0;
  float4_t acc[TM][TN];
  contract<C>(acc, wb, w_at, xb, x_at, 32 * st.x, st.y, lds + wv * (C::D * C::STAGE), l16, g);
  sum_tiles<C>(acc, lds, tid, wv, l16, g, [&](int at, float2 o, int p, int t) {
    const int row = rb + 16 * (at / TN) + t, n = nb + 16 * (at % TN) + 2 * p;
    if (row >= row_end || n >= N) return;  // (N is a multiple of 8)
    if (epi == 1 || epi == 2) {
      int b = b0, first = b0 * Tp;  // (turned rows are their sequence's new rows alone: Tp = T)
      if (!ragged) {
        b = row / Tp;
        first = b * Tp;
      }
      o = rope_turn(o, rope_angle((a.rope_pos0 ? a.rope_pos0[b] : 0) + row - first, a.rope_freq[(n % a.d_rope) / 2]));
    }
    const size_t to = (size_t)row * N + n;
    if (epi == 3) *reinterpret_cast<float2*>(reinterpret_cast<float*>(sg.C) + to) = o;
    else if (epi == 2) *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(sg.C) + to) = pack_bf16x2(o.x, o.y);
    else *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(sg.C) + to) = pack_f16x2(sg.scale * o.x, sg.scale * o.y);
  });
}

template <class C>
hipError_t ring_as(const GemmArgs& args, hipStream_t st) {
  static DeviceSet lds_allowed;
  const hipError_t e = allow_lds(&gemm_ring_kernel<C>, C::BYTES, lds_allowed);
  if (e != hipSuccess) return e;
  GemmArgs a = args;
  constexpr int BM = 16 * C::TM;
  const int Tp = a.rows.past + a.rows.T, per_seq = (Tp + BM - 1) / BM;
  const bool ragged = a.rows.n_new || a.rows.pos0;
  a.col_blocks = gemm_col_blocks(a, 16 * C::TN);
  a.row_blocks = (unsigned)(ragged && !a.rows.zeros ? a.M / Tp * per_seq : (a.M + BM - 1) / BM);
  hipLaunchKernelGGL(gemm_ring_kernel<C>, dim3(ring_grid((unsigned)a.col_blocks, a.row_blocks)), dim3(C::NT), C::BYTES, st, a, per_seq);
  return hipGetLastError();
}

template <RingType TYPE>
hipError_t ring_typed(const GemmArgs& a, hipStream_t st) {
  const long long tiles = gemm_ring_tiles(a);
  if (tiles <= kRingSmall) return ring_as<RingTile<1, 1, 4, 4, TYPE>>(a, st);
  if (tiles <= kRingMedium) return ring_as<RingTile<2, 1, 4, 4, TYPE>>(a, st);
  return ring_as<RingTile<2, 2, 4, 4, TYPE>>(a, st);
}

}  // namespace

hipError_t launch_gemm_ring(const GemmArgs& a, hipStream_t st) {
  return a.in_bf16 ? ring_typed<kRingBf16>(a, st) : ring_typed<kRingF16>(a, st);
}

}  // namespace mtla
