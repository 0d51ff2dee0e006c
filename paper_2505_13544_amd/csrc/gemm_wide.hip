// Matrix products C = A W^T with many rows and columns (gfx950): one workgroup per compute unit walks its share of the
// 256 x 256 tiles as one stream of stages; what a last round would leave most units idle for is cut smaller.
//
// What bounds it is power: the chip holds about 1.9 PFLOP/s of 16x16x32 products alone (random operands; 2.4 of zeros), and every
// byte through LDS and from L2 costs clock.  With the matrix pipes busy 54 % of the time it ran at 2.2 GHz, at 67 % at 2.0.  So:
//   * 16x16x32 instructions; the 32x32x16 form gave 1.26 PFLOP/s under the same load
//   * one stream per unit, the next tile's operands on their way while a tile leaves, no barrier around its way out
//   * one barrier per stage, in the middle of its products, operands read ahead through a ring of registers
//   * both halves of a 128-byte line asked for together (with 64 bytes of each row at a time the loads alone took 274 us
//     of the 385 below, now 235), a quarter of a pair of stages at a time
// Measured (us; before: one tile a workgroup, two barriers' worth of reads in front of the products): 32768 x 3584 x 2048 bf16
// 452 -> 378; 32768 x 2048 x 2048 with fp32 results 286 -> 236; 32768 x 4096 x 512 171 -> 136; 8192^3 918 -> 770 (1.43
// PFLOP/s); 33 ragged row blocks x 4096 x 512 51 -> 42; 20 ragged row blocks 39 -> 28, of which the cut last round is 6.
#include <type_traits>

#include "bounds.h"
#include "gemm_jobs.h"
#include "lds_stream.h"
#include "mtla_device.h"
#include "mtla_kernels.h"

namespace mtla {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

constexpr int kTile = kWideTile, kWideThreads = 512, kWideWaves = 8;
constexpr int kBK = 32, kSlots = 5;        // k of a stage, stages in LDS
constexpr int kPark = 4096;                // bytes a wavefront's results pass through on their way out

// Where the rows are, the same for every job of the launch.  Lane i stands for sequences i * per .. + per - 1: the blocks of
// 256 rows that they use, and those of all sequences up to them.
struct WideRows {
  int used, blocks, upto, n_rb, per, pitch;  // used: rows of sequence i (per = 1); pitch: rows from one sequence to the next
};
__device__ __forceinline__ int used_rows(const GemmArgs& a, int b) {
  const GemmRows& q = a.rows;
  if (!q.pos0 && !q.n_new) return a.M;
  return (q.pos0 ? slots_inside(load_uniform_i32(q.pos0, b), q.stride, q.past) : 0) +
         (q.n_new ? new_rows(load_uniform_i32(q.n_new, b), q.T) : q.T);
}
struct WideLanes {  // the record, lane by lane
  const GemmArgs& a;
  const WideRows& r;
  int per, pitch;
  __device__ __forceinline__ int lane_of(int block) const { return __builtin_ctzll(__ballot(block < r.upto)); }
  __device__ __forceinline__ int upto(int at) const { return __builtin_amdgcn_readlane(r.upto, at); }
  __device__ __forceinline__ int blocks(int at) const { return __builtin_amdgcn_readlane(r.blocks, at); }
  __device__ __forceinline__ int used(int at) const { return __builtin_amdgcn_readlane(r.used, at); }
  __device__ __forceinline__ int used_rows(int b) const { return mtla::used_rows(a, b); }
};
__device__ __forceinline__ WideTile tile_at(const GemmArgs& a, const WideRows& r, const WideWalk& w) {
  WideTile t = wide_tile(a, WideLanes{a, r, r.per, r.pitch}, w);
  t.rb = __builtin_amdgcn_readfirstlane(t.rb);  // (the loads' bases have to be scalars)
  t.row_end = __builtin_amdgcn_readfirstlane(t.row_end);
  return t;
}

// A stream of BM x BN tiles.  Eight wavefronts, each with 64 columns of the tile.
template <bool BF16, int BM, int BN>
struct WideStream {
  static constexpr int WCOLS = BN / 64, WROWS = kWideWaves / WCOLS, WM = BM / WROWS, JM = WM / 16, IN = 4;
  static constexpr int W_BYTES = BN * kBK * 2, STAGE = W_BYTES + BM * kBK * 2;
  static constexpr int NW = BN / 128, NC = NW + BM / 128;  // 1 KB chunks of a stage a wavefront brings: the weights', all
  static constexpr int HALF = (NC + 1) / 2;                // chunks of a part, each for two stages: the other part has the rest
  static constexpr int LA = JM < 4 ? JM - 1 : 3;           // row operands read ahead
  static_assert((LA & (LA + 1)) == 0 && STAGE * kSlots <= 160 * 1024, "geometry");

  const GemmArgs& a;
  const WideRows& rows;
  unsigned char* lds;
  int lane, wv;
  // the load side runs ahead of the products: its place, its slot, its addresses
  WideWalk ld_walk;
  unsigned step;             // jobs from one tile of this workgroup to its next
  int quad;                  // 128-row and 128-column part of the job that is this stream's tile (2 row part + column part)
  int n_st, ld_st, to_ask;   // stages of a tile, stage of the tile that is asked for next, stages not asked for yet
  uint32_t ld_slot, off[NC];
  uint64_t base_w, base_a;

  __device__ __forceinline__ WideTile tile(const WideWalk& w) const {
    WideTile t = tile_at(a, rows, w);
    t.rb += 128 * (quad >> 1);
    t.nb += 128 * (quad & 1);
    return t;
  }

  // Part i (of two, in turn) of the next two stages.  A chunk is 16 rows of 64 bytes; both stages' halves of the rows'
  // 128-byte lines are asked for together, so that the second finds the line in L1, and the parts are spread over
  // two stages' time: the path from L2 takes 64 bytes a clock, and two thirds of that is what the products need.
  __device__ __forceinline__ void issue(int i) {
    if (i == 0 && ld_st == 0) {
      const WideTile t = tile(ld_walk);
      const int N = a.seg[t.z].N, K = a.K, prow = lane >> 2;
      const uint32_t src = 16u * (uint32_t)((lane & 3) ^ swz_rows16<4>(prow));
      base_w = (uint64_t)(uintptr_t)a.seg[t.z].W + (uint64_t)t.nb * (uint32_t)K * 2u;
      base_a = (uint64_t)(uintptr_t)a.A + (uint64_t)t.rb * (uint32_t)K * 2u;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int row = 16 * (wv + 8 * (c < NW ? c : c - NW)) + prow;
        const int last = c < NW ? N - 1 - t.nb : t.row_end - 1 - t.rb;  // rows past it: a readable duplicate
        off[c] = (uint32_t)(row < last ? row : last) * (uint32_t)K * 2u + src;
      }
    }
    const uint32_t next = ld_slot + 1 == kSlots ? 0 : ld_slot + 1;
    const uint32_t base = (uint32_t)(uintptr_t)(lds_byte_ptr)lds + (uint32_t)wv * 1024u;
#pragma unroll
    for (int c = i ? HALF : 0; c < (i ? NC : HALF); ++c) {
      const uint32_t at = c < NW ? 8192u * c : W_BYTES + 8192u * (c - NW);
      const uint64_t from = c < NW ? base_w : base_a;
      load_to_lds_16(reinterpret_cast<const void*>(from), off[c], base + ld_slot * (uint32_t)STAGE + at);
      load_to_lds_16(reinterpret_cast<const void*>(from + 2 * kBK), off[c], base + next * (uint32_t)STAGE + at);
    }
    if (i == 0) return;
    ld_slot = next + 1 == kSlots ? 0 : next + 1;
    base_w += 4 * kBK;
    base_a += 4 * kBK;
    to_ask -= 2;
    if ((ld_st += 2) == n_st) {
      ld_st = 0;
      ld_walk.advance(step, (unsigned)a.col_blocks, (unsigned)rows.n_rb);
    }
  }

  __device__ __forceinline__ void begin(WideWalk first, unsigned step_, int quad_, int n_jobs) {
    ld_walk = first;
    step = step_;
    quad = quad_;
    n_st = a.K / kBK;
    ld_st = 0;
    ld_slot = 0;
    to_ask = n_jobs * n_st;
#pragma unroll 1
    for (int i = 0; i < 2; ++i) {  // (a tile has four stages at least)
      issue(0);
      issue(1);
    }
  }

  // The results of 32 rows x 128 bytes at a time through the wavefront's own 4 KB of `park`, so that memory sees whole
  // lines.  Results of more than kStreamOut bytes go past the caches' usual replacement: written back in bursts as the tiles end
  // they stall every unit at once (32768 x 2048 x 2048 with fp32 results: 281 us with ordinary stores, 249 with these).
  // Smaller ones stay where the next kernel finds them (keys and values of 4.6 K rows, 37 MB: streamed, the attention behind them
  // took 7 us more).
  template <int EPI>
  __device__ __forceinline__ void way_out(const WideTile& t, const float4_t (&acc)[JM][IN], unsigned char* park) {
    constexpr int ES = EPI == 3 ? 4 : 2, COLS = 128 / ES;  // columns of a pass: 128 bytes a row
    int ln = lane;  // (what depends on the lane is formed here, not kept in registers through the products)
    asm volatile("" : "+v"(ln));
    const int l16 = ln & 15, g = ln >> 4;
    const int wn = 64 * (wv % WCOLS), wm = WM * (wv / WCOLS);
    const GemmSegment& sg = a.seg[t.z];
    const int N = sg.N;
    const float sc = sg.scale;
    const uint32_t pitch = (uint32_t)N * ES;
    const int n_rows = t.row_end - t.rb < BM ? t.row_end - t.rb : BM;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<unsigned char*>(sg.C) + (size_t)t.rb * pitch, 0, (int)((uint32_t)n_rows * pitch), 0x00027000);
#pragma unroll
    for (int j = 0; j < JM / 2; ++j) {
#pragma unroll
      for (int p = 0; p < 64 / COLS; ++p) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          const int row = 16 * jj + l16;
          [[maybe_unused]] int grow = t.rb + wm + 32 * j + row;
          if constexpr (EPI == 1 || EPI == 2) grow = grow < t.row_end ? grow : t.row_end - 1;
#pragma unroll
          for (int i = 0; i < COLS / 16; ++i) {
            const int ii = COLS / 16 * p + i;
            float4_t o = acc[2 * j + jj][ii];
            if constexpr (EPI == 1 || EPI == 2) {  // rotation: the lane's columns are two pairs of one head
              const int jn = (t.nb + wn + 16 * ii + 4 * g) % a.d_rope;
              const float4_t cs = *reinterpret_cast<const float4_t*>(a.rope_cs + (size_t)grow * (a.d_rope / 2) + jn / 2);
              o = float4_t{o[0] * cs[0] - o[1] * cs[1], o[0] * cs[1] + o[1] * cs[0], o[2] * cs[2] - o[3] * cs[3], o[2] * cs[3] + o[3] * cs[2]};
            }
            if constexpr (EPI == 3) {
              *reinterpret_cast<float4_t*>(park + row * 128 + (((4 * i + g) ^ (row & 7)) << 4)) = o;
            } else {
              uint2 two;
              if constexpr (EPI == 2) two = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
              else two = make_uint2(pack_f16x2(sc * o[0], sc * o[1]), pack_f16x2(sc * o[2], sc * o[3]));
              *reinterpret_cast<uint2*>(park + row * 128 + (((2 * i + (g >> 1)) ^ (row & 7)) << 4) + 8 * (g & 1)) = two;
            }
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {  // 8 rows of 128 bytes a store
          const int row = 8 * k + (ln >> 3), piece = ln & 7;
          const u32x4_t v = *reinterpret_cast<const u32x4_t*>(park + row * 128 + ((piece ^ (row & 7)) << 4));
          const int col = t.nb + wn + COLS * p + piece * (16 / ES);
          // Always issued, so that the waits for loads behind them can count them: a row past the tile's last lies behind
          // the buffer's end, a column past N is sent there, and the hardware drops both.
          const uint32_t at = (uint32_t)(wm + 32 * j + row) * pitch + (uint32_t)col * ES;
          const int to = (int)(col < N ? at : 0xffffff00u);
          if (a.stream_out) __builtin_amdgcn_raw_buffer_store_b128(v, rs, to, 0, 2 /* nt */);
          else __builtin_amdgcn_raw_buffer_store_b128(v, rs, to, 0, 0);
        }
      }
    }
  }
  __device__ __forceinline__ void leave(const WideTile& t, const float4_t (&acc)[JM][IN], unsigned char* parks) {
    unsigned char* park = parks + wv * kPark;
    const int epi = a.seg[t.z].epi;
    if (epi == 3) way_out<3>(t, acc, park);
    else if (BF16 && epi == 1) way_out<1>(t, acc, park);
    else if (BF16 && epi == 2) way_out<2>(t, acc, park);
    else way_out<0>(t, acc, park);
  }

  // The products of n_jobs tiles from `walk` on, behind begin().  `before_last` is called in front of the last tile's way
  // out, where all slots but the last (which the results pass through) are free; `stores`: of another stream, issued since begin().
  template <class F>
  __device__ __forceinline__ void run(WideWalk walk, int n_jobs, int stores, F&& before_last) {
    const int l16 = lane & 15, g = lane >> 4;
    const uint32_t f0 = (uint32_t)(l16 * 64 + ((g ^ swz_rows16<4>(l16)) << 4));  // row l16 of a 16-row tile, piece g
    const unsigned char* wl = lds + 64 * (wv % WCOLS) * 64 + f0;
    const unsigned char* al = lds + W_BYTES + WM * (wv / WCOLS) * 64 + f0;
    auto read_w = [&](int at, int i) -> u32x4_t { return *reinterpret_cast<const u32x4_t*>(wl + at * STAGE + i * 1024); };
    auto read_a = [&](int at, int j) -> u32x4_t { return *reinterpret_cast<const u32x4_t*>(al + at * STAGE + j * 1024); };
    float4_t acc[JM][IN];
    u32x4_t ar[LA + 1], w0[IN], w1[IN];
    int slot = 0;  // of the stage being multiplied

    // One stage: JM x 4 products of 16 x 16 x 32.  The rows' operands are read LA ahead through a ring, the weights' a stage ahead.
    // The stage's last reads are over before its last LA rows of products: there the workgroup meets, once a stage, its slot
    // may be filled again, and the next stage, landed by now, is read beside the products that are left.
    auto stage = [&](auto first, const u32x4_t (&w)[IN], u32x4_t (&wnext)[IN], auto&& meet, auto&& refill) {
      constexpr bool FIRST = decltype(first)::value;
      constexpr int MEET = JM - 1 - LA;
      const int next = slot + 1 == kSlots ? 0 : slot + 1;
#pragma unroll
      for (int j = 0; j < JM; ++j) {
        if (j <= MEET) ar[(j + LA) & LA] = read_a(slot, j + LA);
        __builtin_amdgcn_sched_barrier(0);
        const u32x4_t av = ar[j & LA];
#pragma unroll
        for (int i = 0; i < IN; ++i) {
          const float4_t c = FIRST ? float4_t{0.f, 0.f, 0.f, 0.f} : acc[j][i];
          if constexpr (BF16)
            acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[i]), __builtin_bit_cast(bf16x8_t, av), c, 0, 0, 0);
          else
            acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, w[i]), __builtin_bit_cast(f16x8_t, av), c, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (j == MEET) {
          meet();
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          barrier_only();
          refill();
#pragma unroll
          for (int i = 0; i < IN; ++i) wnext[i] = read_w(next, i);
        }
        if (j >= MEET && j < JM - 1) ar[(j - MEET) & LA] = read_a(next, j - MEET);
        __builtin_amdgcn_sched_barrier(0);
      }
      slot = next;
    };

    // the first pair of stages: behind it the second pair and another stream's stores
    if (stores == 0) wait_loads_but<2 * NC>();
    else if (stores == 16) wait_loads_but<2 * NC + 16>();
    else wait_loads_but<2 * NC + 32>();
    barrier_only();
#pragma unroll
    for (int i = 0; i < IN; ++i) w0[i] = read_w(0, i);
#pragma unroll
    for (int j = 0; j < LA; ++j) ar[j] = read_a(0, j);
    for (int tile_i = 0;; ++tile_i) {
      const WideTile cur = tile(walk);
      auto none = [&]() {};
      auto ask0 = [&]() {
        if (to_ask > 0) issue(0);
      };
      auto ask1 = [&]() {
        if (to_ask > 0) issue(1);
      };
      // The next pair of stages, this wavefront's part: behind it the first part of the pair after it ...
      auto landed = [&]() {
        if (to_ask <= 0) wait_loads_but<0>();
        else wait_loads_but<2 * HALF>();
      };
      // ... and, in a tile's first stages, the stores of the tile before.
      auto landed_first = [&]() {
        if (to_ask <= 0) wait_loads_but<0>();
        else if (stores == 0) wait_loads_but<2 * HALF>();
        else if (stores == 16) wait_loads_but<2 * HALF + 16>();
        else wait_loads_but<2 * HALF + 32>();
      };
      stage(std::true_type(), w0, w1, none, ask0);
      stage(std::false_type(), w1, w0, landed_first, ask1);
      for (int st = 2; st < n_st; st += 2) {
        stage(std::false_type(), w0, w1, none, ask0);
        stage(std::false_type(), w1, w0, landed, ask1);
      }
      if (tile_i + 1 == n_jobs) {
        before_last();
        leave(cur, acc, lds + (160 * 1024 - kWideWaves * kPark));
        return;
      }
      leave(cur, acc, lds + (slot == 0 ? kSlots - 1 : slot - 1) * STAGE);  // through the slot that was read last
      static_assert(JM == 8 || (BM < 256 || BN < 256), "only 256 x 256 streams have several tiles");
      stores = a.seg[cur.z].epi == 3 ? 32 : 16;
      walk.advance(step, (unsigned)a.col_blocks, (unsigned)rows.n_rb);
    }
  }
};

template <bool BF16>
__global__ __launch_bounds__(kWideThreads, 2) void gemm_wide_kernel(GemmArgs a) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[160 * 1024];
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);

  const bool ragged = a.rows.n_new || a.rows.pos0;
  WideRows rows;
  rows.pitch = ragged ? a.rows.past + a.rows.T : a.M;
  const int n_seq = ragged ? a.M / rows.pitch : 1;
  rows.per = (n_seq + kWave - 1) / kWave;
  rows.used = rows.blocks = 0;
  for (int b = lane * rows.per; b < n_seq && b < (lane + 1) * rows.per; ++b) {
    rows.used = used_rows(a, b);
    rows.blocks += (rows.used + kTile - 1) / kTile;
  }
  rows.upto = wave_scan(rows.blocks);
  rows.n_rb = __builtin_amdgcn_readlane(rows.upto, kWave - 1);

  if (ragged && a.rows.zeros) {  // zeros behind every sequence's last block
    for (int b = 0; b < n_seq; ++b) {
      const int r0 = (used_rows(a, b) + kTile - 1) / kTile * kTile;
      if (r0 >= rows.pitch) continue;
      for (int z = 0; z < a.n_seg; ++z) {
        const size_t row_bytes = (size_t)a.seg[z].N * (a.seg[z].epi == 3 ? 4 : 2);
        unsigned char* p = reinterpret_cast<unsigned char*>(a.seg[z].C) + ((size_t)b * rows.pitch + r0) * row_bytes;
        const size_t n16 = (size_t)(rows.pitch - r0) * row_bytes / 16;
        for (size_t i = (size_t)blockIdx.x * kWideThreads + tid; i < n16; i += (size_t)kWideWgs * kWideThreads)
          reinterpret_cast<u32x4_t*>(p)[i] = u32x4_t{0u, 0u, 0u, 0u};
      }
    }
  }
  if (rows.n_rb <= 0) return;  // no rows

  const unsigned gx = (unsigned)a.col_blocks, n_rb = (unsigned)rows.n_rb;
  const WideShare sh = wide_share(blockIdx.x, gx, n_rb);
  WideWalk at{0u, 0u};
  at.advance(sh.first, gx, n_rb);
  WideWalk part_at{0u, 0u};
  if (sh.cut) part_at.advance(sh.cut_job, gx, n_rb);

  WideStream<BF16, 256, 256> s{a, rows, lds, lane, wv};
  WideStream<BF16, 256, 128> s2{a, rows, lds, lane, wv};
  WideStream<BF16, 128, 128> s4{a, rows, lds, lane, wv};
  bool empty = false;
  auto begin_part = [&]() {
    if (!sh.cut) return;
    // (a part without rows or columns: nothing to do, and none to clear either)
    const WideTile t = tile_at(a, rows, part_at);
    empty = t.rb + 128 * (sh.part >> 1) >= t.row_end || t.nb + 128 * (sh.part & 1) >= a.seg[t.z].N;
    if (empty) return;
    if (sh.cut == 4) s4.begin(part_at, 0u, sh.part, 1);
    else s2.begin(part_at, 0u, sh.part, 1);
  };
  auto nothing = [&]() {};
  int stores = 0;
  if (sh.n_jobs > 0) {
    s.begin(at, sh.step, 0, sh.n_jobs);
    s.run(at, sh.n_jobs, 0, begin_part);
    WideWalk last = at;
    last.advance((unsigned)(sh.n_jobs - 1) * sh.step, gx, n_rb);
    stores = a.seg[tile_at(a, rows, last).z].epi == 3 ? 32 : 16;
  } else {
    begin_part();
  }
  if (!sh.cut || empty) return;
  if (sh.cut == 4) s4.run(part_at, 1, stores, nothing);
  else s2.run(part_at, 1, stores, nothing);
}

}  // namespace

bool gemm_wide_supported(const GemmArgs& a) {
  return a.K >= 128 && a.K % 64 == 0;
}

hipError_t launch_gemm_wide(const GemmArgs& args, hipStream_t st) {
  GemmArgs a = args;
  a.col_blocks = 0;
  size_t out_bytes = 0;
  for (int i = 0; i < a.n_seg; ++i) {
    a.col_blocks += (a.seg[i].N + kTile - 1) / kTile;
    out_bytes += (size_t)a.M * a.seg[i].N * (a.seg[i].epi == 3 ? 4 : 2);
  }
  a.stream_out = out_bytes > kStreamOut;
  if (a.in_bf16) hipLaunchKernelGGL(gemm_wide_kernel<true>, dim3(kWideWgs), dim3(kWideThreads), 0, st, a);
  else hipLaunchKernelGGL(gemm_wide_kernel<false>, dim3(kWideWgs), dim3(kWideThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace mtla
