// Which tiles a matrix product of a prefill takes: host arithmetic on its sizes, so that a test can hold it to the times it stands for.
#pragma once
#include <cmath>

namespace mtla {

// 256 x 256 to 64 x 64: gemm_nt_kernel; behind them the streams of gemm_wide.hip (kWide).
struct GemmTile {
  int bm, bn;
  float base, round, k;  // us: `base` fills and empties the units, a round takes round + k K
};
constexpr GemmTile kGemmTiles[] = {
    {256, 256, 5.f, 4.7f, 0.028f}, {256, 128, 5.f, 2.5f, 0.0152f}, {128, 128, 3.2f, 0.5f, 0.0112f}, {64, 64, 2.2f, 0.5f, 0.004f}};
enum { kWide = 4 };

// Tiles that form the angles of the rows they turn (why these: GemmGeom); the others read them from a table.
constexpr bool gemm_own_angles(int bm, int bn) { return bm == 64 && bn == 64; }

// Products with turned rows (ways out 1 and 2).  A row's position is its place in its sequence, found from where that begins: sequences
// are their new rows alone, and with lengths a block of rows is one sequence's.
template <class Args>
bool gemm_turns(const Args& a) {
  for (int i = 0; i < a.n_seg; ++i)
    if (a.seg[i].epi == 1 || a.seg[i].epi == 2) return true;
  return false;
}
template <class Args>
bool gemm_turned_rows_supported(const Args& a) {
  return !gemm_turns(a) || (!a.rows.pos0 && a.rows.past == 0 && !a.rows.zeros && a.rows.T >= 1);
}

// Column blocks of a launch with tiles of bn columns (a segment starts a block of its own).
template <class Args>
int gemm_col_blocks(const Args& a, int bn) {
  int n = 0;
  for (int i = 0; i < a.n_seg; ++i) n += (a.seg[i].N + bn - 1) / bn;
  return n;
}

// Small products (gemm_ring.hip): 16 x 16 tiles of outputs, as many as the sequences may have.  Up to kRingSmall of them one a workgroup,
// up to kRingMedium two, beyond four.  us of a whole layer over short prompts, without / with them for all its products up to 2000 tiles:
// 8 heads x 64, r = 256, 33 tokens 31.9 / 26.7, 129 (594 tiles) 33.4 / 28.0, 257 (1122) 34.2 / 31.1, 400 (1650) 36.0 / 33.8; 16 x 128, r = 512,
// 17 tokens 49.9 / 36.0, 64 (912) 52.1 / 40.6, 129 (2052) 52.0 / 50.1; 32 x 128, 33 tokens (1260) 70.4 / 58.6.  Up to 3000 tiles: 400 tokens of
// the first 34.0, but 2 x 300 36.6 / 38.6, 200 of the second 53.3 / 56.7, 100 of the third 75.9 / 81.2.
constexpr int kRingSmall = 400, kRingMedium = 600, kRingMost = 2000;
template <class Args>
long long gemm_ring_tiles(const Args& a) {
  const bool ragged = (a.rows.n_new || a.rows.pos0) && !a.rows.zeros;
  const int Tp = a.rows.past + a.rows.T;
  const long long rows = ragged ? (long long)(a.M / Tp) * ((Tp + 15) / 16) : ((long long)a.M + 15) / 16;
  return rows * gemm_col_blocks(a, 16);
}
template <class Args>
bool gemm_ring_pays(const Args& a) {
  return gemm_ring_tiles(a) <= kRingMost;
}

// The time of a product in tiles i, as measured on rows in use x 1024 to 4096 columns.  A round is a tile for each of the 256
// units.  us at K = 512 / 2048: 64 x 64 one round 4.9 / 12, two 7.0 / 20, three 9.8 / 28; 128 x 128 one 9 / 25, two 14.5 / 44; the
// streams, whose last round is cut into halves or quarters of a tile where that fills it: a quarter round 10 / 24, half a one
// 13.5 / 35, one 22 / 60, eight 136 / 480.  With ragged rows the number of row blocks is not known here: three quarters of the
// most, and half a block more per sequence, or half a round where blocks may hold rows of several.
template <class Args>
float gemm_tile_cost(const Args& a, int i) {
  const bool ragged = a.rows.n_new || a.rows.pos0;
  const int Tp = ragged ? a.rows.past + a.rows.T : a.M;
  const float n_seq = ragged ? (float)(a.M / Tp) : 1.f, K = (float)a.K;
  // a ragged launch with as many jobs as this may find them all: it is not taken for less than a round
  auto rounds_of = [&](int bm, int bn, bool packed) -> float {
    // (rows that are not packed: every sequence starts a block of its own, however short it is)
    const float cols = (float)gemm_col_blocks(a, bn);
    const float most = packed || !ragged ? (float)((a.M + bm - 1) / bm) : n_seq * (float)((Tp + bm - 1) / bm);
    if (!ragged) return cols * most / 256.f;
    if (cols * most <= 256.f) return cols * most / 256.f;
    return packed ? 0.75f * cols * most / 256.f + 0.5f : cols * fmaxf(0.75f * (float)a.M / (float)bm + 0.5f * n_seq, n_seq) / 256.f;
  };
  if (i == kWide) {
    const float rounds = rounds_of(256, 256, false), left = rounds - floorf(rounds), whole = left > 0.5f ? ceilf(rounds) : floorf(rounds);
    float cost = 5.f + whole * (4.4f + 0.0246f * K);
    if (left > 0.25f && left <= 0.5f) cost += 1.2f + 0.0142f * K;
    else if (left > 0.f && left <= 0.25f) cost += 0.0097f * K;
    return cost;
  }
  const GemmTile& t = kGemmTiles[i];
  float of = rounds_of(t.bm, t.bn, a.rows.zeros);
  if (ragged && t.bm == 256) {
    // A row block's tiles are one XCD's: few blocks of many rows leave some XCDs two and others one (7 sequences of 137 to 551
    // rows, 2112 columns, K = 1024: 14 blocks in 256 x 128 tiles 36.4 us, 22 in 128 x 128 25.8)
    const float cols = (float)gemm_col_blocks(a, t.bn), blocks = 256.f * of / cols;
    if (blocks >= 8.f) of = ceilf(blocks / 8.f) * cols / 32.f;
  }
  const float rounds = ceilf(of);
  float cost = t.base + rounds * (t.round + t.k * K);
  if (t.bm == 64 && rounds > 2.f) cost += 0.6f;  // (two fit on a unit)
  return cost;
}

// The least of them, and whose it is.
template <class Args>
float gemm_cost(const Args& a, bool wide_supported, int& pick) {
  float best = 0.f;
  pick = 0;
  for (int i = 0; i <= kWide; ++i) {
    if (i == kWide && !wide_supported) break;
    const float cost = gemm_tile_cost(a, i);
    if (i == 0 || cost < best) {
      best = cost;
      pick = i;
    }
  }
  return best;
}

// What a call becomes: the small products; or tiles, with the narrowest product in a launch of its own if that saves time (64 columns
// beside 3584 at 32768 rows open half a round of 256 x 256 tiles more).  `part`: of a call that was split.  A part is tiles whatever its size:
// that is what its time was compared as, and the small products of 64 columns beside thousands of rows read every row for few of them
// and form every angle anew (us of that part, 64 x 64 tiles / 32 x 32 of the small products: 8000 rows, K = 1536 12.9 / 35.6; K = 4096 28.2 / 79.3).
struct GemmPlan {
  bool ring;
  int pick, alone;  // tile; the product by itself or -1
};
template <class Args>
void gemm_without(const Args& a, int alone, Args& one, Args& rest) {
  one = rest = a;
  one.n_seg = 1;
  one.seg[0] = a.seg[alone];
  rest.n_seg = a.n_seg - 1;
  for (int i = alone; i + 1 < a.n_seg; ++i) rest.seg[i] = a.seg[i + 1];
}
template <class Args, class Wide>
GemmPlan gemm_plan(const Args& a, bool part, Wide wide_supported) {
  GemmPlan p{!part && gemm_ring_pays(a), 0, -1};
  if (p.ring) return p;
  const float whole = gemm_cost(a, wide_supported(a), p.pick);
  if (a.n_seg < 2) return p;
  int least = 0, p1 = 0, p2 = 0;
  for (int i = 1; i < a.n_seg; ++i)
    if (a.seg[i].N < a.seg[least].N) least = i;
  Args one, rest;
  gemm_without(a, least, one, rest);
  if (gemm_cost(one, wide_supported(one), p1) + gemm_cost(rest, wide_supported(rest), p2) < whole) p.alone = least;
  return p;
}

}  // namespace mtla
