"""The rule that picks the tiles of a prefill's matrix products (csrc/gemm_tiles.h), compiled and run on the host: its estimates stand for the
measured times that its comment gives, and it picks the faster tiles where both sides were measured."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13544_amd", "csrc")

PROGRAM = r"""
#include "gemm_tiles.h"
#include <cstdio>
#include <vector>
using namespace mtla;
struct Args {
  int M, K, n_seg;
  struct { int N, epi; } seg[4];
  struct { const int *pos0, *n_new; int past, T, zeros; } rows;
};
static int some;
Args equal(int M, int N, int K) { return Args{M, K, 1, {{N, 0}}, {nullptr, nullptr, 0, 1, 0}}; }
Args ragged(int n_seq, int past, int T, std::vector<int> N, int K, int zeros = 0) {
  Args a{n_seq * (past + T), K, (int)N.size(), {}, {past ? &some : nullptr, &some, past, T, zeros}};
  for (size_t i = 0; i < N.size(); ++i) a.seg[i].N = N[i];
  return a;
}
int failed;
void near(const char* what, float estimate, float measured) {   // the estimates choose between neighbours that lie 1.2 and more apart
  if (std::fabs(estimate - measured) <= 0.15f * measured) return;
  std::printf("%s: %.1f us estimated, %.1f measured\n", what, estimate, measured);
  ++failed;
}
void picks(const char* what, const Args& a, int tile, bool wide = true) {
  int pick = -1;
  gemm_cost(a, wide, pick);
  if (pick == tile) return;
  std::printf("%s: tiles %d\n", what, pick);
  ++failed;
}
int main() {
  const struct { int tile, rows, cols; float us512, us2048; const char* what; } kMeasured[] = {
      {3, 1024, 1024, 4.9f, 12.f, "64 x 64, one round"}, {3, 2048, 1024, 7.0f, 20.f, "64 x 64, two"}, {3, 3072, 1024, 9.8f, 28.f, "64 x 64, three"},
      {2, 2048, 2048, 9.f, 25.f, "128 x 128, one round"}, {2, 4096, 2048, 14.5f, 44.f, "128 x 128, two"},
      {kWide, 1024, 4096, 10.f, 24.f, "streams, a quarter round"}, {kWide, 2048, 4096, 13.5f, 35.f, "streams, half a round"},
      {kWide, 4096, 4096, 22.f, 60.f, "streams, one round"}, {kWide, 32768, 4096, 136.f, 480.f, "streams, eight"}};
  for (const auto& m : kMeasured) {
    near(m.what, gemm_tile_cost(equal(m.rows, m.cols, 512), m.tile), m.us512);
    near(m.what, gemm_tile_cost(equal(m.rows, m.cols, 2048), m.tile), m.us2048);
  }
  picks("1000 rows x 1024 columns", equal(1000, 1024, 512), 3);                 // (256 tiles: 4.9 us)
  picks("7 sequences of up to 551 rows", ragged(7, 0, 551, {2112}, 1024), 2);   // 36.4 us in 256 x 128 tiles, 25.8
  picks("32768 x 3584 x 2048", equal(32768, 3584, 2048), kWide);                // 452 us in 256 x 256 tiles, 378
  picks("32768 x 4096 x 512", equal(32768, 4096, 512), kWide);                  // 171, 136
  picks("a contraction that is no multiple of 64", equal(32768, 4096, 2080), 0, false);
  // two sequences of 510 new rows behind up to 1500 slots, 16 heads x 128: what the GPU's test of their starts relies on
  picks("two chunks", ragged(2, 1500, 510, {2048, 2048}, 512), kWide);
  // whatever the sizes, the estimate is of a tile that there is, and never grows when rows are taken away
  for (int M : {1, 63, 64, 65, 500, 5000, 50000})
    for (int N : {8, 64, 72, 1000, 4096})
      for (int K : {64, 512, 4096}) {
        int p = -1, q = -1;
        const float a = gemm_cost(equal(M, N, K), true, p), b = gemm_cost(equal(2 * M, N, K), true, q);
        if (p < 0 || p > kWide || !(a > 0.f) || a > b) {
          std::printf("%d x %d x %d: %f, %f\n", M, N, K, a, b);
          ++failed;
        }
      }
  // rows that are turned: new rows of sequences alone, in blocks of one sequence each
  auto turned = [&](const char* what, Args a, int epi, bool taken) {
    a.seg[a.n_seg - 1].epi = epi;
    if (gemm_turned_rows_supported(a) == taken) return;
    std::printf("turned rows, %s\n", what);
    ++failed;
  };
  turned("all rows", equal(100, 64, 64), 1, true);
  turned("lengths", ragged(3, 0, 40, {512, 64}, 64), 2, true);
  turned("rows behind a past", ragged(3, 5, 40, {512, 64}, 64), 2, false);
  turned("blocks of several sequences", ragged(3, 0, 40, {512, 64}, 64, 1), 1, false);
  turned("none turned", ragged(3, 5, 40, {512, 64}, 64, 1), 3, true);
  // the product that is launched by itself, and its parts, which are tiles however few they have: a layer's q, q^R, c and k^R
  auto wide = [](const Args&) { return true; };
  auto splits = [&](const char* what, const Args& a, int alone, int tile) {
    const GemmPlan whole = gemm_plan(a, false, wide);
    bool good = !whole.ring && whole.alone == alone;
    if (good && alone >= 0) {
      Args one, rest;
      gemm_without(a, alone, one, rest);
      const GemmPlan p = gemm_plan(one, true, wide), q = gemm_plan(rest, true, wide);
      good = one.n_seg == 1 && rest.n_seg == a.n_seg - 1 && one.seg[0].N == a.seg[alone].N && !p.ring && p.pick == tile && p.alone < 0 && !q.ring;
      for (int i = 0; i < rest.n_seg; ++i) good = good && rest.seg[i].N == a.seg[i + (i >= alone)].N;
    }
    if (good) return;
    std::printf("%s: ring %d, alone %d\n", what, whole.ring, whole.alone);
    ++failed;
  };
  auto layer = [](int n_seq, int T, int heads, int d_head, int r) { return ragged(n_seq, 0, T, {heads * d_head, heads * d_head / 2, r, d_head / 2}, heads * d_head); };
  splits("2 x 4000 rows, 12 heads x 128", layer(2, 4000, 12, 128, 256), 3, 3);   // 2000 tiles of 16 x 16: 12.9 us in 64 x 64, 35.6 as small products
  splits("6000 rows, 16 heads x 128", layer(1, 6000, 16, 128, 512), 3, 3);       // 14.4, 33.5
  splits("2 x 4000 rows, 32 heads x 128", layer(2, 4000, 32, 128, 512), 3, 3);   // 28.2, 79.3
  splits("1000 rows, 8 heads x 64", layer(1, 1000, 8, 64, 256), -1, 0);
  // the small products, and where they end: whole layers over short prompts, as measured with and without them
  auto small = [&](const char* what, const Args& a, bool ring, int tile = -1) {
    const GemmPlan p = gemm_plan(a, false, wide);
    if (p.ring == ring && p.ring == (gemm_ring_tiles(a) <= kRingMost) && (ring || tile < 0 || (p.pick == tile && p.alone < 0))) return;
    std::printf("%s: ring %d, %lld tiles, pick %d\n", what, p.ring, gemm_ring_tiles(a), p.pick);
    ++failed;
  };
  small("33 tokens, 8 heads x 64", layer(1, 33, 8, 64, 256), true);      // 31.9 us without, 26.7
  small("129 tokens, 8 heads x 64", layer(1, 129, 8, 64, 256), true);    // 33.4, 28.0
  small("400 tokens, 8 heads x 64", layer(1, 400, 8, 64, 256), true);    // 36.0, 33.8
  small("2 x 300 tokens, 8 heads x 64", layer(2, 300, 8, 64, 256), false);   // 36.6, 38.6
  small("64 tokens, 16 heads x 128", layer(1, 64, 16, 128, 512), true);      // 52.1, 40.6
  small("200 tokens, 16 heads x 128", layer(1, 200, 16, 128, 512), false);   // 53.3, 56.7
  small("33 tokens, 32 heads x 128", layer(1, 33, 32, 128, 512), true);      // 70.4, 58.6
  small("100 tokens, 32 heads x 128", layer(1, 100, 32, 128, 512), false);   // 75.9, 81.2
  small("129 rows x 512 columns", equal(129, 512, 512), true);
  small("one row", equal(1, 8, 32), true);
  small("2000 tiles", equal(800, 640, 512), true);
  small("2050 tiles", equal(801, 656, 512), false);
  // tiles with rows of several sequences that form their own angles (tests/test_gpu_layer_prefill_angles.py): 5 sequences, 8 heads x 64, r = 256
  for (int d_rope : {32, 64})
    for (int tokens : {1, 13, 33, 64, 65, 100, 120}) {
      Args a = equal(5 * tokens, 512, 128);
      a.n_seg = 4;
      a.seg[1].N = 8 * d_rope;
      a.seg[1].epi = 1;
      a.seg[2].N = 256;
      a.seg[3].N = d_rope;
      a.seg[3].epi = 2;
      a.rows.T = tokens;
      small("rows of several sequences", a, tokens < 100, 3);
    }
  for (int i = 0; i < kWide; ++i) failed += gemm_own_angles(kGemmTiles[i].bm, kGemmTiles[i].bn) != (i == 3);
  return failed ? 1 : 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_estimates_stand_for_measured_times(tmp_path):
    (tmp_path / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main")], check=True)
    run = subprocess.run([str(tmp_path / "main")], timeout=60, capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
