"""The list of jobs of the streamed matrix products (csrc/gemm_jobs.h, csrc/bounds.h), compiled and walked on the host: whatever
the starts and lengths of the sequences are, every tile that holds rows in use is taken once, by one workgroup, and none lies
outside the rows and columns that there are."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13544_amd", "csrc")

PROGRAM = r"""
#include "bounds.h"
#include "gemm_jobs.h"
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <tuple>
#include <vector>
using namespace mtla;

struct Args {
  struct { int N; } seg[4];
  int n_seg, col_blocks, M;
  struct { int past, T, stride, zeros; } rows;
};
#define CHECK(x) do { if (!(x)) { std::printf("case %d: %s\n", g_case, #x); std::exit(1); } } while (0)
int g_case;

struct Rows {                       // the kernel's record, lane by lane
  const Args& a;
  const std::vector<int>*pos0, *n_new;
  int per, pitch, n_rb;
  int v_used[64], v_blocks[64], v_upto[64];
  int lane_of(int block) const {
    for (int i = 0; i < 64; ++i) if (block < v_upto[i]) return i;
    CHECK(!"a block that no lane stands for");
    return 0;
  }
  int upto(int i) const { return v_upto[i]; }
  int blocks(int i) const { return v_blocks[i]; }
  int used(int i) const { return v_used[i]; }
  int used_rows(int b) const {
    if (!pos0 && !n_new) return a.M;
    CHECK(b >= 0 && (size_t)b < (pos0 ? pos0 : n_new)->size());
    return (pos0 ? slots_inside((*pos0)[b], a.rows.stride, a.rows.past) : 0) + (n_new ? new_rows((*n_new)[b], a.rows.T) : a.rows.T);
  }
};

void walk(const Args& a, const std::vector<int>* pos0, const std::vector<int>* n_new) {
  const bool ragged = pos0 || n_new;
  const int pitch = ragged ? a.rows.past + a.rows.T : a.M, n_seq = ragged ? a.M / pitch : 1;
  Rows r{a, pos0, n_new, (n_seq + 63) / 64, pitch, 0, {}, {}, {}};
  std::vector<int> used(n_seq);
  for (int i = 0, sum = 0; i < 64; ++i) {
    for (int b = i * r.per; b < n_seq && b < (i + 1) * r.per; ++b) {
      used[b] = r.v_used[i] = r.used_rows(b);
      CHECK(used[b] >= 0 && used[b] <= pitch);
      r.v_blocks[i] += (used[b] + 255) / 256;
    }
    r.v_upto[i] = sum += r.v_blocks[i];
  }
  r.n_rb = r.v_upto[63];
  CHECK(r.n_rb >= 0);
  std::map<std::tuple<int, int, int>, int> taken;   // (first row, first column, segment) of a quarter -> how often
  auto take = [&](const WideTile& t, int dr, int dc) {
    if (t.rb + dr >= t.row_end || t.nb + dc >= a.seg[t.z].N) return;  // a part without rows or columns
    ++taken[{t.rb + dr, t.nb + dc, t.z}];
  };
  if (r.n_rb > 0) {
    const unsigned gx = a.col_blocks, n_rb = r.n_rb;
    for (unsigned w = 0; w < (unsigned)kWideWgs; ++w) {
      const WideShare sh = wide_share(w, gx, n_rb);
      auto tile = [&](const WideWalk& at) {
        const WideTile t = wide_tile(a, r, at);
        const int b = t.rb / pitch;
        CHECK(t.rb >= 0 && b < n_seq && t.rb % pitch < used[b] && t.rb % pitch % 256 == 0);
        CHECK(t.row_end == b * pitch + (a.rows.zeros ? pitch : used[b]) && t.row_end <= a.M);
        CHECK(t.z >= 0 && t.z < a.n_seg && t.nb >= 0 && t.nb < a.seg[t.z].N);
        return t;
      };
      WideWalk at{0u, 0u};
      at.advance(sh.first, gx, n_rb);
      CHECK((unsigned long long)sh.n_jobs <= (unsigned long long)gx * n_rb);
      for (int i = 0; i < sh.n_jobs; ++i, at.advance(sh.step, gx, n_rb)) {
        const WideTile t = tile(at);
        for (int q = 0; q < 4; ++q) take(t, 128 * (q >> 1), 128 * (q & 1));
      }
      if (sh.cut) {
        WideWalk c{0u, 0u};
        c.advance(sh.cut_job, gx, n_rb);
        const WideTile t = tile(c);
        take(t, 128 * (sh.part >> 1), 128 * (sh.part & 1));
        if (sh.cut == 2) take(t, 128 + 128 * (sh.part >> 1), 128 * (sh.part & 1));
      }
    }
  }
  size_t expected = 0;
  for (int b = 0; b < n_seq; ++b)
    for (int row = 0; row < used[b]; row += 256)
      for (int h = 0; h < 256; h += 128) {
        if (b * pitch + row + h >= b * pitch + (a.rows.zeros ? pitch : used[b])) continue;
        for (int z = 0; z < a.n_seg; ++z)
          for (int col = 0; col < a.seg[z].N; col += 128) {
            const auto it = taken.find({b * pitch + row + h, col, z});
            CHECK(it != taken.end() && it->second == 1);
            ++expected;
          }
      }
  CHECK(taken.size() == expected);
}

int main() {
  std::mt19937 g(7);
  auto in = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(g); };
  for (g_case = 0; g_case < 600; ++g_case) {
    Args a{};
    a.n_seg = in(1, 4);
    for (int z = 0; z < a.n_seg; ++z) {
      a.seg[z].N = 8 * in(1, in(0, 1) ? 40 : 400);
      a.col_blocks += (a.seg[z].N + 255) / 256;
    }
    a.rows.stride = in(1, 4);
    a.rows.past = in(0, 2) ? in(0, 2000) : 0;
    a.rows.T = in(1, in(0, 1) ? 20 : 1500);
    a.rows.zeros = in(0, 3) == 0;
    const int n_seq = in(0, 2) ? in(1, 20) : in(60, 200);   // more sequences than lanes among them
    a.M = n_seq * (a.rows.past + a.rows.T);
    std::vector<int> pos0(n_seq), n_new(n_seq);
    const int all = a.rows.past * a.rows.stride;
    for (int b = 0; b < n_seq; ++b) {
      const int bad[] = {-1, -4096, INT_MIN, all + a.rows.stride, INT_MAX};
      pos0[b] = g_case % 3 == 0 && in(0, 2) == 0 ? bad[in(0, 4)] : in(0, all + a.rows.stride - 1);
      n_new[b] = in(0, 5) == 0 ? (in(0, 1) ? -in(0, 3000) : a.rows.T + in(0, 9)) : in(0, a.rows.T);
      if (g_case % 7 == 0) n_new[b] = b % 3 ? 0 : n_new[b];  // empty ones
    }
    walk(a, a.rows.past ? &pos0 : (in(0, 1) ? &pos0 : nullptr), in(0, 2) ? &n_new : nullptr);
  }
  // one sequence of 510 new rows that starts far below zero, 1500 past slots, 32 column blocks: once about 2^32 row blocks
  g_case = -1;
  Args a{{{4096}, {4096}}, 2, 32, 2010, {1500, 510, 2, 0}};
  std::vector<int> pos0{-4096};
  walk(a, &pos0, nullptr);
  for (int p : {0, 1, 5, 2999, 3000, 3001, 3002, INT_MAX, -1, -4096, INT_MIN})
    if (slots_inside(p, 2, 1500) != start_inside(p, 2, 1500) / 2 || slots_inside(p, 2, 1500) != (p < 0 || p > 3001 ? 1500 : p / 2)) return 2;
  if (new_rows(-3, 510) != 0 || new_rows(INT_MIN, 510) != 0 || new_rows(511, 510) != 510 || new_rows(7, 510) != 7) return 3;
  return 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_every_tile_is_taken_once_and_none_lies_outside(tmp_path):
    (tmp_path / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main")], check=True)
    run = subprocess.run([str(tmp_path / "main")], timeout=100, capture_output=True, text=True)
    assert run.returncode == 0, run.stdout + run.stderr
