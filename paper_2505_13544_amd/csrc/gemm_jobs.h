// The list of jobs of the streamed matrix products (gemm_wide.hip) and who takes which: plain arithmetic, without device code,
// so that the host can walk the same list.
//
// A job is a 256 x 256 tile.  Column blocks are those of the segments, one segment behind the other; row blocks those that the
// sequences use, each sequence's from its first row on.
#pragma once

namespace mtla {

constexpr int kWideTile = 256, kWideWgs = 256;

// A place in the list of jobs: groups of four column blocks (the last one: what is left) slowest, then the row blocks, then the
// blocks of the group, so that the jobs side by side on an XCD share their operands in its L2.
struct WideWalk {
  unsigned first, rem;                     // first column block of the group, place in the group
  [[gnu::always_inline]] constexpr unsigned size(unsigned gx) const { return gx - first < 4u ? gx - first : 4u; }
  [[gnu::always_inline]] constexpr void advance(unsigned n, unsigned gx, unsigned n_rb) {
    rem += n;
    while (first + 4u < gx && rem >= 4u * n_rb) {
      rem -= 4u * n_rb;
      first += 4u;
    }
  }
};

// The jobs of a workgroup.  An XCD (workgroup w runs on XCD w % 8) takes an eighth of the list, its 32 workgroups every 32nd
// job of that.  The jobs of a last round that would leave half of them idle or more are cut into halves or quarters.
struct WideShare {
  unsigned first, step;                    // whole tiles: jobs first, first + step, ..
  int n_jobs;                              // so many
  unsigned cut, cut_job;                   // behind them, if cut: this job's part ..
  int part;                                // .. a half (cut 2: column half `part`) or a quarter (cut 4: 2 row half + column half)
};
[[gnu::always_inline]] constexpr WideShare wide_share(unsigned workgroup, unsigned gx, unsigned n_rb) {
  const unsigned xcd = workgroup & 7u, wi = workgroup >> 3, nwg = kWideWgs / 8;
  const unsigned long long total = (unsigned long long)gx * n_rb;
  const unsigned lo = (unsigned)(total * xcd / 8u), n = (unsigned)(total * (xcd + 1) / 8u) - lo;
  const unsigned left = n % nwg, cut = left == 0 ? 0 : (left <= nwg / 4 ? 4 : (left <= nwg / 2 ? 2 : 0));
  const unsigned whole = cut ? n - left : n;
  const bool part = cut && wi < left * cut;
  return WideShare{lo + wi,
                   nwg,
                   wi < whole ? (int)((whole - wi + nwg - 1) / nwg) : 0,
                   part ? cut : 0u,
                   part ? lo + whole + (cut == 4 ? wi >> 2 : wi >> 1) : 0u,
                   part ? (int)(cut == 4 ? wi & 3u : wi & 1u) : 0};
}

struct WideTile {
  int rb, row_end, nb, z;                  // first row, row behind the last, first column, segment
};
// The tile at a place.  Rows: where the rows are, with lane i standing for sequences i * per .. + per - 1 (upto(i): the blocks
// of all sequences up to them, blocks(i): theirs, used(i): the rows in use of sequence i if per = 1, used_rows(b): of sequence b,
// lane_of(block): the first lane whose upto() is above it).
template <class Args, class Rows>
[[gnu::always_inline]] constexpr WideTile wide_tile(const Args& a, const Rows& r, const WideWalk& w) {
  const unsigned gsz = w.size((unsigned)a.col_blocks);
  const unsigned ib = gsz == 4u ? w.rem >> 2 : (gsz == 3u ? w.rem / 3u : (gsz == 2u ? w.rem >> 1 : w.rem));
  const int at = r.lane_of((int)ib);
  int block = (int)ib - (r.upto(at) - r.blocks(at));
  int b = at, used = r.used(at);
  if (r.per > 1) {
    b = at * r.per;
    used = r.used_rows(b);
    while (block >= (used + kWideTile - 1) / kWideTile) {
      block -= (used + kWideTile - 1) / kWideTile;
      used = r.used_rows(++b);
    }
  }
  const int rb = b * r.pitch + block * kWideTile, row_end = b * r.pitch + (a.rows.zeros ? r.pitch : used);
  int cb = (int)(w.first + (w.rem - ib * gsz)), z = 0;
  for (int n = (a.seg[0].N + kWideTile - 1) / kWideTile; z + 1 < a.n_seg && cb >= n; n = (a.seg[z].N + kWideTile - 1) / kWideTile) {
    cb -= n;
    ++z;
  }
  return WideTile{rb, row_end, cb * kWideTile, z};
}

}  // namespace mtla
