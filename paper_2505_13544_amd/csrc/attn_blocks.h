// Which row block of which (sequence, head) pair a workgroup of the prefill attention takes: plain arithmetic, without device code, so
// that the host can walk the same list.
#pragma once

namespace mtla {

constexpr int kAttnRows = 128;  // query rows of a block; of a small one half
constexpr int kXcds = 8;        // workgroup w runs on XCD w % 8

// Pairs of an XCD, and how many of them are side by side (`group`).  A group's blocks go out heaviest first (a block walks the columns
// in front of its last row), all pairs' of one place in the sequence before the next; the next group's heavy ones then meet this one's light
// ones.  A heavy and a light block for every workgroup instead, as many columns for each, left units idle behind ragged prompts (7
// of 1287 to 2574 rows, 8 heads x 128, s = 2, 115 -> 99 us a pass; 3 of 3000, 16 x 64, 103 -> 85), and all pairs in one group had the heavy
// blocks of all in step: 8 prompts of 2048, 16 heads x 128, groups of 2, 4, 8, 16: 235, 228, 234, 245 us (4096: 555, 556, 568, 588; 1024: 111, 106,
// 113, 116); 8 of 4096, 8 x 64, s = 1, groups of 4 and 8: 237 and 230.  Groups are as equal as whole pairs allow (72 pairs at d_head 128: 5 and 4).
// `at_once`: blocks of 128 rows, heads of 128, no cache in front of them (behind one all blocks are heavy), and no more of them than the chip holds side by side: there is no next round for a group to
// meet, and all heavy ones first leave a unit's second place to a light one.  Groups / one: 8 of 6 to 257, 16 heads (384 blocks) 55.3 / 51.6, 5 of 700, 16 heads
// (480) 72.1 / 69.4, 8 of 10 to 400, 12 heads (384) 48.0 / 46.4, 8 of 400, 16 heads (512) 67.9 / 66.6; but 8 of 1000, 12 heads (768) 81.4 / 86.0, and with
// blocks of 64, one of 1000, 16 heads (256) 48.9 / 52.4.  (d_head 64, three on a unit: no difference up to 1024 blocks.)
[[gnu::always_inline]] constexpr int attn_pairs(int pairs) { return (pairs + kXcds - 1) / kXcds; }  // of an XCD
constexpr int attn_group(int pairs, int d_head, bool at_once) {
  const int per = attn_pairs(pairs), about = d_head <= 64 ? 8 : 4, groups = per / about > 1 && !at_once ? per / about : 1;
  return (per + groups - 1) / groups;
}
constexpr bool attn_at_once(int rows, int pairs, int n_blocks, int d_head, int past) {
  return rows == kAttnRows && d_head > 64 && past == 0 && (long long)pairs * n_blocks <= 512;
}

// Rows of a block of the plain form.  Where a unit has one block of 128 or none, the heaviest one's chain is the pass, and half the rows
// in each wavefront shorten it (every pair of tiles is still read by all wavefronts, so with more blocks than that the LDS is what they
// wait for).  us a pass, 128 rows / 64: 2048 tokens, 8 heads x 128 (128 blocks of 128 rows) 55.3 / 48.6, 16 heads (256) 60.4 / 55.4, 24 heads (384) 71.6
// / 68.7, but 3 of 1024 (384) 60.4 / 61.7 and 2 of 2048 (512) 75.6 / 77.5; d_head 64, whose blocks take half the LDS: 4096 x 8 heads (256) 57.3 / 49.1, 2 of
// 3072 (384) 56.1 / 51.3, 32 of 256 (512) 40.1 / 38.7, 8 of 500, 20 heads, s = 1 (640) 53.9 / 52.3, 5 of 900, 16 heads, s = 2
// (640) 50.7 / 51.3, of 225 to 900 45.6 / 44.2, but 5 of 2000 (640) 59.8 / 62.0, s = 1, 1024 blocks 127.7 / 146.6.  Behind `past` slots of a cache all blocks are heavy: 2 of 512, 16 x 128
// (128) 50.7 / 45.0, 8 of 128 (128) 117.4 / 114.0, 12 of 128 (192) 150.0 / 159.2; d_head 64, 16 of 128 (128) 63.2 / 55.6, 32 of 128 (256) 81.8 / 79.5, of 65 64.0 / 65.4; the longer the
// past, the more of the pass is those reads: behind 4000 slots, 8 x 64, times of 64 rows over those of 128 at 128, 160, 192 and 256 blocks 0.90, 0.99, 1.03 and 1.03.
// And up to 64 rows the other half of a block would be empty: 64 prompts of 64, 16 x 128 78.4 / 73.6; 48 behind a cache 307 / 299.
[[gnu::always_inline]] constexpr int attn_rows(int T, int pairs, int d_head, int past) {
  const long long blocks = (long long)((T + kAttnRows - 1) / kAttnRows) * pairs;
  const int most = d_head <= 64 ? (past == 0 ? (T <= 1100 ? 640 : 512) : (past <= 2048 ? 240 : 160)) : (past == 0 ? 256 : 128);
  return T <= kAttnRows / 2 || blocks <= most ? kAttnRows / 2 : kAttnRows;
}

// Whether a unit is kept to two blocks of 128 rows (heads of 64 and their registers leave room for three).  With a few more blocks than two a unit all are
// there from the start, and the unit that got three heavy ones is last; two at a time, the third goes to whoever is done.  It shows where a block
// walks many columns.  us a pass, three / two a unit: one prompt of 4000, 20 heads (640 blocks), s = 1 116.6 / 111.5, s = 2 79.4 / 76.4, s = 4 61.7 / 64.8; of 4700, 16 heads (592), s = 4 61.2
// / 59.9; 2 of 3200, 16 heads (800), s = 1 105.1 / 98.9, s = 4 60.3 / 62.7; 2 of 1900, 20 heads (600), s = 2 57.0 / 56.1; 5 of 900, 16 heads (640), s = 1 58.7 / 60.0; beyond, 2 of 4000,
// 20 heads (1280) 106.9 / 110.1.
[[gnu::always_inline]] constexpr bool attn_two_a_unit(int rows, int pairs, int n_blocks, int T, int s, int d_head, int past) {
  const long long blocks = (long long)pairs * n_blocks;
  return rows == kAttnRows && d_head <= 64 && past == 0 && blocks > 512 && blocks <= (s <= 2 ? 800 : 600) && T >= 950LL * s;
}

struct AttnBlock {
  int pair, block;  // pair: head + n_heads * sequence; may be past the last one
};
[[gnu::always_inline]] constexpr AttnBlock attn_block(unsigned workgroup, int pairs, int n_blocks, int group) {
  const int per = attn_pairs(pairs), i = (int)(workgroup / kXcds), first = i / (group * n_blocks) * group;
  const int size = per - first < group ? per - first : group, rest = i - first * n_blocks;
  return AttnBlock{kXcds * (first + rest % size) + (int)(workgroup % kXcds), n_blocks - 1 - rest / size};
}

}  // namespace mtla
