// Which row block of which (sequence, head) pair a workgroup of the prefill attention takes: plain arithmetic, without device code, so
// that the host can walk the same list.
#pragma once

namespace mtla {

constexpr int kAttnRows = 128;  // query rows of a block
constexpr int kXcds = 8;        // workgroup w runs on XCD w % 8

// Pairs of an XCD, and how many of them are side by side (`group`).  A group's blocks go out heaviest first (a block walks the columns
// in front of its last row), all pairs' of one place in the sequence before the next; the next group's heavy ones then meet this one's light
// ones.  A heavy and a light block for every workgroup instead, as many columns for each, left units idle behind ragged prompts (7
// of 1287 to 2574 rows, 8 heads x 128, s = 2, 115 -> 99 us a pass; 3 of 3000, 16 x 64, 103 -> 85), and all pairs in one group had the heavy
// blocks of all in step: 8 prompts of 2048, 16 heads x 128, groups of 2, 4, 8, 16: 235, 228, 234, 245 us (4096: 555, 556, 568, 588; 1024: 111, 106,
// 113, 116); 8 of 4096, 8 x 64, s = 1, groups of 4 and 8: 237 and 230.  Groups are of equal size, so that the last one is no smaller.
[[gnu::always_inline]] constexpr int attn_pairs(int pairs) { return (pairs + kXcds - 1) / kXcds; }  // of an XCD
constexpr int attn_group(int pairs, int d_head) {
  const int per = attn_pairs(pairs), about = d_head <= 64 ? 8 : 4, groups = per / about > 1 ? per / about : 1;
  return (per + groups - 1) / groups;
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
