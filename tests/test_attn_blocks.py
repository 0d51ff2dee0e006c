"""The order in which the workgroups of the prefill attention take row blocks (csrc/attn_blocks.h), walked on the host: every block of
every (sequence, head) pair once, the blocks of a pair on one XCD, a group's blocks heaviest first; and how many rows a block has."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13544_amd", "csrc")
SOURCE = """
#include "attn_blocks.h"
extern "C" int group_of(int pairs, int d_head, int at_once) { return mtla::attn_group(pairs, d_head, at_once); }
extern "C" int at_once(int rows, int pairs, int n_blocks, int d_head, int past) { return mtla::attn_at_once(rows, pairs, n_blocks, d_head, past); }
extern "C" int rows_of(int T, int pairs, int d_head, int past) { return mtla::attn_rows(T, pairs, d_head, past); }
extern "C" int two_a_unit(int rows, int pairs, int n_blocks, int T, int s, int d_head, int past) { return mtla::attn_two_a_unit(rows, pairs, n_blocks, T, s, d_head, past); }
extern "C" void block_of(unsigned w, int pairs, int n_blocks, int group, int* out) {
  const mtla::AttnBlock b = mtla::attn_block(w, pairs, n_blocks, group);
  out[0] = b.pair;
  out[1] = b.block;
}
"""


@pytest.fixture(scope="module")
def blocks(tmp_path_factory):
    where = tmp_path_factory.mktemp("blocks")
    (where / "b.cpp").write_text(SOURCE)
    so = str(where / "b.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", str(where / "b.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("pairs", [1, 7, 8, 9, 56, 60, 72, 128, 224])
@pytest.mark.parametrize("n_blocks", [1, 2, 3, 16, 21, 32, 65])
@pytest.mark.parametrize("d_head", [64, 128])
@pytest.mark.parametrize("at_once", [0, 1])
def test_every_block_once(blocks, pairs, n_blocks, d_head, at_once):
    per, group = (pairs + 7) // 8, blocks.group_of(pairs, d_head, at_once)
    assert 1 <= group <= per
    assert not at_once or group == per
    out, seen = (ctypes.c_int * 2)(), {}
    for w in range(8 * per * n_blocks):
        blocks.block_of(w, pairs, n_blocks, group, out)
        assert 0 <= out[0] < 8 * per and 0 <= out[1] < n_blocks and out[0] % 8 == w % 8
        assert (out[0], out[1]) not in seen
        seen[out[0], out[1]] = w
    # on an XCD: group after group, of a group block after block from the last one on, of a block place all pairs of the group
    for xcd in range(8):
        order = [seen[8 * (first + i) + xcd, x] for first in range(0, per, group) for x in reversed(range(n_blocks)) for i in range(min(group, per - first))]
        assert order == sorted(order)


@pytest.mark.parametrize("pairs,d_head,group", [(8, 128, 1), (32, 128, 4), (56, 128, 7), (64, 128, 4), (72, 128, 5), (128, 128, 4), (128, 64, 8),
                                                (120, 64, 15), (224, 64, 10)])
def test_pairs_side_by_side(blocks, pairs, d_head, group):
    assert blocks.group_of(pairs, d_head, 0) == group


@pytest.mark.parametrize("lens,heads,d_head,one_group", [((8, 257), 16, 128, True), ((5, 700), 16, 128, True), ((8, 400), 12, 128, True), ((8, 400), 16, 128, True),
                                                         ((8, 1000), 12, 128, False), ((1, 1000), 16, 128, False), ((8, 257), 16, 64, False)])
def test_one_group_where_all_blocks_are_there_at_once(blocks, lens, heads, d_head, one_group):
    B, T = lens
    rows = blocks.rows_of(T, B * heads, d_head, 0)
    assert bool(blocks.at_once(rows, B * heads, -(-T // rows), d_head, 0)) == one_group
    assert not blocks.at_once(rows, B * heads, -(-T // rows), d_head, 1)


# prompts, rows of each, heads, d_head, slots of a past, and the rows of a block that were the faster ones
@pytest.mark.parametrize("B,T,heads,d_head,past,rows", [
    (1, 2048, 8, 128, 0, 64), (1, 2048, 16, 128, 0, 64), (3, 1024, 16, 128, 0, 128), (2, 2048, 16, 128, 0, 128), (64, 64, 16, 128, 0, 64),
    (64, 65, 16, 128, 0, 128), (1, 4096, 8, 64, 0, 64), (2, 3072, 8, 64, 0, 64), (32, 256, 8, 64, 0, 64), (8, 500, 20, 64, 0, 64), (8, 1100, 8, 64, 0, 64), (5, 2000, 8, 64, 0, 128), (4, 4096, 8, 64, 0, 128),
    (2, 512, 16, 128, 1000, 64), (8, 128, 16, 128, 4000, 64), (12, 128, 16, 128, 1000, 128), (48, 64, 16, 128, 4000, 64),
    (16, 128, 8, 64, 4000, 64), (32, 65, 8, 64, 4000, 128), (24, 128, 8, 64, 4000, 128), (16, 256, 8, 64, 4000, 128), (28, 128, 8, 64, 1000, 64),
    (32, 65, 8, 64, 1000, 128)])
def test_rows_of_a_block(blocks, B, T, heads, d_head, past, rows):
    assert blocks.rows_of(T, B * heads, d_head, past) == rows


@pytest.mark.parametrize("B,T,heads,s,d_head,two", [(1, 4000, 20, 1, 64, True), (1, 4000, 20, 2, 64, True), (1, 4000, 20, 4, 64, False), (1, 4700, 16, 4, 64, True), (2, 3200, 16, 1, 64, True),
                                                    (2, 1900, 20, 2, 64, True), (5, 900, 16, 1, 64, False), (2, 4000, 20, 2, 64, False), (1, 4000, 20, 1, 128, False),
                                                    (1, 4000, 8, 1, 64, False)])
def test_two_blocks_a_unit(blocks, B, T, heads, s, d_head, two):
    rows = blocks.rows_of(T, B * heads, d_head, 0)
    assert bool(blocks.two_a_unit(rows, B * heads, -(-T // rows), T, s, d_head, 0)) == two
    assert not blocks.two_a_unit(rows, B * heads, -(-T // rows), T, s, d_head, 1)
