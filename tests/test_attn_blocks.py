"""The order in which the workgroups of the prefill attention take row blocks (csrc/attn_blocks.h), walked on the host: every block of
every (sequence, head) pair once, the blocks of a pair on one XCD, a group's blocks heaviest first."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13544_amd", "csrc")
SOURCE = """
#include "attn_blocks.h"
extern "C" int group_of(int pairs, int d_head) { return mtla::attn_group(pairs, d_head); }
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


@pytest.mark.parametrize("pairs", [1, 7, 8, 9, 56, 60, 128, 224])
@pytest.mark.parametrize("n_blocks", [1, 2, 3, 16, 21, 32, 65])
@pytest.mark.parametrize("d_head", [64, 128])
def test_every_block_once(blocks, pairs, n_blocks, d_head):
    per, group = (pairs + 7) // 8, blocks.group_of(pairs, d_head)
    assert 1 <= group <= per
    out, seen = (ctypes.c_int * 2)(), {}
    for w in range(8 * per * n_blocks):
        blocks.block_of(w, pairs, n_blocks, group, out)
        assert 0 <= out[0] < 8 * per and 0 <= out[1] < n_blocks and out[0] % 8 == w % 8
        assert (out[0], out[1]) not in seen
        seen[out[0], out[1]] = w
    for pair in range(8 * per):
        order = [seen[pair, x] for x in range(n_blocks)]
        assert order == sorted(order, reverse=True)
