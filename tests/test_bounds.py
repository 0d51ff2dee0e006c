"""What lengths and starts out of the caller's arrays count as (csrc/bounds.h), compiled and run on the host, and that the kernels take
them through it."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13544_amd", "csrc")

PROGRAM = r"""
#include "bounds.h"
#include <climits>
#include <initializer_list>
using namespace mtla;
int main() {
  for (int s : {1, 2, 3, 5, 16})
    for (int slots : {1, 2, 15, 16, 640}) {
      const long long cap = (long long)slots * s;
      for (int len = -3 * s; len <= cap + 3 * s; ++len) {
        const long long in = len < 0 ? 0 : (len > cap ? cap : len);   // the nearer end of what the capacity allows
        if (live_slots(len, s, slots) != (in + s - 1) / s) return 1;
      }
      for (int len : {INT_MAX, INT_MAX - 1}) if (live_slots(len, s, slots) != slots) return 2;
      for (int len : {INT_MIN, INT_MIN + 1}) if (live_slots(len, s, slots) != 0) return 3;
    }
  if (append_status(0, 1, 2, 1) != 0 || append_status(1, 1, 2, 1) != 0 || append_status(2, 1, 2, 1) != 3 || append_status(-1, 1, 2, 1) != 1 ||
      append_status(INT_MIN, 1, 1, INT_MAX) != 1 || append_status(INT_MAX, 1, 1, INT_MAX) != 3 || append_status(INT_MAX - 1, 1, 1, INT_MAX) != 0)
    return 5;
  return live_slots(INT_MAX, 1, INT_MAX) == INT_MAX && live_slots(INT_MAX, 16, INT_MAX / 16) == INT_MAX / 16 ? 0 : 4;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_lengths(tmp_path):
    (tmp_path / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main")], check=True)
    assert subprocess.run([str(tmp_path / "main")], timeout=60).returncode == 0


def test_kernels_take_lengths_through_it():
    # every decode kernel that reads seq_len, and the beam reordering: no count of slots that the capacity does not bound
    counted = re.compile(r"(seq_len\[[^\]]*\]|\blen) \+ (a\.)?stride - 1\) / ")
    users = set()
    for name in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, name)).read()
        if name.endswith(".hip"):
            assert not counted.search(text), name
        if "live_slots(" in text:
            users.add(name)
    assert {"append.hip", "attn_cols.hip", "attn_f32.hip", "attn_mfma.hip", "attn_valu.hip", "attn_whole.hip", "combine_mfma.hip",
            "proj.hip"} <= users
