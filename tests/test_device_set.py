"""Set-up that belongs to a device (csrc/device_set.h: the permission of a kernel to take more than 64 KB of LDS) is remembered
for that device and for no other, compiled and run on the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13544_amd", "csrc")

PROGRAM = r"""
#include "device_set.h"
#include <thread>
#include <vector>
int main() {
  mtla::DeviceSet s;
  for (int d = -1; d < 70; ++d) if (s.has(d)) return 1;
  s.add(0);
  s.add(5);
  for (int d = -1; d < 70; ++d) if (s.has(d) != (d == 0 || d == 5)) return 2;
  s.add(64);                                     // past the last one that is kept, and no device at all
  s.add(-1);
  for (int d = -1; d < 70; ++d) if (s.has(d) != (d == 0 || d == 5)) return 3;
  std::vector<std::thread> t;
  for (int d = 0; d < 64; d += 2) t.emplace_back([&s, d] { s.add(d); s.add(d + 1); });
  for (auto& x : t) x.join();
  for (int d = -1; d < 70; ++d) if (s.has(d) != (d >= 0 && d < 64)) return 4;
  mtla::DeviceSet other;
  return other.has(0) ? 5 : 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_devices_are_remembered_one_by_one(tmp_path):
    (tmp_path / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-pthread", "-I", CSRC, str(tmp_path / "main.cpp"), "-o",
                    str(tmp_path / "main")], check=True)
    assert subprocess.run([str(tmp_path / "main")], timeout=60).returncode == 0


def test_no_launcher_remembers_for_the_whole_process():
    for name in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, name)).read()
        assert "static bool" not in text, name
        calls = text.count("hipFuncSetAttribute(")
        assert calls == (1 if name == "mtla_kernels.h" else 0), name   # all through allow_lds
