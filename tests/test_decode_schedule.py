"""The rule that picks the schedule of a decode step's attention (csrc/decode_schedule.h), compiled and run on the host: where both schedules were
measured it takes the faster one, and below eight tiles a unit, where the balanced one's outputs are less exact, it takes chunks."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13544_amd", "csrc")
SOURCE = """
#include "decode_schedule.h"
extern "C" int chunk(int max_batch, int max_slots) { return mtla::decode_chunk(max_batch, max_slots); }
extern "C" int balanced(int r, int n_heads, int batch, int max_slots, int chunk, int chunk_set, int n_cu) {
  return mtla::decode_balanced(r, n_heads, batch, max_slots, chunk, chunk_set, n_cu);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    where = tmp_path_factory.mktemp("schedule")
    (where / "s.cpp").write_text(SOURCE)
    so = str(where / "s.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", str(where / "s.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


def takes(rule, r, heads, batch, max_batch, max_slots, n_cu=256):
    return bool(rule.balanced(r, heads, batch, max_slots, rule.chunk(max_batch, max_slots), 0, n_cu))


# r, heads, sequences of the call, of the session, slots, us a step in chunks and balanced (256 units, heads of 64 but where 16 or 32 at r >= 256: 128)
MEASURED = [
    (128, 8, 32, 32, 1024, 12.8, 16.4), (128, 8, 100, 100, 1000, 17.2, 20.0), (128, 8, 112, 112, 1024, 17.6, 21.3), (128, 8, 256, 256, 640, 19.9, 24.9),
    (128, 8, 128, 256, 1024, 18.8, 22.1), (128, 8, 24, 128, 2048, 15.9, 19.0), (128, 8, 36, 256, 1024, 15.7, 16.5), (128, 8, 2, 14, 16384, 15.6, 19.5), (128, 8, 256, 256, 512, 18.5, 23.3),
    (128, 8, 14, 28, 8192, 21.6, 20.6), (128, 8, 448, 448, 512, 31.9, 28.7), (128, 8, 90, 512, 1024, 21.1, 20.2), (128, 8, 40, 512, 1024, 19.8, 16.7),
    (128, 8, 6, 64, 8192, 19.6, 16.6), (128, 16, 208, 208, 1024, 31.4, 27.9), (128, 20, 112, 112, 1024, 24.2, 30.5), (128, 20, 56, 224, 1024, 20.2, 21.8),
    (128, 20, 256, 256, 1024, 33.1, 46.9), (128, 20, 64, 256, 1024, 21.4, 22.9), (128, 20, 16, 16, 8192, 26.6, 22.9), (128, 20, 32, 224, 1024, 19.2, 18.3), (128, 20, 36, 256, 1024, 20.6, 18.7),
    (128, 20, 40, 512, 1024, 27.8, 19.5), (128, 32, 6, 64, 8192, 27.6, 20.2),
    (256, 8, 32, 32, 1024, 16.1, 18.7), (256, 8, 64, 64, 1024, 19.6, 22.5), (256, 8, 100, 100, 1000, 23.4, 25.0), (256, 8, 128, 128, 1024, 25.2, 27.1),
    (256, 8, 4, 16, 8192, 18.1, 20.1), (256, 8, 2, 8, 16384, 19.2, 23.5), (256, 16, 32, 128, 1024, 20.2, 21.8), (256, 16, 100, 100, 1000, 26.3, 28.3),
    (256, 8, 256, 256, 768, 37.2, 32.9), (256, 8, 256, 256, 1504, 52.0, 46.8), (256, 16, 256, 256, 2048, 66.8, 45.6), (256, 8, 256, 256, 512, 25.5, 28.2),
    (256, 8, 96, 96, 1024, 26.8, 24.7), (256, 8, 40, 160, 1024, 20.4, 19.5), (256, 8, 160, 160, 1024, 33.7, 29.9), (256, 8, 24, 128, 2048, 24.0, 21.7),
    (256, 8, 40, 512, 1024, 30.9, 19.0), (256, 8, 90, 512, 1024, 32.6, 25.1), (256, 8, 6, 64, 8192, 31.3, 20.6), (256, 16, 40, 512, 1024, 36.4, 22.6),
    (256, 32, 32, 32, 1024, 29.6, 26.4), (256, 32, 100, 100, 1000, 47.8, 35.2), (256, 20, 40, 512, 1024, 46.7, 24.4),
    (512, 20, 16, 16, 1024, 24.9, 28.4),
    (512, 32, 2, 2, 12000, 36.3, 38.5), (512, 16, 24, 24, 1000, 28.8, 29.0), (256, 32, 24, 24, 1000, 23.2, 24.4),
    (512, 16, 32, 32, 1024, 31.8, 29.1), (512, 16, 24, 128, 2048, 42.4, 32.5), (512, 32, 50, 50, 1000, 72.1, 44.2), (512, 32, 6, 64, 8192, 90.1, 31.8),
]


@pytest.mark.parametrize("r,heads,batch,max_batch,max_slots,chunks,balanced", MEASURED)
def test_takes_the_faster_one(rule, r, heads, batch, max_batch, max_slots, chunks, balanced):
    assert takes(rule, r, heads, batch, max_batch, max_slots) == (balanced < chunks)


@pytest.mark.parametrize("r", [64, 128, 256, 512])
@pytest.mark.parametrize("heads", [1, 16, 17, 32])
def test_small_calls_take_chunks(rule, r, heads):
    for batch, max_slots in ((1, 32752), (31, 1040), (127, 256), (2047, 16), (63, 511), (24, 1000), (12, 2600), (8, 4000)):
        assert -(-max_slots // 16) * batch < 8 * 256
        for max_batch in (batch, 4 * batch, 65535):
            assert not rule.balanced(r, heads, batch, max_slots, rule.chunk(max_batch, max_slots), 0, 256)
        for chunk in (32, 1024):
            assert not rule.balanced(r, heads, batch, max_slots, chunk, 1, 256)


@pytest.mark.parametrize("r", [64, 128, 256, 512])
@pytest.mark.parametrize("n_cu", [1, 32, 256, 1024])
def test_border(rule, r, n_cu):
    # r = 64, and any chunk of the caller's: eight tiles a unit, with nothing else asked
    for batch in (8 * n_cu - 1, 8 * n_cu, 8 * n_cu + 1, 64 * n_cu):
        for chunk in (32, 64, 4096):
            assert bool(rule.balanced(r, 8, batch, 16, chunk, 1, n_cu)) == (batch >= 8 * n_cu)
        assert bool(rule.balanced(64, 8, batch, 16, 64, 0, n_cu)) == (batch >= 8 * n_cu)


def test_sizes_at_the_limits(rule):
    assert rule.chunk(1, 1) == 64 and rule.chunk(512, 64) == 64 and rule.chunk(513, 64) == 128 and rule.chunk(65535, 2 ** 31 - 1) == 1024
    for r in (64, 128, 256, 512):
        assert rule.balanced(r, 8, 65535, 2 ** 31 - 1, 1024, 0, 256) == 1
        assert rule.balanced(r, 32, 65535, 2 ** 31 - 1, 32, 1, 256) == 1
