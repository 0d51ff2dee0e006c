"""The prefill attention (attn_explicit_kernel in csrc/prefill_explicit.hip) as tests/test_gemm_stream_model.py has the products: who
writes and reads which of its four LDS buffers between which meetings, over the two row blocks of a workgroup; and which rows of a
sequence's keys and values it reads for which start, against those that the launches in front of it wrote."""
import os
import subprocess

import pytest

from tests.test_gemm_stream_model import Wave, check

BYTES, BUFFERS = 20 * 1024, 4


def blocks_of(wave, tiles, reads, wait=0):
    """reads(block, t): whether the wavefront multiplies the pair of tiles from t on (none above its rows); every wavefront asks for
    its part of every tile.  wait: loads left in flight by the wait of a step."""
    for k, n in enumerate(tiles):
        def issue(t):
            wave.load(t % BUFFERS * BYTES, (t % BUFFERS + 1) * BYTES, (k, t), 1)
        wave.meet()                              # the buffers of the block before are read
        if n > 0:
            issue(0)
            issue(1)
        for t in range(0, n, 2):
            wave.wait_but(wait)
            wave.meet()
            if t + 2 < n:
                issue(t + 2)
                issue(t + 3)
            if reads(k, t):
                for u in (0, 1):
                    wave.now((t + u) % BUFFERS * BYTES, ((t + u) % BUFFERS + 1) * BYTES, (k, t + u))
    wave.wait_but(0)


@pytest.mark.parametrize("first", [0, 1, 2, 3, 4, 5, 7, 8, 33])
@pytest.mark.parametrize("second", [None, 0, 1, 2, 3, 6])
def test_lds_of_the_two_blocks(first, second):
    tiles = [first] if second is None else [first, second]
    writer = Wave()
    blocks_of(writer, tiles, lambda k, t: True)
    check(writer.accesses)
    # a wavefront that skips the steps above its rows, beside one that does not: the same meetings
    skips = Wave()
    blocks_of(skips, tiles, lambda k, t: t < tiles[k] // 2)
    assert skips.space == writer.space
    check(writer.accesses + [a for a in skips.accesses if not a["write"]])


def test_the_model_sees_a_step_that_waits_for_one_load_less():
    wave = Wave()
    blocks_of(wave, [6, 2], lambda k, t: True, wait=1)
    with pytest.raises(AssertionError):
        check(wave.accesses)


@pytest.fixture(scope="module")
def inside(tmp_path_factory):
    """start_inside of csrc/bounds.h, compiled for the host."""
    where = tmp_path_factory.mktemp("bounds")
    header = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_13544_amd", "csrc", "bounds.h")
    (where / "b.cpp").write_text(
        "#define __host__\n#define __device__\n#define __forceinline__ inline\n#include <cstdint>\n#include \"%s\"\n"
        "extern \"C\" long long inside(int p, int s, int n) { return mtla::start_inside(p, s, n); }\n" % header)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(where / "b.so"), str(where / "b.cpp")], check=True)
    import ctypes
    f = ctypes.CDLL(str(where / "b.so")).inside
    f.restype = ctypes.c_longlong
    return f


@pytest.mark.parametrize("s,past_pitch,T", [(1, 0, 300), (1, 70, 129), (2, 150, 255), (3, 40, 200), (4, 33, 128), (16, 5, 140)])
def test_rows_read_are_rows_written(inside, s, past_pitch, T):
    for start in (-4096, -1, 0, 1, s, past_pitch * s // 2 + 1, past_pitch * s, past_pitch * s + 1, 2 ** 31 - 1):
        p0 = inside(start, s, past_pitch)
        assert 0 <= p0 < (past_pitch + 1) * s    # (the slot in progress may hold tokens)
        j0 = past = p0 // s
        for used in {1, T // 2 + 1, T}:
            written = past + used                # the staging launch and the product: slots of the past, then the new rows
            assert written <= past_pitch + T
            for m0 in range(0, used, 128):
                n_cols = (p0 + min(m0 + 128, used) - 1) // s
                cols = range(-(-n_cols // 32) * 32 + 32)
                rows = [c if c < j0 else past + c * s + s - 1 - p0 for c in (min(c, n_cols - 1) for c in cols)] if n_cols else []
                own = [past + min(m, used - 1) for m in range(m0, m0 + 128)]
                assert all(0 <= row < written for row in rows + own), (start, used, m0)
                # every column that a row sees is one that closed before it
                assert all(row < past or row - past < min(m0 + 128, used) - 1 for row in rows), (start, used, m0)
