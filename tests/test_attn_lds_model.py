"""The prefill attention (attn_explicit_kernel in csrc/prefill_explicit.hip) as tests/test_gemm_stream_model.py has the products: who
writes and reads which of its four LDS buffers between which meetings, while a block's queries and own rows change lanes in them, its tiles pass
through and its outputs leave through them; and which rows of a sequence's keys and values it reads for which start, against those that
the launches in front of it wrote."""
import os
import subprocess

import pytest

from tests.test_gemm_stream_model import Wave, check

KB, BUFFERS, WAVES = 1024, 4, 4


class Geometry:
    """TileGeom<d_head, d_rope>: bytes of a tile, of a wavefront's part of a pair of them, and what passes through that part."""

    def __init__(self, d_head, d_rope):
        self.tile = 32 * 2 * (2 * d_head + d_rope)
        self.own = 2 * self.tile // WAVES
        self.turn = KB * ((d_head + d_rope) // 32 + d_head // 32)   # 16 rows' queries and values, 64 bytes a piece
        self.leave = 16 * d_head * 4                                 # 16 rows' outputs
        assert self.turn <= self.own and self.leave <= self.own


def a_block(wave, g, n, reads, *, wait=0, drained=True, leave=lambda n: ~(n - 1) & 2 if n > 0 else 0):
    """One workgroup: n tiles; reads(t): whether the wavefront multiplies the pair of tiles from t on (none above its rows); every wavefront asks
    for its part of every tile.  wait: loads left in flight by the wait of a step; drained: the turns are over when the wavefront meets the others;
    leave(n): first buffer of the pair that the outputs leave through."""
    def issue(t):
        wave.load(t % BUFFERS * g.tile, (t % BUFFERS + 1) * g.tile, t, 1)

    def pass_through(first, size, tag):          # every wavefront its own part, written and read in its own order
        for w in range(WAVES):
            at = first * g.tile + w * g.own
            wave.now(at, at + size, (tag, w), write=True)

    if n > 0:
        issue(0)
        issue(1)
    pass_through(2, g.turn, "rows")
    if not drained:
        for a in wave.accesses[-WAVES:]:
            a["last"] += 1
    for t in range(0, n, 2):
        wave.wait_but(wait)
        wave.meet()
        if t + 2 < n:
            issue(t + 2)
            issue(t + 3)
        if reads(t):
            for u in (0, 1):
                wave.now((t + u) % BUFFERS * g.tile, ((t + u) % BUFFERS + 1) * g.tile, t + u)
    pass_through(leave(n), g.leave, "outputs")
    wave.wait_but(0)


GEOMETRIES = [(128, 64), (128, 32), (64, 64), (64, 32)]
TILES = [0, 1, 2, 3, 4, 5, 6, 7, 8, 33]


@pytest.mark.parametrize("d_head,d_rope", GEOMETRIES)
@pytest.mark.parametrize("n", TILES)
def test_lds_of_a_block(d_head, d_rope, n):
    g = Geometry(d_head, d_rope)
    wave = Wave()
    a_block(wave, g, n, lambda t: True)
    check(wave.accesses)
    # a wavefront that skips the steps above its rows, beside one that does not: the same meetings
    skips = Wave()
    a_block(skips, g, n, lambda t: t < n // 2)
    assert skips.space == wave.space
    check(wave.accesses + [a for a in skips.accesses if not a["write"]])


@pytest.mark.parametrize("mistake", [dict(wait=1), dict(drained=False), dict(leave=lambda n: (n - 1) & 2)])
def test_the_model_sees_a_mistake(mistake):
    # a step that waits for one load less; turns that are still under way when their place is filled; outputs in the pair that is being read
    wave = Wave()
    a_block(wave, Geometry(128, 64), 6, lambda t: True, **mistake)
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
            for m0, rows_of_block in [(m, 128) for m in range(0, used, 128)] + [(m, 64) for m in range(0, used, 64)]:
                n_cols = (p0 + min(m0 + rows_of_block, used) - 1) // s
                cols = range(-(-n_cols // 32) * 32 + 32)
                rows = [c if c < j0 else past + c * s + s - 1 - p0 for c in (min(c, n_cols - 1) for c in cols)] if n_cols else []
                own = [past + min(m, used - 1) for m in range(m0, m0 + rows_of_block)]
                assert all(0 <= row < written for row in rows + own), (start, used, m0)
                # every column that a row sees is one that closed before it
                assert all(row < past or row - past < min(m0 + rows_of_block, used) - 1 for row in rows), (start, used, m0)
