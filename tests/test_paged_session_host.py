"""The host side of PagedSession without a GPU: buffers in host memory, launches replaced by records of their arguments."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2505_13544_amd import binding as B
from paper_2505_13544_amd import session as S


class Launches:
    def __init__(self):
        self.capturing, self.fail, self.forks = False, 0, []

    def fork(self, ctx, c, kr, table, tail, lens, src, fresh, batch, *dst):
        if isinstance(self.fail, Exception):
            raise self.fail
        if not self.fail:
            ints = lambda at: list((ctypes.c_int32 * batch).from_address(at))
            self.forks.append((ints(src), ints(fresh)))
        return self.fail


@pytest.fixture
def launches(monkeypatch):
    class Event:
        def record(self, stream):
            pass

        def synchronize(self):
            pass

    rec, empty = Launches(), torch.empty
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: None)
    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch, "empty", lambda *a, pin_memory=False, **k: empty(*a, **k))
    monkeypatch.setattr(S, "_raw_stream", lambda device: 0)
    monkeypatch.setattr(torch._C, "_cuda_isCurrentStreamCapturing", lambda: rec.capturing)
    monkeypatch.setattr(B.Context, "workspace_init", lambda *a: None)
    monkeypatch.setattr(B.calls, "mtla_cache_fork_paged", rec.fork)
    return rec


def make(max_batch=4, n_pages=24, order=None):
    return S.PagedSession(n_heads=2, d_head=64, r=64, d_rope=32, d_hyper=16, stride=2, max_batch=max_batch, max_slots=64,
                          page_slots=16, n_pages=n_pages, device="cpu", page_order=order)


def grow(s, n_new):
    s.reserve(n_new)
    s.h_len[:len(n_new)] += np.asarray(n_new)


def state(s):
    k = s._book
    assert (k.table, k.next_table) == (s.h_table.ctypes.data, s._h_next[0].ctypes.data)
    assert (k.len, k.next_len) == (s.h_len.ctypes.data, s._h_next[1].ctypes.data)
    assert np.array_equal(np.bincount(s.h_table[s.h_table >= 0], minlength=s.n_pages), s.refs)
    assert sorted(s.free) == np.flatnonzero(s.refs == 0).tolist()
    return s.h_table.tolist(), s.h_len.tolist(), s.refs.tolist(), s.free.tolist(), s.table.data_ptr(), s.table.tolist()


def test_bookkeeping_is_refused_while_the_stream_is_captured(launches):
    s = make()
    grow(s, [40, 7, 0, 33])
    was = state(s)
    launches.capturing = True
    with pytest.raises(RuntimeError, match="captur"):
        s.fork([0, 0, 1, 3])
    with pytest.raises(RuntimeError, match="captur"):
        s.reserve([64, 64, 64, 64])
    assert state(s) == was and not launches.forks
    s.reserve([1, 1, 0, 0])                       # the pages are there already: nothing to copy, a step can be captured
    launches.capturing = False
    s.reserve([64, 64, 64, 64])
    assert np.array_equal(s.table.numpy()[s.h_table >= 0], s.h_table[s.h_table >= 0])
    s.fork([0, 0, 1, 3])
    assert len(launches.forks) == 1 and state(s) != was


@pytest.mark.parametrize("n_pages", [10, 11, 24])            # the ring nearly used up, and with room
def test_a_fork_whose_launch_fails_changes_nothing(launches, n_pages):
    rng = np.random.default_rng(n_pages)
    s = make(n_pages=n_pages, order=rng.permutation(n_pages))
    grow(s, [35, 5, 0, 30])                                   # pages 2, 1, 0, 1
    for src in ([0, 0, 1, 3], [3, 1, 0], [0, 1, 2, 3], [2, 2, 2, 2], [0]):
        was = state(s)
        for launches.fail in (B.MTLA_ERR_HIP, TypeError("an argument")):
            with pytest.raises((B.MtlaError, TypeError)):
                s.fork(src)
            assert state(s) == was
        launches.fail = 0
        s.fork(src)
        state(s)
        expected = [was[1][b] for b in src] + [0] * (4 - len(src))
        assert s.h_len.tolist() == expected and launches.forks[-1][0] == src
        grow(s, [4] * 4)


def test_what_a_fork_and_a_reserve_take(launches):
    s = make(n_pages=40)
    s.reserve([])                                             # nothing to do
    s.reserve(torch.tensor([3, 3, 3, 3]))
    s.h_len[:] = 3

    class Number:
        def __int__(self):
            return 1

    s.fork([Number(), 0])
    assert launches.forks.pop()[0] == [1, 0]
    for src in ([0, 1, 1, 3], (0, 1, 1, 3), range(4), (x for x in [3, 2, 1, 0]), np.array([2, 2, 2, 2]), torch.tensor([0, 1])):
        s.fork(src)
        state(s)
    assert [f[0] for f in launches.forks] == [[0, 1, 1, 3], [0, 1, 1, 3], [0, 1, 2, 3], [3, 2, 1, 0], [2, 2, 2, 2], [0, 1]]
    was, pinned = state(s), s._picks.host.copy()
    for bad in ([], [0] * 5, [0] * 9):                        # a pinned slot holds four sources and four pages
        with pytest.raises(IndexError):
            s.fork(bad)
    assert np.array_equal(s._picks.host, pinned)
    for bad in ([4], [-1]):
        with pytest.raises(IndexError):
            s.fork(bad)
    assert state(s) == was
