"""The library's page bookkeeping (host only) against a plain walk over Python lists and dicts."""
import numpy as np
import pytest

from paper_2505_13544_amd import binding as B


class Book:
    def __init__(self, max_batch, max_slots, page_slots, stride, n_pages):
        pages = -(-max_slots // page_slots)
        self.table, self.next_table = (np.full((max_batch, pages), -1, np.int32) for _ in range(2))
        self.len, self.next_len = (np.zeros(max_batch, np.int64) for _ in range(2))
        self.refs, self.ring = np.zeros(n_pages, np.int32), np.arange(n_pages, dtype=np.int32)
        at = lambda x: x.ctypes.data
        self.c = B.mtla_page_book(at(self.table), at(self.next_table), at(self.len), at(self.next_len), at(self.refs),
                                  at(self.ring), 0, n_pages, max_batch, pages, n_pages, page_slots, stride, max_slots)

    def reserve(self, n_new):
        n = np.asarray(n_new, np.int32)
        return B.lib.mtla_pages_reserve(self.c, n.ctypes.data, len(n))

    def fork(self, src):
        src, fresh = np.asarray(src, np.int32), np.zeros(len(src), np.int32)
        rc = B.lib.mtla_pages_fork(self.c, src.ctypes.data, len(src), fresh.ctypes.data)
        if rc == 0:
            self.table, self.next_table = self.next_table, self.table
            self.len, self.next_len = self.next_len, self.len
        return rc, fresh


def check_counts(k):
    """Every page is named refs[p] times, and the ring holds exactly the pages nobody names."""
    named = np.bincount(k.table[k.table >= 0], minlength=len(k.refs))
    assert np.array_equal(named, k.refs)
    free = [int(k.ring[(k.c.free_head + i) % len(k.ring)]) for i in range(k.c.free_count)]
    assert sorted(free) == np.flatnonzero(named == 0).tolist()


@pytest.mark.parametrize("batch,page_slots,stride", [(1, 16, 1), (7, 16, 2), (12, 64, 3)])
def test_pages_of_a_random_beam_search(batch, page_slots, stride):
    max_slots = 5 * page_slots
    k = Book(batch, max_slots, page_slots, stride, batch * 7)
    rng = np.random.default_rng(batch)
    for step in range(200):
        room = max_slots * stride - int(k.len.max())
        if room <= 0:
            break
        n_new = rng.integers(0, min(room, page_slots) + 1, batch)
        before = k.table.copy()
        filled = k.reserve(n_new)
        assert filled == int(((before < 0) & (k.table >= 0)).sum()) and np.array_equal(before[before >= 0], k.table[before >= 0])
        k.len[:] += n_new
        for b in range(batch):
            need = -(-(-(-int(k.len[b]) // stride)) // page_slots)
            assert (k.table[b, :need] >= 0).all()
        check_counts(k)
        src = rng.integers(0, batch, rng.integers(1, batch + 1)) if step % 3 else rng.permutation(batch)
        old, old_len = k.table.copy(), k.len.copy()
        rc, fresh = k.fork(src)
        assert rc == 0
        for b, s in enumerate(src):
            pw = min(int(old_len[s]) // stride, max_slots - 1) // page_slots
            assert np.array_equal(k.table[b, :pw], old[s, :pw]) and k.table[b, pw] == fresh[b] and (k.table[b, pw + 1:] == -1).all()
            assert k.len[b] == old_len[s]
            alone = int((src == s).sum()) == 1 and old[s, pw] >= 0
            assert (fresh[b] == old[s, pw]) if alone else (fresh[b] not in old[old >= 0])
        assert (k.table[len(src):] == -1).all() and (k.len[len(src):] == 0).all()
        check_counts(k)


def test_refused_calls_change_nothing():
    k = Book(2, 32, 16, 1, 3)
    assert k.reserve([17, 1]) == 3
    k.len[:] = [17, 1]
    state = lambda: (k.table.tolist(), k.len.tolist(), k.refs.tolist(), k.c.free_count)
    was = state()
    assert k.reserve([0, 16]) == -2 and state() == was          # no page left
    assert k.fork([0, 0])[0] == -2 and state() == was           # two continuations need two pages of their own
    assert k.fork([0, 2])[0] == -1 and k.fork([-1])[0] == -1 and state() == was
    assert k.reserve([1, 1, 1]) == -1
