"""A model of who writes and reads which byte of LDS when in the streamed matrix products (WideStream in csrc/gemm_wide.hip), walked over
stage counts, job counts, ways out and cut last tiles.  Eight wavefronts run one program and meet once a stage, so an access
is placed by the meetings it lies between: a load to LDS from the meeting behind which it is asked for to the one in front of
which its wavefront has waited for it (the vector-memory counter goes down in order, loads and stores alike), a read to the one in front
of which reads are over.  Two accesses in the space between the same two meetings may happen in either order: none of
them may be a write beside another one or beside a read of the same byte, and a read has to find its own stage's bytes."""
import itertools

import pytest

KB, SLOTS, LDS = 1024, 5, 160 * 1024
PARK = 8 * 4096


class Wave:
    """One wavefront's program: accesses [first, last] space between meetings, and its vector-memory operations in flight."""

    def __init__(self):
        self.space, self.queue, self.accesses = 0, [], []

    def load(self, lo, hi, tag, count):
        access = dict(lo=lo, hi=hi, tag=tag, write=True, first=self.space, last=None)
        self.accesses.append(access)
        self.queue += [access] * count

    def stores(self, n):
        self.queue += [None] * n

    def wait_but(self, n):
        done, self.queue = self.queue[:len(self.queue) - n], self.queue[len(self.queue) - n:]
        for access in done:
            if access is not None and not any(access is left for left in self.queue):
                access["last"] = self.space

    def now(self, lo, hi, tag, write=False):
        self.accesses.append(dict(lo=lo, hi=hi, tag=tag, write=write, first=self.space, last=self.space))

    def meet(self):
        self.space += 1


class Stream:
    """WideStream<.., BM, BN>: the same numbers and the same order of operations."""

    def __init__(self, wave, name, bm, bn):
        self.wave, self.name = wave, name
        self.w_bytes = bn * 64
        self.stage_bytes = self.w_bytes + bm * 64
        self.nc = bn // 128 + bm // 128          # 1 KB chunks a wavefront brings of a stage
        self.half = (self.nc + 1) // 2           # of a part, each for two stages
        assert self.stage_bytes * SLOTS <= LDS and self.nc * 8 * KB == self.stage_bytes

    def issue(self, i):
        nxt = (self.slot + 1) % SLOTS
        chunks = range(self.half, self.nc) if i else range(self.half)
        for c in chunks:                         # eight wavefronts' chunks: 8 KB of the stage
            for slot, stage in ((self.slot, self.asked), (nxt, self.asked + 1)):
                self.wave.load(slot * self.stage_bytes + 8 * KB * c, slot * self.stage_bytes + 8 * KB * (c + 1), (self.name, stage), 1)
        if i == 0:
            return
        self.slot, self.asked, self.to_ask = (nxt + 1) % SLOTS, self.asked + 2, self.to_ask - 2

    def begin(self, n_jobs, n_st):
        self.n_jobs, self.n_st, self.slot, self.asked, self.to_ask = n_jobs, n_st, 0, 0, n_jobs * n_st
        for _ in range(2):
            self.issue(0)
            self.issue(1)

    def run(self, stores, stores_of, before_last=lambda: None):
        """stores: of another stream, issued since begin(); stores_of(job): of a job's way out."""
        wave = self.wave
        wave.wait_but(2 * self.nc + stores)
        wave.meet()
        slot = stage = 0

        def multiply(wait, part):
            nonlocal slot, stage
            wave.now(slot * self.stage_bytes, (slot + 1) * self.stage_bytes, (self.name, stage))  # its reads are over at its meeting
            if wait:
                wave.wait_but(wait())
            wave.meet()
            if self.to_ask > 0:
                self.issue(part)
            slot, stage = (slot + 1) % SLOTS, stage + 1

        landed = lambda: 0 if self.to_ask <= 0 else 2 * self.half
        for job in range(self.n_jobs):
            multiply(None, 0)
            multiply(lambda: 0 if self.to_ask <= 0 else 2 * self.half + stores, 1)
            for _ in range(2, self.n_st, 2):
                multiply(None, 0)
                multiply(landed, 1)
            last = job + 1 == self.n_jobs
            if last:
                before_last()
            park = LDS - PARK if last else (slot - 1) % SLOTS * self.stage_bytes  # of all wavefronts; each passes its own 4 KB
            wave.now(park, park + PARK, (self.name, "park", job), write=True)
            stores = stores_of(job)
            wave.stores(stores)
            assert last or self.stage_bytes == PARK


def check(accesses):
    assert all(a["last"] is not None for a in accesses), "something in flight at the end"
    for a, b in itertools.combinations(accesses, 2):
        if a["lo"] < b["hi"] and b["lo"] < a["hi"] and (a["write"] or b["write"]):
            assert a["last"] < b["first"] or b["last"] < a["first"], (a, b)
    writes = [a for a in accesses if a["write"]]
    for a in accesses:
        if not a["write"]:
            for byte in range(a["lo"], a["hi"], 8 * KB):
                before = [w for w in writes if w["lo"] <= byte < w["hi"] and w["last"] < a["first"]]
                assert max(before, key=lambda w: w["last"])["tag"] == a["tag"], a


@pytest.mark.parametrize("n_st", [4, 6, 8, 10, 12, 14, 16, 32])
@pytest.mark.parametrize("n_jobs", [0, 1, 2, 3, 6])
@pytest.mark.parametrize("cut", [0, 2, 4])
def test_lds_of_a_workgroup(n_st, n_jobs, cut):
    for ways in itertools.product((16, 32), repeat=min(n_jobs, 3)):
        stores_of = lambda job: ways[job % len(ways)]
        wave = Wave()
        part = Stream(wave, "part", 256 if cut == 2 else 128, 128) if cut else None
        start_part = lambda: part and part.begin(1, n_st)
        if n_jobs:
            whole = Stream(wave, "whole", 256, 256)
            whole.begin(n_jobs, n_st)
            whole.run(0, stores_of, start_part)
        else:
            start_part()
        if part:
            part.run(stores_of(n_jobs - 1) if n_jobs else 0, lambda job: 16)
        wave.wait_but(0)
        check(wave.accesses)


def test_the_model_sees_a_wait_that_is_short():
    class Short(Stream):
        def __init__(self, *args):
            super().__init__(*args)
            self.half += 1                       # (a wait for fewer loads than there are)

        def issue(self, i):
            self.half -= 1
            super().issue(i)
            self.half += 1

    wave = Wave()
    stream = Short(wave, "whole", 256, 256)
    stream.begin(2, 8)
    stream.run(0, lambda job: 16)
    wave.wait_but(0)
    with pytest.raises(AssertionError):
        check(wave.accesses)
