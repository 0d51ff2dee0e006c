"""GPU parity of the decode kernels that take a whole (sequence, head) in one workgroup, at the edges of their tiles, of their
steps of 64 slots and of the capacity up to which they are taken, against the float64 oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import harness as H

pytestmark = pytest.mark.gpu


def _workload(dtype, n_heads, d_head, r, stride, plen, steps=2):
    return W.WORKLOADS["speech_bf16" if dtype == "bf16" else "tiny_f32"].scaled(
        name=f"whole_{dtype}_{r}", batch=len(plen), d_model=96, n_heads=n_heads, d_head=d_head, r=r, d_rope=d_head // 2, stride=stride,
        prefix=(1, max(plen)), steps=steps, seed=300 + r + n_heads)


@pytest.mark.parametrize("dtype,n_heads,d_head,r,stride,plen", [
    ("bf16", 8, 64, 128, 1, (1, 14, 15, 16, 62, 63, 64, 65, 127, 128, 318)),      # four wavefronts, 320 slots
    ("bf16", 8, 64, 128, 1, (1, 2, 16, 17, 127, 128, 129, 130, 255, 257, 765, 766)),  # eight, 768: the most there
    ("bf16", 21, 64, 128, 2, (1, 2, 31, 33, 126, 127, 128, 129, 300, 400, 508)),  # more than 16 heads
    ("bf16", 9, 64, 128, 1, tuple(range(1, 138, 3))),                             # two heads a workgroup, one left over
    ("bf16", 11, 64, 128, 2, tuple(range(1, 700, 10))),                           # four, three left over; eight wavefronts
    ("bf16", 31, 64, 128, 1, tuple(range(1, 319, 8))),                            # more workgroups than compute units
    ("bf16", 8, 64, 256, 1, (1, 15, 17, 63, 65, 129, 191, 193, 510)),
    ("bf16", 8, 64, 256, 1, (1, 31, 33, 127, 129, 255, 256, 257, 385, 638)),      # eight wavefronts, the most there
    ("bf16", 7, 64, 256, 1, tuple(range(2, 90, 2))),
    ("bf16", 13, 64, 256, 3, tuple(range(1, 220, 4))),
    ("bf16", 5, 128, 256, 2, (1, 3, 127, 129, 383, 510, 1022)),
    ("bf16", 13, 128, 256, 1, tuple(range(1, 383, 17))),
    ("bf16", 3, 64, 512, 1, (1, 64, 129, 254, 382)),
    ("bf16", 4, 128, 512, 1, (1, 16, 62, 63, 64, 65, 128, 129, 382)),
    ("bf16", 15, 128, 512, 2, tuple(range(1, 160, 8))),
    ("bf16", 1, 128, 128, 3, (1, 2, 3, 4, 190, 191, 192, 193, 194)),
    ("bf16", 18, 128, 128, 1, tuple(range(1, 400, 25))),
    ("f32", 4, 64, 64, 1, (1, 7, 8, 9, 63, 64, 65, 500, 766)),
    ("f32", 3, 128, 128, 2, (1, 15, 17, 129, 700)),                            # two passes over the output columns
    ("f32", 8, 64, 256, 1, (1, 31, 33, 64, 300, 510)),
])
def test_slots_around_tiles_and_steps(dtype, n_heads, d_head, r, stride, plen):
    plen = np.array(plen, np.int32)
    wl = _workload(dtype, n_heads, d_head, r, stride, plen)
    H.run_decode_parity(wl, prefix_lens=plen)
    H.run_decode_parity(wl, prefix_lens=plen, fused_step=True)


@pytest.mark.parametrize("dtype,r", [("bf16", 256), ("bf16", 512), ("f32", 128)])
def test_stale_rows_and_empty_sequences(dtype, r):
    # rows no slot stands for hold NaN, in a sequence's first step and behind it; a sequence without a slot gives zeros
    plen = np.array([0, 1, 17, 64, 70, 130], np.int32)
    wl = _workload(dtype, 6, 64, r, 1, plen, steps=1)
    wts = W.make_weights(wl)
    toks = [W.make_tokens(wl, wts, b, 0, max(int(n), 1)) for b, n in enumerate(plen)]
    sess = H.make_session(wl)
    H.upload_weights(sess, wts)
    sess.cache_c.fill_(float("nan"))
    sess.cache_kr.fill_(float("nan"))
    c, kr = (H.to_device(H.pad_stack([getattr(t, f)[:n] for t, n in zip(toks, plen)], int(plen.max())), wl.dtype) for f in ("c", "kr"))
    sess.append(c, kr, n_new=torch.from_numpy(plen).cuda())
    ob = H.OracleBatch.new(wl, wts)
    q, q_rope = (H.to_device(np.stack([getattr(t, f)[-1] for t in toks]), wl.dtype) for f in ("q", "q_rope"))
    out = torch.full((len(plen), wl.n_heads, wl.d_head), 9.0, device="cuda")
    lat, lse = torch.full((len(plen), wl.n_heads, r), 9.0, device="cuda"), torch.full((len(plen), wl.n_heads), 9.0, device="cuda")
    sess.decode(q, q_rope, out=out, out_latent=lat, lse=lse)
    assert torch.all(out[0] == 0) and torch.all(lat[0] == 0) and torch.all(lse[0] == -float("inf"))
    for b in range(1, len(plen)):
        n = int(plen[b])
        ob.append(b, toks[b].c[:n], toks[b].kr[:n])
        o_ref, ol_ref, lse_ref, _ = ob.decode(b, toks[b].q[-1], toks[b].q_rope[-1])
        assert H.max_err(out[b], o_ref) <= H.TOL[dtype] and H.max_err(lse[b], lse_ref) <= H.TOL[dtype], b
        H.check_latent(np.abs(lat[b].cpu().numpy().astype(np.float64) - ol_ref), ob.caches[b].arrays()[0], wl.dtype, f"sequence {b}")


@pytest.mark.parametrize("dtype,r", [("bf16", 256), ("f32", 64)])
def test_reference_moves_between_steps(dtype, r):
    # logits far apart, so that a later step tops the weights' reference: the same from the split schedule
    wl = _workload(dtype, 8, 64, r, 1, (250, 250, 250), steps=1)
    wts = W.make_weights(wl)
    toks = [W.make_tokens(wl, wts, b, 0, 250) for b in range(wl.batch)]
    d = {f: H.to_device(np.stack([getattr(t, f) for t in toks]), wl.dtype) for f in ("q", "q_rope", "c", "kr")}
    outs = []
    for chunk in (None, 128):
        sess = H.make_session(wl, decode_chunk=chunk)
        H.upload_weights(sess, wts)
        sess.append(d["c"], d["kr"])
        out = torch.zeros(wl.batch, wl.n_heads, wl.d_head, device="cuda")
        sess.decode(64 * d["q"][:, -1].contiguous(), 64 * d["q_rope"][:, -1].contiguous(), out=out)
        outs.append(out.cpu())
    assert torch.isfinite(outs[0]).all()
    assert (outs[0] - outs[1]).abs().max() <= (H.TOL["bf16"] if dtype == "bf16" else 64 * H.TOL["f32"])  # (logits 64 times as large)


@pytest.mark.parametrize("dtype,r", [("bf16", 256), ("f32", 64)])
def test_a_chunk_set_to_the_default_value_is_set(dtype, r):
    # the caller's chunk keeps the split form, which gives the static schedule's bits; restoring the default leaves it again
    wl = _workload(dtype, 8, 64, r, 1, (120, 37, 64), steps=1)
    wts = W.make_weights(wl)
    toks = [W.make_tokens(wl, wts, b, 0, 120) for b in range(wl.batch)]
    d = {f: H.to_device(np.stack([getattr(t, f) for t in toks]), wl.dtype) for f in ("q", "q_rope", "c", "kr")}
    default = H.make_session(wl).ctx.get_decode_chunk()
    outs = []
    for chunk, schedule, restore in ((None, 0, False), (None, 1, False), (default, 0, False), (default, 0, True)):
        sess = H.make_session(wl, decode_chunk=chunk, decode_schedule=schedule)
        if restore:
            sess.ctx.set_decode_chunk(0)
        H.upload_weights(sess, wts)
        sess.append(d["c"], d["kr"])
        out = torch.zeros(wl.batch, wl.n_heads, wl.d_head, device="cuda")
        sess.decode(d["q"][:, -1].contiguous(), d["q_rope"][:, -1].contiguous(), out=out)
        outs.append(out)
    assert not torch.equal(outs[0], outs[1])   # (two forms, two orders of summation)
    assert torch.equal(outs[2], outs[1]) and torch.equal(outs[3], outs[0])
