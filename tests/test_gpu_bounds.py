"""Lengths outside what a session can hold, as a caller that writes seq_len itself may leave them: every decode kernel takes them for the
nearer end of the range, so that no row of another sequence, and nothing behind the arrays, is read."""
import pytest
import torch

import workloads as W
from tests import harness as H
from tests.test_gpu_paged import make_paged

pytestmark = pytest.mark.gpu

SLOTS, STRIDE = 70, 2   # no multiple of a tile or a chunk
CAP = SLOTS * STRIDE
LENGTHS = [CAP + 1, 10 ** 9, -7, -2 ** 31, 33, 2 ** 31 - 1]
INSIDE = [CAP, CAP, 0, 0, 33, CAP]


@pytest.mark.parametrize("dtype,n_heads,r,chunk,schedule,page_slots", [
    ("bf16", 8, 256, None, 0, 0),    # one workgroup a sequence and head
    ("bf16", 9, 128, None, 0, 0),
    ("bf16", 8, 256, 64, 1, 0),      # split, short chunks
    ("bf16", 24, 128, 32, 1, 0),     # static, two head tiles
    ("bf16", 8, 512, None, 2, 0),    # balanced, columns split
    ("bf16", 8, 64, None, 2, 0),     # balanced, r = 64
    ("bf16", 40, 64, 32, 0, 0),      # vector kernel
    ("f32", 4, 64, None, 0, 0),      # one workgroup a sequence and head
    ("f32", 4, 128, 32, 0, 0),
    ("bf16", 8, 256, None, 0, 16),   # paged
    ("bf16", 8, 256, 64, 1, 32),
    ("bf16", 20, 128, None, 2, 16),
])
def test_decode_takes_a_length_outside_for_the_nearer_end(dtype, n_heads, r, chunk, schedule, page_slots):
    wl = W.WORKLOADS["speech_bf16" if dtype == "bf16" else "tiny_f32"].scaled(
        name="bounds", batch=len(LENGTHS), d_model=64, n_heads=n_heads, d_head=64, r=r, d_rope=32, stride=STRIDE, prefix=4, steps=1, seed=9)
    kw = dict(max_slots=SLOTS, decode_chunk=chunk, decode_schedule=schedule)
    n_pages = len(LENGTHS) * -(-SLOTS // max(page_slots, 1))
    sess = make_paged(wl, page_slots=page_slots, n_pages=n_pages, **kw) if page_slots else H.make_session(wl, **kw)
    H.upload_weights(sess, W.make_weights(wl))
    g = torch.Generator(device="cuda").manual_seed(9)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=g).to(sess.tdt)
    for t in (sess.pool_c, sess.pool_kr) if page_slots else (sess.cache_c, sess.cache_kr):
        t.copy_(rand(*t.shape))
    if page_slots:
        sess.table.copy_(torch.randperm(n_pages, device="cuda", generator=g).to(torch.int32).view(sess.table.shape))
    q, q_rope = rand(wl.batch, n_heads, 64), rand(wl.batch, n_heads, 32)
    got = []
    for lengths in (INSIDE, LENGTHS):
        sess.seq_len.copy_(torch.tensor(lengths, dtype=torch.int32))
        out = torch.full((wl.batch, n_heads, 64), 9.0, device="cuda")
        lat, lse = torch.full((wl.batch, n_heads, r), 9.0, device="cuda"), torch.full((wl.batch, n_heads), 9.0, device="cuda")
        sess.decode(q, q_rope, out=out, out_latent=lat, lse=lse)
        got.append((out, lat, lse))
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert torch.isfinite(got[0][0]).all() and torch.all(got[0][0][2] == 0) and torch.all(got[0][2][3] == -float("inf"))


@pytest.mark.parametrize("call,dtype,d_head,d_hyper", [
    ("step", "bf16", 64, 64), ("step", "bf16", 96, 64), ("step", "f32", 64, 64), ("append", "bf16", 64, 64), ("append", "bf16", 64, 40),
    ("append", "f32", 64, 64), ("prefill", "bf16", 64, 64), ("prefill", "bf16", 64, 40), ("layer_step", "bf16", 64, 64),
    ("layer_prefill", "bf16", 64, 64)])
@pytest.mark.parametrize("length", [-1, -37, -2 ** 31])
def test_append_refuses_a_length_below_zero(call, dtype, d_head, d_hyper, length):
    # status 1, that sequence as it was; the others, whose rows lie in front of and behind its own, as without it
    wl = W.WORKLOADS["speech_bf16" if dtype == "bf16" else "tiny_f32"].scaled(
        name="bounds_append", batch=3, d_model=64, n_heads=4, d_head=d_head, r=128, d_rope=32, d_hyper=d_hyper, stride=STRIDE, prefix=4,
        steps=1, seed=8)
    wts = W.make_weights(wl)
    T = 1 if "step" in call else 21
    states = []
    for middle in (4, length):
        sess = H.make_session(wl, max_slots=SLOTS)
        wts_G = torch.randn(SLOTS, d_hyper, generator=torch.Generator().manual_seed(1)).numpy()
        sess.set_weights(hyp_A=wts.hyp_A, hyp_G=wts_G, w_uk=wts.w_uk_lib, w_uv=wts.w_uv_lib)
        g = torch.Generator(device="cuda").manual_seed(8)
        rand = lambda *s: torch.randn(*s, device="cuda", generator=g).to(sess.tdt)
        for t in (sess.cache_c, sess.cache_kr, sess.tail_c):
            t.copy_(rand(*t.shape))
        sess.seq_len.copy_(torch.tensor([5, middle, 9], dtype=torch.int32))
        before = [t.clone() for t in (sess.cache_c, sess.cache_kr, sess.tail_c, sess.seq_len)]
        c, kr, q, q_rope = rand(3, T, 128), rand(3, T, 32), rand(3, T, 4, d_head), rand(3, T, 4, 32)
        out = torch.zeros(3, T, 4, d_head, device="cuda")
        if call == "step":
            sess.step(c[:, 0].contiguous(), kr[:, 0].contiguous(), q[:, 0].contiguous(), q_rope[:, 0].contiguous(), out=out[:, 0])
        elif call == "append":
            sess.append(c, kr)
        elif call == "prefill":
            keep = sess.prefill_chunk(q, q_rope, c, kr, out=out, max_past_slots=6)
        else:
            lw = W.make_layer_weights(wl, wts)
            sess.set_layer_weights(w_q=lw.w_q, w_qr=lw.w_qr, w_r=lw.w_r, w_kr=lw.w_kr, w_o=lw.w_o)
            out, x = torch.zeros(3, T, 64, device="cuda"), rand(3, T, 64)
            if call == "layer_step":
                sess.layer_step(x[:, 0].contiguous(), y=out[:, 0])
            else:
                keep = sess.layer_prefill(x, y=out, max_past_slots=6)
        torch.cuda.synchronize()
        after = [t.clone() for t in (sess.cache_c, sess.cache_kr, sess.tail_c, sess.seq_len)]
        states.append(after + [out])
        assert sess.device_status() == (0 if middle >= 0 else 1)
        if middle < 0:
            for a, b in zip(before, after):
                assert torch.equal(a[1], b[1])
    for a, b in zip(*states):
        assert torch.equal(a[0], b[0]) and torch.equal(a[2], b[2])
    assert torch.isfinite(states[1][4][[0, 2]].float()).all()
