"""Prefills of so many tokens that a workgroup of their front launch appends several chunks of 32 tokens (more than 1024 chunks in all
at r = 64 and 128, 768 at 256, 512 at 512): the one-call prefill and whole-layer prefill, from inside a slot, against the float64
oracle.  The RoPE queries are four times the row's own RoPE key, so that most of a row's weight is on its own running state (0.99 at the
median, 0.5 or more for nine rows of ten): an output is off by what its row of C_hat' is off.  Sequences 3 .. are copies of
sequence 3, whose outputs and states must be its, bit for bit."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import mtla_oracle as O
from tests import harness as H
from tests.test_gpu_layer_prefill import _oracle_cache, _oracle_rows, _setup

pytestmark = pytest.mark.gpu

START, T = 37, 2080
SHAPES = [(1, 64, 17), (2, 128, 16), (3, 256, 12), (2, 512, 9), (16, 64, 17)]


def _lens(batch):
    lens = np.full(batch, START + T, np.int32)
    lens[:3] = START + T - 1, START + 31, START  # runs out in the last chunk, inside the first one, before the call
    return lens


def _copies(rows, batch):
    return np.stack(rows + [rows[3]] * (batch - 4))


def _tolerance(stride):
    return H.TOL["bf16"] * max(1.0, stride / 3)  # (as the header gives it: a cache row is a sum of `stride` weighted latents)


def _same_copies(sess, lens, stride, outs):
    for out in outs:
        assert torch.equal(out[4:], out[3:4].expand_as(out[4:]))
    n = -(-int(lens[3]) // stride)
    for x in (sess.cache_c[:, :n], sess.cache_kr[:, :n], sess.tail_c):
        assert torch.equal(x[4:], x[3:4].expand_as(x[4:]))


@pytest.mark.parametrize("stride,r,batch", SHAPES)
def test_prefill_step(stride, r, batch):
    wl = W.WORKLOADS["speech_bf16"].scaled(name="groups", batch=batch, d_model=64, n_heads=2, d_head=64, r=r, d_rope=32, stride=stride,
                                           prefix=START + T, steps=0, seed=20 + stride + r)
    wts = W.make_weights(wl)
    toks = [W.make_tokens(wl, wts, b, 0, START + T) for b in range(4)]
    qr = [W.storage_round(np.repeat(4 * t.kr[:, None], wl.n_heads, 1), wl.dtype) for t in toks]
    lens = _lens(batch)
    sess = H.make_session(wl)
    H.upload_weights(sess, wts)
    ob = H.OracleBatch.new(wl, wts, batch=4)
    refs, w_refs = [], []
    for b in range(4):
        n = lens[b]
        w_refs.append(ob.append(b, toks[b].c[:n], toks[b].kr[:n])[0])
        refs.append(O.prefill_attn(toks[b].q[:n], qr[b][:n], toks[b].c[:n], toks[b].kr[:n], wts.w_uk, wts.w_uv, stride,
                                   O.softmax_scale(wl.d_head), hyp_A=wts.hyp_A, hyp_a=None, hyp_G=wts.hyp_G)[0])
    for a, m in ((0, START), (START, T)):
        put = lambda rows: H.to_device(_copies([x[a:a + m] for x in rows], batch), wl.dtype)
        out = torch.empty(batch, m, wl.n_heads, wl.d_head, dtype=torch.float32, device="cuda")
        w = torch.zeros(batch, m, dtype=torch.float32, device="cuda")
        n_new = np.clip(lens - a, 0, m)
        keep = sess.prefill_chunk(put([t.q for t in toks]), put(qr), put([t.c for t in toks]), put([t.kr for t in toks]), out=out,
                                  max_past_slots=a // stride, n_new=torch.from_numpy(n_new).cuda(), w_out=w)
        assert sess.device_status() == 0
        del keep
        for b in range(4):
            n = int(n_new[b])
            if n:
                assert H.max_err(out[b, :n], refs[b][a:a + n]) <= _tolerance(stride), (a, b)
                assert H.max_err(w[b, :n], w_refs[b][a:a + n]) <= H.TOL_W, (a, b)
    _same_copies(sess, lens, stride, (out, w))
    H.check_cache(sess, ob)
    assert sess.seq_len.cpu().tolist() == lens.tolist()


@pytest.mark.parametrize("stride,r,batch", SHAPES)
def test_layer_prefill(stride, r, batch):
    wl = W.WORKLOADS["speech_bf16"].scaled(name="lp_groups", batch=batch, d_model=64, n_heads=2, d_head=64, r=r, d_rope=32, stride=stride,
                                           prefix=START + T, steps=0, seed=50 + stride + r)
    wts, lw, sess, okw = _setup(wl)
    lw.w_qr = np.tile(4 * lw.w_kr, (wl.n_heads, 1))
    sess.set_layer_weights(w_q=lw.w_q, w_qr=lw.w_qr, w_r=lw.w_r, w_kr=lw.w_kr, w_o=lw.w_o)
    xs = [W.make_x(wl, b, 0, START + T) for b in range(4)]
    lens = _lens(batch)
    refs = [_oracle_rows(wl, wts, lw, okw, xs[b][:lens[b]]) for b in range(4)]
    for a, m in ((0, START), (START, T)):
        y = torch.empty(batch, m, wl.d_model, dtype=torch.float32, device="cuda")
        n_new = np.clip(lens - a, 0, m)
        keep = sess.layer_prefill(H.to_device(_copies([x[a:a + m] for x in xs], batch), wl.dtype), y=y, max_past_slots=a // stride,
                                  n_new=torch.from_numpy(n_new).cuda())
        assert sess.device_status() == 0
        del keep
        for b in range(4):
            n = int(n_new[b])
            if n:
                assert H.max_err(y[b, :n], refs[b][a:a + n]) <= _tolerance(stride), (a, b)
    _same_copies(sess, lens, stride, (y,))
    ob = H.OracleBatch.new(wl, wts, batch=4)
    for b in range(4):
        _oracle_cache(wl, wts, lw, okw, ob, b, xs[b][:lens[b]])
    H.check_cache(sess, ob, kr_exact=False)
    assert sess.seq_len.cpu().tolist() == lens.tolist()
