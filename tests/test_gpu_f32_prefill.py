"""fp32 storage: the bulk append on the matrix cores and the parallel form, at the edges of their tiles (16 rows or columns, 8
slots and 16 tokens per append workgroup, 32 x 64 key / value tiles, a block from either end of a sequence), against the
float64 oracle.  Bound: the fp32 tolerance of the other tests, which is for values of order 1, times the largest value: an output is
a mean of values under weights whose relative error is that of their logit, a sum of at most 576 products."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import mtla_oracle as O
from tests import harness as H
from tests.test_gpu_prefill import _gpu_prefill, _prefill_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,lens,heads,d_head,r,d_rope,stride", [
    (1, (1, 0, 1), 4, 64, 64, 32, 2),             # one row
    (16, (16, 15, 1), 4, 64, 64, 32, 1),          # one block: no second one
    (17, (17, 16, 2), 8, 64, 128, 32, 2),         # one row in the second block
    (33, (33, 32, 31), 3, 64, 256, 64, 3),        # three blocks: the middle one alone; columns of the product not a multiple of 64
    (65, (65, 64, 48), 8, 64, 256, 32, 4),
    (130, (130, 97, 0), 4, 32, 512, 64, 16),      # an empty sequence, the widest latent, the longest stride of the matrix-core append
    (49, (49, 47, 34), 2, 32, 64, 32, 1),         # the narrowest rows: eight of them a load
    (641, (641, 16, 333), 2, 64, 64, 32, 1),      # few workgroups and many columns: operands as they are multiplied
    (322, (322, 321, 0), 4, 32, 128, 32, 1),
    (32, (32, 17, 1), 4, 64, 64, 32, 2),          # hardly any rows: likewise
    (81, (81, 17, 80), 2, 128, 64, 64, 2),        # one block a workgroup
    (500, (500, 479, 3), 8, 128, 128, 32, 2),     # heads of 128: more workgroups than have their next tile ahead (24 x 32)
    (290, (290, 273, 16), 16, 128, 64, 64, 1),    # 48 x 19
    (40, (40, 39, 5), 4, 64, 64, 32, 17),         # stride beyond the matrix-core append
])
def test_rows_at_the_edges(T, lens, heads, d_head, r, d_rope, stride):
    wl = W.WORKLOADS["tiny_f32"].scaled(name="f32_edges", batch=3, d_model=64, n_heads=heads, d_head=d_head, r=r, d_rope=d_rope,
                                        stride=stride, prefix=T, steps=0, seed=5 + T)
    wts = W.make_weights(wl)
    toks, d = _prefill_inputs(wl, wts, T)
    sess, w, out, lat = _gpu_prefill(wl, wts, d, T, np.array(lens, np.int32))
    ob = H.OracleBatch.new(wl, wts)
    for b, n in enumerate(lens):
        w_ref, _ = ob.append(b, toks[b].c[:n], toks[b].kr[:n])
        if n:
            assert np.abs(w[b, :n].cpu().numpy() - w_ref).max() <= H.TOL_W
            o_ref, ol_ref, _, _ = O.prefill_attn(toks[b].q[:n], toks[b].q_rope[:n], toks[b].c[:n], toks[b].kr[:n], wts.w_uk, wts.w_uv,
                                                stride, O.softmax_scale(d_head), hyp_A=wts.hyp_A, hyp_a=None, hyp_G=wts.hyp_G)
            assert H.max_err(out[b, :n], o_ref) <= H.TOL["f32"] * max(1.0, np.abs(o_ref).max())
            assert H.max_err(lat[b, :n], ol_ref) <= H.TOL["f32"] * max(1.0, np.abs(ol_ref).max())
        assert torch.all(out[b, n:] == 0) and torch.all(lat[b, n:] == 0)
    H.check_cache(sess, ob)
    assert sess.seq_len.cpu().tolist() == list(lens) and sess.device_status() == 0


@pytest.mark.parametrize("stride,pieces", [(2, (3, 40, 1, 17)), (1, (7, 8, 9, 33)), (5, (81, 2, 90)), (16, (130, 1, 140)), (20, (41, 60))])
def test_bulk_append_continues(stride, pieces):
    # pieces that end inside a slot, in and behind the first group of eight slots; equal to the appends token by token up to the
    # order of the logit's sum
    n = sum(pieces)
    wl = W.WORKLOADS["tiny_f32"].scaled(name="f32_pieces", batch=2, d_model=64, r=128, stride=stride, prefix=n, steps=0, seed=9)
    wts = W.make_weights(wl)
    toks = [W.make_tokens(wl, wts, b, 0, n) for b in range(2)]
    sess = H.make_session(wl)
    H.upload_weights(sess, wts)
    ob = H.OracleBatch.new(wl, wts)
    t = 0
    for k, m in enumerate(pieces):
        cut = lambda f: H.to_device(np.stack([getattr(x, f)[t:t + m] for x in toks]), "f32")
        w = torch.zeros(2, m, device="cuda")
        sess.append(cut("c"), cut("kr"), w_out=w)
        for b in range(2):
            w_ref, _ = ob.append(b, toks[b].c[t:t + m], toks[b].kr[t:t + m])
            assert np.abs(w[b].cpu().numpy() - w_ref).max() <= H.TOL_W
        t += m
        H.check_cache(sess, ob, what=f"piece {k}")


@pytest.mark.parametrize("stride,batch", [(1, 40), (3, 40), (4, 3), (4, 40), (8, 40), (16, 40)])
def test_bulk_append_groups_of_slots(stride, batch):
    # one call, whose workgroups take one to eight slots by the stride and the number of them, and pieces of 25 tokens (up to two chunks of
    # one workgroup): the same bits
    wl = W.WORKLOADS["tiny_f32"].scaled(name="f32_groups", batch=batch, d_model=64, n_heads=1, d_head=64, r=64, d_rope=32, stride=stride,
                                        prefix=230, steps=0, seed=stride)
    wts = W.make_weights(wl)
    g = torch.Generator(device="cuda").manual_seed(batch)
    c, kr = (torch.randn(batch, 230, n, generator=g, device="cuda") for n in (wl.r, wl.d_rope))
    sess, w = [H.make_session(wl) for _ in range(2)], [torch.zeros(batch, 230, device="cuda") for _ in range(2)]
    for s, x, step in zip(sess, w, (225, 25)):
        H.upload_weights(s, wts)
        for a, e in [(0, 5)] + [(t, min(t + step, 230)) for t in range(5, 230, step)]:
            piece = torch.zeros(batch, e - a, device="cuda")
            s.append(c[:, a:e].contiguous(), kr[:, a:e].contiguous(), w_out=piece)
            x[:, a:e] = piece
        assert s.device_status() == 0
    n = -(-230 // stride)
    assert torch.equal(w[0], w[1]) and torch.equal(sess[0].tail_c, sess[1].tail_c)
    assert torch.equal(sess[0].cache_c[:, :n], sess[1].cache_c[:, :n]) and torch.equal(sess[0].cache_kr[:, :n], sess[1].cache_kr[:, :n])
    ob = H.OracleBatch.new(wl, wts)
    for b in range(0, batch, 13):
        w_ref, _ = ob.append(b, c[b].cpu().numpy(), kr[b].cpu().numpy())
        assert np.abs(w[0][b].cpu().numpy() - w_ref).max() <= H.TOL_W


@pytest.mark.parametrize("batch,T,lens", [
    (40, 5, None), (40, 5, "ragged"),    # blocks of the key / value product over several sequences
    (7, 56, "ragged"), (7, 57, "ragged"),  # the longest that are one sequence to it; a sequence's own blocks
    (5, 65, None), (33, 1, None),
])
def test_rows_of_several_sequences_in_a_block(batch, T, lens):
    wl = W.WORKLOADS["tiny_f32"].scaled(name="f32_short", batch=batch, d_model=64, n_heads=3, d_head=64, r=128, d_rope=32, stride=2,
                                        prefix=T, steps=0, seed=60 + T)
    wts = W.make_weights(wl)
    g = np.random.default_rng(batch + T)
    n = np.full(batch, T, np.int32) if lens is None else g.integers(0, T + 1, batch).astype(np.int32)
    toks, d = _prefill_inputs(wl, wts, T)
    w = torch.rand(batch, T, device="cuda", generator=torch.Generator(device="cuda").manual_seed(T))
    sess = H.make_session(wl)
    H.upload_weights(sess, wts)
    out = torch.empty(batch, T, wl.n_heads, wl.d_head, device="cuda")
    lat = torch.empty(batch, T, wl.n_heads, wl.r, device="cuda")
    keep = sess.prefill(d["q"], d["q_rope"], d["c"], d["kr"], w, out=out, out_latent=lat,
                        seq_lens=None if lens is None else torch.from_numpy(n).cuda())
    torch.cuda.synchronize()
    del keep
    for b in range(batch):
        m = int(n[b])
        assert torch.all(out[b, m:] == 0) and torch.all(lat[b, m:] == 0)
        if m:
            o_ref, ol_ref, _, _ = O.prefill_attn(toks[b].q[:m], toks[b].q_rope[:m], toks[b].c[:m], toks[b].kr[:m], wts.w_uk, wts.w_uv,
                                                 wl.stride, O.softmax_scale(wl.d_head), w=w[b, :m].cpu().numpy())
            assert H.max_err(out[b, :m], o_ref) <= H.TOL["f32"] * max(1.0, np.abs(o_ref).max())
            assert H.max_err(lat[b, :m], ol_ref) <= H.TOL["f32"] * max(1.0, np.abs(ol_ref).max())


@pytest.mark.parametrize("stride,at,d_head", [(2, 163, 64), (3, 141, 64), (5, 150, 32), (16, 163, 64)])
def test_infinite_latents_leave_the_rows_far_before_them_alone(stride, at, d_head):
    # An infinite element of a token's latent: rows of blocks of 16 that end before it are what they are without it, also where their
    # tile of closed chunks is shared with a block behind it.
    T = 300
    wl = W.WORKLOADS["tiny_f32"].scaled(name="f32_inf", batch=1, d_model=64, n_heads=2, d_head=d_head, r=128, d_rope=32, stride=stride,
                                        prefix=T, steps=0, seed=90 + stride)
    wts = W.make_weights(wl)
    _, d = _prefill_inputs(wl, wts, T)
    w = torch.rand(1, T, device="cuda", generator=torch.Generator(device="cuda").manual_seed(stride))
    sess = H.make_session(wl)
    H.upload_weights(sess, wts)

    def attend():
        out, lat = (torch.empty(1, T, wl.n_heads, n, device="cuda") for n in (wl.d_head, wl.r))
        keep = sess.prefill(d["q"], d["q_rope"], d["c"], d["kr"], w, out=out, out_latent=lat)
        torch.cuda.synchronize()
        del keep
        return out, lat

    want = attend()
    d["c"][0, at, 5] = float("inf")
    for got, ref in zip(attend(), want):
        assert torch.equal(got[:, :at // 16 * 16], ref[:, :at // 16 * 16])
