"""GPU parity of the prefill kernels at the edges of their tiles: the form with the latent-space output (32-column tiles, 128-row
blocks), the plain form in blocks of 64 and of 128 rows (an even and an odd number of tiles, none at all), and the matrix
products at each of their tile sizes with rows left out."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import mtla_oracle as O
from tests import harness as H
from tests.test_gpu_prefill import _gpu_prefill, _prefill_inputs

pytestmark = pytest.mark.gpu


def _check(lens, n_heads, d_head, r, d_rope, stride, latent, which=None, q_scale=1.0):
    T = max(lens)
    wl = W.WORKLOADS["speech_bf16"].scaled(name="pf_edge", batch=len(lens), d_model=64, n_heads=n_heads, d_head=d_head, r=r,
                                           d_rope=d_rope, stride=stride, prefix=T, steps=0, seed=900 + T)
    wts = W.make_weights(wl)
    toks, d = _prefill_inputs(wl, wts, T)
    d["q"] *= q_scale
    _, w, out, lat = _gpu_prefill(wl, wts, d, T, np.array(lens, np.int32), want_latent=latent)
    for b in which or range(len(lens)):
        n = lens[b]
        o_ref, ol_ref, _, Cp = O.prefill_attn(q_scale * toks[b].q[:n], toks[b].q_rope[:n], toks[b].c[:n], toks[b].kr[:n],
                                              wts.w_uk, wts.w_uv, stride, O.softmax_scale(wl.d_head),
                                              hyp_A=wts.hyp_A, hyp_a=None, hyp_G=wts.hyp_G)
        assert H.max_err(out[b, :n], o_ref) <= H.TOL["bf16"], b
        assert torch.all(out[b, n:] == 0)
        if latent:
            H.check_latent(np.abs(lat[b, :n].cpu().numpy().astype(np.float64) - ol_ref), Cp, "bf16", f"sequence {b}")
            assert torch.all(lat[b, n:] == 0)


@pytest.mark.parametrize("n_heads,d_head,r,d_rope,stride,lens,q_scale", [
    (3, 128, 512, 64, 1, (1, 32, 33, 34), 1.0),              # no tile, one, one and a column
    (3, 128, 512, 64, 1, (127, 128, 129, 257), 1.0),         # ends of row blocks; blocks of padding only
    (2, 64, 64, 32, 2, (64, 65, 66, 300), 1.0),              # the narrowest latents
    (5, 64, 512, 64, 3, (96, 97, 98, 99), 1.0),
    (9, 128, 64, 32, 2, (193,), 1.0),                        # r below d_head
    (1, 128, 256, 64, 16, (500, 17, 16), 1.0),               # the widest chunk
    (2, 64, 128, 64, 1, (160, 150), 4.0),                    # logits far above the own column's: references move
])
def test_latent_form(n_heads, d_head, r, d_rope, stride, lens, q_scale):
    _check(lens, n_heads, d_head, r, d_rope, stride, True, q_scale=q_scale)


@pytest.mark.parametrize("n_heads,d_head,r,d_rope,stride,lens", [
    (3, 64, 128, 32, 1, (1, 2, 32, 33, 64, 65, 128, 129)),   # blocks of 64 rows; 0, 1, 2, 3 tiles, full and begun
    (3, 128, 512, 64, 2, (64, 65, 66, 127, 130, 255, 256, 257)),
    (2, 128, 256, 32, 16, (513, 512, 511, 1)),
])
def test_plain_form(n_heads, d_head, r, d_rope, stride, lens):
    _check(lens, n_heads, d_head, r, d_rope, stride, False)


@pytest.mark.parametrize("n_heads,d_head,r,d_rope,stride,lens,which", [
    (32, 128, 256, 64, 2, (64, 65, 66, 127, 130, 255, 256, 257), (1, 3, 4, 6, 7)),  # as above, with enough blocks for 128 rows each
    (32, 64, 64, 32, 1, (32, 33, 64, 65, 128, 129, 160, 1), (1, 4, 5, 6)),
    (8, 128, 128, 64, 2, (64, 63, 1) + (64,) * 37, (0, 1, 2, 39)),                  # many, but of 64 rows: one small block
])
def test_plain_form_rows_of_a_block(n_heads, d_head, r, d_rope, stride, lens, which):
    lens = lens if d_head == 128 else lens + tuple(reversed(lens))
    _check(lens, n_heads, d_head, r, d_rope, stride, False, which=which)


def test_plain_form_many_blocks_and_large_products():
    # 1440 blocks of 128 rows in groups of pairs, most of them padding, an odd number a pair; the key and value products take
    # their largest tiles, with most sequences' rows left out
    lens = [640, 639, 513, 1] + [5] * 43 + [130]
    _check(lens, 6, 64, 256, 32, 2, False, which=(0, 1, 2, 3, 47))


@pytest.mark.parametrize("n_heads,d_head,r,stride,lens,which", [
    (12, 64, 512, 2, (1400, 1399, 257, 1), (1, 2, 3)),       # one round of tiles, cut into halves
    (32, 128, 128, 3, (900, 899, 513, 1), (2, 3)),           # whole rounds and a rest; the shortest contraction
    (18, 64, 128, 2, (769, 768, 767, 640), (0, 3)),          # columns that end inside a tile, at its half
    (8, 64, 256, 2, (600,) * 40 + (257, 1) * 13, (39, 40, 65)),  # more sequences than lanes
])
def test_streamed_products(n_heads, d_head, r, stride, lens, which):
    _check(lens, n_heads, d_head, r, 32, stride, False, which=which)


@pytest.mark.parametrize("bits", [14.5, 16.0])
@pytest.mark.parametrize("latent", [False, True])
def test_own_column_far_above_the_others(latent, bits):
    # An even row's own key and the odd rows' keys (stride 2: the final ones) have opposite signs in one element of the RoPE
    # part, so the row's own logit is `bits` (in units of log2) above every other column's: the other weights are subnormal
    # fp16 numbers, and the 1536 and more of a late row are 6.6e-2 (14.5) and 2.3e-2 (16) of the normaliser.  Were they dropped
    # from it, or from the sum of the values (the latents have a mean of one, so that it is no sum of independent ones), the
    # outputs would be off by that share.
    T, stride = 4096, 2
    wl = W.WORKLOADS["speech_bf16"].scaled(name="pf_own", batch=1, d_model=64, n_heads=2, d_head=64, r=64, d_rope=32, stride=stride,
                                           prefix=T, steps=0, seed=977)
    wts = W.make_weights(wl)
    toks, _ = _prefill_inputs(wl, wts, T)
    t, scale = toks[0], O.softmax_scale(wl.d_head)
    c, q, kr, q_rope = H.bf16_round(t.c + 1.0), 0.0625 * t.q, np.array(t.kr), np.zeros_like(t.q_rope)
    kr[0::2, 0], kr[1::2, 0] = 1.0, -1.0
    q_rope[..., 0] = H.bf16_round(bits * np.log(2.0) / (2 * scale))
    d = {f: H.to_device(x[None].astype(np.float32), wl.dtype) for f, x in (("q", q), ("q_rope", q_rope), ("c", c), ("kr", kr))}
    _, w, out, lat = _gpu_prefill(wl, wts, d, T, np.array([T], np.int32), want_latent=latent)
    late = np.arange(3072, T, 2)                             # of the late rows those whose own value is largest
    weight = w[0].double().cpu().numpy()
    rows = [0, 2, 64, 126, 128, 1022, 1024, 2050] + sorted(late[np.argsort(weight[late])[-8:]].tolist())
    o_ref, ol_ref, _, Cp = O.prefill_attn(q, q_rope, c, kr, wts.w_uk, wts.w_uv, stride, scale, hyp_A=wts.hyp_A, hyp_a=None,
                                          hyp_G=wts.hyp_G, rows=rows)
    others = np.einsum("n,hnk->hk", Cp[1:T:2].mean(0), wts.w_uv)
    for value in (o_ref[-8:], others):                       # what dropping them would cost shows
        assert np.abs(value).max() * 1536 * 2.0 ** -bits > 2 * H.TOL["bf16"]
    assert H.max_err(out[0, rows], o_ref) <= H.TOL["bf16"]
    if latent:
        H.check_latent(np.abs(lat[0, rows].cpu().numpy().astype(np.float64) - ol_ref), Cp, "bf16", "own column")


def test_outputs_past_the_caches():
    # 172 MB of outputs in one call, which leave past the caches, and the sequences one at a time, whose 34 MB do not: a row's sums are the
    # same but for the references of the blocks of rows it is in, a tenth of the bound on any row; blocks cut by a sequence's end and by T
    B, T, nh, dh = 5, 2105, 32, 128
    lens = np.array([T, T - 1, 17, 0, 1040], np.int32)
    wl = W.WORKLOADS["speech_bf16"].scaled(name="streamed", batch=B, d_model=64, n_heads=nh, d_head=dh, r=128, d_rope=64, stride=4, prefix=1, steps=0, seed=5)
    wts = W.make_weights(wl, max_slots=-(-T // 4))
    g = torch.Generator(device="cuda").manual_seed(8)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.bfloat16)
    d = dict(q=n(B, T, nh, dh), q_rope=n(B, T, nh, 64), c=n(B, T, 128), kr=n(B, T, 64))
    _, _, out, _ = _gpu_prefill(wl, wts, d, T, lens, want_latent=False)
    for b in range(B):
        one = {k: v[b:b + 1].contiguous() for k, v in d.items()}
        _, _, ref, _ = _gpu_prefill(wl.scaled(batch=1), wts, one, T, lens[b:b + 1], want_latent=False)
        assert torch.isfinite(out[b]).all() and (out[b] - ref[0]).abs().max() <= H.TOL["bf16"] / 10
        assert torch.all(out[b, lens[b]:] == 0)


def test_latent_outputs_of_medium_size():
    # 43 MB of outputs in one call, which stay in the caches, and the sequences one at a time, whose 14 MB leave past them: the same blocks
    B, T, nh, dh = 3, 700, 16, 64
    lens = np.array([T, 0, 129], np.int32)
    wl = W.WORKLOADS["speech_bf16"].scaled(name="medium", batch=B, d_model=64, n_heads=nh, d_head=dh, r=256, d_rope=32, stride=3, prefix=1, steps=0, seed=6)
    wts = W.make_weights(wl, max_slots=-(-T // 3))
    g = torch.Generator(device="cuda").manual_seed(9)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.bfloat16)
    d = dict(q=n(B, T, nh, dh), q_rope=n(B, T, nh, 32), c=n(B, T, 256), kr=n(B, T, 32))
    _, _, out, lat = _gpu_prefill(wl, wts, d, T, lens, want_latent=True)
    for b in range(B):
        one = {k: v[b:b + 1].contiguous() for k, v in d.items()}
        _, _, ref, ref_lat = _gpu_prefill(wl.scaled(batch=1), wts, one, T, lens[b:b + 1], want_latent=True)
        assert torch.equal(out[b], ref[0]) and torch.equal(lat[b], ref_lat[0])
        assert torch.isfinite(lat[b]).all() and torch.all(lat[b, lens[b]:] == 0) and torch.all(out[b, lens[b]:] == 0)
