"""GPU parity of the prefill kernels at the edges of their tiles: the form with the latent-space output (32-column tiles, 128-row
blocks), the plain form with and without paired row blocks (an even and an odd number of tiles, none at all), and the matrix
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
    (3, 64, 128, 32, 1, (1, 2, 32, 33, 64, 65, 128, 129)),   # unpaired blocks; 0, 1, 2, 3 tiles, full and begun
    (3, 128, 512, 64, 2, (64, 65, 66, 127, 130, 255, 256, 257)),
    (2, 128, 256, 32, 16, (513, 512, 511, 1)),
])
def test_plain_form(n_heads, d_head, r, d_rope, stride, lens):
    _check(lens, n_heads, d_head, r, d_rope, stride, False)


def test_plain_form_paired_blocks_and_large_products():
    # more than 512 pairs of row blocks, an odd number of blocks (the last one has no partner); the key and value products take
    # their largest tiles, with most sequences' rows left out
    lens = [640, 639, 513, 1] + [5] * 43 + [130]
    _check(lens, 6, 64, 256, 32, 2, False, which=(0, 1, 2, 3, 47))
