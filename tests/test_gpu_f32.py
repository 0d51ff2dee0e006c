"""fp32 storage on the matrix cores, at the edges of its tiles, against the float64 oracle (1e-5)."""
import numpy as np
import pytest

import workloads as W
from oracle import mtla_oracle as O
from tests import harness as H
from tests.test_gpu_prefill import _gpu_prefill, _prefill_inputs

pytestmark = pytest.mark.gpu


# heads around the tile of 16; d_head with and without a fixed number of pieces per lane; every latent width;
# more sequences than the absorption takes at once; chunks that leave wavefronts without a tile
@pytest.mark.parametrize("n_heads,d_head,r,d_rope,chunk", [(1, 32, 64, 64, 64), (16, 64, 128, 32, 32), (17, 96, 256, 64, 64),
                                                           (33, 64, 512, 32, 128), (3, 128, 512, 64, 96)])
def test_f32_decode_edges(n_heads, d_head, r, d_rope, chunk):
    wl = W.WORKLOADS["tiny_f32"].scaled(name=f"f32_{n_heads}_{r}", batch=9, d_model=64, n_heads=n_heads, d_head=d_head, r=r,
                                        d_rope=d_rope, stride=2, prefix=(0, 270), steps=3, seed=40 + n_heads)
    plen = np.array([0, 1, 2, 31, 32, 33, 127, 200, 270], np.int32)
    H.run_decode_parity(wl, prefix_lens=plen, decode_chunk=chunk)
    H.run_decode_parity(wl, prefix_lens=plen, decode_chunk=chunk, fused_step=True)


@pytest.mark.parametrize("d_head,d_rope,r,stride,T", [(32, 64, 64, 1, 33), (64, 32, 256, 2, 97), (64, 64, 512, 3, 64),
                                                      (128, 32, 128, 4, 131), (128, 64, 256, 5, 1), (96, 32, 128, 2, 40)])
def test_f32_prefill_edges(d_head, d_rope, r, stride, T):
    wl = W.WORKLOADS["tiny_f32"].scaled(name="pf32", batch=3, d_model=64, n_heads=5, d_head=d_head, r=r, d_rope=d_rope,
                                        stride=stride, prefix=T, steps=0, seed=60 + T)
    wts = W.make_weights(wl)
    toks, d = _prefill_inputs(wl, wts, T)
    seq_lens = np.array([T, T // 2, 0], np.int32)
    for want_latent in (False, True):
        _, w, out, lat = _gpu_prefill(wl, wts, d, T, seq_lens, want_latent)
        for b in range(wl.batch):
            n = int(seq_lens[b])
            if n:
                o_ref, ol_ref, _, _ = O.prefill_attn(toks[b].q[:n], toks[b].q_rope[:n], toks[b].c[:n], toks[b].kr[:n],
                                                     wts.w_uk, wts.w_uv, stride, O.softmax_scale(d_head), hyp_A=wts.hyp_A,
                                                     hyp_a=None, hyp_G=wts.hyp_G)
                assert H.max_err(out[b, :n], o_ref) <= H.TOL["f32"]
                assert lat is None or H.max_err(lat[b, :n], ol_ref) <= H.TOL["f32"]
            assert (out[b, n:] == 0).all() and (lat is None or (lat[b, n:] == 0).all())
