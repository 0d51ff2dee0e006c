"""GPU parity of the projections' rotation where tiles form their own angles: pieces without a list of lengths, so that a
tile holds rows of several sequences, each continuing from another position.  Up to 65 tokens the products are the small ones of 16 x 16
tiles and more (gemm_ring_kernel), from 100 on 64 x 64 tiles (gemm_nt_kernel; tests/test_gemm_tiles.py holds the rule to that).
Outputs and cache against the float64 oracle, within the 2e-2 of bf16."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import harness as H
from tests.test_gpu_layer_prefill import _oracle_cache, _oracle_rows, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_rope", [32, 64])
@pytest.mark.parametrize("tokens", [1, 13, 33, 64, 65, 100, 120])
def test_tiles_with_rows_of_several_sequences(d_rope, tokens):
    starts = np.array([40, 3, 0, 57, 22], dtype=np.int32)
    wl = W.WORKLOADS["speech_bf16"].scaled(name="lp_angles", batch=len(starts), d_model=128, d_rope=d_rope, stride=3, prefix=180,
                                           steps=0, seed=300 + d_rope + tokens)
    wts, lw, sess, okw = _setup(wl)
    xs = [W.make_x(wl, b, 0, int(starts[b]) + tokens) for b in range(wl.batch)]
    first = np.full((wl.batch, int(starts.max()), wl.d_model), np.nan)
    for b, n in enumerate(starts):
        first[b, :n] = xs[b][:n]
    y = torch.empty(first.shape, dtype=torch.float32, device="cuda")
    keep = [sess.layer_prefill(H.to_device(first, wl.dtype), y=y, n_new=torch.from_numpy(starts).cuda())]
    y = torch.empty(wl.batch, tokens, wl.d_model, dtype=torch.float32, device="cuda")
    x = np.stack([xs[b][starts[b]:] for b in range(wl.batch)])
    keep.append(sess.layer_prefill(H.to_device(x, wl.dtype), y=y, max_past_slots=int(starts.max()) // wl.stride))
    torch.cuda.synchronize()
    for b in range(wl.batch):
        err = H.max_err(y[b], _oracle_rows(wl, wts, lw, okw, xs[b])[starts[b]:])
        assert err <= H.TOL["bf16"], (b, err)
    assert sess.device_status() == 0
    ob = H.OracleBatch.new(wl, wts)
    for b in range(wl.batch):
        _oracle_cache(wl, wts, lw, okw, ob, b, xs[b])
    H.check_cache(sess, ob, what="after both pieces", kr_exact=False)
