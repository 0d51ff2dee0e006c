"""Decode calls below eight tiles a unit keep their partials in fp32: with queries of zero every weight is
one and the latent output the mean of the rows, which partials in half would miss by 2^-12 of them and more."""
import numpy as np
import pytest
import torch

from paper_2505_13544_amd.session import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_heads,r,batch,slots", [(17, 512, 9, 2064),   # 1161 tiles
                                                   (32, 512, 31, 1040),  # 2015
                                                   (20, 512, 7, 4096),   # 1792
                                                   (16, 512, 23, 1400), (20, 256, 31, 1040), (16, 256, 31, 1040), (8, 128, 31, 1040)])
def test_partials_in_fp32(n_heads, r, batch, slots):
    s = Session(n_heads=n_heads, d_head=64, r=r, d_rope=32, d_hyper=64, stride=1, max_batch=batch, max_slots=slots, dtype="bf16")
    g = torch.Generator(device="cuda").manual_seed(r + n_heads)
    s.cache_c.copy_(torch.randn(batch, slots, r, generator=g, device="cuda") + 1.0)
    s.cache_kr.copy_(torch.randn(batch, slots, 32, generator=g, device="cuda"))
    w = np.ones((n_heads, r, 64), np.float32)
    s.set_weights(hyp_A=np.zeros((64, r), np.float32), hyp_G=np.zeros((slots, 64), np.float32), w_uk=w, w_uv=w.transpose(0, 2, 1))
    lens = np.linspace(1, slots, batch).astype(np.int32)
    lens[1], lens[2] = 0, slots
    s.seq_len.copy_(torch.from_numpy(lens))
    q, q_rope = torch.zeros(batch, n_heads, 64, device="cuda").bfloat16(), torch.zeros(batch, n_heads, 32, device="cuda").bfloat16()
    out, latent = torch.empty(batch, n_heads, 64, device="cuda"), torch.empty(batch, n_heads, r, device="cuda")
    s.decode(q, q_rope, out=out, out_latent=latent)
    for b, n in enumerate(lens):
        ref = s.cache_c[b, :n].double().mean(0) if n else torch.zeros(r, dtype=torch.float64, device="cuda")
        # sums of up to 4096 fp32 terms of about one, in any order: below 1e-5
        assert (latent[b].double() - ref).abs().max().item() <= 1e-5, b
    assert s.device_status() == 0
