"""bf16 bulk append: workgroups that take several chunks of 32 tokens, slots that end in, at and behind a chunk's end.  A token's
weight and its place in the sum do not depend on how the tokens are divided into calls, so one call of many tokens leaves, bit for
bit, what several of fewer leave (whose workgroups take a chunk each; those are held to the oracle by the other tests)."""
import numpy as np
import pytest
import torch

import workloads as W
from tests import harness as H

pytestmark = pytest.mark.gpu


def _append(wl, wts, start, pieces, c, kr, lens, given):
    sess = H.make_session(wl)
    H.upload_weights(sess, wts)
    w, slots, t = [], [], 0
    for m in (start,) + pieces:
        n_new = torch.from_numpy(np.clip(lens - t, 0, m).astype(np.int32)).cuda()
        w_out = torch.zeros(wl.batch, m, dtype=torch.float32, device="cuda")
        slot_out = torch.full((wl.batch, m), -1, dtype=torch.int32, device="cuda")
        sess.append(c[:, t:t + m].contiguous(), kr[:, t:t + m].contiguous(), n_new=n_new, w_out=w_out, slot_out=slot_out,
                    w_override=None if given is None else given[:, t:t + m].contiguous())
        w.append(w_out)
        slots.append(slot_out)
        t += m
    assert sess.device_status() == 0 and sess.seq_len.cpu().tolist() == lens.tolist()
    return sess, torch.cat(w, 1), torch.cat(slots, 1)


@pytest.mark.parametrize("stride,r,d_rope,batch,given", [(1, 64, 32, 17, False), (2, 512, 64, 16, False), (3, 128, 32, 16, False),
                                                         (5, 256, 64, 16, True), (16, 64, 32, 18, False), (2, 64, 32, 3, False),
                                                         (1, 512, 64, 3, False), (1, 128, 32, 3, True)])
def test_one_call_of_many_tokens_equals_several(stride, r, d_rope, batch, given):
    start, T = 37, 2080  # from inside a slot (stride 1: none, and of 3 sequences 16 slots a workgroup); more than one chunk a workgroup from 8 sequences on
    wl = W.WORKLOADS["speech_bf16"].scaled(name="append_groups", batch=batch, d_model=64, r=r, d_rope=d_rope, stride=stride,
                                           prefix=start + T, steps=0, seed=40 + stride)
    wts = W.make_weights(wl)
    g = torch.Generator(device="cuda").manual_seed(stride)
    c = torch.randn(batch, start + T, r, generator=g, device="cuda").bfloat16()
    kr = torch.randn(batch, start + T, d_rope, generator=g, device="cuda").bfloat16()
    w = torch.rand(batch, start + T, generator=g, device="cuda") if given else None
    lens = np.full(batch, start + T)
    lens[:3] = start + T - 1, start + 31, start  # runs out in the last chunk, inside the first one, before the call
    one, w1, s1 = _append(wl, wts, start, (T,), c, kr, lens, w)
    some, w2, s2 = _append(wl, wts, start, (333, 2, 32, 800, T - 333 - 2 - 32 - 800), c, kr, lens, w)
    torch.cuda.synchronize()
    assert torch.equal(w1, w2) and torch.equal(s1, s2)
    live = torch.arange(one.max_slots, device="cuda")[None] * stride < torch.from_numpy(lens).cuda()[:, None]
    for a, b in ((one.cache_c, some.cache_c), (one.cache_kr, some.cache_kr)):
        assert torch.equal(a[:batch][live], b[:batch][live])
    assert torch.equal(one.tail_c[:batch], some.tail_c[:batch])


@pytest.mark.parametrize("r", [64, 128, 256, 512])
@pytest.mark.parametrize("d_hyper", [16, 32, 48, 64])
def test_infinite_latents_saturate_the_weight(r, d_hyper):
    # An infinite element whose column of hyp_A is positive, under positive rows of hyp_G: the logit is that infinity, the weight 1
    # or 0, also where the hyper-network has fewer rows than the matrix operands; the other tokens' weights are finite.
    wl = W.WORKLOADS["speech_bf16"].scaled(name="append_inf", batch=2, d_model=64, r=r, d_hyper=d_hyper, stride=2, prefix=40, steps=0)
    sess = H.make_session(wl)
    H.upload_weights(sess, W.make_weights(wl))
    g = torch.Generator(device="cuda").manual_seed(r + d_hyper)
    c = torch.randn(2, 40, r, generator=g, device="cuda").bfloat16()
    kr = torch.randn(2, 40, wl.d_rope, generator=g, device="cuda").bfloat16()
    col = r - 3
    sess.hyp_A[:, col] = 0.5
    sess.hyp_G.abs_().add_(0.01)
    c[0, 3, col] = float("inf")
    c[1, 33, col] = float("-inf")
    w = torch.full((2, 40), -1.0, device="cuda")
    sess.append(c, kr, w_out=w)
    assert w[0, 3] == 1 and w[1, 33] == 0
    w[0, 3], w[1, 33] = 0.5, 0.5
    assert torch.all((w >= 0) & (w <= 1))
