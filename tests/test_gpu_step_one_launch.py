"""fp32 decode steps of few short sequences run as one launch, in which a sequence's workgroups count themselves in the workspace
header and the last one writes the state.  Bit for bit what the append and the attention as separate calls give: the sums are the
same, in the same order."""
import pytest
import torch

import workloads as W
from tests import harness as H

pytestmark = pytest.mark.gpu


def _pair(batch, heads, d_head, r, d_rope, stride, slots, lens, seed=3):
    wl = W.WORKLOADS["tiny_f32"].scaled(name="one_launch", batch=batch, d_model=64, n_heads=heads, d_head=d_head, r=r, d_rope=d_rope,
                                        stride=stride, prefix=1, steps=0, seed=seed)
    wts = W.make_weights(wl, max_slots=slots)  # (a row of hyp_G for every slot of the session)
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda")
    pre, pre_kr = n(batch, max(1, max(lens)), r), n(batch, max(1, max(lens)), d_rope)
    sess = [H.make_session(wl, max_slots=slots) for _ in range(2)]
    for s in sess:
        H.upload_weights(s, wts)
        s.append(pre, pre_kr, n_new=torch.tensor(lens, dtype=torch.int32, device="cuda"))
    tok = lambda: (n(batch, 1, r), n(batch, 1, d_rope), n(batch, heads, d_head), n(batch, heads, d_rope))
    out = lambda: (torch.zeros(batch, heads, d_head, device="cuda"), torch.zeros(batch, heads, r, device="cuda"), torch.zeros(batch, heads, device="cuda"))
    return sess, tok, out


@pytest.mark.parametrize("batch,heads,d_head,r,d_rope,stride,slots,lens", [
    (1, 1, 64, 64, 32, 1, 3, (0,)),                            # an empty sequence, one workgroup, full after three tokens
    (3, 4, 64, 64, 32, 2, 66, (0, 127, 128)),                  # the 64th and 65th slot, the second step of the walk
    (2, 8, 128, 256, 64, 3, 130, (191, 384)),                  # the second one fills up on the way
    (5, 3, 64, 128, 64, 4, 40, (1, 63, 64, 65, 160)),          # the last is full from the start
    (56, 4, 64, 64, 32, 2, 20, tuple(i % 39 for i in range(56))),
    (2, 8, 128, 128, 64, 3, 130, (191, 384)),                  # heads of 128 (at r = 256: two launches)
    (56, 3, 64, 64, 32, 2, 20, tuple(i % 39 for i in range(56))),  # as many sequences as there are counters
    (57, 4, 64, 64, 32, 2, 20, tuple(i % 39 for i in range(57))),  # one more than there are counters: two launches
])
def test_equals_append_then_attend(batch, heads, d_head, r, d_rope, stride, slots, lens):
    (a, b), tok, out = _pair(batch, heads, d_head, r, d_rope, stride, slots, lens)
    full = False
    for _ in range(5):
        c, kr, q, qr = tok()
        oa, ob = out(), out()
        a.step(c, kr, q, qr, out=oa[0], out_latent=oa[1], lse=oa[2])
        b.append(c, kr)
        b.decode(q, qr, out=ob[0], out_latent=ob[1], lse=ob[2])
        for x, y in zip(oa, ob):
            assert torch.equal(x, y)
        assert torch.equal(a.seq_len, b.seq_len) and torch.equal(a.tail_c, b.tail_c)
        for i, n in enumerate(a.seq_len.cpu().tolist()):
            k = -(-n // stride)
            assert torch.equal(a.cache_c[i, :k], b.cache_c[i, :k]) and torch.equal(a.cache_kr[i, :k], b.cache_kr[i, :k])
        sa, sb = a.device_status(), b.device_status()
        assert sa == sb
        full |= sa != 0
    assert full == any(n + 5 > slots * stride for n in lens)


def test_graph_replays_beside_other_forms():
    # a captured step replayed between eager steps of the same workspace that take other kernels (a chunk set by the caller)
    (a, b), tok, out = _pair(3, 4, 64, 64, 32, 2, 60, (5, 50, 0))
    c, kr, q, qr = tok()
    o = out()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    len0, tail0 = a.seq_len.clone(), a.tail_c.clone()
    with torch.cuda.stream(side):
        a.step(c, kr, q, qr, out=o[0], out_latent=o[1], lse=o[2])
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.step(c, kr, q, qr, out=o[0], out_latent=o[1], lse=o[2])
    a.seq_len.copy_(len0)
    a.tail_c.copy_(tail0)
    for i in range(6):
        for dst, src in zip((c, kr, q, qr), tok()):
            dst.copy_(src)
        ref = out()
        if i % 2:
            a.ctx.set_decode_chunk(64)
            a.step(c, kr, q, qr, out=o[0], out_latent=o[1], lse=o[2])
            a.ctx.set_decode_chunk(0)
            tol = 1e-5
        else:
            graph.replay()
            tol = 0.0
        b.append(c, kr)
        b.decode(q, qr, out=ref[0], out_latent=ref[1], lse=ref[2])
        for x, y in zip(o, ref):
            assert (x - y).abs().max() <= tol * max(1.0, float(y.abs().max()))
        assert torch.equal(a.seq_len, b.seq_len) and torch.equal(a.tail_c, b.tail_c)
    assert a.device_status() == 0
