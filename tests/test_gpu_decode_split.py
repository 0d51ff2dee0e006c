"""GPU parity of the decode kernel for short chunks (64 slots a step, rows and weights shared through LDS) at the edges of its
tiles and steps, and of the front kernel's column blocks, against the float64 oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from paper_2505_13544_amd.session import PagedSession, Session
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_heads,r,d_rope,chunk", [(1, 64, 64, 64), (16, 64, 32, 320), (8, 256, 32, 64), (9, 128, 64, 96),
                                                    (15, 512, 64, 128), (16, 256, 64, 32), (3, 512, 32, 320)])
def test_slots_around_tiles_and_steps(n_heads, r, d_rope, chunk):
    # the last step begins a tile, fills it, leaves wavefronts without a slot; chunks of half a step and of several
    plen = np.array([1, 15, 16, 17, 63, 64, 65, 128, 129, 319, 321, 340], np.int32)
    wl = W.WORKLOADS["speech_bf16"].scaled(name=f"split_{r}_{chunk}", batch=len(plen), d_model=96, n_heads=n_heads, d_head=64, r=r,
                                           d_rope=d_rope, stride=1, prefix=(1, 340), steps=2, seed=60 + r + chunk)
    H.run_decode_parity(wl, prefix_lens=plen, decode_chunk=chunk, decode_schedule=1)


@pytest.mark.parametrize("n_heads,r,d_rope,chunk", [(17, 64, 32, 64), (32, 128, 64, 96), (24, 256, 32, 160), (31, 256, 64, 32),
                                                    (32, 512, 64, 64), (20, 512, 32, 96)])
def test_two_head_tiles(n_heads, r, d_rope, chunk):
    # more than sixteen heads: a wavefront's logits are those of one head tile and two of a step's four slot tiles
    plen = np.array([1, 15, 17, 32, 33, 48, 63, 64, 65, 97, 161, 200], np.int32)
    wl = W.WORKLOADS["speech_bf16"].scaled(name=f"split2_{r}_{chunk}", batch=len(plen), d_model=96, n_heads=n_heads, d_head=64, r=r,
                                           d_rope=d_rope, stride=1, prefix=(1, 200), steps=2, seed=60 + r + chunk)
    H.run_decode_parity(wl, prefix_lens=plen, decode_chunk=chunk, decode_schedule=1)


@pytest.mark.parametrize("n_heads,r,d_rope,chunk", [(16, 64, 64, 192), (8, 128, 32, 160), (16, 128, 64, 320), (17, 64, 32, 160), (32, 128, 32, 160),
                                                    (20, 128, 64, 128)])
def test_rows_that_travel_a_step_ahead(n_heads, r, d_rope, chunk):
    # narrow latents, chunks of several steps: two places for rows in turn, whose last step may hold up to 32 slots; the same over pages
    # and over one stored copy of the first 100 slots, bit for bit; rows that no sequence holds are no numbers
    lens = np.array([100, 1, 63, 64, 65, 96, 97, 128, 129, 160, 161, 192, 193, 225, 320, 321, 350], np.int32)
    B, slots, shared_slots = len(lens), 352, 100
    wl = W.WORKLOADS["speech_bf16"].scaled(name=f"ahead_{r}_{chunk}", batch=B, d_model=96, n_heads=n_heads, d_head=64, r=r, d_rope=d_rope, stride=1,
                                           prefix=(1, 350), steps=2, seed=90 + r + chunk)
    H.run_decode_parity(wl, prefix_lens=lens, decode_chunk=chunk, decode_schedule=1)
    kw = dict(n_heads=n_heads, d_head=64, r=r, d_rope=d_rope, d_hyper=64, stride=1, max_batch=B, max_slots=slots, dtype="bf16", decode_chunk=chunk,
              decode_schedule=1)
    flat, paged, shared = Session(**kw), PagedSession(page_slots=32, n_pages=B * slots // 32, **kw), Session(**kw)
    g = torch.Generator(device="cuda").manual_seed(r + chunk)
    n = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    c, kr = n(B, 350, r), n(B, 350, d_rope)
    c[:, :shared_slots], kr[:, :shared_slots] = c[:1, :shared_slots].clone(), kr[:1, :shared_slots].clone()
    wts = W.make_weights(wl, max_slots=slots)
    outs = []
    for s in (flat, paged, shared):
        H.upload_weights(s, wts)
        for cache in (s.pool_c, s.pool_kr) if s is paged else (s.cache_c, s.cache_kr):
            cache.fill_(float("nan"))
        s.append(c, kr, n_new=lens.tolist() if s is paged else torch.from_numpy(lens).cuda())
    shared.share_prefix(torch.zeros(B, dtype=torch.int32, device="cuda"), torch.from_numpy(np.minimum(lens, shared_slots)).cuda())
    shared.cache_c[1:, :shared_slots] = float("nan")
    q, q_rope = n(B, n_heads, 64), n(B, n_heads, d_rope)
    for s in (flat, paged, shared):
        out = torch.empty(B, n_heads, 64, device="cuda")
        s.decode(q, q_rope, out=out)
        outs.append(out)
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


def test_more_pieces_than_one_round_of_the_merge():
    # 29 pieces a row, dealt to the wavefronts of the combine's one-row form; rows with none, one and a few of them
    plen = np.array([1, 33, 130, 900], np.int32)
    wl = W.WORKLOADS["speech_bf16"].scaled(name="split_pieces", batch=len(plen), d_model=96, n_heads=8, d_head=64, r=256, d_rope=32,
                                           stride=1, prefix=(1, 900), steps=2, seed=83)
    H.run_decode_parity(wl, prefix_lens=plen, decode_chunk=32, decode_schedule=1)


@pytest.mark.parametrize("r,schedule", [(64, 1), (128, 1), (128, 2)])
def test_pieces_dealt_to_parts_of_a_wavefront(r, schedule):
    # narrow latents: sixteen groups (r = 64) or eight (r = 128) merge a row; rows with none, one, a few and all of 29 pieces
    plen = np.array([1, 33, 130, 900], np.int32)
    wl = W.WORKLOADS["speech_bf16"].scaled(name=f"split_narrow_{r}_{schedule}", batch=len(plen), d_model=96, n_heads=8, d_head=64, r=r, d_rope=32,
                                           stride=1, prefix=(1, 900), steps=2, seed=84)
    H.run_decode_parity(wl, prefix_lens=plen, decode_chunk=32 if schedule == 1 else 64, decode_schedule=schedule)


@pytest.mark.parametrize("batch,schedule", [(1, 2), (3, 1), (16, 2), (65, 1), (67, 2)])
def test_wide_merge_of_eight_wavefronts(batch, schedule):
    # r = 512 with heads of 128: a row a workgroup and sixteen, the last tile nearly empty, rows with no and with more than one round of pieces
    plen = np.array([400, 1, 65] * 23, np.int32)[:batch]
    wl = W.WORKLOADS["speech_bf16"].scaled(name=f"merge8_{batch}", batch=batch, d_model=96, n_heads=3, d_head=128, r=512, d_rope=64, stride=1,
                                           prefix=(1, 400), steps=1, seed=85)
    H.run_decode_parity(wl, prefix_lens=plen, decode_chunk=32 if schedule == 1 else 64, decode_schedule=schedule)


def test_reference_moves_between_steps():
    # logits far apart: the weights' reference moves from step to step of one chunk; chunks of one step never move theirs
    wl = W.WORKLOADS["speech_bf16"].scaled(name="split_far", batch=3, d_model=96, n_heads=8, d_head=64, r=256, d_rope=32, stride=1,
                                           prefix=320, steps=1, seed=71)
    wts = W.make_weights(wl)
    toks = [W.make_tokens(wl, wts, b, 0, 320) for b in range(wl.batch)]
    d = {f: H.to_device(np.stack([getattr(t, f) for t in toks]), wl.dtype) for f in ("q", "q_rope", "c", "kr")}
    outs = []
    for chunk in (64, 320):
        sess = H.make_session(wl, decode_chunk=chunk, decode_schedule=1)
        H.upload_weights(sess, wts)
        sess.append(d["c"], d["kr"])
        out = torch.zeros(wl.batch, wl.n_heads, wl.d_head, device="cuda")
        sess.decode(64 * d["q"][:, -1].contiguous(), 64 * d["q_rope"][:, -1].contiguous(), out=out)
        outs.append(out.cpu())
    assert torch.isfinite(outs[0]).all()
    assert (outs[0] - outs[1]).abs().max() <= H.TOL["bf16"]
