"""The binding's native call path (csrc/pycall.cpp): what it takes for an address and what it refuses, no GPU needed."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2505_13544_amd import binding as B

GOOD = dict(n_heads=8, d_head=64, r=256, d_rope=32, d_hyper=64, stride=2, max_batch=16, max_slots=640, dtype="bf16")


def _append(n_new):
    # batch 0: what gets as far as the library is refused there, before anything is enqueued
    ctx = B.Context(**GOOD)
    return ctx.cache_append_status(1024, 1024, 1024, 1024, 1024, 1024, n_new, 1, 0, 1024, None, 1024, None, None, None, 1024)


@pytest.mark.parametrize("host", [np.array([1, 2], np.int32), np.int32(4), b"abcd", bytearray(8), memoryview(b"abcd"),
                                  (ctypes.c_int32 * 2)(1, 2), ctypes.c_void_p(4096), [1, 2], 1.0],
                         ids=lambda h: type(h).__name__)
def test_host_memory_is_no_device_address(host):
    with pytest.raises(AttributeError):
        _append(host)


def test_addresses():
    class Has:
        def data_ptr(self):
            return 4096

    for a in (None, 4096, torch.zeros(4, dtype=torch.int32), Has()):
        assert _append(a) == B.MTLA_ERR_INVALID_ARG


def test_a_page_book_is_the_structure():
    # an empty structure reaches the library, which refuses it; other memory does not
    assert B.calls.mtla_pages_reserve(B.mtla_page_book(), None, 1) == -1
    assert B.calls.mtla_pages_reserve(None, None, 1) == -1
    for book in (bytes(ctypes.sizeof(B.mtla_page_book)), bytearray(8), np.zeros(4, np.int32), 4096):
        with pytest.raises((TypeError, BufferError)):
            B.calls.mtla_pages_reserve(book, None, 1)
    with pytest.raises(AttributeError):   # the host arrays beside it are addresses
        B.calls.mtla_pages_reserve(B.mtla_page_book(), np.zeros(4, np.int32), 1)


def _layer_step(lw):
    ctx = B.Context(**GOOD)
    return ctx.layer_decode_step_status(lw, 1024, 1024, 1024, 1024, 1024, 1024, None, 1024, 1024, 1024, 0, 1024, None, 1024, 1024)


LAYER = dict(w_q=1024, w_qr=1024, w_r=1024, w_kr=1024, w_o=1024, d_model=512)


@pytest.mark.parametrize("key", sorted(LAYER))
def test_a_missing_layer_weight_is_named(key):
    with pytest.raises(KeyError, match=key):
        _layer_step({k: v for k, v in LAYER.items() if k != key})


def test_layer_weights_are_a_mapping():
    from types import MappingProxyType
    for lw in (LAYER, dict(LAYER, ln_gamma=None, ln_beta=1024, ln_eps=1e-5, rope_base=1e4), MappingProxyType(LAYER)):
        assert _layer_step(lw) == B.MTLA_ERR_INVALID_ARG   # batch 0
    for bad in (None, 1024, [1024], b"abcd"):             # memory that is no mapping is never read as a structure
        with pytest.raises(TypeError):
            _layer_step(bad)
    for k, v in (("d_model", None), ("d_model", 512.0), ("ln_eps", None), ("rope_base", "10000")):
        with pytest.raises(TypeError):
            _layer_step(dict(LAYER, **{k: v}))
