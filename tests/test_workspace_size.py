"""Workspace sizes that callers may have allocated stay enough (split-K takes its room inside them)."""
import ctypes

import pytest

from paper_2403_12900_amd.binding import make_config
from paper_2403_12900_amd.configs import LLAMA2_7B, LLAMA2_13B, LLAMA2_70B, TINY, ModelConfig
from tests.test_abi_host import HOST_LIB


def _lib():
    lib = ctypes.CDLL(HOST_LIB)
    lib.sprh_workspace_bytes.restype = ctypes.c_size_t
    return lib


# 32 slots of at most 1024 positions, 512 KV blocks, as first laid out for attention's KV splits alone.
@pytest.mark.parametrize("model,nbytes", [(TINY, 75561984), (LLAMA2_7B, 18303480832), (LLAMA2_13B, 33408484352),
                                          (LLAMA2_70B, 144599204864)])
def test_workspace_is_no_larger(model, nbytes):
    assert _lib().sprh_workspace_bytes(ctypes.byref(make_config(model, 32, 1024, 512))) <= nbytes


@pytest.mark.parametrize("heads,kv_heads,head_dim,d_ff,vocab", [(1, 1, 64, 8, 16), (1, 1, 64, 1 << 20, 1 << 20), (16, 1, 64, 4096, 1 << 24),
                                                                (64, 64, 128, 11008, 32000)])
def test_room_holds_every_row_of_a_pass(heads, kv_heads, head_dim, d_ff, vocab):
    """At least one KV split per row of the largest pass, and every attention counter, whatever the other sizes are."""
    m = ModelConfig(n_layers=1, d_model=64, n_heads=heads, n_kv_heads=kv_heads, head_dim=head_dim, d_ff=d_ff, vocab=vocab)
    floats, counters = ctypes.c_size_t(), ctypes.c_int()
    _lib().sprh_split_room(ctypes.byref(make_config(m, 64, 64, 64)), ctypes.byref(floats), ctypes.byref(counters))
    assert floats.value >= 1024 * heads * (head_dim + 4)
    assert counters.value >= 64 * kv_heads
