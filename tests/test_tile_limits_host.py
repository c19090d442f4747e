"""Sizes the tile kernel cannot address are refused on the host, before any GPU work."""
import ctypes

import pytest

import paper_2502_14317_amd as pc

ONE = ctypes.c_void_p(256)            # never dereferenced: the call is refused first
SHAPE = -2
WS = 1 << 62


def _attn(n_q, n_seg, k_t, heads, with_self, D=128):
    s = ONE if with_self else None
    return pc.lib().pc_parallel_attn(ONE, ONE, ONE, None, 0, s, s, 1, n_q, n_seg, k_t, heads, heads, D, 0, 1e4, 0.0,
                                     ONE, None, ONE, WS, None)


def _attn8(n_q, n_seg, k_t, cap, heads, with_self, D=128):
    s, t = ONE if with_self else None, ONE if cap else None
    return pc.lib().pc_parallel_attn_fp8(ONE, ONE, ONE, ONE, ONE, None, 0, t, t, t, cap, s, s, 1, n_q, n_seg, k_t,
                                         heads, heads, D, 0, 1e4, 0.0, ONE, None, ONE, WS, None)


@pytest.mark.parametrize("heads", [65536, 1 << 18])
def test_self_segment_of_too_many_heads(heads):
    assert _attn(65, 0, 1, heads, True) == SHAPE
    assert _attn8(65, 0, 1, 0, heads, True) == SHAPE


def test_segments_of_too_many_tiles():
    k_t = 65535 * 64 + 1
    assert _attn(65, 1, k_t, 1, False) == SHAPE
    assert _attn8(65, 1, k_t, 0, 1, False) == SHAPE
    assert _attn8(65, 0, 1, k_t, 1, False) == SHAPE
