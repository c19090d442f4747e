"""Argument errors of the one-call entry points (a layer, a decoding step over either cache): all of them are found on
the host, before any launch, and an argument list that is right up to its workspace ends in the workspace error."""
import ctypes

import pytest

import paper_2502_14317_amd as pc

ONE, ODD = ctypes.c_void_p(256), ctypes.c_void_p(264)          # never dereferenced
NULL, SHAPE, WORKSPACE = -1, -2, -3

LAYER = dict(shape=None, q=ONE, k=ONE, v=ONE, chunk_lens=None, first_len=64, keep_chunks=2, keep_tokens=8, calibrated=0, lam=0.5,
             class_lo=0, class_hi=4, o=ONE, lse=ONE, k_rope=ONE, tok_score=ONE, chunk_score=ONE, chunk_idx=ONE, chunk_top=None,
             tok_idx=ONE, tok_cnt=None, kc=ONE, vc=ONE, global_o=ONE, global_lse=None, ws=ONE, ws_bytes=0, stream=None)
LAYER_SHAPE = dict(n_chunks=2, chunk_len=64, query_len=16, n_q_heads=8, n_kv_heads=2, head_dim=128, obs_window=8, rope_base=1e4,
                   softmax_scale=0.0)
STEP = dict(q=ONE, k_new=ONE, v_new=ONE, batch=2, n_seg=3, k_t=64, n_q_heads=8, n_kv_heads=2, head_dim=128, pos=10, rope_base=1e4,
            softmax_scale=0.0, kc=ONE, vc=ONE, seg_len=ONE, seg_len_per_head=0, out=ONE, lse_out=None, ws=ONE, ws_bytes=0, stream=None)
STEP8 = dict(q=ONE, k_new=ONE, v_new=ONE, k8=ONE, v8=ONE, k_scale=ONE, v_scale=ONE, seg_len=None, seg_len_per_head=0, k_tail=ONE,
             v_tail=ONE, tail_len=ONE, tail_cap=32, batch=2, n_seg=3, k_t=64, n_q_heads=8, n_kv_heads=2, head_dim=128, pos=10,
             rope_base=1e4, softmax_scale=0.0, out=ONE, lse_out=None, ws=ONE, ws_bytes=0, stream=None)


def _layer(**change):
    fields = dict(LAYER_SHAPE, **{k: v for k, v in change.items() if k in LAYER_SHAPE})
    shape = pc.make_shape(*[fields[k] for k in ("n_chunks", "chunk_len", "query_len", "n_q_heads", "n_kv_heads", "head_dim",
                                                "obs_window", "rope_base")])
    shape.softmax_scale = fields["softmax_scale"]
    args = dict(LAYER, shape=ctypes.byref(shape), **{k: v for k, v in change.items() if k not in LAYER_SHAPE})
    return pc.lib().pc_layer_forward(*args.values())


def _call(fn, base):
    return lambda **change: getattr(pc.lib(), fn)(*dict(base, **change).values())


_step, _step8 = _call("pc_decode_step", STEP), _call("pc_decode_step_fp8", STEP8)
nan, inf = float("nan"), float("inf")


@pytest.mark.parametrize("want,changes", [
    (WORKSPACE, [{}, {"ws": None, "ws_bytes": 1 << 40}, {"ws": ctypes.c_void_p(128), "ws_bytes": 1 << 40}, {"query_len": 2},
                 {"calibrated": 1, "tok_cnt": ONE}, {"chunk_lens": ONE, "first_len": 0}]),
    (NULL, [{"shape": None}] + [{k: None} for k in ("q", "k", "v", "o", "lse", "k_rope", "tok_score", "chunk_score", "chunk_idx",
                                                    "tok_idx", "kc", "vc", "global_o")] + [{"calibrated": 1}]),
    (SHAPE, [{"n_chunks": 0}, {"head_dim": 96}, {"n_q_heads": 7}, {"rope_base": 0.5}, {"softmax_scale": -1.0}, {"obs_window": 0},
             {"obs_window": 81}, {"obs_window": 17, "chunk_lens": ONE}, {"first_len": -1}, {"first_len": 65}, {"keep_chunks": 0},
             {"keep_chunks": 3}, {"keep_tokens": 0}, {"keep_tokens": 65}, {"chunk_len": 32769, "first_len": 0}, {"n_chunks": 4097},
             {"query_len": 0}, {"calibrated": 1, "tok_cnt": ONE, "lam": nan}, {"calibrated": 1, "tok_cnt": ONE, "class_lo": 5},
             {"calibrated": 1, "tok_cnt": ONE, "class_hi": 65}, {"calibrated": 1, "tok_cnt": ONE, "class_lo": -1}]
     + [{k: ODD} for k in ("q", "k", "v", "o", "k_rope", "kc", "vc", "global_o")]),
])
def test_layer(want, changes):
    for change in changes:
        if change == {"shape": None}:
            assert pc.lib().pc_layer_forward(*dict(LAYER, shape=None).values()) == want
        else:
            assert _layer(**change) == want, change


COMMON_SHAPE = [{"batch": -1}, {"batch": 0}, {"k_t": 0}, {"n_kv_heads": 0}, {"n_q_heads": 7}, {"head_dim": 96}, {"rope_base": 0.5},
                {"rope_base": inf}, {"rope_base": nan}, {"softmax_scale": -1.0}, {"softmax_scale": nan}, {"seg_len_per_head": 2},
                {"k_t": (1 << 24) + 1}, {"batch": (1 << 20) + 1}, {"q": ODD}, {"out": ODD}]
# more than 16 heads a group (the tile path) and rows that arrive rotated (no base needed)
COMMON_OK = [{}, {"n_q_heads": 64}, {"pos": -1, "rope_base": 0.0}, {"ws": None, "ws_bytes": 1 << 40}]


@pytest.mark.parametrize("want,changes", [
    (WORKSPACE, COMMON_OK + [{"n_seg": 1}, {"seg_len_per_head": 1}]),
    (NULL, [{k: None} for k in ("q", "k_new", "v_new", "kc", "vc", "seg_len", "out")]),
    (SHAPE, COMMON_SHAPE + [{"n_seg": 0}, {"kc": ODD}, {"vc": ODD}, {"seg_len": ctypes.c_void_p(258)}, {"k_new": ctypes.c_void_p(257)}]),
])
def test_step(want, changes):
    for change in changes:
        assert _step(**change) == want, change


@pytest.mark.parametrize("want,changes", [
    (WORKSPACE, COMMON_OK + [{"n_seg": 0, "k8": None, "v8": None, "k_scale": None, "v_scale": None}, {"seg_len": ONE, "seg_len_per_head": 1}]),
    (NULL, [{k: None} for k in ("q", "k_new", "v_new", "k8", "v8", "k_scale", "v_scale", "k_tail", "v_tail", "tail_len", "out")]),
    (SHAPE, COMMON_SHAPE + [{"n_seg": -1}, {"tail_cap": 0}, {"tail_cap": (1 << 24) + 1}, {"k8": ODD}, {"v8": ODD}, {"k_tail": ODD},
                            {"v_tail": ODD}, {"tail_len": ctypes.c_void_p(258)}]),
])
def test_step_8bit(want, changes):
    for change in changes:
        assert _step8(**change) == want, change


@pytest.mark.parametrize("fn", [_step, _step8])
def test_tile_limits_of_a_step(fn):
    """Beyond 16 heads a group the tile kernel's limits hold, and are looked at before the new row is stored."""
    enough = dict(n_q_heads=64, ws_bytes=1 << 62)
    assert fn(k_t=65535 * 64 + 1, **enough) == SHAPE
    if fn is _step8:
        assert fn(tail_cap=65535 * 64 + 1, **enough) == SHAPE


def test_workspaces_of_refused_shapes_are_zero():
    bad = pc.make_shape(2, 64, 16, 7, 2, 128, 8, 1e4)
    good = pc.make_shape(2, 64, 16, 8, 2, 128, 8, 1e4)
    assert pc.pc_layer_workspace_bytes(bad, 2, 8) == 0 and pc.pc_layer_workspace_bytes(good, 2, 0) == 0
    assert pc.pc_layer_workspace_bytes(good, 2, 8) > pc.pc_chunk_prefill_workspace_bytes(good)
    assert pc.pc_decode_step_workspace_bytes(0, 3, 64, 8, 2, 128) == 0
    assert pc.pc_decode_step_fp8_workspace_bytes(2, 3, 64, -1, 8, 2, 128) == 0
    assert pc.pc_decode_step_workspace_bytes(2, 3, 64, 8, 2, 128) > pc.pc_parallel_attn_workspace_bytes(2, 1, 3, 64, 8, 2, 128, 0)
