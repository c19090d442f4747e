"""A workspace serves every call that is no larger in any size than the one it was sized for: the sizes
the library asks for never fall where a size grows.  Host only."""
import paper_2502_14317_amd as pc


def _assert_rising(sizes, what):
    top, at = 0, None
    for key, n in sizes:
        assert n > 0, (what, key)
        assert n >= top, f"{what}: {key} needs {n} bytes, {at} needs {top}"
        top, at = n, key


def _score_sizes(shapes, fn):
    return [(s[:3] + s[6:7], fn(pc.make_shape(*s, 1e4))) for s in shapes]


def test_score_workspace_rises_with_chunks_and_rows():
    """Few and many voting columns, through the point where the key blocks double."""
    for fn in (pc.pc_chunk_query_scores_workspace_bytes, pc.pc_chunk_prefill_workspace_bytes):
        for hq, hkv, d, w, wq, obs in ((14, 2, 64, 1280, 512, 512), (16, 2, 128, 512, 512, 512), (12, 2, 64, 64, 512, 512),
                                       (32, 1, 128, 3000, 100, 100), (8, 8, 64, 100, 28, 28), (16, 2, 64, 100, 28, 28)):
            _assert_rising(_score_sizes([(c, w, wq, hq, hkv, d, obs) for c in range(1, 300)], fn), (fn, hq, hkv, "chunks"))
            for c in (1, 10):
                rows = sorted({1, 2, *range(64, 20000, 61)})
                _assert_rising(_score_sizes([(c, n, wq, hq, hkv, d, obs) for n in rows], fn), (fn, hq, hkv, c, "rows"))
                _assert_rising(_score_sizes([(c, w, wq, hq, hkv, d, n) for n in range(1, wq + 1)], fn),
                               (fn, hq, hkv, c, "voting rows"))


def test_tile_attention_workspace_rises_with_every_size():
    """Batch, query rows, segments, keys, tail and self segment, where the number of parts the keys are cut
    into goes up and down."""
    a, a8 = pc.pc_parallel_attn_workspace_bytes, pc.pc_parallel_attn_fp8_workspace_bytes
    for hq, hkv, d in ((32, 8, 128), (32, 32, 128), (8, 8, 64), (64, 8, 128), (3, 1, 64)):
        for s in (False, True):
            for n_q, n_seg, k_t in ((512, 8, 2048), (64, 4, 300), (100, 32, 1000)):
                _assert_rising([(b, a(b, n_q, n_seg, k_t, hq, hkv, d, s)) for b in range(1, 65)], (hq, s, "batch"))
                _assert_rising([(b, a8(b, n_q, n_seg, k_t, 200, hq, hkv, d, s)) for b in range(1, 65)], (hq, s, "batch, 8 bit"))
            for b in (1, 3, 8):
                _assert_rising([(n, a(b, n, 8, 2048, hq, hkv, d, s)) for n in range(17, 2100, 5)], (hq, s, b, "rows"))
                _assert_rising([(n, a(b, 200, n, 500, hq, hkv, d, s)) for n in range(1, 100)], (hq, s, b, "segments"))
                _assert_rising([(n, a(b, 200, 3, n, hq, hkv, d, s)) for n in range(1, 6000, 31)], (hq, s, b, "keys"))
                _assert_rising([(n, a8(b, 200, 3, 100, n, hq, hkv, d, s)) for n in range(1, 6000, 31)], (hq, s, b, "tail"))
                assert a(b, 200, 3, 500, hq, hkv, d, True) >= a(b, 200, 3, 500, hq, hkv, d, False)
