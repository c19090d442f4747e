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
