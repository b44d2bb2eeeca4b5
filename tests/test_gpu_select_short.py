"""Selection of one short sequence: the forms of pooling (in one workgroup's LDS, by many workgroups) and of ranking (by
one wave, by counting, by classes) at their edges, against the oracle (Sec. 3.2.3)."""
import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T, chunk, window, rate", [
    (1, 1, 1, 1.0), (7, 8, 13, 0.5), (64, 1, 1, 0.1), (65, 1, 3, 0.9), (255, 1, 13, 0.3), (256, 1, 5, 0.01), (257, 1, 5, 0.3),
    (2047, 7, 13, 0.3), (2048, 8, 13, 0.2), (2048, 1, 1, 0.05), (2048, 9, 4095, 0.5), (2048, 256, 13, 0.3), (1500, 257, 13, 0.5),
    (2049, 8, 13, 0.2), (2049, 9, 13, 0.2), (8192, 32, 13, 0.1), (8191, 32, 13, 1.0), (8193, 33, 13, 0.1),
])
@pytest.mark.parametrize("kind", ["plain", "ties", "nan"])
def test_one_short_sequence(T, chunk, window, rate, kind):
    rng = np.random.default_rng(T + chunk)
    x = np.exp(2.0 * rng.standard_normal(T)).astype(np.float32) / 16000
    if kind == "ties":
        x = (np.round(x * 4e4) / 4e4).astype(np.float32)
    if kind == "nan":
        x[T // 2] = np.nan
    cu = np.array([0, T], dtype=np.int32)
    sel = hp.gpu_pool_select(x, cu, chunk, window, rate)
    if kind == "nan":
        assert sel.cu_keep.cpu().tolist() == [0, -1] and (sel.kept_idx == -1).all()
        return
    kept, cu_keep, cs, _ = orc.pool_select(x, cu, chunk, window, rate)
    assert sel.cu_keep.cpu().tolist() == cu_keep.tolist()
    np.testing.assert_array_equal(sel.chunk_scores.cpu().numpy()[:len(cs)], cs.astype(np.float32))
    got = sel.kept_idx.cpu().numpy()
    # (chunk means are the oracle's to a rounding of fp64: what ties in exact arithmetic may differ there)
    hp.selection_matches(got, sel.cu_keep.cpu().numpy(), x, cu, chunk, window, rate, 1e-12)
    assert (got[int(cu_keep[1]):] == -1).all()
    few = hp.gpu_pool_select(x, cu, chunk, window, rate, capacity=max(1, len(kept) // 2), want_chunk_scores=False)
    np.testing.assert_array_equal(few.kept_idx.cpu().numpy(), got[:max(1, len(kept) // 2)])


@pytest.mark.parametrize("T, window", [(1600, 4095), (1601, 16001), (1601, 15999), (1700, 159), (1700, 161), (2048, 35), (2048, 37),
                                       (2048, 2 ** 31 - 1)])
@pytest.mark.parametrize("chunk", [1, 7, 32, 256])
def test_wide_windows(T, window, chunk):
    """On both sides of the line between pooling by one workgroup and by many: the same chunk scores, the oracle's."""
    x = np.exp(2.0 * np.random.default_rng(T + window).standard_normal(T)).astype(np.float32) / 16000
    cu = np.array([0, T], dtype=np.int32)
    sel = hp.gpu_pool_select(x, cu, chunk, window, 0.3)
    _, cu_keep, cs, _ = orc.pool_select(x, cu, chunk, min(window, 2 * T + 1), 0.3)
    assert sel.cu_keep.cpu().tolist() == cu_keep.tolist()
    np.testing.assert_allclose(sel.chunk_scores.cpu().numpy()[:len(cs)], cs.astype(np.float32), rtol=2e-7)   # (fp64 means, rounded)
    hp.selection_matches(sel.kept_idx.cpu().numpy(), sel.cu_keep.cpu().numpy(), x, cu, chunk, min(window, 2 * T + 1), 0.3, 1e-12)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 1024, 1025, 2048])
@pytest.mark.parametrize("chunk, T", [(1, 0), (8, 0), (40, 0), (300, -7)])
def test_forms_of_ranking_at_their_edges(n, chunk, T):
    """So many chunks (the last one cut short where T says so), a tenth, half and all of them kept, ties among them."""
    T = n * chunk + (T if n * chunk > 7 else 0)
    x = np.exp(np.random.default_rng(n + chunk).standard_normal(T)).astype(np.float32) / 16000
    x = np.repeat(x[::4], 4)[:T] if chunk == 1 and n > 2 else x          # equal scores in fours
    cu = np.array([0, T], dtype=np.int32)
    for rate in (0.1, 0.5, 1.0):
        kept, cu_keep, _, _ = orc.pool_select(x, cu, chunk, 1, rate)
        sel = hp.gpu_pool_select(x, cu, chunk, 1, rate, want_chunk_scores=False)
        assert sel.cu_keep.cpu().tolist() == cu_keep.tolist()
        got = sel.kept_idx.cpu().numpy()
        if chunk == 1:                                                   # (the scores themselves: no rounding at all)
            np.testing.assert_array_equal(got[:len(kept)], kept)
        hp.selection_matches(got, sel.cu_keep.cpu().numpy(), x, cu, chunk, 1, rate, 1e-12)


@pytest.mark.parametrize("chunk", [1 << 30, 2 ** 31 - 1001, 2 ** 31 - 500, 2 ** 31 - 1])
@pytest.mark.parametrize("lens", [(1000,), (2047,), (1000, 0, 1, 1700)])
def test_chunks_longer_than_any_sequence(chunk, lens):
    """One chunk a sequence, all of it kept, up to the longest chunk an int holds."""
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    x = np.random.default_rng(7).random(T).astype(np.float32)
    for want_chunk_scores in (False, True):
        sel = hp.gpu_pool_select(x, cu, chunk, 1, 0.3, want_chunk_scores=want_chunk_scores)
        assert sel.cu_keep.cpu().tolist() == cu.tolist()
        assert sel.kept_idx.cpu().tolist() == list(range(T))
