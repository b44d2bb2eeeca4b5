"""GPU parity of sp_pool_select at the sizes where its kernels change form (chunks held in registers up to 16384 per
sequence, few per workgroup or one long one, with and without the chunk scores) against the fp64 oracle."""
import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def _scores(n, seed, kind):
    g = np.random.default_rng(seed)
    if kind == "ties":     # few distinct values: equal chunk scores everywhere, also at the threshold
        return g.integers(1, 4, size=n).astype(np.float32)
    if kind == "wide":     # the sign-and-exponent byte differs
        return (10.0 ** g.uniform(-37, 37, size=n)).astype(np.float32)
    return np.exp(2.0 * g.standard_normal(n)).astype(np.float32) / 16000.0


@pytest.mark.parametrize("kind", ["plain", "ties", "wide"])
@pytest.mark.parametrize("lens, chunk, window, rate", [
    ((1,), 1, 1, 0.5),
    ((1025,), 1, 1, 0.1),                                   # two rows per wave
    ((2048,), 1, 5, 0.3), ((2049,), 1, 5, 0.3),             # the single-sequence kernel's largest, the general path
    ((0, 1, 1024, 1025, 4096, 4097, 63, 16384, 16385), 1, 3, 0.2),  # all register sizes and one beyond
    ((300, 0, 7, 5000), 7, 13, 0.25),                       # chunks that do not divide a workgroup, short last ones
    ((1000, 3, 700), 255, 9, 0.4), ((1000, 3, 700), 256, 9, 0.4), ((1000, 3, 700), 257, 9, 0.4),  # long chunks
    ((900,), 300, 1001, 0.5),                               # a window longer than the sequence
    ((40,) * 70, 16, 13, 1.0),                              # everything kept, more sequences than a wave
])
def test_selection_at_the_edges(lens, chunk, window, rate, kind):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    sc = _scores(int(cu[-1]), len(lens) + chunk, kind)
    kept_o, cu_keep_o, cs_o, _ = orc.pool_select(sc, cu, chunk, window, rate)
    for want_chunk_scores in (False, True):
        for _ in range(2):
            sel = hp.gpu_pool_select(sc, cu, chunk, window, rate, want_chunk_scores=want_chunk_scores)
            cu_keep, n = sel.cu_keep.cpu().numpy(), len(kept_o)
            kept = sel.kept_idx.cpu().numpy()
            assert (cu_keep == cu_keep_o).all()
            assert (kept[:n] == kept_o).all() and (kept[n:] == -1).all()
            if want_chunk_scores:
                np.testing.assert_allclose(sel.chunk_scores.cpu().numpy()[:len(cs_o)], cs_o.astype(np.float32), rtol=1e-6)


@pytest.mark.parametrize("want_chunk_scores", [False, True])
@pytest.mark.parametrize("lens", [(3000,), (500, 20000, 7)])
def test_a_nan_score_is_answered_in_band(lens, want_chunk_scores):
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    sc = _scores(int(cu[-1]), 3, "plain")
    sc[min(700, len(sc) - 1)] = np.nan
    sel = hp.gpu_pool_select(sc, cu, 1, 1, 0.2, want_chunk_scores=want_chunk_scores)
    assert (sel.cu_keep.cpu().numpy()[1:] == -1).all() and (sel.kept_idx.cpu().numpy() == -1).all()
