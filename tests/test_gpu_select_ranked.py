"""The k-th chunk among chunks whose scores lie close together (Sec. 3.2.3): a cluster of as many as are ranked among
themselves, one fewer and one more, its least, middle and largest member the last one kept, ties in it, in every form of
the selection (one sequence, batches, chunks per thread)."""
import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, B", [(300, 1), (1024, 1), (2048, 1), (700, 3), (3000, 2), (9000, 2)])
@pytest.mark.parametrize("cluster", [1, 2, 63, 64, 65, 128, 200])
@pytest.mark.parametrize("ties", [1, 3])
def test_close_scores(n, B, cluster, ties):
    rng = np.random.default_rng(n + cluster)
    above = (n - cluster) // 3
    # values in [1, 2): the cluster a few units in the last place wide at 1.5, the others at least 1 / 32 away from it
    x = np.concatenate([1.54 + 0.45 * rng.random(above), 1.5 + (np.arange(cluster) // ties) * 2.0 ** -23,
                        1.0 + 0.45 * rng.random(n - cluster - above)]).astype(np.float32)
    cu = np.arange(0, n * B + 1, n, dtype=np.int32)
    for last in sorted({1, cluster // 2 + 1, cluster}):
        scores = np.concatenate([rng.permutation(x) for _ in range(B)])
        rate = (above + last - 0.5) / n                     # keeps above + last chunks
        kept, cu_keep, _, _ = orc.pool_select(scores, cu, 1, 1, rate)
        sel = hp.gpu_pool_select(scores, cu, 1, 1, rate, want_chunk_scores=False)
        assert sel.cu_keep.cpu().tolist() == cu_keep.tolist() == [b * (above + last) for b in range(B + 1)]
        np.testing.assert_array_equal(sel.kept_idx.cpu().numpy()[:len(kept)], kept)


@pytest.mark.parametrize("lens", [(1024, 0), (1025, 0, 0), (1000, 24), (1000, 25), (4096, 0), (0, 4097), (2000, 2096, 0), (1, 1, 1, 1, 1024)])
@pytest.mark.parametrize("chunk", [1, 3])
def test_batches_at_the_edges_of_what_a_kernel_holds(lens, chunk):
    """All tokens of the batch decide which kernel runs: sequences of as many chunks as it holds, and one more."""
    cu = np.concatenate([[0], np.cumsum(np.array(lens) * chunk)]).astype(np.int32)
    scores = np.random.default_rng(len(lens)).random(int(cu[-1])).astype(np.float32)
    kept, cu_keep, _, _ = orc.pool_select(scores, cu, chunk, 1, 0.3)
    for want_chunk_scores in (False, True):
        sel = hp.gpu_pool_select(scores, cu, chunk, 1, 0.3, want_chunk_scores=want_chunk_scores)
        assert sel.cu_keep.cpu().tolist() == cu_keep.tolist()
        hp.selection_matches(sel.kept_idx.cpu().numpy()[:len(kept)], cu_keep, scores, cu, chunk, 1, 0.3, 1e-12)
