"""Selection and gather of batches on either side of the number of sequences whose offsets are searched in LDS, of the number
one wave adds up, with empty sequences among them (Sec. 3.2.3 and 3.2.4 of arXiv 2502.02789; oracle)."""
import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [2, 63, 64, 65, 254, 255, 256, 257])
@pytest.mark.parametrize("chunk,window", [(1, 1), (16, 5), (300, 3)])
def test_kept_sets_and_positions(B, chunk, window):
    import torch
    from paper_2502_02789_amd import device as dev
    rng = np.random.default_rng(B * 1000 + chunk)
    lens = rng.integers(0, 90, size=B)
    lens[rng.integers(0, B)] = 700
    lens[rng.integers(0, B)] = 0
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    scores = rng.standard_normal(T).astype(np.float32) ** 2
    ids = rng.integers(0, 1000, size=T).astype(np.int32)
    want_idx, want_cu = orc.pool_select(scores, cu, chunk, window, 0.3)[:2]
    n = int(want_cu[-1])
    for table in (True, False):  # chunks numbered without gaps, as the caller who wants their scores gets them, and not
        sel = hp.gpu_pool_select(scores, cu, chunk, window, 0.3, want_chunk_scores=table)
        np.testing.assert_array_equal(sel.cu_keep.cpu().numpy(), want_cu)
        np.testing.assert_array_equal(sel.kept_idx.cpu().numpy()[:n], want_idx)
    got_ids, got_pos, decode, _ = dev.Gatherer(sel, token_ids=torch.from_numpy(ids).cuda()).run()
    owner = np.repeat(np.arange(B), np.diff(want_cu))
    np.testing.assert_array_equal(got_ids.cpu().numpy()[:n], ids[want_idx])
    np.testing.assert_array_equal(got_pos.cpu().numpy()[:n], want_idx - cu[owner])
    np.testing.assert_array_equal(decode.cpu().numpy(), lens)


@pytest.mark.parametrize("B", [2, 64, 65])
def test_one_invalid_score_keeps_nothing(B):
    lens = np.full(B, 50)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    scores = np.ones(int(cu[-1]), dtype=np.float32)
    scores[int(cu[-1]) - 7] = np.nan
    sel = hp.gpu_pool_select(scores, cu, 4, 1, 0.5, want_chunk_scores=False)
    assert sel.cu_keep.cpu().numpy()[0] == 0 and (sel.cu_keep.cpu().numpy()[1:] == -1).all()
