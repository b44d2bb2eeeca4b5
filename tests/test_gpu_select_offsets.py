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


@pytest.mark.parametrize("B,embed", [(1, 0), (3, 0), (255, 0), (256, 0), (3, 64)])
def test_gather_from_a_list_that_ends_with_the_last_kept_index(B, embed):
    """sp_gather with a list of exactly cu_keep[B] indices and outputs of more room: what lies behind the list (here indices
    that no prompt has) goes nowhere, and the outputs behind the kept tokens stay as they were."""
    import torch
    from paper_2502_02789_amd import binding as sp
    rng = np.random.default_rng(B)
    lens = rng.integers(0, 40, size=B)
    lens[0] = 900
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    kept, cu_keep = orc.pool_select(rng.random(T).astype(np.float32), cu, 8, 3, 0.2)[:2]
    ids = rng.integers(0, 100, size=T).astype(np.int32)
    table = rng.integers(0, 2 ** 15, size=(100, embed or 8)).astype(np.int16)
    n, cap = len(kept), len(kept) + 1500
    room = torch.full((n + 2000,), 2 ** 31 - 1, dtype=torch.int32, device="cuda")
    room[:n] = torch.from_numpy(kept.astype(np.int32)).cuda()
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = {k: torch.full((cap,), -7, dtype=torch.int32, device="cuda") for k in ("kept_pos", "kept_ids")}
    decode = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    rows = torch.full((cap, embed), 7, dtype=torch.int16, device="cuda").view(torch.bfloat16) if embed else None
    keep = [dev(cu), dev(cu_keep.astype(np.int32)), room[:n], dev(ids), dev(table).view(torch.bfloat16) if embed else None]
    sp.sp_gather(sp.make_gather_args(keep[0], keep[1], keep[2], out["kept_pos"], decode, token_ids=keep[3],
                                     kept_ids=out["kept_ids"], embed=keep[4], out_embed=rows))
    want_ids, want_pos, want_decode, want_rows = orc.gather(kept, cu_keep, cu, ids, table.view(np.uint16))
    np.testing.assert_array_equal(out["kept_ids"].cpu().numpy()[:n], want_ids)
    np.testing.assert_array_equal(out["kept_pos"].cpu().numpy()[:n], want_pos)
    np.testing.assert_array_equal(decode.cpu().numpy(), want_decode)
    assert (out["kept_ids"][n:] == -7).all() and (out["kept_pos"][n:] == -7).all()
    if embed:
        np.testing.assert_array_equal(rows.view(torch.int16).cpu().numpy().view(np.uint16)[:n], want_rows)
        assert (rows.view(torch.int16)[n:] == 7).all()
