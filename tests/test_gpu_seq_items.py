"""The single-pass kernel for few query rows at the edges of its 32-key items and of the pairs they are held in: a wave with
one item more than another, an odd number of items, a ragged first one, waves without keys; four and eight rows, both head
dims, contiguous and paged (Sec. 3.2 equation of arXiv 2502.02789, fp64 oracle)."""
import math

import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import helpers as hp
from tests import test_gpu_fp8_cache as fp8
from tests.test_gpu_batch_single_pass import _check
from tests.test_unit_deal import _stretch, lib  # noqa: F401 (lib: a fixture)

pytestmark = pytest.mark.gpu

# items of 32 keys, dealt to eight waves: 1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 32, 33 and one key more or fewer
LENS = tuple(32 * i + e for i in (1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 32, 33) for e in (-1, 0, 1)) + (1, 0, 5, 2047)


@pytest.mark.parametrize("paged", [0, 16])
@pytest.mark.parametrize("shape", [dict(H=4, H_kv=1, N=1, d=128), dict(H=4, H_kv=1, N=2, d=64), dict(H=8, H_kv=1, N=1, d=128),
                                   dict(H=3, H_kv=1, N=1, d=64)])
def test_items_and_pairs(shape, paged):
    w = synth.scaled(synth.workload(4), seqlens=LENS, L=8, salient_frac=0.02, salient_run=1, **shape)
    inp = synth.make_qk(w)
    scale = 1.0 / math.sqrt(w.d)
    for mode in (orc.LAYER_MAX, orc.LAYER_MEAN):
        want, want_lse = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], scale, mode)
        if paged:
            pools, table = hp.paged_copy(inp["k"], inp["cu_seqlens"], paged, seed=3)
            got, lse = hp.gpu_score_paged(inp["q"], pools, table, inp["cu_seqlens"], w.H_kv, scale, mode, max_seqlen=2047)
        else:
            got, lse = hp.gpu_score(inp["q"], inp["k"], inp["cu_seqlens"], w.H_kv, scale, mode, max_seqlen=2047)
        hp.assert_scores_close(got, want, f"{shape} mode={mode} paged={paged}")
        np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-4)


@pytest.mark.parametrize("n_queries,mode,layers", [
    (1, orc.LAYER_MAX, 32), (1, orc.LAYER_MEAN, 32), (1, orc.LAYER_MEAN, 128),  # (mean: in rounds, and in stretches of layers)
    (4, orc.LAYER_MAX, 32), (8, orc.LAYER_MAX, 32), (8, orc.LAYER_MEAN, 32)])
def test_stretches_of_equal_cost(n_queries, mode, layers):
    """Enough slabs for every workgroup to get a stretch of them: sequences that one workgroup has several of, that several
    share, that are empty, and one that breaks the promise (NaN, and nobody else is touched)."""
    lens = (700, 1, 0, 33, 650, 64, 300, 0, 257) * 6 + (699,)
    over = 8193 if n_queries == 1 else 4097 if n_queries == 2 else 3073
    for all_lens in (lens, lens[:20] + (over,) + lens[20:]):
        w = synth.scaled(synth.workload(4), seqlens=all_lens, L=layers, H=16, H_kv=4, N=n_queries, d=64, salient_frac=0.02, salient_run=1)
        inp = synth.make_qk(w)
        scale = 1.0 / math.sqrt(w.d)
        want, want_lse = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], scale, mode)
        got, lse = hp.gpu_score(inp["q"], inp["k"], inp["cu_seqlens"], w.H_kv, scale, mode, max_seqlen=700)
        cu = np.asarray(inp["cu_seqlens"])
        ok = np.ones(len(got), dtype=bool)
        if len(all_lens) > len(lens):
            ok[cu[20]:cu[21]] = False
            assert np.isnan(got[~ok]).all() and np.isnan(lse[:, 20]).all()
        hp.assert_scores_close(got[ok], want[ok], f"{n_queries} mode={mode}")
        keep = [b for b in range(len(all_lens)) if all_lens[b] != over]
        np.testing.assert_allclose(lse[:, keep], want_lse[:, keep], rtol=0, atol=2e-4)


@pytest.mark.parametrize("shape, bits, paged", [
    (dict(H=16, N=2, d=64), 16, 16), (dict(H=16, N=2, d=64), 8, 0), (dict(H=32, N=1, d=128), 16, 0), (dict(H=32, N=1, d=128), 8, 16),  # eight rows
    (dict(H=16, N=1, d=128, L=28), 16, 16), (dict(H=16, N=1, d=64, L=28), 8, 16),                                                      # four
    (dict(H=16, N=8, d=128), 16, 16), (dict(H=16, N=8, d=128), 8, 0), (dict(H=16, N=8, d=64), 8, 16),  # the kernel for 32 rows, four ...
    (dict(H=32, N=4, d=128), 16, 0), (dict(H=32, N=4, d=128), 8, 16), (dict(H=32, N=4, d=64), 16, 16)])  # ... and eight heads per KV head
def test_stretches_in_every_form_of_the_kernels(lib, shape, bits, paged):  # noqa: F811
    """Eight and 32 rows, both head dims, pages and 8-bit keys; the batch is one that is cut into stretches."""
    lens = (700, 1, 0, 33, 650, 64, 300, 0, 257) * 6 + (699,)
    w = synth.scaled(synth.workload(4), seqlens=lens, salient_frac=0.02, salient_run=1, **dict(dict(L=16, H_kv=4), **shape))
    rows = (4 if w.H <= 16 else 8) * w.N
    assert _stretch(lib, lens, w.L, w.H_kv, fp8=int(bits == 8), d=w.d, N=w.N, limit=8192 if rows <= 4 else 4096 if rows <= 8 else 3072) != 0
    if bits == 8:
        fp8._check(w, orc.LAYER_MAX, False, max_seqlen=700, paged=paged)
    else:
        _check(w, synth.make_qk(w), orc.LAYER_MAX, max_seqlen=700, paged=paged)
