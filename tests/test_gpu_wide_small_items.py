"""GPU parity of the kernels with 32 query rows per KV head where a ring item is two loads (8-bit keys, d = 64): the waits for
single items at starts, ends and in slabs of few tiles per wave, on the three kernels that share the stream, against
the fp64 oracle (Sec. 3.2 equation, Sec. 3.2.2)."""
import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import test_gpu_fp8_cache as fp8
from tests.test_gpu_batch_single_pass import _check
from tests.test_gpu_wide_passes import _check_paged

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [orc.LAYER_MAX, orc.LAYER_MEAN])
@pytest.mark.parametrize("lens, kw", [
    ((1, 31, 33, 65, 0, 97, 255, 256, 257, 289, 513, 769, 1025, 1600), dict(max_seqlen=1600)),   # whole sequences
    ((40, 300, 7, 1000, 290), dict(max_seqlen=1000, paged=16)),
    ((3500,), {}),                                                                               # teams: 1 to 7 items a wave
    ((9001,), dict(exclusive_device=False)),
    ((33, 4500, 300), dict(max_seqlen=4500)),                                                    # two passes
])
def test_items_of_two_loads(lens, kw, mode):
    w = synth.scaled(synth.workload(4), seqlens=lens, L=3, H=32, H_kv=8, N=8, d=64, salient_frac=0.02, salient_run=1)
    fp8._check(w, mode, False, **kw)


@pytest.mark.parametrize("page", [8, 16, 32, 128])
@pytest.mark.parametrize("lens", [(1700,), (4501,)])         # two passes of a short prompt of few slabs; teams
@pytest.mark.parametrize("bits, d", [(16, 64), (16, 128), (8, 64), (8, 128)])
def test_pages_smaller_and_larger_than_an_item(bits, d, lens, page):
    """Items of 32 keys in four pages to a quarter of one, the last page cut short."""
    w = synth.scaled(synth.workload(3), seqlens=lens, L=2, H=8, H_kv=2, N=8, d=d, salient_run=1)
    _check_paged(w, synth.make_qk(w), orc.LAYER_MAX, bits, page)


@pytest.mark.parametrize("page", [8, 32, 128])
@pytest.mark.parametrize("lens, max_seqlen", [((300, 33, 0, 1, 1000, 129), 1000), ((300, 4100, 1, 65), 4100)])
@pytest.mark.parametrize("d", [64, 128])
def test_pages_in_batches(d, lens, max_seqlen, page):
    w = synth.scaled(synth.workload(4), seqlens=lens, L=3, H=16, H_kv=4, N=8, d=d, salient_frac=0.02, salient_run=1)
    nv = np.arange(1, len(lens) + 1, dtype=np.int32)
    inp = synth.make_qk(w)
    for mode in (orc.LAYER_MAX, orc.LAYER_MEAN):
        _check(w, inp, mode, max_seqlen=max_seqlen, paged=page, n_valid=nv)
        fp8._check(w, mode, False, max_seqlen=max_seqlen, paged=page, n_valid=nv)
