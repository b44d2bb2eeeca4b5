"""GPU parity of the kernels with 32 query rows per KV head where a ring item is two loads (8-bit keys, d = 64): the waits for
single items at starts, ends and in slabs of few tiles per wave, on the three kernels that share the stream, against
the fp64 oracle (Sec. 3.2 equation, Sec. 3.2.2)."""
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import test_gpu_fp8_cache as fp8

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
