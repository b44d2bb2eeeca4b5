"""GPU parity of the two-pass kernels for many query rows per KV head (long prompts on a shared device, batches with
long sequences) against the fp64 oracle, element by element (Sec. 3.2 equation, Sec. 3.2.2)."""
import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import test_gpu_fp8_cache as fp8
from tests.test_gpu_batch_single_pass import _check, _lens

pytestmark = pytest.mark.gpu

MODES = [orc.LAYER_MAX, orc.LAYER_MEAN]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [
    dict(tokens=3073, L=4, H=32, H_kv=8, N=8, d=128),    # one key more than the single-pass kernel holds
    dict(tokens=4096, L=2, H=16, H_kv=4, N=8, d=64),     # a full piece
    dict(tokens=4097, L=3, H=6, H_kv=2, N=5, d=128),     # three heads padded to four, two pieces
    dict(tokens=12345, L=2, H=64, H_kv=8, N=4, d=64),    # eight heads per KV head
    dict(tokens=8225, L=5, H=8, H_kv=1, N=3, d=128),     # few slabs, ragged pieces
    dict(tokens=5001, L=3, H=4, H_kv=1, N=8, d=64),      # results that outweigh the keys
])
def test_one_prompt_on_a_shared_device(shape, mode):
    shape = dict(shape)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), salient_run=1, **shape)
    inp = synth.make_qk(w)
    _check(w, inp, mode, max_seqlen=0, exclusive_device=False)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("d", [64, 128])
def test_batch_with_long_sequences(d, mode):
    """Empty sequences, one key, the edges of tiles, items and 2048-key pieces; valid query counts; pages."""
    lens = (0, 1, 31, 32, 33, 65, 2047, 2048, 2049, 0, 4097, 513) + _lens(d, 12, 1, 300)
    w = synth.scaled(synth.workload(4), seqlens=lens, L=3, H=8, H_kv=2, N=8, d=d, salient_frac=0.02, salient_run=1)
    inp = synth.make_qk(w)
    nv = np.random.default_rng(d).integers(1, 9, size=len(lens)).astype(np.int32)
    _check(w, inp, mode, max_seqlen=5000, n_valid=nv)    # a stated length beyond what the single-pass kernel holds
    _check(w, inp, mode, max_seqlen=5000, paged=16)


@pytest.mark.parametrize("mode", MODES)
def test_batch_of_one_slab(mode):
    """Next to no slabs: pieces of 256 keys."""
    w = synth.scaled(synth.workload(4), seqlens=(5000, 0, 255, 256, 257, 3100), L=1, H=4, H_kv=1, N=8, d=64, salient_frac=0.02, salient_run=1)
    inp = synth.make_qk(w)
    _check(w, inp, mode, max_seqlen=5000)
    _check(w, inp, mode, max_seqlen=5000, paged=16)
    fp8._check(w, mode, False, max_seqlen=5000)


@pytest.mark.parametrize("d, paged", [(64, 0), (128, 0), (64, 16), (128, 8)])
def test_8_bit_cache(d, paged):
    w = synth.scaled(synth.workload(3), seqlens=(300, 4500, 7), L=2, H=32, H_kv=8, N=8, d=d, salient_run=1)
    for mode in MODES:
        fp8._check(w, mode, False, paged=paged, max_seqlen=4500)


@pytest.mark.parametrize("mode", MODES)
def test_8_bit_cache_eight_heads_per_kv_head(mode):
    for d in (64, 128):
        w = synth.scaled(synth.workload(3), seqlens=(300, 4500, 7), L=2, H=32, H_kv=4, N=4, d=d, salient_run=1)
        fp8._check(w, mode, False, paged=16 if d == 64 else 0, max_seqlen=4500)
