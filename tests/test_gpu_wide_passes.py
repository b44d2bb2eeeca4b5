"""GPU parity of the two-pass kernels for many query rows per KV head (batches with long sequences, short prompts of few
slabs on a shared device, prompts longer than the teams of workgroups hold) against the fp64 oracle, element by element
(Sec. 3.2 equation, Sec. 3.2.2)."""
import math

import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import helpers as hp
from tests import test_gpu_fp8_cache as fp8
from tests.test_gpu_batch_single_pass import _check, _lens

pytestmark = pytest.mark.gpu

MODES = [orc.LAYER_MAX, orc.LAYER_MEAN]


# One sequence comes here without the promise of an idle device where it has up to 3072 keys and fewer than 64 (layer, KV head)
# slabs (more go to the kernels for whole sequences and to the teams), and with any promise beyond 131072 keys.
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [
    dict(tokens=3072, L=4, H=32, H_kv=8, N=8, d=128),
    dict(tokens=2049, L=2, H=16, H_kv=4, N=8, d=64),
    dict(tokens=1000, L=3, H=6, H_kv=2, N=5, d=128),     # three heads padded to four
    dict(tokens=3001, L=2, H=64, H_kv=8, N=4, d=64),     # eight heads per KV head
    dict(tokens=2500, L=5, H=8, H_kv=1, N=3, d=128),     # few slabs, ragged pieces
    dict(tokens=33, L=3, H=4, H_kv=1, N=8, d=64),        # results that outweigh the keys
])
def test_one_short_prompt_of_few_slabs(shape, mode):
    """bf16 and 8-bit keys, contiguous and paged."""
    shape = dict(shape)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), salient_run=1, **shape)
    inp = synth.make_qk(w)
    _check(w, inp, mode, max_seqlen=0, exclusive_device=False)
    fp8._check(w, mode, False, exclusive_device=False)
    for bits, page in ((16, 8), (8, 16)):
        _check_paged(w, inp, mode, bits, page)


def _check_paged(w, inp, mode, bits, page):
    import torch
    from paper_2502_02789_amd import device as dev
    keys, k_scale = synth.quantize_k_fp8(inp["k"]) if bits == 8 else (inp["k"], None)
    scale = 1.0 / math.sqrt(w.d)
    want, want_lse = orc.token_importance(inp["q"], keys, inp["cu_seqlens"], scale, mode, **(dict(k_scale=k_scale) if bits == 8 else {}))
    pools, table = hp.paged_copy(keys, inp["cu_seqlens"], page, seed=page, fill=0x7E if bits == 8 else 0x7F00)
    s = dev.Scorer(dev.bf16_from_bits(inp["q"]), [torch.from_numpy(p).cuda() if bits == 8 else dev.bf16_from_bits(p) for p in pools],
                   torch.from_numpy(np.asarray(inp["cu_seqlens"], dtype=np.int32)).cuda(), H_kv=w.H_kv, scale=scale, layer_reduce=mode,
                   want_lse=True, block_table=torch.from_numpy(table).cuda(), page_size=page, total_tokens=w.T, exclusive_device=False,
                   k_scale=None if k_scale is None else torch.from_numpy(np.ascontiguousarray(k_scale)).cuda())
    s.scores.fill_(float("nan"))
    s.run()
    s.check()
    hp.assert_scores_close(s.scores.cpu().numpy(), want, f"{w.name} {bits} bits, pages of {page}, mode={mode}")
    np.testing.assert_allclose(s.lse.cpu().numpy(), want_lse, rtol=0, atol=2e-4)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("tokens, N, H, H_kv, bits", [
    (131073, 8, 4, 1, 16),      # a key more than the teams hold
    (140007, 4, 16, 2, 8),      # eight heads per KV head
    (65537, 12, 4, 2, 16),      # more than eight queries, two heads: the teams end at 65536, the tiled kernels take it
])
def test_one_prompt_longer_than_the_teams_hold(tokens, N, H, H_kv, bits, mode):
    """Against the plain kernels on the same buffers, with and without the promise of an idle device."""
    import torch
    from paper_2502_02789_amd import device as dev
    w = synth.scaled(synth.workload(3), seqlens=(tokens,), L=1, H=H, H_kv=H_kv, N=N, d=64, salient_run=1)
    inp = synth.make_qk(w)
    keys, k_scale = synth.quantize_k_fp8(inp["k"]) if bits == 8 else (inp["k"], None)
    for exclusive in (False, True):
        s = dev.Scorer(dev.bf16_from_bits(inp["q"]), [torch.from_numpy(k).cuda() if bits == 8 else dev.bf16_from_bits(k) for k in keys],
                       torch.tensor([0, tokens], dtype=torch.int32).cuda(), H_kv=H_kv, scale=1.0 / math.sqrt(w.d), layer_reduce=mode,
                       want_lse=True, exclusive_device=exclusive,
                       k_scale=None if k_scale is None else torch.from_numpy(np.ascontiguousarray(k_scale)).cuda())
        got = []
        for general in (False, True):
            s.scores.fill_(float("nan"))
            s.run(general=general)
            s.check()
            got.append((s.scores.cpu().numpy(), s.lse.cpu().numpy()))
        hp.assert_scores_close(got[0][0], got[1][0], f"{tokens} keys, {N} queries, mode={mode}")
        np.testing.assert_allclose(got[0][1], got[1][1], rtol=0, atol=2e-4)


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
