"""GPU parity of the single-pass kernel for short prompts with look-ahead (nine to 32 query rows per KV head, all
logits of a sequence on chip) against the fp64 oracle, element by element (Sec. 3.2 equation, Sec. 3.2.2)."""
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
# empty, one key, the edges of 32- and 64-key tiles, waves without a tile, all eight waves with a ragged last one
LENS = (0, 1, 31, 32, 33, 63, 64, 65, 127, 129, 255, 256, 257, 500, 512, 513, 1029, 1100)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [
    dict(H=8, H_kv=2, N=8, d=128),      # Llama-shaped draft, eight look-ahead steps: all 32 columns
    dict(H=8, H_kv=2, N=8, d=64),
    dict(H=6, H_kv=2, N=5, d=128),      # three heads padded to four, unused query slots
    dict(H=4, H_kv=2, N=3, d=64),       # two heads padded to four
    dict(H=16, H_kv=2, N=4, d=128),     # eight heads per KV head
    dict(H=10, H_kv=2, N=3, d=64),      # five heads padded to eight
])
def test_batch_with_look_ahead(shape, mode):
    w = synth.scaled(synth.workload(4), seqlens=LENS, L=4, salient_frac=0.02, salient_run=1, **shape)
    inp = synth.make_qk(w)
    _check(w, inp, mode, max_seqlen=1100)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("longest", [2048, 2049, 2304, 2305, 3072, 3073])
def test_edges_of_what_the_registers_hold(longest, d, mode):
    """Up to 2304 keys (bf16, d = 128) or 2048 the running maximum over a unit's slabs is all in registers, up to 3072
    partly in memory (units of one slab and of several); one more and the other kernels take over."""
    for B_small, L in ((2, 4), (40, 8)):
        w = synth.scaled(synth.workload(4), seqlens=(longest, longest - 31) + _lens(longest, B_small, 1, 90), L=L,
                         H=8, H_kv=2, N=8, d=d, salient_frac=0.02, salient_run=1)
        _check(w, synth.make_qk(w), mode, max_seqlen=longest)


@pytest.mark.parametrize("mode", MODES)
def test_valid_query_counts_pages_and_many_units(mode):
    """Enough sequences that a workgroup walks over many units of several slabs."""
    w = synth.scaled(synth.workload(4), seqlens=_lens(17, 80, 1, 400), L=12, H=8, H_kv=2, N=8, salient_frac=0.02, salient_run=1)
    inp = synth.make_qk(w)
    nv = np.random.default_rng(18).integers(1, 9, size=80).astype(np.int32)
    _check(w, inp, mode, max_seqlen=400, n_valid=nv)
    _check(w, inp, mode, max_seqlen=400, n_valid=nv, paged=16)
    _check(w, inp, mode, max_seqlen=400, paged=8)
    _check(w, inp, mode, max_seqlen=3000, paged=128)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("n_keys", [1, 300, 2048, 3001])
def test_one_prompt_with_look_ahead(n_keys, mode):
    w = synth.scaled(synth.workload(3), seqlens=(n_keys,), L=8, N=8)
    inp = synth.make_qk(w)
    a = _check(w, inp, mode, max_seqlen=0, exclusive_device=True)
    b = _check(w, inp, mode, max_seqlen=0, exclusive_device=False)
    assert (a.view(np.uint32) == b.view(np.uint32)).all()   # the flag does not matter here
    _check(w, inp, mode, max_seqlen=0, paged=16)


def test_a_sequence_longer_than_the_kernel_holds_gets_nan_scores():
    lens = _lens(10, 20, 50, 400)
    w = synth.scaled(synth.workload(4), seqlens=lens[:9] + (3073,) + lens[10:], L=8, H=8, H_kv=2, N=8)
    inp = synth.make_qk(w)
    scale = 1.0 / math.sqrt(w.d)
    want, _ = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], scale, orc.LAYER_MAX)
    got, lse = hp.gpu_score(inp["q"], inp["k"], inp["cu_seqlens"], w.H_kv, scale, orc.LAYER_MAX, max_seqlen=400)
    cu = np.asarray(inp["cu_seqlens"])
    inside = np.zeros(len(got), dtype=bool)
    inside[cu[9]:cu[10]] = True
    assert np.isnan(got[inside]).all() and np.isnan(lse[:, 9]).all()
    hp.assert_scores_close(got[~inside], want[~inside], "the other sequences")


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [dict(H=8, N=8), dict(H=16, N=4), dict(H=6, N=3)])   # four, eight and three per KV head
def test_8_bit_cache(heads, d, mode):
    """Slots of two and four 32-key tiles: the edges of tiles and slots, paged and not."""
    w = synth.scaled(synth.workload(4), seqlens=LENS, L=4, H_kv=2, d=d, salient_frac=0.02, salient_run=1, **heads)
    for paged in (0, 16):
        fp8._check(w, mode, False, max_seqlen=1100, paged=paged)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("longest", [2048, 2049, 3072])
def test_8_bit_cache_at_the_edges_of_what_the_registers_hold(longest, d, mode):
    """Units of several slabs whose running maxima are read back beyond 2048 keys, with whole and ragged last slots."""
    w = synth.scaled(synth.workload(4), seqlens=(longest, longest - 31, longest - 97) + _lens(longest, 77, 1, 90), L=8,
                     H=8, H_kv=2, N=8, d=d, salient_frac=0.02, salient_run=1)
    fp8._check(w, mode, False, max_seqlen=longest)
    fp8._check(w, mode, False, max_seqlen=longest, paged=16)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("n_keys", [2047, 2048, 2081, 3072, 3073])
def test_one_prompt_of_many_slabs_with_and_without_the_promise(n_keys, mode):
    """128 slabs: on an idle device from 2048 keys on in teams of two workgroups, else a workgroup to a slab; the workspace handed on
    from call to call either way."""
    w = synth.scaled(synth.workload(3), seqlens=(n_keys,), L=32, H=16, H_kv=4, N=8, d=64)
    inp = synth.make_qk(w)
    a = _check(w, inp, mode, max_seqlen=0, exclusive_device=True)
    b = _check(w, inp, mode, max_seqlen=0, exclusive_device=False)
    np.testing.assert_allclose(a, b, rtol=2e-5)
    import torch
    from paper_2502_02789_amd import device as dev
    cu = torch.from_numpy(inp["cu_seqlens"]).cuda()
    s = dev.Scorer(dev.bf16_from_bits(inp["q"]), [dev.bf16_from_bits(k) for k in inp["k"]], cu, H_kv=w.H_kv, scale=1.0 / math.sqrt(w.d),
                   layer_reduce=mode, keep_workspace=True)
    for _ in range(3):
        assert np.array_equal(s.run().cpu().numpy(), a)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("lens, L, H_kv, N", [
    ((300,), 24, 8, 8), ((300,), 28, 8, 8), ((2500,), 28, 8, 8),  # 192 and 224 results a tile: a step of eight rows a thread and a part of one
    ((90,), 17, 8, 5), ((33,), 33, 8, 3),                         # queries that do not divide the rows of a step, one result beyond two steps
    ((500,), 5, 16, 8), ((500,), 11, 6, 8), ((500,), 16, 4, 8),   # parts of a layer: two steps of eight, fewer than eight, four
    (_lens(3, 60, 1, 90), 12, 2, 8), (_lens(4, 20, 1, 300), 16, 4, 4),  # whole layers and halves of layers as parts
])
def test_merge_of_results(lens, L, H_kv, N, mode):
    w = synth.scaled(synth.workload(4), seqlens=lens, L=L, H=4 * H_kv, H_kv=H_kv, N=N, d=64, salient_frac=0.02, salient_run=1)
    _check(w, synth.make_qk(w), mode, max_seqlen=max(lens))


@pytest.mark.parametrize("n_keys, L, H_kv, N, waits", [
    (2047, 16, 8, 8, False), (2800, 16, 8, 8, True), (2048, 36, 8, 8, True), (3072, 24, 8, 8, False), (2048, 15, 8, 8, False),
    (3073, 24, 8, 8, True), (500, 8, 8, 8, False), (500, 7, 8, 8, True), (3000, 40, 8, 1, False)])
def test_which_calls_may_wait_on_the_promise_of_an_idle_device(n_keys, L, H_kv, N, waits):
    """With no polls allowed a call that waits for other workgroups has NaN scores, the others do not notice."""
    import torch
    from paper_2502_02789_amd import binding as sp, device as dev
    g = torch.Generator(device="cuda")
    g.manual_seed(n_keys)
    q = torch.randn((L, 1, N, 4 * H_kv, 64), device="cuda", generator=g).to(torch.bfloat16)
    ks = [torch.randn((n_keys, H_kv, 64), device="cuda", generator=g).to(torch.bfloat16) for _ in range(L)]
    s = dev.Scorer(q, ks, torch.tensor([0, n_keys], dtype=torch.int32, device="cuda"), H_kv=H_kv, scale=0.125, exclusive_device=True)
    before = sp.sp_set_wait_budget(0)
    try:
        got = s.run().clone()
        torch.cuda.synchronize()
    finally:
        sp.sp_set_wait_budget(before)
    assert bool(torch.isnan(got).all()) if waits else bool(torch.isfinite(got).all())


@pytest.mark.parametrize("n_keys, L, H_kv, N, d", [(2100, 32, 8, 8, 128), (2100, 32, 8, 4, 128), (2100, 16, 8, 8, 64), (2700, 16, 8, 8, 64), (3073, 16, 8, 8, 64)])
def test_kept_workspace_handed_on_between_kinds_of_cache(n_keys, L, H_kv, N, d):
    """Calls of one shape on a bf16 and on an 8-bit cache, in turn on one workspace that is kept: the scores of calls that keep nothing."""
    import torch
    from paper_2502_02789_amd import binding as sp, device as dev
    g = torch.Generator(device="cuda")
    g.manual_seed(n_keys + N)
    q = torch.randn((L, 1, N, 4 * H_kv, d), device="cuda", generator=g).to(torch.bfloat16)
    ks = [torch.randn((n_keys, H_kv, d), device="cuda", generator=g) for _ in range(L)]
    cu = torch.tensor([0, n_keys], dtype=torch.int32, device="cuda")
    kw = dict(H_kv=H_kv, scale=d ** -0.5, exclusive_device=True)
    both = [dev.Scorer(q, [k.to(torch.bfloat16) for k in ks], cu, **kw), dev.Scorer(q, [k.to(torch.float8_e4m3fn).view(torch.uint8) for k in ks], cu, **kw)]
    want = [s.run().clone() for s in both]
    room = torch.empty(max(s.workspace.numel() for s in both), dtype=torch.uint8, device="cuda")
    for s in both:
        s.args.d_workspace, s.args.workspace_bytes = room.data_ptr(), room.numel()
    both[0].run()
    for i in (1, 0, 0, 1, 1, 0):
        both[i].args.flags = sp.SP_SCORE_EXCLUSIVE_DEVICE | sp.SP_SCORE_WORKSPACE_KEPT
        both[i].scores.fill_(-1.0)
        sp.sp_score(both[i].args, None)
        assert torch.equal(both[i].scores, want[i]), i
