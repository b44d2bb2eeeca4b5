"""GPU parity of the single-pass kernel for one long prompt (small teams of workgroups exchange row statistics;
SP_SCORE_EXCLUSIVE_DEVICE) against the fp64 oracle, element by element (Sec. 3.2 equation, Sec. 3.2.2), at the edges
of its cut into members, teams and units."""
import math

import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import helpers as hp
from tests import test_gpu_fp8_cache as fp8
from tests.test_gpu_batch_single_pass import _check

pytestmark = pytest.mark.gpu

MODES = [orc.LAYER_MAX, orc.LAYER_MEAN]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [
    dict(tokens=3073, L=4, H=32, H_kv=8, N=8, d=128),    # the shortest prompt: more members than the keys need, ...
    dict(tokens=3100, L=1, H=32, H_kv=8, N=8, d=64),     # ... so few slabs that most members have no keys at all
    dict(tokens=4097, L=32, H=8, H_kv=4, N=5, d=64),     # two heads padded to four, a member with one key
    dict(tokens=4096, L=24, H=48, H_kv=16, N=8, d=64),   # three heads padded to four, several slabs per unit, full members
    dict(tokens=6150, L=8, H=64, H_kv=8, N=4, d=128),    # eight heads per KV head
    dict(tokens=5000, L=6, H=40, H_kv=8, N=3, d=64),     # five heads padded to eight, units that do not divide evenly
    dict(tokens=9000, L=3, H=32, H_kv=8, N=1, d=128),    # one query
    dict(tokens=9000, L=1, H=16, H_kv=4, N=8, d=128),    # as many slabs as teams
    dict(tokens=16000, L=4, H=4, H_kv=1, N=8, d=128),
    dict(tokens=3100, L=1, H=4, H_kv=1, N=2, d=64),      # one slab: three of four teams idle, members without keys
    dict(tokens=33000, L=3, H=4, H_kv=1, N=8, d=64),
])
def test_one_long_prompt(shape, mode):
    shape = dict(shape)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), salient_run=1, **shape)
    inp = synth.make_qk(w)
    _check(w, inp, mode, max_seqlen=0, exclusive_device=True)
    if w.T == 4097:
        for page in (8, 64):
            _check(w, inp, mode, max_seqlen=0, paged=page)


def test_valid_query_count_and_head_major_cache():
    w = synth.scaled(synth.workload(3), seqlens=(7001,), L=5, H=16, H_kv=4, N=8, salient_run=1)
    inp = synth.make_qk(w)
    scale = 1.0 / math.sqrt(w.d)
    nv = np.array([3], dtype=np.int32)
    want, _ = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], scale, orc.LAYER_MAX, nv)
    for head_major in (False, True):
        got, _ = hp.gpu_score(inp["q"], inp["k"], inp["cu_seqlens"], w.H_kv, scale, orc.LAYER_MAX, n_valid=nv, head_major=head_major)
        hp.assert_scores_close(got, want, f"head_major={head_major}")


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("d, paged", [(64, 0), (128, 0), (64, 16), (128, 8)])
def test_8_bit_cache(d, paged, mode):
    w = synth.scaled(synth.workload(3), seqlens=(5003,), L=4, H=32, H_kv=8, N=8, d=d, salient_run=1)
    fp8._check(w, mode, False, paged=paged)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("d, paged", [(64, 0), (64, 16), (128, 8)])
def test_8_bit_cache_eight_heads_per_kv_head(d, paged, mode):
    w = synth.scaled(synth.workload(3), seqlens=(5003,), L=4, H=32, H_kv=4, N=4, d=d, salient_run=1)
    fp8._check(w, mode, False, paged=paged)


@pytest.mark.parametrize("d, bits, paged", [(128, 16, 0), (64, 16, 0), (128, 8, 0), (64, 8, 0), (128, 16, 16), (64, 16, 64), (64, 8, 16)])
@pytest.mark.parametrize("shape", [
    dict(tokens=33001, L=19, H=4, H_kv=1, N=8),    # eight teams: two rounds of whole layers, three layers left over
    dict(tokens=32801, L=10, H=8, H_kv=2, N=3),    # one round, two layers left over, cut in halves
    dict(tokens=66007, L=9, H=8, H_kv=1, N=2),     # four teams on two dies each, eight heads per KV head
])
def test_mean_over_whole_layers_and_left_over_parts(shape, d, bits, paged):
    """At least as many layers as teams: a team adds each of its layers to what it stored before (the read-back on whole
    and ragged slots of one, two and four tiles), the layers left over are merged from parts."""
    shape = dict(shape)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), d=d, salient_run=1, **shape)
    if bits == 8:
        fp8._check(w, orc.LAYER_MEAN, False, paged=paged)
    else:
        _check(w, synth.make_qk(w), orc.LAYER_MEAN, max_seqlen=0, paged=paged, exclusive_device=True)


@pytest.mark.parametrize("mode", MODES)
def test_kept_workspace_and_changed_inputs_over_consecutive_calls(mode):
    """Both copies of the exchange lines in turn, on other keys each time."""
    import torch
    from paper_2502_02789_amd import device as dev
    w = synth.scaled(synth.workload(3), seqlens=(4500,), L=4, H=32, H_kv=8, N=8, d=64, salient_run=1)
    inp = synth.make_qk(w)
    scale = 1.0 / math.sqrt(w.d)
    ks = [dev.bf16_from_bits(k) for k in inp["k"]]
    s = dev.Scorer(dev.bf16_from_bits(inp["q"]), ks, torch.from_numpy(np.asarray(inp["cu_seqlens"], dtype=np.int32)).cuda(),
                   H_kv=w.H_kv, scale=scale, layer_reduce=mode, keep_workspace=True)
    for turn in range(5):
        keys = [np.roll(k, 37 * turn, axis=0) for k in inp["k"]]
        for t, k in zip(ks, keys):
            t.copy_(dev.bf16_from_bits(k))
        want, _ = orc.token_importance(inp["q"], keys, inp["cu_seqlens"], scale, mode)
        s.scores.fill_(float("nan"))
        s.run()
        s.check()
        hp.assert_scores_close(s.scores.cpu().numpy(), want, f"call {turn}")


def test_kept_workspace_shared_by_two_kinds_of_cache():
    """SP_SCORE_WORKSPACE_KEPT asks for the same shape, not for the same kind of cache: calls on a bf16 and on an 8-bit
    cache take turns on one workspace (their results are cut differently, 40 groups and ten)."""
    import torch
    from paper_2502_02789_amd import binding as sp, device as dev
    w = synth.scaled(synth.workload(3), seqlens=(17000,), L=5, H=32, H_kv=8, N=1, d=64, salient_run=1)
    inp = synth.make_qk(w)
    scale = 1.0 / math.sqrt(w.d)
    codes, k_scale = synth.quantize_k_fp8(inp["k"])
    kw = dict(H_kv=w.H_kv, scale=scale, layer_reduce=orc.LAYER_MEAN)
    q, cu = dev.bf16_from_bits(inp["q"]), torch.from_numpy(np.asarray(inp["cu_seqlens"], dtype=np.int32)).cuda()
    both = [dev.Scorer(q, [dev.bf16_from_bits(k) for k in inp["k"]], cu, **kw),
            dev.Scorer(q, [torch.from_numpy(c).cuda() for c in codes], cu, k_scale=torch.from_numpy(k_scale).cuda(), **kw)]
    want = [orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], scale, orc.LAYER_MEAN)[0],
            orc.token_importance(inp["q"], codes, inp["cu_seqlens"], scale, orc.LAYER_MEAN, k_scale=k_scale)[0]]
    room = torch.empty(max(s.workspace.numel() for s in both), dtype=torch.uint8, device="cuda")
    for turn in range(6):
        s = both[turn % 2]
        s.args.d_workspace, s.args.workspace_bytes = room.data_ptr(), room.numel()
        s.args.flags = sp.SP_SCORE_EXCLUSIVE_DEVICE | (sp.SP_SCORE_WORKSPACE_KEPT if turn else 0)
        s.scores.fill_(float("nan"))
        sp.sp_score(s.args)
        sp.sp_score_check(s.args)
        hp.assert_scores_close(s.scores.cpu().numpy(), want[turn % 2], f"turn {turn}")


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [
    dict(tokens=9001, L=3, H=8, H_kv=4, N=12, d=128),      # two heads per KV head
    dict(tokens=8193, L=4, H=4, H_kv=4, N=9, d=128),       # one
    dict(tokens=5003, L=2, H=16, H_kv=8, N=16, d=64),      # two tiles per slot; all 32 columns
    dict(tokens=20001, L=9, H=2, H_kv=1, N=13, d=128),     # 32 members, eight teams: whole layers and a part (mean)
    dict(tokens=17000, L=9, H=4, H_kv=2, N=16, d=64),      # ... with ragged slots of two tiles
    dict(tokens=100, L=4, H=8, H_kv=4, N=9, d=128),        # shorter than a member
])
def test_more_than_eight_queries(shape, mode):
    """One or two heads per KV head with nine to sixteen queries: the heads padded to two, four 32-key tiles per wave."""
    shape = dict(shape)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), salient_run=1, **shape)
    inp = synth.make_qk(w)
    nv = np.array([w.N - 2], dtype=np.int32)
    _check(w, inp, mode, max_seqlen=0, n_valid=nv, exclusive_device=True)
    _check(w, inp, mode, max_seqlen=0, paged=16)
    if w.T < 10000:
        fp8._check(w, mode, False, paged=0)
        fp8._check(w, mode, False, n_valid=nv, paged=16)
