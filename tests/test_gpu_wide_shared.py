"""One long prompt without SP_SCORE_EXCLUSIVE_DEVICE: the teams of workgroups run without the promise of an idle device,
and a call whose waits give up completes itself in its second launch (Sec. 3.2 equation, Sec. 3.2.2)."""
import math

import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def _scorer(w, inp, mode, bits=16, page=0, n_valid=None, exclusive_device=False):
    import torch
    from paper_2502_02789_amd import device as dev
    kw, k, k_scale = {}, inp["k"], None
    if bits == 8:
        k, k_scale = synth.quantize_k_fp8(k)
        k_scale = torch.from_numpy(np.ascontiguousarray(k_scale)).cuda()
    if page:
        k, table = hp.paged_copy(k, inp["cu_seqlens"], page, seed=page, fill=0x7E if bits == 8 else 0x7F00)
        kw = dict(block_table=torch.from_numpy(table).cuda(), page_size=page, total_tokens=w.T)
    ks = [torch.from_numpy(x).cuda() if bits == 8 else dev.bf16_from_bits(x) for x in k]
    nv = None if n_valid is None else torch.tensor([n_valid], dtype=torch.int32).cuda()
    return dev.Scorer(dev.bf16_from_bits(inp["q"]), ks, torch.tensor([0, w.T], dtype=torch.int32).cuda(), H_kv=w.H_kv,
                      scale=1.0 / math.sqrt(w.d), layer_reduce=mode, want_lse=True, n_valid=nv, k_scale=k_scale,
                      exclusive_device=exclusive_device, **kw)


@pytest.mark.parametrize("shape, opt", [
    (dict(tokens=3073, L=4, N=8), {}),                                       # members with next to no keys, few slabs
    (dict(tokens=4097, L=24, H=8, H_kv=4, N=5, d=64), dict(page=16)),        # one key in the last piece
    (dict(tokens=6150, L=8, H=64, H_kv=8, N=4), dict(mode=orc.LAYER_MEAN)),  # whole layers and parts of layers
    (dict(tokens=9000, L=3, H=16, H_kv=4, N=1), dict(mode=orc.LAYER_MEAN)),  # few rows: logits were kept in memory
    (dict(tokens=5003, L=36, N=8, d=64), dict(mode=orc.LAYER_MEAN, bits=8)),
    (dict(tokens=16385, L=2, N=2, H=8, H_kv=8), dict(bits=8, page=64)),
    (dict(tokens=7001, L=5, H=8, H_kv=4, N=12), dict(n_valid=7)),            # heads padded to two columns
    (dict(tokens=40000, L=1, H=4, H_kv=1, N=8, d=64), {}),                   # members without keys: nobody to wait for them
])
def test_a_call_whose_waits_give_up_completes_itself(shape, opt):
    """The same bits whether every wait is answered (bound as it is), none (bound 0: the second launch does the work) or
    the device is promised exclusive; the plain kernels' scores and log-sum-exps to tolerance."""
    from paper_2502_02789_amd import binding as sp
    shape, opt = dict(shape), dict(opt)
    mode = opt.pop("mode", orc.LAYER_MAX)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), salient_run=1, **shape)
    inp = synth.make_qk(w)
    s = _scorer(w, inp, mode, **opt)

    def call(**kw):
        s.scores.fill_(float("nan"))
        s.lse.fill_(float("nan"))
        s.run(**kw)
        s.check()                                   # (a call without the flag never reports a time-out)
        return s.scores.cpu().numpy(), s.lse.cpu().numpy()

    want, want_lse = call(general=True)
    first = call()
    hp.assert_scores_close(first[0], want, f"{w.name} {opt}")
    np.testing.assert_allclose(first[1], want_lse, rtol=0, atol=2e-4)
    before = sp.sp_set_wait_budget(0)
    try:
        runs = [call(), call()]
    finally:
        sp.sp_set_wait_budget(before)
    runs.append(call())
    e = _scorer(w, inp, mode, exclusive_device=True, **opt)
    e.run()
    e.check()
    runs.append((e.scores.cpu().numpy(), e.lse.cpu().numpy()))
    for scores, lse in runs:
        assert np.array_equal(scores, first[0]) and np.array_equal(lse, first[1])


@pytest.mark.parametrize("shape, opt", [
    (dict(tokens=9000, L=8, N=8), {}),
    (dict(tokens=6150, L=12, H=64, H_kv=8, N=4), dict(mode=orc.LAYER_MEAN)),          # parts of layers
    (dict(tokens=5003, L=75, H=8, H_kv=2, N=8, d=64), dict(mode=orc.LAYER_MEAN, bits=8)),   # sums over layers, then parts
    (dict(tokens=40000, L=1, H=4, H_kv=1, N=8, d=64), {}),                            # members without keys
])
def test_a_call_some_of_whose_waits_give_up_completes_itself(shape, opt):
    """Few looks allowed: some workgroups get their team's lines, others give up, in the first slab or a later one, with
    valid slabs folded and sums written; the same bits as with every wait answered."""
    from paper_2502_02789_amd import binding as sp
    shape, opt = dict(shape), dict(opt)
    mode = opt.pop("mode", orc.LAYER_MAX)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), salient_run=1, **shape)
    s = _scorer(w, synth.make_qk(w), mode, **opt)

    def call():
        s.scores.fill_(float("nan"))
        s.lse.fill_(float("nan"))
        s.run()
        s.check()
        return s.scores.cpu().numpy(), s.lse.cpu().numpy()

    want = call()
    assert np.isfinite(want[0]).all()
    for looks in (1, 2, 3, 5, 10, 20, 50):
        before = sp.sp_set_wait_budget(looks)
        try:
            runs = [call() for _ in range(3)]
        finally:
            sp.sp_set_wait_budget(before)
        for scores, lse in runs:
            assert np.array_equal(scores, want[0]) and np.array_equal(lse, want[1]), looks


@pytest.mark.parametrize("mode", [orc.LAYER_MAX, orc.LAYER_MEAN])
@pytest.mark.parametrize("shape", [
    dict(tokens=3073, L=4, H=32, H_kv=8, N=8, d=128),    # one key more than the kernel for whole sequences holds
    dict(tokens=4096, L=2, H=16, H_kv=4, N=8, d=64),     # full shares
    dict(tokens=4097, L=3, H=6, H_kv=2, N=5, d=128),     # three heads padded to four
    dict(tokens=12345, L=2, H=64, H_kv=8, N=4, d=64),    # eight heads per KV head
    dict(tokens=8225, L=5, H=8, H_kv=1, N=3, d=128),     # few slabs, ragged shares
    dict(tokens=5001, L=3, H=4, H_kv=1, N=8, d=64),      # results that outweigh the keys
])
def test_one_prompt_on_a_shared_device(shape, mode):
    """The teams against the oracle."""
    shape = dict(shape)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), salient_run=1, **shape)
    inp = synth.make_qk(w)
    want, want_lse = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], 1.0 / math.sqrt(w.d), mode)
    got, lse = hp.gpu_score(inp["q"], inp["k"], inp["cu_seqlens"], w.H_kv, 1.0 / math.sqrt(w.d), mode, exclusive_device=False)
    hp.assert_scores_close(got, want, f"{w.name} mode={mode}")
    np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-4)


def test_calls_on_four_streams_at_once():
    """Four calls in flight together, each with a workspace of its own, more workgroups than the device holds."""
    import torch
    w = synth.scaled(synth.workload(3), seqlens=(20000,), L=4, salient_run=1)
    inp = synth.make_qk(w)
    calls = [(_scorer(w, dict(inp, q=np.roll(inp["q"], i, axis=0)), orc.LAYER_MAX), torch.cuda.Stream()) for i in range(4)]
    want = []
    for s, _ in calls:
        s.run()
        torch.cuda.synchronize()
        want.append(s.scores.clone())
        s.scores.fill_(float("nan"))
    torch.cuda.synchronize()
    for _ in range(6):
        for s, stream in calls:
            with torch.cuda.stream(stream):
                s.run()
    torch.cuda.synchronize()
    for (s, _), x in zip(calls, want):
        assert torch.equal(s.scores, x)


@pytest.mark.parametrize("mode", [orc.LAYER_MAX, orc.LAYER_MEAN])
@pytest.mark.parametrize("shape", [dict(tokens=3072, L=7, N=8), dict(tokens=2051, L=5, H=16, H_kv=2, N=4, d=64)])
def test_short_prompts_of_few_slabs_stay_on_two_passes(shape, mode):
    """One sequence on the two-pass kernels: up to 3072 keys and fewer than 64 slabs, against the oracle."""
    shape = dict(shape)
    w = synth.scaled(synth.workload(3), seqlens=(shape.pop("tokens"),), salient_run=1, **shape)
    inp = synth.make_qk(w)
    want, want_lse = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], 1.0 / math.sqrt(w.d), mode)
    got, lse = hp.gpu_score(inp["q"], inp["k"], inp["cu_seqlens"], w.H_kv, 1.0 / math.sqrt(w.d), mode, exclusive_device=False)
    hp.assert_scores_close(got, want, f"{w.name} mode={mode}")
    np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-4)


def test_other_work_on_most_compute_units_does_not_hold_a_call_up():
    """200 compute units held by another stream leave no team of sixteen complete: the call must give up waiting as a
    whole and soon.  256 workgroups on 56 compute units are five rounds, and both launches work: ten times the undisturbed
    call, and the wait.  (Measured 10 times; 36 when every workgroup waited out a bound of its own.)"""
    import torch
    from paper_2502_02789_amd import binding as sp, device as dev, probe
    T, L, H, H_kv, d = 9000, 32, 32, 8, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q = torch.randn((L, 1, 8, H, d), generator=g, device="cuda").to(torch.bfloat16)
    k = [torch.randn((T, H_kv, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(L)]
    s = dev.Scorer(q, k, torch.tensor([0, T], dtype=torch.int32, device="cuda"), H_kv=H_kv, scale=1.0 / math.sqrt(d),
                   layer_reduce=sp.SP_LAYER_MAX, exclusive_device=False)
    lib, other = probe.load_library(), torch.cuda.Stream()
    start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))

    def call(held):
        torch.cuda.synchronize()
        s.scores.fill_(float("nan"))
        if held:
            assert lib.sp_probe_occupy(held, 65536, 30000, other.cuda_stream) == 0
        torch.cuda._sleep(200000)
        start.record()
        s.run()
        end.record()
        end.synchronize()
        assert not held or not other.query()                        # (the other work is still there)
        torch.cuda.synchronize()
        return start.elapsed_time(end), s.scores.cpu().numpy()

    call(0)
    alone = sorted((call(0) for _ in range(5)), key=lambda x: x[0])[2]
    beside = sorted((call(200) for _ in range(3)), key=lambda x: x[0])[1]
    assert np.array_equal(beside[1], alone[1])
    assert beside[0] < 20 * alone[0], (beside[0], alone[0])


@pytest.mark.parametrize("tokens", [3073, 9001, 16383])
@pytest.mark.parametrize("L, H, H_kv, N", [(1, 4, 1, 1), (2, 4, 1, 8), (1, 8, 2, 8), (8, 16, 4, 1), (11, 3, 1, 3)])
@pytest.mark.parametrize("mode", [orc.LAYER_MAX, orc.LAYER_MEAN])
def test_merge_of_few_results(tokens, L, H, H_kv, N, mode):
    """One to 33 rows of results a tile: on both sides of what a small workgroup of the merge reads in one step."""
    w = synth.scaled(synth.workload(3), seqlens=(tokens,), salient_run=1, L=L, H=H, H_kv=H_kv, N=N, d=64)
    inp = synth.make_qk(w)
    want, want_lse = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], 1.0 / math.sqrt(w.d), mode)
    got, lse = hp.gpu_score(inp["q"], inp["k"], inp["cu_seqlens"], w.H_kv, 1.0 / math.sqrt(w.d), mode, exclusive_device=False)
    hp.assert_scores_close(got, want, f"{w.name} mode={mode}")
    np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-4)
