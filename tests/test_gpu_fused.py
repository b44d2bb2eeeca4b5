"""GPU parity of sp_score_pool_select (one short prompt scored and selected in a single launch)
against the oracle, and against the separate calls."""
import ctypes as C
import math

import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def _run_fused(w, inp, mode, chunk, window, rate, n_valid=None, head_major=False):
    import torch
    from paper_2502_02789_amd import device as dev
    q = dev.bf16_from_bits(inp["q"])
    if head_major:
        ks = [dev.bf16_from_bits(np.ascontiguousarray(k.transpose(1, 0, 2))).permute(1, 0, 2) for k in inp["k"]]
    else:
        ks = [dev.bf16_from_bits(k) for k in inp["k"]]
    cu = torch.from_numpy(inp["cu_seqlens"]).cuda()
    nv = None if n_valid is None else torch.tensor([n_valid], dtype=torch.int32, device="cuda")
    s = dev.Scorer(q, ks, cu, H_kv=w.H_kv, scale=1.0 / math.sqrt(w.d), layer_reduce=mode, n_valid=nv, want_lse=True)
    sel = dev.Selector(s.scores, cu, chunk=chunk, pool_window=window, keep_rate=rate, want_chunk_scores=True)
    s.scores.fill_(float("nan"))
    dev.score_pool_select(s, sel)
    torch.cuda.synchronize()
    return s, sel


@pytest.mark.parametrize("mode", [orc.LAYER_MAX, orc.LAYER_MEAN])
@pytest.mark.parametrize("case", [
    dict(number=1),                                                    # the tiny workload as it is
    dict(number=1, seqlens=(2048,), L=3),                              # as many keys as one workgroup takes
    dict(number=1, seqlens=(1,)),                                      # a single key
    dict(number=1, seqlens=(1333,), H=8, H_kv=2, N=2, n_valid=1),      # eight rows per KV head, one valid query
    dict(number=3, seqlens=(777,), L=2, H=8, H_kv=8, N=8, n_valid=5),  # head dim 128, one head per KV head
    dict(number=1, seqlens=(1100,), H=8, H_kv=1, N=2, n_valid=2),      # sixteen rows: every column of the operand
    dict(number=3, seqlens=(2000,), L=2, H=4, H_kv=2, N=3, n_valid=2), # head dim 128, six rows
    dict(number=1, seqlens=(333,), L=5, H=6, H_kv=2, N=4, n_valid=3),  # three heads per KV head, more pairs than waves take at once
    dict(number=1, seqlens=(600,), H=4, H_kv=1, N=1, chunk=1, window=1, rate=0.1),   # the raw variant
    dict(number=1, seqlens=(1500,), chunk=48, window=7, rate=0.33, head_major=True),
])
def test_fused_short_prompt_against_oracle(case, mode):
    case = dict(case)
    number = case.pop("number")
    n_valid = case.pop("n_valid", None)
    head_major = case.pop("head_major", False)
    base = synth.workload(number)
    chunk, window, rate = case.pop("chunk", base.chunk), case.pop("window", base.pool_window), case.pop("rate", base.keep_rate)
    w = synth.scaled(base, salient_frac=0.02, salient_run=1, **case) if case else base
    inp = synth.make_qk(w)
    scale = 1.0 / math.sqrt(w.d)
    nv = None if n_valid is None else np.array([n_valid], dtype=np.int32)
    want, want_lse = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], scale, mode, nv)
    s, sel = _run_fused(w, inp, mode, chunk, window, rate, n_valid, head_major)
    got = s.scores.cpu().numpy()
    hp.assert_scores_close(got, want, f"fused {w.name} {case} mode={mode}")
    np.testing.assert_allclose(s.lse.cpu().numpy(), want_lse, rtol=0, atol=2e-4)
    # stage-isolated: the oracle's selection on these very scores must be identical
    kept_o, cu_keep_o, cs_o, _ = orc.pool_select(got, inp["cu_seqlens"], chunk, window, rate)
    n = int(sel.cu_keep[1])
    assert sel.cu_keep.cpu().tolist() == cu_keep_o.tolist()
    assert (sel.kept_idx[:n].cpu().numpy() == kept_o).all() and (sel.kept_idx[n:] == -1).all()
    np.testing.assert_array_equal(sel.chunk_scores.cpu().numpy()[:len(cs_o)], cs_o.astype(np.float32))
    # end to end against the oracle's own scores: differences only inside the tolerance window
    hp.selection_matches(sel.kept_idx[:n].cpu().numpy(), sel.cu_keep.cpu().numpy(), want, inp["cu_seqlens"], chunk,
                         window, rate, hp.SCORE_RTOL)


@pytest.mark.parametrize("chunk", [1, 4, 15, 16, 32, 1023, 2 ** 31 - 500, 2 ** 31 - 1])
@pytest.mark.parametrize("d", [64, 128])
def test_forms_of_ranking_and_long_chunks(chunk, d):
    """1000 and 1024 tokens in 1000 chunks to one, ranked by classes, by counting and by one wave; chunks longer than the prompt."""
    for T in (1000, 1024):
        w = synth.scaled(synth.workload(1), seqlens=(T,), d=d, salient_frac=0.02, salient_run=1)
        s, sel = _run_fused(w, synth.make_qk(w), orc.LAYER_MAX, chunk, 5, 0.3)
        got = s.scores.cpu().numpy()
        kept, cu_keep, cs, _ = orc.pool_select(got, np.array([0, T], dtype=np.int32), min(chunk, T), 5, 0.3)
        assert sel.cu_keep.cpu().tolist() == cu_keep.tolist()
        np.testing.assert_allclose(sel.chunk_scores.cpu().numpy()[:len(cs)], cs.astype(np.float32), rtol=2e-7)
        hp.selection_matches(sel.kept_idx.cpu().numpy()[:len(kept)], cu_keep, got, np.array([0, T], dtype=np.int32), min(chunk, T), 5, 0.3, 1e-12)


def test_fused_equals_the_separate_calls():
    import torch
    from paper_2502_02789_amd import device as dev
    w = synth.workload(1)
    inp = synth.make_qk(w)
    s, sel = _run_fused(w, inp, orc.LAYER_MAX, w.chunk, w.pool_window, w.keep_rate)
    fused_scores = s.scores.clone()
    fused_kept = sel.kept_idx.clone()
    s.run()
    sel.run()
    torch.cuda.synchronize()
    np.testing.assert_allclose(fused_scores.cpu().numpy(), s.scores.cpu().numpy(), rtol=1e-4, atol=1e-12)
    assert (fused_kept == sel.kept_idx).all()


def test_fused_refuses_what_one_workgroup_cannot_hold():
    import torch
    from paper_2502_02789_amd import binding as sp, device as dev
    lib = sp.load_library()
    for changes in (dict(seqlens=(2049,)), dict(seqlens=(300, 200)), dict(seqlens=(500,), H=8, H_kv=1, N=3),
                    dict(seqlens=(500,), N=9)):
        w = synth.scaled(synth.workload(1), **changes)
        inp = synth.make_qk(w)
        q = dev.bf16_from_bits(inp["q"])
        ks = [dev.bf16_from_bits(k) for k in inp["k"]]
        cu = torch.from_numpy(inp["cu_seqlens"]).cuda()
        s = dev.Scorer(q, ks, cu, H_kv=w.H_kv, scale=0.125)
        sel = dev.Selector(s.scores, cu, chunk=32, pool_window=13, keep_rate=0.25)
        s.scores.fill_(-3.0)
        assert lib.sp_score_pool_select(C.byref(s.args), C.byref(sel.args), None) == sp.SP_EUNSUPPORTED, changes
        torch.cuda.synchronize()
        assert (s.scores == -3.0).all() and (sel.kept_idx == -1).all()
    # mismatched halves are an argument error
    w = synth.workload(1)
    inp = synth.make_qk(w)
    cu = torch.from_numpy(inp["cu_seqlens"]).cuda()
    s = dev.Scorer(dev.bf16_from_bits(inp["q"]), [dev.bf16_from_bits(k) for k in inp["k"]], cu, H_kv=w.H_kv, scale=0.125)
    other = torch.zeros(w.T, dtype=torch.float32, device="cuda")
    sel = dev.Selector(other, cu, chunk=32, pool_window=13, keep_rate=0.25)
    assert lib.sp_score_pool_select(C.byref(s.args), C.byref(sel.args), None) == sp.SP_EINVAL


@pytest.mark.parametrize("mode", [orc.LAYER_MAX, orc.LAYER_MEAN])
@pytest.mark.parametrize("N", [1, 2])
def test_probabilities_in_the_subnormal_range(N, mode):
    """One key takes all the attention, the others are 88 to 100 below it: probabilities of 6e-39 to 2e-44, which fp32 has with
    fewer bits, but has; the kept tokens are those with the largest, not the first ones."""
    w = synth.scaled(synth.workload(1), seqlens=(200,), H=4, H_kv=1, N=N, d=64, salient_frac=0.02, salient_run=1)
    inp = synth.make_qk(w)
    bits = lambda x: (np.float32(x).view(np.uint32) >> 16).astype(np.uint16)  # (of values that bf16 has)
    inp["q"][:] = 0
    inp["q"][..., 0], inp["q"][..., 1] = bits(8.0), bits(0.5)                # times 1 / sqrt(d): 1 and 1 / 16
    below = np.arange(w.T)[::-1].astype(np.float32)
    for k in inp["k"]:
        k[:] = 0
        k[1:, :, 0] = bits(-88.0)
        k[1:, :, 1] = bits(-below)[1:, None]
    want, _ = orc.token_importance(inp["q"], inp["k"], inp["cu_seqlens"], 1.0 / math.sqrt(w.d), mode)
    assert 1e-44 < want.min() and want[1:].max() < 1.1e-38
    s, sel = _run_fused(w, inp, mode, 1, 1, 0.3)
    got = s.scores.cpu().numpy().astype(np.float64)
    # 2^-149 is the spacing there: half of it a probability, half again the average over layers and queries; logits of 145 in
    # base 2 rounded to 2^-24
    np.testing.assert_allclose(got, want, rtol=2e-5, atol=1.5 * 2.0 ** -149)
    assert sel.kept_idx[:60].cpu().tolist() == [0] + list(range(141, 200))
