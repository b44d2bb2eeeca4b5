"""GPU: finite queries and keys whose product does not fit fp32 (a logit of -inf, as a key that is meant to be ignored has)
on every route of sp_score, against the fp64 oracle (Sec. 3.2 equation, Sec. 3.2.2): such a key has probability 0 and
takes nothing from the others, wherever it sits in a lane's, a wave's or a workgroup's share of the keys."""
import math

import numpy as np
import pytest

from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import synth
from tests import helpers as hp

pytestmark = pytest.mark.gpu

BF16_1E25, BF16_MINUS_1E25 = 0x6904, 0xE904


@pytest.mark.parametrize("ignored", ["first", "last", "middle"])
@pytest.mark.parametrize("route", [
    dict(lens=(3000,), L=8, H=32, H_kv=8, N=8, d=128),                                # whole sequence in a workgroup, 32 columns
    dict(lens=(3000,), L=8, H=32, H_kv=8, N=8, d=64),
    dict(lens=(5000,), L=4, H=32, H_kv=8, N=8, d=128),                                # teams of workgroups
    dict(lens=(5000,), L=4, H=32, H_kv=8, N=8, d=64),
    dict(lens=(5000,), L=4, H=32, H_kv=8, N=8, d=128, exclusive_device=False),        # teams without the promise of an idle device
    dict(lens=(3000,), L=4, H=32, H_kv=8, N=8, d=128, exclusive_device=False),        # two passes, query tile once per workgroup
    dict(lens=(5000, 700), L=4, H=32, H_kv=8, N=8, d=64, max_seqlen=5000),
    dict(lens=(2500, 700) * 8, L=8, H=8, H_kv=2, N=1, d=128, max_seqlen=2500),        # whole sequence in a workgroup, four rows
    dict(lens=(5000, 700), L=2, H=32, H_kv=8, N=8, d=128),                            # two passes over tiles
    dict(lens=(5000, 700), L=2, H=32, H_kv=8, N=1, d=128),                            # kept logits
    dict(lens=(5000, 700), L=2, H=8, H_kv=2, N=2, d=64, general=True),                # the plain kernels
])
def test_keys_whose_logits_overflow(route, ignored):
    r = dict(route)
    lens, kw = r.pop("lens"), {k: r.pop(k) for k in ("exclusive_device", "max_seqlen", "general") if k in r}
    w = synth.scaled(synth.workload(4), seqlens=lens, salient_frac=0.02, salient_run=1, **r)
    inp = synth.make_qk(w)
    inp["q"][..., 0] = BF16_1E25
    cu = np.asarray(inp["cu_seqlens"])
    for k in inp["k"]:
        k[..., 0] = 0
        for b, m in enumerate(lens):
            lo, hi = dict(first=(0, 2 * m // 3), last=(m // 3, m), middle=(m // 5, 4 * m // 5))[ignored]
            k[cu[b] + lo:cu[b] + hi, :, 0] = BF16_MINUS_1E25
    scale = 1.0 / math.sqrt(w.d)
    want, want_lse = orc.token_importance(inp["q"], inp["k"], cu, scale, orc.LAYER_MAX)
    got, lse = hp.gpu_score(inp["q"], inp["k"], cu, w.H_kv, scale, orc.LAYER_MAX, **kw)
    hp.assert_scores_close(got, want, f"{route} {ignored}")
    np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-4)
