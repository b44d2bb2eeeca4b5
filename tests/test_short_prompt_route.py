"""Which kernel one prompt of 2048 to 3072 keys takes on an idle device (no GPU needed: the size of the workspace shows it): a workgroup
to a slab as without the promise, or two."""
import ctypes as C

import pytest

from paper_2502_02789_amd import binding as sp


def _bytes(flags, **kw):
    a = sp.ScoreArgs()
    for k, v in dict(dict(B=1, N=8, L=32, H_kv=8, d=128, T=2048, page_size=0, flags=flags, k_token_stride=1024, k_head_stride=128), **kw).items():
        setattr(a, k, v)
    a.H = 4 * a.H_kv
    return sp.load_library().sp_score_workspace_bytes(C.byref(a))


FP8, MEAN = dict(k_dtype=sp.SP_K_FP8_E4M3), dict(layer_reduce=sp.SP_LAYER_MEAN)


@pytest.mark.parametrize("cache", [{}, FP8])
@pytest.mark.parametrize("two, shape", [
    (True, {}), (True, MEAN), (True, dict(T=3072)), (False, dict(N=4, T=2500)), (False, dict(N=6)),  # every round full both ways
    (False, dict(d=64)), (True, dict(d=64, T=2800)),
    (False, dict(L=24)), (False, dict(L=24, T=3072)), (False, dict(L=24, N=4, T=2500)), (False, dict(L=28, d=64)), (False, dict(L=17)),  # a round more
    (True, dict(L=16)), (True, dict(L=16, **MEAN)), (True, dict(L=36)), (True, dict(L=48)),  # half a round saved
    (False, dict(L=36, **MEAN)), (False, dict(L=40, N=4, **MEAN)),
    (False, dict(L=16, d=64)), (False, dict(L=16, d=64, T=2350, **MEAN)), (True, dict(L=16, d=64, T=2400)),
    (False, dict(T=2047)), (False, dict(L=15)), (False, dict(L=8))])
def test_two_workgroups_to_a_slab(two, shape, cache):
    """The same way for both kinds of cache and whether or not the workspace is kept: a workspace that one such call leaves may be handed to
    another as kept."""
    promised, not_promised = _bytes(sp.SP_SCORE_EXCLUSIVE_DEVICE, **shape, **cache), _bytes(0, **shape, **cache)
    assert promised > 0 and not_promised > 0
    assert (promised != not_promised) == two
    assert _bytes(sp.SP_SCORE_EXCLUSIVE_DEVICE | sp.SP_SCORE_WORKSPACE_KEPT, **shape, **cache) == promised
