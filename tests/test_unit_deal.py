"""The even cut of a batch's slabs among the workgroups (sp_unit_deal.h), on the CPU: the stretches as the kernel walks over
them take every grain of every sequence once, in order; the results of a sequence are numbered without gaps and fit what is
laid out for them; no workgroup has more than its share by more than a grain of the longest sequence it meets."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

from paper_2502_02789_amd import binding as sp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "sp_unit_deal.h"
extern "C" int deal(const sp_score_args* a, int W, int limit, int whole, long* stretch, int* grains, int* extra) {
  int n = 0;
  const sp::UnitDeal d = sp::make_unit_deal(a, W, limit, whole != 0, &n);
  *stretch = d.stretch; *grains = d.grains; *extra = d.extra;
  return n;
}
// stretch [first, end) of workgroup w in sequence b, and the workgroup of its first grain
extern "C" void stretch_of(const sp_score_args* a, int W, int limit, int whole, int w, int b, int cu_b, int M, int* out) {
  int n = 0;
  const sp::UnitDeal d = sp::make_unit_deal(a, W, limit, whole != 0, &n);
  const long at = d.start(cu_b, b), c = d.cost(M);
  out[0] = d.first_grain(w, at, c); out[1] = d.first_grain(w + 1, at, c); out[2] = d.owner(at, c, 0);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    path = tmp_path_factory.mktemp("deal")
    cxx = shutil.which("g++") or shutil.which("c++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    (path / "shim.cpp").write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2502_02789_amd", "csrc"), "shim.cpp", "-o", "shim.so"], cwd=path, check=True)
    return C.CDLL(str(path / "shim.so"))


def _cases():
    rng = random.Random(7)
    for _ in range(60):
        B = rng.choice([1, 2, 5, 16, 22, 64, 100])
        hi = rng.randint(200, 3072)
        lens = [rng.choice([0, 1, rng.randint(1, hi), rng.randint(hi // 2, hi), hi]) for _ in range(B)]
        yield lens, hi, rng.choice([8, 16, 32, 80, 128]), rng.choice([1, 4, 8]), rng.choice([64, 128]), rng.choice([0, 1]), rng.choice([256, 304, 64])


@pytest.mark.parametrize("whole", [0, 1])
def test_every_grain_once(lib, whole):
    dealt = 0
    for lens, hi, L, H_kv, d, fp8, W in _cases():
        B, T, limit = len(lens), sum(lens), 3072
        a = sp.ScoreArgs()
        for k, v in dict(B=B, N=8, L=L, H=4 * H_kv, H_kv=H_kv, d=d, T=T, max_seqlen=hi, k_dtype=fp8).items():
            setattr(a, k, v)
        stretch, grains, extra = C.c_long(), C.c_int(), C.c_int()
        n_groups = lib.deal(C.byref(a), W, limit, whole, C.byref(stretch), C.byref(grains), C.byref(extra))
        if stretch.value == 0:
            continue
        dealt += 1
        assert grains.value == (L if whole else L * H_kv)
        cu = [0]
        for m in lens:
            cu.append(cu[-1] + m)
        taken, groups, load = [0] * B, [0] * B, [0] * W
        out = (C.c_int * 3)()
        for w in range(W):
            for b in range(B):
                lib.stretch_of(C.byref(a), W, limit, whole, w, b, cu[b], lens[b], out)
                g0, g1, first = out
                assert 0 <= g0 <= g1 <= grains.value
                load[w] += 2 * (g1 - g0) * (lens[b] + extra.value)
                if g0 == g1:
                    assert not 0 < g0 < grains.value    # nobody in the middle of a sequence without a grain of it
                    continue
                assert g0 == taken[b] and w - first == groups[b]  # in order, numbered without gaps
                taken[b], groups[b] = g1, groups[b] + 1
        assert taken == [grains.value] * B
        assert max(groups) <= n_groups <= W
        assert max(load) <= stretch.value + 2 * (max(lens) + extra.value)
    assert dealt >= 10 if not whole else dealt >= 3


def _stretch(lib, lens, L, H_kv, longest=0, fp8=0, d=128, N=8, limit=3072, W=256):
    a = sp.ScoreArgs()
    for k, v in dict(B=len(lens), N=N, L=L, H=4 * H_kv, H_kv=H_kv, d=d, T=sum(lens), max_seqlen=longest or max(lens), k_dtype=fp8).items():
        setattr(a, k, v)
    stretch, grains, extra = C.c_long(), C.c_int(), C.c_int()
    lib.deal(C.byref(a), W, limit, 0, C.byref(stretch), C.byref(grains), C.byref(extra))
    return stretch.value


@pytest.mark.parametrize("fp8", [0, 1])
@pytest.mark.parametrize("B, lo, hi, stretches", [
    (32, 200, 1000, False), (64, 100, 700, False), (96, 64, 308, False), (128, 72, 268, False),  # whole rounds of short prompts
    (40, 100, 700, True), (48, 200, 1000, True), (100, 100, 300, True), (22, 1400, 2100, True),   # a round partly filled
    (16, 300, 3000, True), (8, 200, 1277, True), (64, 1024, 3072, True), (32, 1000, 1500, True)])  # few prompts, long ones
def test_whole_rounds_of_short_prompts_stay_rounds(lib, B, lo, hi, stretches, fp8):
    rng = random.Random(B)
    lens = [hi] + [rng.randint(lo, hi) for _ in range(B - 1)]
    assert (_stretch(lib, lens, 32, 8, fp8=fp8) != 0) == stretches
    assert (_stretch(lib, lens, 32, 8, fp8=fp8, d=64) != 0) == (stretches or B < 96)  # (a slab takes half the time)


@pytest.mark.parametrize("L, stretches", [(32, False), (33, False), (36, False), (47, False), (48, True), (64, True)])
def test_one_sequence_is_cut_into_stretches_from_three_slabs_for_two_workgroups_on(lib, L, stretches):
    assert (_stretch(lib, [2300], L, 8) != 0) == stretches
