"""How long a call without the promise of an idle device waits for the members of a team (sp_wide_team_plan.h), on the CPU: at
least a pass over the keys at the pace a compute unit streams them undisturbed, so that teams that are done can make room
for members that are kept out, and no more than three (and the tail of another stream's kernel), so that waiting never
costs much more than giving up does."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

from paper_2502_02789_amd import binding as sp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "sp_wide_team_plan.h"
extern "C" int patience(const sp_score_args* a, int wgs, long long* us, int* slabs, int* chunk) {
  const sp::WideTeamPlan pl = sp::make_wide_team_plan(a, wgs);
  if (!pl.ok) return 0;
  *us = sp::wide_team_patience_us(pl, a);
  *slabs = (pl.deal.n_slabs + pl.deal.teams - 1) / pl.deal.teams;
  *chunk = pl.chunk;
  return 1;
}
"""


@pytest.mark.parametrize("wgs", [256, 128, 32])
@pytest.mark.parametrize("bits", [16, 8])
def test_between_one_and_three_passes(tmp_path, wgs, bits):
    cxx = shutil.which("g++") or shutil.which("c++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    (tmp_path / "shim.cpp").write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2502_02789_amd", "csrc"), "shim.cpp", "-o", "shim.so"], cwd=tmp_path, check=True)
    lib = C.CDLL(str(tmp_path / "shim.so"))
    rng = random.Random(11)
    seen = 0
    for _ in range(400):
        a = sp.ScoreArgs()
        for k, v in dict(B=1, N=8, L=rng.randint(1, 128), H=32, H_kv=8, d=rng.choice([64, 128]), T=int(3073 * 43 ** rng.random()),
                         k_dtype=sp.SP_K_FP8_E4M3 if bits == 8 else sp.SP_K_BF16, layer_reduce=rng.choice([0, 1])).items():
            setattr(a, k, v)
        us, slabs, chunk = C.c_longlong(), C.c_int(), C.c_int()
        if not lib.patience(C.byref(a), wgs, C.byref(us), C.byref(slabs), C.byref(chunk)):
            continue
        seen += 1
        # undisturbed: 25 KB a us and workgroup (8-bit keys 19, which arithmetic holds up), 1.7 us for the end of a slab
        call = slabs.value * (1.7 + chunk.value * a.d * bits / 8 / (25e3 if bits == 16 else 19e3))
        assert call < us.value < 60 + 3 * call, (a.T, a.L, a.d, us.value, call)
    assert seen > 100
