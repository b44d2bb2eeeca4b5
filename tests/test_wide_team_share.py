"""The members' keys in the cut of one long prompt (sp_wide_team_plan.h), on the CPU: whole 32-key tiles that cover the prompt
and fit what a member has room for, no member but the last ones short of any."""
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
extern "C" void plan(const sp_score_args* a, int wgs, int* out) {
  const sp::WideTeamPlan pl = sp::make_wide_team_plan(a, wgs);
  out[0] = pl.ok; out[1] = pl.lgP; out[2] = pl.chunk; out[3] = pl.share;
}
"""


@pytest.mark.parametrize("wgs", [256, 128, 32])
def test_shares_cover_the_prompt(tmp_path, wgs):
    cxx = shutil.which("g++") or shutil.which("c++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    (tmp_path / "shim.cpp").write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2502_02789_amd", "csrc"), "shim.cpp", "-o", "shim.so"], cwd=tmp_path, check=True)
    lib = C.CDLL(str(tmp_path / "shim.so"))
    rng = random.Random(3)
    shapes = [(T, n) for T in (3073, 4096, 4097, 16384, 16385, 32768, 33000, 65536, 65537, 100000, 131072) for n in (8, 12)]
    for T, n in shapes + [(int(3073 * 43 ** rng.random()), 8) for _ in range(300)]:
        a = sp.ScoreArgs()
        for k, v in dict(B=1, N=n, L=rng.randint(1, 80), H=16, H_kv=8, d=128, T=T).items():
            setattr(a, k, v)
        out = (C.c_int * 4)()
        lib.plan(C.byref(a), wgs, out)
        ok, lgP, chunk, share = out
        if not ok:                                                  # refused: only what no team holds
            assert T > min(64, wgs) * (2048 if n <= 8 else 1024), (T, n)
            continue
        P = 1 << lgP
        assert share % 32 == 0 and share <= chunk and P * share >= T, (T, n, lgP, share)
        assert (T + P - 1) // P > share - 32, (T, n, lgP, share)    # not a tile more than needed
        keys = [max(0, min(T - m * share, share)) for m in range(P)]  # as the kernel has it
        assert sum(keys) == T and keys == sorted(keys, reverse=True), (T, n, lgP, share)
        assert sum(0 < k < share for k in keys) <= 1, (T, n, lgP, share)  # full ones, at most one cut short, then empty ones
