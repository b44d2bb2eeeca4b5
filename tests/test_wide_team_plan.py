"""The cut of one long prompt into members, teams and runs of (layer, KV head) slabs (sp_wide_team_plan.h), walked on the
CPU with the functions that the kernel walks it with."""
import ctypes as C
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

from paper_2502_02789_amd import binding as sp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "sp_wide_team_plan.h"
// out: ok, lgP, chunk, teams, run, rounds, part, n_groups, plain_groups, gpl; per slab: the team, its place in the team's
// order, the number of the run, the first slab of the run
extern "C" int wgs_of(int compute_units) { return sp::wide_team_wgs(compute_units); }
extern "C" int walk(const sp_score_args* a, int wgs, int* out, int* team_of, int* place_of, int* run_of, int* first_of) {
  const sp::WideTeamPlan pl = sp::make_wide_team_plan(a, wgs);
  const int fields[] = {pl.ok, pl.lgP, pl.chunk, pl.deal.teams, pl.deal.run, pl.deal.rounds, pl.deal.part, pl.n_groups, pl.plain_groups, pl.gpl};
  for (int i = 0; i < 10; ++i) out[i] = fields[i];
  if (!pl.ok) return 0;
  int visits = 0;
  for (int t = 0; t < pl.deal.teams; ++t) {
    int place = 0;
    for (int q = 0;; ++q) {
      const int s0 = pl.deal.start(t, q), s1 = pl.deal.end(q, s0);
      if (s0 >= pl.deal.n_slabs) break;
      for (int s = s0; s < s1; ++s, ++visits) { team_of[s] = t; place_of[s] = place++; run_of[s] = q; first_of[s] = s0; }
    }
  }
  return visits;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    where = tmp_path_factory.mktemp("plan")
    (where / "shim.cpp").write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2502_02789_amd", "csrc"), "shim.cpp", "-o", "shim.so"], cwd=where, check=True)
    lib = C.CDLL(str(where / "shim.so"))

    def run(wgs=256, **fields):
        a = sp.ScoreArgs()
        for k, v in dict(dict(B=1, N=8, L=32, H=32, H_kv=8, d=128, T=32768, k_token_stride=1024, k_head_stride=128, scale=0.1), **fields).items():
            setattr(a, k, v)
        n = a.L * a.H_kv
        arrays = [np.full(n, -1, dtype=np.int32) for _ in range(4)]
        out = np.zeros(10, dtype=np.int32)
        ptr = lambda x: x.ctypes.data_as(C.POINTER(C.c_int))  # noqa: E731
        visits = lib.walk(C.byref(a), wgs, ptr(out), *[ptr(x) for x in arrays])
        p = dict(zip("ok lgP chunk teams run rounds part n_groups plain_groups gpl".split(), (int(x) for x in out)))
        p.update(visits=visits, slabs=n, **dict(zip("team place run_of first".split(), arrays)))
        return p
    run.wgs_of = lib.wgs_of
    return run


def _shapes():
    rng = random.Random(7)   # (prompts of more than 3072 keys: few slabs are taken beyond)
    fixed = [dict(L=L, H_kv=K, T=T) for L in (1, 2, 16, 24, 28, 32, 33, 36, 48, 80, 128) for K in (1, 2, 4, 5, 8, 16) for T in (3073, 9000, 32768, 131072)]
    drawn = [dict(L=rng.randint(1, 128), H_kv=rng.randint(1, 32), T=int(3073 * 43 ** rng.random())) for _ in range(400)]
    return [dict(s, H=s["H_kv"] * 4, layer_reduce=m) for s in fixed + drawn for m in (sp.SP_LAYER_MAX, sp.SP_LAYER_MEAN)]


@pytest.mark.parametrize("wgs", [256, 128, 64, 32])
def test_every_slab_and_key_is_taken_once(walk, wgs):
    for shape in _shapes():
        p = walk(wgs, **shape)
        if not p["ok"]:
            assert shape["T"] > 2048 * min(64, wgs), shape
            continue
        P = 1 << p["lgP"]
        assert p["visits"] == p["slabs"] and (p["team"] >= 0).all(), shape
        assert P * p["teams"] == wgs and p["chunk"] % 256 == 0 and p["chunk"] <= 2048 and P * p["chunk"] >= shape["T"], shape
        if shape["layer_reduce"] == sp.SP_LAYER_MAX:
            assert p["n_groups"] == len(set(p["team"])) and set(p["team"]) == set(range(p["n_groups"])), shape
            continue
        # mean: whole layers in the rounds (summed per team), then parts that lie in one layer, a group each
        K, base = shape["H_kv"], p["rounds"] * p["run"] * p["teams"]
        assert p["run"] == K and K % p["part"] == 0 and p["gpl"] == K // p["part"], shape
        assert (p["first"][:base] == np.arange(base) // K * K).all(), shape
        assert (p["first"][base:] == base + np.arange(p["slabs"] - base) // p["part"] * p["part"]).all(), shape
        assert p["plain_groups"] == (p["teams"] if p["rounds"] else 0), shape
        assert p["n_groups"] == p["plain_groups"] + (p["slabs"] - base) // p["part"], shape


def test_maximum_over_layers_even_shares_close_together(walk):
    """No team has a slab more than another needs, and teams that have come equally far are in the same few layers (a pass
    over new buffers pays for every page that is met for the first time)."""
    for shape in _shapes():
        if shape["layer_reduce"] != sp.SP_LAYER_MAX:
            continue
        p = walk(**shape)
        if not p["ok"]:
            continue
        counts = np.bincount(p["team"], minlength=p["teams"])
        assert counts.max() == -(-p["slabs"] // p["teams"]), shape
        for k in range(counts.max()):
            at = np.flatnonzero(p["place"] == k)
            assert at.max() - at.min() < 4 * p["teams"], shape


def test_mean_over_layers_even_shares(walk):
    """Layer counts that the number of teams does not divide: what a busiest team has beyond its share costs no more than
    the results that even shares would cost (a part of a layer is a result of its own: eight times its bytes in keys)."""
    for L in range(1, 129):
        for T in (3073, 4000, 9000, 16000, 32768, 131072):
            for bits in (16, 8):
                p = walk(L=L, T=T, layer_reduce=sp.SP_LAYER_MEAN, k_dtype=sp.SP_K_FP8_E4M3 if bits == 8 else sp.SP_K_BF16)
                share = -(-p["slabs"] // p["teams"])
                busiest = np.bincount(p["team"], minlength=p["teams"]).max()
                result = 8 * 4 * 8 / (128 * bits / 8)               # slabs' time for a part's result
                assert busiest <= share + 1 + result * share, (L, T, bits, busiest, share)
                if L >= p["teams"]:                                 # whole layers to everybody, few left over
                    assert busiest <= share + 4, (L, T, bits, busiest, share)


def test_more_than_eight_queries(walk):
    """One or two heads per KV head leave room for sixteen queries (padded to four they would not); three do not."""
    for heads, N in ((1, 9), (1, 16), (2, 9), (2, 12), (2, 16)):
        for T in (3073, 8193, 16384, 32768, 65536):
            for mean in (sp.SP_LAYER_MAX, sp.SP_LAYER_MEAN):
                p = walk(H=8 * heads, N=N, T=T, layer_reduce=mean)
                assert p["ok"] and p["visits"] == p["slabs"] and p["chunk"] <= 1024 and (p["chunk"] << p["lgP"]) >= T, (heads, N, T)
    assert not walk(H=16, N=12, T=65537)["ok"] and not walk(H=24, N=9, T=9000)["ok"]


def test_workgroups_by_compute_units(walk):
    """The whole chip and its partitions; every workgroup has a compute unit of its own."""
    assert [walk.wgs_of(n) for n in (256, 304, 255, 128, 64, 32, 31, 8)] == [256, 256, 128, 128, 64, 32, 0, 0]
    assert not walk(0)["ok"]
