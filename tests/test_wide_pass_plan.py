"""The cut of the two-pass kernels for up to 32 query rows per KV head (sp_wide_pass_plan.h), on the CPU: places for the
pieces of every sequence, and enough units for the device where the prompt has the keys."""
import ctypes as C
import os
import random
import shutil
import subprocess

import pytest

from paper_2502_02789_amd import binding as sp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "sp_wide_pass_plan.h"
extern "C" void plan(const sp_score_args* a, int* out) {
  const sp::WidePassPlan pl = sp::make_wide_pass_plan(a);
  out[0] = pl.chunk; out[1] = pl.slots; out[2] = pl.per; out[3] = pl.n_groups; out[4] = pl.gpl;
}
extern "C" int first_place(int seq0, int b, int chunk) { return sp::pass_first_place(seq0, b, chunk); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    where = tmp_path_factory.mktemp("plan")
    (where / "shim.cpp").write_text(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2502_02789_amd", "csrc"), "shim.cpp", "-o", "shim.so"], cwd=where, check=True)
    return C.CDLL(str(where / "shim.so"))


def _plan(lib, **fields):
    a = sp.ScoreArgs()
    for k, v in dict(dict(B=1, N=8, L=32, H=32, H_kv=8, d=128), **fields).items():
        setattr(a, k, v)
    out = (C.c_int * 5)()
    lib.plan(C.byref(a), out)
    return dict(zip(("chunk", "slots", "per", "n_groups", "gpl"), out))


def _shapes(n):
    rng = random.Random(11)
    for _ in range(n):
        yield rng, dict(L=rng.choice([1, 1, 2, 3, 16, 32, 80]), H_kv=rng.choice([1, 1, 2, 4, 5, 8]), N=rng.randint(1, 8), d=rng.choice([64, 128]),
                        k_dtype=rng.choice([sp.SP_K_BF16, sp.SP_K_FP8_E4M3]), layer_reduce=rng.choice([sp.SP_LAYER_MAX, sp.SP_LAYER_MEAN]))


def test_every_piece_has_a_place_of_its_own(lib):
    for rng, shape in _shapes(600):
        B = rng.choice([1, 1, 2, 5, 40])
        lens = [rng.choice([0, 1, 31, 255, 256, 257, 2048, 4097, int(300 * 100 ** rng.random())]) for _ in range(B)]
        lens[0] = max(lens[0], 1)
        p = _plan(lib, B=B, T=sum(lens), **shape)
        assert 0 < p["chunk"] <= 4096 and p["chunk"] % 32 == 0, (shape, lens)
        slabs = shape["L"] * shape["H_kv"]
        assert p["n_groups"] == -(-slabs // p["per"]) and (p["gpl"] == 0 or shape["H_kv"] % p["per"] == 0), (shape, lens)
        free, start = 0, 0
        for b, m in enumerate(lens):
            first = lib.first_place(start, b, p["chunk"])
            assert first >= free, (shape, lens)
            free, start = first + -(-m // p["chunk"]), start + m
        assert free <= p["slots"], (shape, lens)


def test_few_slabs_still_fill_the_device(lib):
    """A third of the 256 workgroups or more have a unit (of 256 keys at least) where there are the keys for it."""
    for rng, shape in _shapes(600):
        slabs = shape["L"] * shape["H_kv"]
        for lens in ([int(1000 * 130 ** rng.random())], [int(1000 * 30 ** rng.random()) for _ in range(rng.randint(2, 6))]):
            T = sum(lens)
            p = _plan(lib, B=len(lens), T=T, **shape)
            units = sum(-(-m // p["chunk"]) for m in lens) * p["n_groups"]
            wave_keys = 8192 // (shape["d"] * (1 if shape["k_dtype"] == sp.SP_K_FP8_E4M3 else 2))
            smallest = max(256, 8 * wave_keys)        # keys that give each of a workgroup's waves something
            most = sum(max(1, m // smallest) for m in lens) * slabs
            assert units >= min(256, most) / 3 or p["per"] > 1, (shape, lens, p)
