"""The gather kernels on the CPU: sp_gather.hip compiled for the host, a std::thread per GPU thread, with inputs that end where
the contract lets them end -- the list of kept indices behind cu_keep[B] entries, the offsets behind B + 1, the token ids behind
T -- in front of a page that cannot be read, and outputs with room for more (Sec. 3.2.4 of arXiv 2502.02789; oracle)."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# what sp_gather.hip uses of the runtime: one launch at a time, blocks one after the other, their threads at once
RUNTIME = r"""
#pragma once
#include <math.h>
#include <pthread.h>
#include <stdint.h>
#include <string.h>
#include <algorithm>
#include <thread>
#include <vector>
#define __global__
#define __device__
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(n)
using std::max;
using std::min;
struct dim3 { unsigned x; dim3(unsigned n = 1) : x(n) {} };
inline thread_local dim3 threadIdx, blockIdx, gridDim;
inline pthread_barrier_t block_barrier;
inline void __syncthreads() { pthread_barrier_wait(&block_barrier); }
inline float __shfl_xor(float v, int, int) { return v; }
inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
typedef void* hipStream_t;
enum hipError_t { hipSuccess };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
template <typename K, typename P>
void launch(K kernel, dim3 grid, dim3 block, const P& p) {
  pthread_barrier_init(&block_barrier, nullptr, block.x);
  for (unsigned b = 0; b < grid.x; ++b) {
    std::vector<std::thread> threads;
    for (unsigned t = 0; t < block.x; ++t)
      threads.emplace_back([=] { threadIdx = t; blockIdx = b; gridDim = grid; kernel(p); });
    for (auto& t : threads) t.join();
  }
  pthread_barrier_destroy(&block_barrier);
}
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, p) launch(kernel, grid, block, p)
"""
# one call, in a process of its own (a read behind an input's end is a fault there)
CALL = r"""
import ctypes as C, mmap, sys
import numpy as np
from oracle import specprefill_oracle as orc
from paper_2502_02789_amd import binding as sp

lib, libc = C.CDLL(sys.argv[1]), C.CDLL(None)
B, spare, D = (int(x) for x in sys.argv[2:5])
held = []
def ends_at_a_page(a):
    a = np.ascontiguousarray(a)
    size = max(1, -(-a.nbytes // mmap.PAGESIZE)) * mmap.PAGESIZE
    m = mmap.mmap(-1, size + mmap.PAGESIZE)
    at = C.addressof(C.c_char.from_buffer(m))
    held.append(m)
    assert libc.mprotect(C.c_void_p(at + size), C.c_size_t(mmap.PAGESIZE), 0) == 0
    C.memmove(at + size - a.nbytes, a.ctypes.data, a.nbytes)
    return at + size - a.nbytes

rng = np.random.default_rng(B)
lens = rng.integers(0, 12, size=B)
lens[0] = 300
cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
scores = rng.random(int(cu[-1])).astype(np.float32)
kept, cu_keep = orc.pool_select(scores, cu, 4, 3, 0.4)[:2]
ids = rng.integers(0, 50, size=int(cu[-1])).astype(np.int32)
table = rng.integers(0, 2 ** 16, size=(50, D or 8)).astype(np.uint16)
n, cap = len(kept), len(kept) + spare
out_ids, out_pos, decode = np.full(cap, -7, np.int32), np.full(cap, -7, np.int32), np.full(B, -7, np.int32)
rows = np.full((cap, D or 8), 7, np.uint16)
a = sp.GatherArgs()
a.B, a.kept_capacity = B, cap
a.d_cu_seqlens, a.d_cu_keep, a.d_kept_idx = ends_at_a_page(cu), ends_at_a_page(cu_keep.astype(np.int32)), ends_at_a_page(kept.astype(np.int32))
a.d_token_ids = ends_at_a_page(ids)
a.d_kept_ids, a.d_kept_pos, a.d_decode_pos = out_ids.ctypes.data, out_pos.ctypes.data, decode.ctypes.data
if D:
    a.V, a.D, a.d_embed, a.d_out_embed = 50, D, ends_at_a_page(table), rows.ctypes.data
assert lib.sp_gather(C.byref(a), None) == 0
want_ids, want_pos, want_decode, want_rows = orc.gather(kept, cu_keep, cu, ids, table)
np.testing.assert_array_equal(out_ids[:n], want_ids)
np.testing.assert_array_equal(out_pos[:n], want_pos)
np.testing.assert_array_equal(decode, want_decode)
assert (out_ids[n:] == -7).all() and (out_pos[n:] == -7).all()
if D:
    np.testing.assert_array_equal(rows[:n], want_rows)
    assert (rows[n:] == 7).all()
print("read in range")
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    path = tmp_path_factory.mktemp("gather")
    (path / "hip").mkdir()
    (path / "hip" / "hip_runtime.h").write_text(RUNTIME)
    clang = "/opt/rocm/llvm/bin/clang++" if os.path.exists("/opt/rocm/llvm/bin/clang++") else shutil.which("clang++")
    subprocess.run([clang, "-x", "c++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread", "-I", str(path), "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "paper_2502_02789_amd", "csrc", "sp_gather.hip"), "-o", str(path / "gather.so")], check=True)
    return str(path / "gather.so")


@pytest.mark.parametrize("B,spare,D", [(1, 0, 0), (1, 3000, 0), (3, 700, 0), (255, 300, 0), (256, 300, 0), (1, 40, 16), (257, 0, 8)])
def test_nothing_behind_the_inputs_is_read(lib, B, spare, D):
    got = subprocess.run([sys.executable, "-c", CALL, lib, str(B), str(spare), str(D)], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert got.returncode == 0 and "read in range" in got.stdout, (got.returncode, got.stderr[-2000:])
