// How the two-pass kernels for up to 32 query rows per KV head (sp_score_wide_passes.hip) cut a call into pieces of
// sequences and runs of (layer, KV head) slabs.  Plain C++: a test without a GPU goes through it.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "specprefill.h"

#ifdef __HIPCC__
#define SP_PLAN_FN __host__ __device__ __forceinline__
#else
#define SP_PLAN_FN inline
#endif

namespace sp {

constexpr int kPassWaves = 8;
constexpr int kPassItemKeys = 32;                                // what a wave takes at a time
constexpr int kPassTiles = 16;                                   // 32-key tiles per wave
constexpr int kPassMaxKeys = kPassTiles * 32 * kPassWaves;       // keys of a piece
constexpr int kPassBatchKeys = 2048;                             // ... where the sequences' lengths are not known here

// the pieces of sequence b, whose first token is seq0, have the places from here on
SP_PLAN_FN int pass_first_place(int seq0, int b, int chunk) { return seq0 / chunk + b; }

struct WidePassPlan { int chunk, slots, per, n_groups, gpl; };

inline WidePassPlan make_wide_pass_plan(const sp_score_args* a) {
  const int slabs = a->L * a->H_kv, round = kPassItemKeys * kPassWaves;
  const bool mean = a->layer_reduce == SP_LAYER_MEAN;
  WidePassPlan best = {};
  int64_t best_cost = INT64_MAX;
  // The cut into pieces and runs of slabs whose rounds over 256 workgroups are fullest: keys of a round's longest
  // unit, plus about 200 keys' time for the end of a slab and 300 for that of a unit, plus its results, written and
  // read back, at three times their bytes.  (Without that term the mean over layers of 24577 keys was cut into 256
  // parts of layers for 8-bit keys, 407 us against 294 with 32, and 16 layers of d = 64 into 128, 202 against 157.
  // Few KV heads are better off here than on the tiled kernels even where results outweigh keys: 16 layers, 2 KV
  // heads of 8-bit d = 64, mean: 55 us against 98.)  For a batch the sequences' lengths are not known here: pieces of
  // one size for all.
  const int64_t result_bytes = 3 * 4 * a->N, key_bytes = a->d * (a->k_dtype == SP_K_FP8_E4M3 ? 1 : 2);
  // One sequence: from as few pieces as hold it to seven more, or, where the slabs are few, to a unit per workgroup (but
  // pieces of 256 keys at least).  A batch: pieces of 2048 keys, halved while the slabs are too few for a unit per
  // workgroup.  (One layer, four heads of one KV head, d = 128: 128K keys in 39 pieces 55 us, in 256 39, on the tiled
  // kernels 42; two prompts of 10000 and 20000 keys 32, 22 and 30.)
  const int n0 = (int)((a->T + kPassMaxKeys - 1) / kPassMaxKeys);
  const int n1 = std::max(n0 + 7, (int)std::min<int64_t>(256 / slabs, a->T / 256));
  for (int n = n0, chunk = kPassBatchKeys; a->B > 1 ? chunk >= 256 : n <= n1; ++n, chunk /= 2) {
    WidePassPlan pl = {};
    pl.chunk = a->B > 1 ? chunk : (int)((a->T + n - 1) / n + 31) / 32 * 32;
    pl.slots = a->B > 1 ? (int)(a->T / chunk) + a->B : (int)((a->T + pl.chunk - 1) / pl.chunk);
    if (a->B > 1 && chunk < kPassBatchKeys && (int64_t)pl.slots * slabs > 256) break;
    const int64_t keys = (int64_t)((pl.chunk + round - 1) / round) * round;
    for (int per = 1; per <= (mean ? a->H_kv : slabs); per = per < 16 ? per + 1 : per + per / 8) {
      if (mean && a->H_kv % per != 0) continue;
      const int groups = (slabs + per - 1) / per;
      const int64_t rounds = ((int64_t)pl.slots * groups + 255) / 256;
      const int64_t cost = rounds * (per * (keys + 200) + 300 + keys * result_bytes / key_bytes);
      if (cost < best_cost) {
        best_cost = cost;
        best = pl;
        best.per = per;
        best.n_groups = groups;
        best.gpl = mean ? a->H_kv / per : 0;
      }
    }
  }
  if (a->B == 1) ++best.slots;  // (the numbering T / chunk + 1 of one sequence)
  return best;
}

}  // namespace sp
