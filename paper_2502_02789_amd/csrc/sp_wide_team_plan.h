// How the single-pass kernel for one long prompt (sp_score_wide_team.hip) cuts a call: the prompt into the members of a
// team, the (layer, KV head) slabs into the teams' runs.  Plain C++ (the host's sizes and the kernel's walk come from the
// same functions, and a test without a GPU goes through them).
#pragma once

#include <stdint.h>

#include <algorithm>

#include "specprefill.h"

#ifdef __HIPCC__  // (as in sp_wide_pass_plan.h)
#define SP_PLAN_FN __host__ __device__ __forceinline__
#else
#define SP_PLAN_FN inline
#endif

namespace sp {

#ifndef SP_TEAM_MAX_WGS
#define SP_TEAM_MAX_WGS 256
#endif
constexpr int kWideTeamDieWGs = 32;      // compute units of a die
constexpr int kWideTeamWaves = 8;
constexpr int kWideTeamMaxPartners = 64;

// The 32 columns are the queries times the heads of a group, padded to 2^this: four or eight, and two where more than eight
// queries leave no room for four.  (32 layers, 8 KV heads of two heads, d = 128, in us: the kernels before the teams of this
// kind, two passes for want of this variant, now: twelve queries on 12000 keys 300, 336, 152; nine on 32K keys 348, 853,
// 366, the one shape tried that is not as fast as it was: half the keys per member, so twice the exchanges.)
inline int wide_team_lg(const sp_score_args* a) {
  const int heads = a->H / a->H_kv;
  return heads > 4 ? 3 : heads <= 2 && a->N > 8 ? 1 : 2;
}
// 32-key tiles per wave: what the registers hold of logits (16 each) and running maxima (16 >> lg each).
constexpr int wide_team_tiles(int lg) { return lg > 1 ? 8 : 4; }

// The slabs are dealt out to the teams in turn: `rounds` rounds of `run` slabs to each team, the others in parts of
// `part`, again in turn.
struct WideTeamDeal {
  int teams, n_slabs, run, rounds, part;
  SP_PLAN_FN int base() const { return rounds * run * teams; }  // slabs of the whole rounds
  // team `team`'s q-th run: where it starts (n_slabs or more: there is none) and ends
  SP_PLAN_FN int start(int team, int q) const {
    return q < rounds ? (q * teams + team) * run : base() + ((q - rounds) * teams + team) * part;
  }
  SP_PLAN_FN int end(int q, int start_) const {
    const int e = start_ + (q < rounds ? run : part);
    return e < n_slabs ? e : n_slabs;
  }
};

// Workgroups of a call, which must all be resident: one per compute unit, as many as a power of two allows (256 on the
// whole chip, 128, 64 or 32 on a partition of it); 0: too few.
inline int wide_team_wgs(int compute_units) {
  int wgs = SP_TEAM_MAX_WGS;
  while (wgs > compute_units) wgs >>= 1;
  return wgs >= kWideTeamDieWGs ? wgs : 0;
}

struct WideTeamPlan {
  bool ok;
  int lgP, chunk;          // members of a team (a power of two), keys a member has room for in whole rounds of its waves
  int share;               // keys of a member, whole 32-key tiles
  WideTeamDeal deal;
  // Groups of the result array.  Maximum over layers: one per team that has a slab.  Mean: the teams' sums over whole
  // layers (plain_groups of them), then the parts of the layers left, gpl of a layer.
  int n_groups, plain_groups, gpl;
};

// Slabs of a run (maximum over layers).  What the teams read at a time is spread over so many layers: with one run
// per team (16 of them at 32K keys, each in two layers of its own) the first pass over new buffers met 1 GB of pages at
// once; with single slabs the teams crowd into one or two layers.  First / later pass of 32K keys (32 layers, 8 KV
// heads, d = 128, eight queries) in us: one slab 403 / 356, two 386 / 341, four 385 / 340, eight 393 / 339, all sixteen
// 429 / 340; 8-bit keys 312 / 259, 290 / 244, 283 / 236, 300 / 238, 300 / 239; 128K keys 1537 / 1409, 1478 / 1345,
// 1486 / 1311, 1556 / 1370, 1535 / 1360 (all 128).
constexpr int kWideTeamRun = 4;

inline WideTeamPlan make_wide_team_plan(const sp_score_args* a, int wgs) {
  WideTeamPlan pl = {};
  const int most_partners = std::min(kWideTeamMaxPartners, wgs);
  if (a->B != 1 || a->rope_theta > 0.f) return pl;
  const int lg = wide_team_lg(a);
  if (a->H / a->H_kv > 8 || (a->N << lg) > 32) return pl;
  const int64_t most = wide_team_tiles(lg) * 32 * kWideTeamWaves;   // keys of a member
  if (a->T <= 0 || a->T > most_partners * most) return pl;
  if (a->k_dtype == SP_K_FP8_E4M3 && a->d_block_table && a->page_size < (a->d == 64 ? 16 : 8)) return pl;
  if (a->k_token_stride > (INT32_MAX / 256)) return pl;  // (a ring slot's keys must span less than 2 GiB)
  const int slabs = a->L * a->H_kv;
  // Short prompts of next to no layers stay on the kernels that also take un-rotated caches: their scores are then bit for
  // bit those of the same cache stored un-rotated.
  if (slabs < 8 && a->T <= 3072) return pl;
  int lgP = 1;
  while ((most << lgP) < a->T) ++lgP;
  // (fewer slabs than teams: more members per team instead, as long as each still has a wave's worth of keys; a single
  // slab is still faster this way than in two passes: one layer, one KV head of four, 32K keys 16 us against 35)
  while ((wgs >> lgP) > slabs && (1 << lgP) < most_partners) ++lgP;
  const int P = 1 << lgP, teams = wgs >> lgP;
  pl.lgP = lgP;
  pl.chunk = (int)(((a->T + P - 1) / P + 255) / 256 * 256);
  // Whole tiles, not whole rounds of the eight waves: fewer keys for the busiest member.  The last members may still have
  // none (3073 keys, 32 members: 24 full shares of 128, one key in another, seven empty ones).  (32 layers, 8 KV heads,
  // d = 128, eight queries, before -> now in us: 33000 keys 407 -> 384, 70000 821 -> 787, 100000 1118 -> 1073, 8-bit keys
  // 269 -> 250 and 565 -> 544 for the first two; where the prompt fills whole rounds nothing changes.)
  pl.share = (int)((a->T + P - 1) / P + 31) / 32 * 32;
  WideTeamDeal& d = pl.deal;
  d.teams = teams;
  d.n_slabs = slabs;
  if (a->layer_reduce == SP_LAYER_MEAN) {
    // Whole layers, in turn, as long as there is one for every team; the layers left over (all of them, if there are
    // fewer than teams) in parts, cut so that the team with the most of them is done soonest: its slabs (with about 200
    // keys' time for the end of each), 300 keys' time for the end of a part and its results at eight times their bytes
    // (written, read back, and they hold up the stream).  Keys are counted in whole rounds of the eight waves, which is how
    // the constants were fitted; by the members' shares the choice is the same for all usual numbers of KV heads (1, 2, 4,
    // 8; 26000 shapes of 3073 to 131072 keys) and another one in fewer than one of 1000 others.  Left over as whole layers,
    // or in the largest parts that give every team one, where there are fewer: 24 layers of 32K keys 328 us against 267, 36
    // layers 492 against 410 (16000 keys 315 against 215), 20 layers of 4 KV heads 114 against 84, 22 layers of 8192 keys
    // with d = 64 68 against 62; the exception among the shapes tried: 33 layers of 4000 keys 86.5 against 88.8.
    d.run = a->H_kv;
    d.rounds = a->L / teams;
    d.part = a->H_kv;
    const int left = a->L - d.rounds * teams;
    const int64_t key_bytes = a->d * (a->k_dtype == SP_K_FP8_E4M3 ? 1 : 2), result_bytes = 8 * 4 * a->N;
    int64_t least = INT64_MAX;
    for (int part = a->H_kv; part >= 1; --part) {
      if (a->H_kv % part != 0) continue;
      const int64_t parts = ((int64_t)left * (a->H_kv / part) + teams - 1) / teams;  // parts of the busiest team
      const int64_t cost = parts * ((part * (pl.chunk + 200) + 300) * key_bytes + pl.chunk * result_bytes);
      if (cost < least) { least = cost; d.part = part; }
    }
    pl.plain_groups = d.rounds > 0 ? teams : 0;
    pl.gpl = a->H_kv / d.part;
    pl.n_groups = pl.plain_groups + (a->L - d.rounds * teams) * pl.gpl;
  } else {
    d.run = std::min(kWideTeamRun, (slabs + teams - 1) / teams);
    d.rounds = slabs / (d.run * teams);
    d.part = std::max(1, (slabs - d.base() + teams - 1) / teams);
    pl.n_groups = d.rounds > 0 ? teams : (slabs + d.part - 1) / d.part;
  }
  pl.ok = true;
  return pl;
}

// How long, in microseconds, a workgroup of a call without the promise of an idle device waits for the lines of a slab
// before the call gives up waiting, as a whole.  What giving up costs is another pass over K, so nobody waits much longer
// than one takes; and not much less either, because that is when the first teams are done and make room for members that
// other work has kept out.  Reckoned with 16 KB of keys a us and workgroup (8-bit keys 12, which arithmetic holds up;
// undisturbed 25 and 19), 3 us for the end of a slab, and 50 us for the tail of another stream's kernel.  (200 compute
// units held by other work, which leaves no team of sixteen complete, us per call: every workgroup with a bound of its own
// of a millisecond and more, one for all of them, two passes: 9000 keys 4492, 1288, 765; 24577 keys 5165, 3188, 1903.  Up
// to 64 held, where teams that are done make room: 176, 176, 270 and 409, 409, 669; 24577 8-bit keys 309, 309, 273, with
// 64 held 307, 308, 449.  Beside 4096^3 products, 3500 keys: 289, 290, 392, the same with 20, 100, 200 and 400 us for a tail.)
inline int64_t wide_team_patience_us(const WideTeamPlan& pl, const sp_score_args* a) {
  const int64_t slabs = (pl.deal.n_slabs + pl.deal.teams - 1) / pl.deal.teams;
  const int64_t slab_bytes = (int64_t)pl.chunk * a->d * (a->k_dtype == SP_K_FP8_E4M3 ? 1 : 2);
  return 50 + slabs * 3 + slabs * slab_bytes / (a->k_dtype == SP_K_FP8_E4M3 ? 12000 : 16000);
}

}  // namespace sp
