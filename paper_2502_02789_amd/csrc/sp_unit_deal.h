// How the single-pass kernels for batches of short prompts (sp_score_seq.hip, sp_score_wide.hip) share a batch out evenly
// without knowing the sequences' lengths on the host: the slabs of all sequences, one behind the other, are cut into as many
// stretches of equal cost as there are workgroups.  Plain C++: host and kernels use the same functions, and a test without
// a GPU goes through them.
//
// A grain is what is not cut: a (layer, KV head) slab, or a whole layer where layers are added up.  A grain of sequence b
// (M keys) costs M + extra, so the first grain of b lies at grains * (cu[b] + extra * b), known from cu alone, and a
// workgroup finds its stretch by itself.  A grain belongs to the stretch that its middle lies in.  All positions are
// doubled, so that they are whole numbers.
//
// Against units of a fixed number of slabs, longest sequences first, in rounds of alternating direction, which leave some
// workgroups a third unit where others have two, need a launch to rank the sequences and write twice as many results (whole
// call, 32 layers, 8 KV heads, d = 128, before -> now in us): 12 prompts of 2656..3949 keys, one query 461 -> 407; 18 of
// 1430..1988 406 -> 338; 22 of 1400..2100, eight queries 499 -> 400; 6 of 858..1723 111 -> 94; 56 of 596..1269, one query 631
// -> 534; 64 of 1024..4096 1671 -> 1655; 16 of 300..3000, eight queries 335 -> 331, 8-bit keys 200 -> 193; 7 of
// 296..2444, 8-bit 67 -> 64.  Where rounds come out even and prompts are short it is the other way round (make_unit_deal).
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

struct UnitDeal {
  int64_t stretch;   // twice the cost of a workgroup's share; 0: dealt out in rounds
  double inverse;    // 1 / stretch
  int grains, slabs; // of a sequence; slabs of a grain
  int extra;         // keys' time that the end of a grain takes

  SP_PLAN_FN int64_t cost(int M) const { return (int64_t)(M > 0 ? M : 0) + extra; }
  // of sequence b's first grain
  SP_PLAN_FN int64_t start(int cu_b, int b) const { return 2 * (int64_t)grains * (cu_b + (int64_t)extra * b); }
  // first grain of a sequence (starting at `at`, cost c a grain) whose middle does not lie in front of workgroup w's
  // stretch: 0 .. grains
  SP_PLAN_FN int first_grain(int w, int64_t at, int64_t c) const {
    const int64_t x = w * stretch - at - c;  // smallest s with 2 s c >= x
    if (x <= 0) return 0;
    if (x > 2 * c * (grains - 1)) return grains;
    int64_t s = (int)((float)(double)x / (float)(double)(2 * c));  // (right to one: fewer than 2^20 grains)
    while (2 * s * c < x) ++s;
    while (s > 0 && 2 * (s - 1) * c >= x) --s;
    return (int)s;
  }
  // the workgroup that has grain s
  SP_PLAN_FN int owner(int64_t at, int64_t c, int s) const {
    const int64_t x = at + (2 * (int64_t)s + 1) * c;
    int64_t w = (int64_t)((double)x * inverse);
    while (w > 0 && w * stretch > x) --w;
    while ((w + 1) * stretch <= x) ++w;
    return (int)w;
  }
};

// Units dealt out in rounds: results per sequence, and slabs per unit (a multiple of `step`).  A unit's end costs several
// microseconds (its results go out, the next unit's table entries come in), so few large units are better as long as the
// workgroups' shares stay even, which takes more units the more sequences of different lengths there are.  Measured best (32 layers,
// 8 KV heads, prompts of 1K to 4K keys): 2 per workgroup (of 256) for 16 prompts, 2 to 4 for 64, 8 for 256.
inline int round_groups(const sp_score_args* a, int step, int* slabs_per_group) {
  const int per_wg = std::min(8, std::max(2, a->B / 32)), slabs = a->L * a->H_kv;
  const int groups = std::max(1, std::min(slabs / step, (256 * per_wg + a->B - 1) / a->B));
  *slabs_per_group = ((slabs + groups - 1) / groups + step - 1) / step * step;
  return (slabs + *slabs_per_group - 1) / *slabs_per_group;
}

// The cut for W workgroups; sequences longer than `limit` keys (what the kernel holds) are not scored.  *n_groups: results a
// sequence may get, one from each workgroup that has a grain of it.  stretch = 0: not worth it, or not possible.
inline UnitDeal make_unit_deal(const sp_score_args* a, int W, int limit, bool whole_layers, int* n_groups) {
  UnitDeal d = {};
  d.slabs = whole_layers ? a->H_kv : 1;
  d.grains = a->L * a->H_kv / d.slabs;
  // (about 1.5 us for the end of a slab, at the 27 GB/s that a workgroup streams; 40 or 400 keys instead of 160: 8 prompts of
  // 200..1277 keys 90 us against 100 and 92, 16 of 300..3000 331 against 335 and 344)
  d.extra = 160 * 256 / (a->d * (a->k_dtype == SP_K_FP8_E4M3 ? 1 : 2));
  *n_groups = 0;
  if (a->T < 1 || d.grains > (1 << 20) || a->T + (int64_t)d.extra * a->B > ((int64_t)1 << 50) / d.grains) return d;
  const int64_t stretch = (2 * d.grains * (a->T + (int64_t)d.extra * a->B) + W - 1) / W;
  const int64_t held = std::min<int64_t>(limit, a->T) + d.extra;
  // Every workgroup between the first and the last that has a grain of a sequence must have one: no grain longer than a stretch.
  if (2 * held > stretch) return d;
  // A stretch is right to half a grain on either side, so four of the longest have to fit (busiest workgroup over 1500 random
  // batches, median against the rounds: three to four 1.10, four to five 0.98, seven to ten 0.96, more 0.79); ten layers (five of
  // them: 64 prompts of 1024..4096 keys, one query, 1730 us against 1673 in rounds).  (Mean over layers in parts of layers, as many as let
  // four fit, every part a unit with a result of its own: 22 prompts of 1400..2100 keys, eight queries, 508 us against 432 in rounds.)
  // One sequence, whose grains are equal: stretches save results, not time, as long as a workgroup has two grains either way (eight
  // queries, d = 64, 1300 keys: 288 slabs 32.9 us against 29.5 in rounds, 384 29.0 and 30.6).
  const int64_t longest = std::min<int64_t>(a->B == 1 ? a->T : a->max_seqlen, a->T) + d.extra;
  if (a->B == 1 ? 2 * (int64_t)d.grains < 3 * (int64_t)W : (whole_layers ? 10 : 4) * 2 * longest > stretch) return d;
  // A slab's time is that of the rounds of 256 keys that a workgroup's waves take, which no sum over the offsets knows: short
  // prompts of different lengths are off by up to half.  Rounds of units even that out where there are many sequences and no round is left partly
  // filled (32, 64, 96 or 128 of them; us, stretches and rounds, 32 layers, 8 KV heads, d = 128: 128 prompts of up to 400 keys,
  // eight queries 1.21 of the time in rounds, 64 of 100..700, four queries 357 and 308, one query and 8-bit keys 303 and 239; 32 of
  // 200..1000, 8-bit 157 and 147); of 1500 keys and more stretches are ahead again (64 of up to 1594 0.97), and with any other number of
  // sequences (40 of 100..700 0.78..0.98, 48 0.75..0.97).  Of d = 64 from 96 sequences on (128 of up to 700, 8-bit 1.08; 32 0.91..1.03, 64
  // 0.93..1.02).
  int per = 1;
  const int groups = round_groups(a, d.slabs, &per);
  if (a->B >= (a->d == 64 ? 96 : 32) && a->max_seqlen <= 1408 && (int64_t)a->B * groups % W == 0) return d;
  d.stretch = stretch;
  d.inverse = 1.0 / (double)stretch;
  *n_groups = (int)std::min<int64_t>(W, 2 * (int64_t)(d.grains - 1) * held / stretch + 2);
  return d;
}

}  // namespace sp
