// Single-pass scorer for one long prompt: small teams of workgroups, each holding ALL logits of its keys for a slab.
//
// Same quantity as the other scoring kernels: row softmax of the stored queries against the prompt keys
// (Sec. 3.2 equation of arXiv 2502.02789), max over heads, max/mean over layers, mean over queries (Sec. 3.2.2).
// Stream, products, statistics and the fold over heads are those of sp_score_wide.hip (sp_wide_core.h).  There one
// workgroup owns a whole prompt; a longer prompt is cut into P pieces of up to 2048 keys (1024 with more than eight
// queries), and the P workgroups of a team walk together over the team's (layer, KV head) slabs:
//
//   * per slab every member publishes ONE 128-byte line, the base-2 log-sum-exps of its keys for the 32 rows (agent
//     scope); its first wave then reads the team's P lines (contiguous) until none is "empty" any more, folds them
//     into the rows' log-sum-exps and hands those to the other waves through LDS;
//   * a slab is 18 us of stream for a workgroup (2048 keys, d = 128) and the ring holds 5 us of it, so the exchange
//     is short against a slab, and the teams, which never meet, drift apart: while one waits the others have the
//     memory.  The next slab's first item is computed while the lines travel, its logits in registers of their own
//     (32K keys 350 -> 339 us), and bf16 keys' other items in turn with the fold of the slab before;
//   * 256 / P teams are dealt the slabs in turn, a few at a time (sp_wide_team_plan.h); a team's maxima go out as one
//     group of the result array, merged by the kernel that merges the units of short prompts.  Mean over layers: whole
//     layers in turn, a team adds their maxima up; the layers left over in parts, each a group of its own.
//
// The lines exist twice: a call works in copy (epoch mod 2) and puts "empty" back into the other one as it publishes,
// so the next call finds it clean; a small kernel sets that up in front of a call that cannot rely on the previous one
// (no SP_SCORE_WORKSPACE_KEPT).  The workgroups of a team must be resident together; every wait is bounded.
//
// On the promise of an idle device (SP_SCORE_EXCLUSIVE_DEVICE) an expired wait turns the call's scores into NaN.  Without
// it the kernel is launched twice: where a workgroup has waited for one slab's lines about as long as the whole call takes
// (wide_team_patience_us) it notes that down for all to see, and from then on nobody waits any more.  The lines of
// statistics still go out for every slab -- a line depends on nothing but the member's own keys -- so after the first
// launch all of them are there, and the second one, which returns at once where nobody gave up, forms all results again
// without any wait.  So nothing depends on what else runs on the device,
// K is read once as a rule and twice at worst, and the scores have the same bits either way.  (Two passes over K before:
// 24577 keys, 32 layers, 8 KV heads, d = 128, eight queries, whole step: 498 -> 290 us; 128K keys 2604 -> 1351; one query on
// 20000 keys, logits kept in memory before, 311 -> 252.  Beside another stream's 4096^3 products: 9000 keys 655 -> 557 us,
// 24577 keys 520 -> 298, 100000 keys 2228 -> 1607, the other stream no slower; four such calls at once on four streams,
// 24577 keys, 504 -> 294 us each.)
//
// Bound by the HBM stream of K for bf16 caches (32 layers, 8 KV heads, d = 128, eight queries, kernel and merge in a filled
// queue: 32K keys 342 us = 6.3 TB/s, mean over layers 30011 keys 319, 8192 keys 99; 16 layers, d = 64, 8K keys 40: two slabs
// per workgroup, their start and end), by latency and vector instructions for 8-bit caches (32K keys 220 us).
// Tried: polling by every wave instead of one and a barrier 355 against 350 us, polls that read the die's own L2 451.
#include <atomic>
#include <mutex>

#include "sp_wide_core.h"
#include "sp_wide_team_plan.h"

namespace sp {

static_assert(kWideTeamWaves == kTiledWaves, "a member's keys are those of its waves");
constexpr uint32_t kEmptyLine = 0xffffffffu;
constexpr int kDefaultSpinBudget = 1 << 16;  // polls per workgroup and call before giving up (~0.1 s)
static std::atomic<int> g_spin_budget{kDefaultSpinBudget};

struct WideTeamDev : TiledDev {
  int lgP, share;          // members of a team (a power of two), keys of a member
  WideTeamDeal deal;
  int spin_budget;
  uint32_t* lines;         // two copies of [slab][member][32]
  size_t copy_words;
  uint32_t* status;        // [epoch & 1] != 0: a wait of this call expired; [2]: epoch, calls since the last fill;
                           // [3] != 0: a wait of a shared call's first launch expired, nobody waits any longer
  int launch;              // kAlone; kFirst and kSecond: the launches of a call without the promise of an idle device
  uint32_t patience;       // kFirst: ticks of the 100 MHz clock that a workgroup waits for the lines of a slab
};
enum { kAlone = 0, kFirst = 1, kSecond = 2 };

// the lines' first copy "empty", status and epoch 0
__global__ __launch_bounds__(256) void wide_team_fill_kernel(uint4* lines, size_t n_vec, uint32_t* status) {
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_vec; i += stride)
    lines[i] = make_uint4(kEmptyLine, kEmptyLine, kEmptyLine, kEmptyLine);
  if (blockIdx.x == 0 && threadIdx.x < 4) status[threadIdx.x] = 0;
}

template <int D, int LG, bool FP8, bool PAGED>
__global__ __launch_bounds__(kTiledThreads) void wide_team_kernel(const WideTeamDev p) {
  extern __shared__ __align__(1024) unsigned char smem[];
  using W = WideKernel<D, LG, FP8, PAGED>;
  constexpr int KEEP = W::KEEP, MAXT = wide_team_tiles(LG);
  using vkeep = typename W::vkeep;
  W w(p, smem);
  const uint32_t lse_lds = (uint32_t)reinterpret_cast<uintptr_t>(smem) + W::kSmem;  // 32 row log-sum-exps
  // The members of a team sit on one die where one has enough compute units (workgroups are dealt out to the dies
  // in turn).  (Measured, whole call: 32K keys, 16 members, next to each other on one die 352 us, over all dies 363; 128K
  // keys, 64 members, on two dies 1457 us, over all dies 1390.)  Without the promise of an idle device eight members on each
  // of as many dies as that takes: workgroups start in their order, so of a call that gets a quarter of every die (four
  // calls at once on four streams) whole teams are resident.  (24577 keys, one call / four at once, us per call: eight on
  // a die 296 / 295, four 305 / 281, two 306 / 289, all on one die 298 / 563; two passes 498 / 504.)
  const int P = 1 << p.lgP, dies = (int)gridDim.x / kWideTeamDieWGs;
  const int most_on_die = p.launch == kAlone && P <= kWideTeamDieWGs ? kWideTeamDieWGs : kWideTeamDieWGs / 4;
  const int over = min(dies, max(1, P / most_on_die)), share = P / over;  // dies of a team, members on each
  const int die = (int)blockIdx.x % dies, nth = (int)blockIdx.x / dies;
  const int place = (die / over * (kWideTeamDieWGs / share) + nth / share) * P + nth % share * over + die % over;
  const int team = place >> p.lgP, member = place & (P - 1);
  const WideTeamDeal& deal = p.deal;
  const bool mean = p.layer_reduce != SP_LAYER_MAX;
  int q = 0, s = deal.start(team, 0), s_end = deal.end(0, s);
  if (s >= deal.n_slabs || (p.launch == kSecond && p.status[3] == 0)) return;
  const uint32_t epoch = __builtin_amdgcn_readfirstlane(p.status[2]);  // (turned by the merge kernel)
  uint32_t* const lines_cur = p.lines + (size_t)(epoch & 1u) * p.copy_words;
  uint32_t* const lines_nxt = p.lines + (size_t)(~epoch & 1u) * p.copy_words;
  if (blockIdx.x == 0 && threadIdx.x == 0) p.status[~epoch & 1u] = 0;  // the next call's status word
  const int key0 = member * p.share;
  const int M = max(0, min((int)p.T - key0, p.share));
  const int nt = w.items_of(M);
  int polls = p.spin_budget;
  bool expired = polls <= 0;

  int l = s / p.H_kv, g = s - l * p.H_kv;
  w.ah = {w.slab_keys(l, g, 0), 0, key0, M, nt};
  w.issue_queries(l, g, 0, 0);
  w.start_stream();
  w.first_queries();

  f32x16 held[MAXT];
  vkeep run[MAXT];
#pragma unroll
  for (int t = 0; t < MAXT; ++t)
#pragma unroll
    for (int k = 0; k < KEEP; ++k) run[t][k] = -INFINITY;

  struct Place { int q, s, s_end, l, g; };  // slab s = (l, g) of the team's q-th run, which ends at s_end
  Place cur = {q, s, s_end, l, g}, nxt = cur;
  auto line_of = [&](int slab) __attribute__((always_inline)) { return lines_cur + ((size_t)slab << (p.lgP + 5)); };
  // the slab behind `cur`: of this run or the team's next one; its requests begin
  auto move_on = [&](int buf) __attribute__((always_inline)) {
    int nq = cur.q, ns = cur.s + 1, ns_end = cur.s_end, nl = cur.l, ng = cur.g + 1;
    if (ng == p.H_kv) { ng = 0; ++nl; }
    if (ns == cur.s_end) {
      ++nq;
      ns = deal.start(team, nq);
      ns_end = deal.end(nq, ns);
      nl = ns / p.H_kv;
      ng = ns - nl * p.H_kv;
    }
    nxt = {nq, ns, ns_end, nl, ng};
    const bool more = nxt.s < deal.n_slabs;
    w.nx.left = 0;
    if (more) {
      w.nx = {w.slab_keys(nxt.l, nxt.g, 0), 0, key0, M, nt};
      w.issue_queries(nxt.l, nxt.g, 0, buf ^ 1);
    }
    w.begin_slab();
    w.slab_scale(cur.l, cur.g);
    return more;
  };
  // this member's statistics of a slab for the others
  auto publish = [&](int slab, float own) __attribute__((always_inline)) {
    if (w.wave == 0) {
      const int ln = W::lane_id();
      if (ln < 32) {  // (-inf -- no key of the prompt in this workgroup -- is a value, not "empty")
        store32_agent(line_of(slab) + member * 32 + ln, __float_as_uint(own));
        lines_nxt[((size_t)slab << (p.lgP + 5)) + member * 32 + ln] = kEmptyLine;
      }
    }
  };
  // the whole team's: the lane's row's base-2 log-sum-exp
  auto team_lse = [&](int slab, int sl, int sg) __attribute__((always_inline)) {
    if (w.wave == 0) {
      const int ln = W::lane_id();
      // Lane ln holds, of load i, rows 4 * (ln % 8) .. + 3 of member i * 8 + ln / 8 (lanes beyond the last member read
      // nothing and get zeros).
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(line_of(slab), 0, (uint32_t)P * 128u, 0x00020000);
      const int loads = P <= 8 ? 1 : P >> 3;
      uint32_t since = 0;  // when this slab's wait began
      float m[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY}, z[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int i0 = 0; i0 < loads; i0 += 4) {  // four loads at a time: more registers are not free
        u32x4 x[4];
        // The loads come before any question: with a way around them the compiler clears and copies x in front of every fold
        // (32 layers, d = 128, us: 128K 8-bit keys 879 -> 863, 32K bf16 keys 342.7 -> 341.3; 16 layers, d = 64, 33000 8-bit
        // keys 141.1 -> 138.9).  One look at most where the wait is given up: what it finds is formed again or refused.
        for (;;) {
          bool empty = false;
          asm volatile("" ::: "memory");  // (a new look at the lines every time)
          uint32_t given_up = 0;
          if (p.launch == kFirst) given_up = __hip_atomic_load(p.status + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            x[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, ln * 16 + (i0 + i) * 1024, 0, /*sc1*/ 16));
#pragma unroll
          for (int i = 0; i < 4; ++i)
            empty |= x[i].x == kEmptyLine || x[i].y == kEmptyLine || x[i].z == kEmptyLine || x[i].w == kEmptyLine;
          if (!__any(empty) || expired || M <= 0) break;  // (a member without keys has no use for the rows' log-sum-exps)
          if (--polls <= 0) expired = true;
          if (p.launch == kFirst) {
            const uint32_t now = (uint32_t)wall_clock64() | 1u;
            if (since == 0) since = now;
            if (__builtin_amdgcn_readfirstlane(given_up) != 0 || now - since > p.patience) expired = true;
            if (expired) __hip_atomic_store(p.status + 3, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          __builtin_amdgcn_s_sleep(2);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float mn = m[c];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((i0 + i) * 8 + (ln >> 3) < P) mn = fmaxf(mn, __uint_as_float(x[i][c]));
          const float ref = (mn == -INFINITY) ? 0.f : mn;
          z[c] *= fast_exp2(m[c] - ref);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((i0 + i) * 8 + (ln >> 3) < P) z[c] += fast_exp2(__uint_as_float(x[i][c]) - ref);
          m[c] = mn;
        }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float mx = fmaxf(m[c], __shfl_xor(m[c], 8, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));  // finite: the prompt is not empty
        z[c] *= fast_exp2(m[c] - mx);
        m[c] = mx;
      }
      u32x4 out;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        z[c] += __shfl_xor(z[c], 8, kWave);
        z[c] += __shfl_xor(z[c], 16, kWave);
        z[c] += __shfl_xor(z[c], 32, kWave);
        out[c] = __float_as_uint(m[c] + __builtin_amdgcn_logf(z[c]));
      }
      if (ln < 8) lds_poke128(lse_lds + ln * 16, out);  // rows 4 * ln .. + 3
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();
    const float lse2 = __uint_as_float(lds_peek(lse_lds + (W::lane_id() & 31) * 4));
    if (p.lse_out && member == 0 && w.wave == 0) w.store_lse(sl, sg, 0, lse2);
    return lse2;
  };
  // log2-probabilities of a held tile; maximum over the heads of a group and over the slabs
  auto fold = [&](auto tc, float c2, float neg_lse2) __attribute__((always_inline)) {
    constexpr int t = decltype(tc)::value;
    float y[KEEP];
    W::fold_heads(held[t], c2, neg_lse2, y);
#pragma unroll
    for (int k = 0; k < KEEP; ++k) run[t][k] = fmaxf(run[t][k], y[k]);
  };
  // The results, behind the fold of slab `of`.  Maximum over layers: one group per team, at its end.  Mean: a run of a round
  // is a layer, whose maxima join the sum in the team's group (registers for the sums would be a quarter of what the logits
  // leave); a part of a layer has a group of its own behind the teams'.
  auto results = [&](const Place& of, bool last) __attribute__((always_inline)) {
    if (!(mean ? of.s + 1 == of.s_end : last)) return;
    const bool sum = mean && of.q < deal.rounds;
    const int group = !mean || sum ? team : p.plain_groups + (of.s - deal.base()) / deal.part;
    const int q_n = W::lane_id() & (W::NS - 1);
    const int64_t step = (int64_t)p.n_groups * p.N * 32;  // from tile to tile
    float* const out = p.group_scores + ((int64_t)((key0 >> 5) + w.wave + (nt - 1) * kTiledWaves) * p.n_groups + group) * p.N * 32 +
                       q_n * 32 + w.fold_key();
    const int64_t back = kTiledWaves * step;              // from one of the wave's tiles to the next
    if (sum) {
      constexpr int STEP = LG == 1 ? 2 : 4;  // tiles whose loads go out together
      wide_static_for<0, MAXT / STEP>([&](auto bc) __attribute__((always_inline)) {
        constexpr int t0 = decltype(bc)::value * STEP;
        vkeep old[STEP];
#pragma unroll
        for (int i = 0; i < STEP; ++i)
#pragma unroll
          for (int k = 0; k < KEEP; ++k) old[i][k] = 0.f;
        if (of.q > 0 && q_n < p.N) {
#pragma unroll
          for (int i = 0; i < STEP; ++i)
            if (t0 + i < nt) old[i] = W::load_keep(out - (t0 + i) * back);
        }
#pragma unroll
        for (int i = 0; i < STEP; ++i)
#pragma unroll
          for (int k = 0; k < KEEP; ++k) run[t0 + i][k] = old[i][k] + fast_exp2(run[t0 + i][k]);
      });
    }
    wide_static_for<0, MAXT>([&](auto tc) __attribute__((always_inline)) {
      constexpr int t = decltype(tc)::value;
      if (q_n < p.N && t < nt) W::store_keep(out - t * back, run[t]);
#pragma unroll
      for (int k = 0; k < KEEP; ++k) run[t][k] = -INFINITY;
    });
  };
  int buf = 0;
  float rm = -INFINITY, rs = 0.f;
  if constexpr (!FP8) {
    // A turn takes a slab's products and, tile by tile in front of them, folds the slab before.  That one's log-sum-exps are
    // waited for behind the first item's products, whose logits have registers of their own until then; the ring is emptied
    // without a stop between slabs.  (With the fold of all tiles as soon as the log-sum-exps are there and the next slab's
    // products behind it, in us: 32 layers of d = 128, 32K keys 349 -> 342, mean over 30011 keys 326 -> 319, 24577 keys
    // without the promise 280 -> 272; 16 layers of d = 64, 33000 keys 133 -> 123.  8-bit keys lose by it, below.)  The first
    // turn has nothing to fold -- its log-sum-exps are infinite, its logits zero --, the last one only that.
#pragma unroll
    for (int t = 0; t < MAXT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) held[t][i] = 0.f;
    Place done = cur;
    bool live = true, folds = false, more = true;
#pragma unroll 1
    for (;;) {
      f32x16 spare;
      rm = -INFINITY;
      rs = 0.f;
      if (live) {
        more = move_on(buf);
        if (nt > 0) spare = w.template item_logits<0>(nt, M, buf, rm, rs);
      }
      float neg_lse2 = -INFINITY;
      if (folds) neg_lse2 = -team_lse(done.s, done.l, done.g);
      wide_static_for<0, MAXT>([&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        if (t < nt) {
          fold(tc, w.c2, neg_lse2);
          if (live) {
            if constexpr (t == 0) held[0] = spare;
            else held[t] = w.template item_logits<t>(nt, M, buf, rm, rs);
          }
        }
      });
      if (folds) results(done, !live);
      if (!live) break;
      publish(cur.s, w.workgroup_lse(rm, rs, buf));
      w.end_slab();
      done = cur;
      cur = nxt;
      folds = true;
      live = more;
      buf ^= 1;
    }
  } else {
    // The first item of the next slab is computed while the lines of this one travel (its logits wait in registers of
    // their own), the other tiles' fold comes before its other products: 8-bit keys, which arithmetic bounds, take 219 us so
    // at 32K keys of 32 layers of d = 128 and 139 at 33000 of 16 layers of d = 64, 227 and 146 in the order above.
    f32x16 spare;
    bool early = false;  // the first item of the slab at hand is in `spare`, its statistics in (rm, rs)
#pragma unroll 1
    for (;;) {
      const bool more = move_on(buf);
      if (early) {
        held[0] = spare;
      } else {
        rm = -INFINITY;
        rs = 0.f;
        if (nt > 0) held[0] = w.template item_logits<0>(nt, M, buf, rm, rs);
      }
      w.template slab_logits<MAXT, 1>(held, nt, M, buf, rm, rs);
      publish(cur.s, w.workgroup_lse(rm, rs, buf));
      const float c2 = w.c2;
      early = more && nt > 0;
      if (early) {
        rm = -INFINITY;
        rs = 0.f;
        w.slab_scale(nxt.l, nxt.g);
        spare = w.template item_logits<0>(nt, M, buf ^ 1, rm, rs);
      }
      const float lse2 = team_lse(cur.s, cur.l, cur.g);
      wide_static_for<0, MAXT>([&](auto tc) __attribute__((always_inline)) {
        if (decltype(tc)::value < nt) fold(tc, c2, -lse2);
      });
      results(cur, !more);
      w.end_slab();
      if (!more) break;
      cur = nxt;
      buf ^= 1;
    }
  }
  if (w.wave == 0 && expired && W::lane_id() == 0) atomicOr(p.status + (p.launch == kFirst ? 3u : epoch & 1u), 1u);
  wait_vmcnt<0>();
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
static size_t copy_bytes(const WideTeamPlan& pl) { return (size_t)pl.deal.n_slabs * 128 << pl.lgP; }
static size_t result_bytes(const WideTeamPlan& pl, const sp_score_args* a) {
  return align_up(sizeof(float) * 32 * (size_t)pl.n_groups * a->N * wide_tiles(a), 256);
}

static WideTeamPlan make_plan(const sp_score_args* a) { return make_wide_team_plan(a, wide_team_wgs(seq_cu_count())); }
bool wide_team_supported(const sp_score_args* a) { return make_plan(a).ok; }
// Workspace: the lines' two copies, the status words, the results.  What a call hands on to the next (lines and status)
// sits where the shape alone says, whatever the cut into result groups, which the kind of cache may change.
size_t wide_team_workspace_bytes(const sp_score_args* a) {
  const WideTeamPlan pl = make_plan(a);
  return pl.ok ? align_up(2 * copy_bytes(pl), 256) + result_bytes(pl, a) + 256 : 0;
}
size_t wide_team_status_offset(const sp_score_args* a) {
  const WideTeamPlan pl = make_plan(a);
  return pl.ok ? align_up(2 * copy_bytes(pl), 256) : 0;
}

template <int D, int LG, bool FP8, bool PAGED>
static sp_status launch_wide_team(const WideTeamDev& dev, hipStream_t stream) {
  auto kernel = wide_team_kernel<D, LG, FP8, PAGED>;
  constexpr int smem = WideKernel<D, LG, FP8, PAGED>::kSmem + 128;
  // once per kernel and device, under a lock: allow the large dynamic LDS size and make sure the whole grid can be
  // resident at once (one workgroup per compute unit)
  static std::mutex mu;
  static bool prepared[kMaxDevices] = {};
  {
    std::lock_guard<std::mutex> lock(mu);
    const int slot = current_device();
    if (!prepared[slot]) {
      int per_cu = 0;
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess ||
          hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kernel), kTiledThreads, smem) != hipSuccess ||
          per_cu < 1)
        return SP_ELAUNCH;
      prepared[slot] = true;
    }
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)(dev.deal.teams << dev.lgP)), dim3(kTiledThreads), smem, stream, dev);
  return launch_status();
}
template <int D, int LG, bool FP8>
static sp_status wide_team_by_pages(const WideTeamDev& dev, hipStream_t stream) {
  return dev.block_table ? launch_wide_team<D, LG, FP8, true>(dev, stream) : launch_wide_team<D, LG, FP8, false>(dev, stream);
}
template <int D>
static sp_status wide_team_by_kind(const sp_score_args* a, const WideTeamDev& dev, hipStream_t stream) {
  const bool fp8 = a->k_dtype == SP_K_FP8_E4M3;
  if (dev.lgG == 1) return fp8 ? wide_team_by_pages<D, 1, true>(dev, stream) : wide_team_by_pages<D, 1, false>(dev, stream);
  if (dev.lgG == 2) return fp8 ? wide_team_by_pages<D, 2, true>(dev, stream) : wide_team_by_pages<D, 2, false>(dev, stream);
  return fp8 ? wide_team_by_pages<D, 3, true>(dev, stream) : wide_team_by_pages<D, 3, false>(dev, stream);
}

sp_status wide_team_score(const sp_score_args* a, hipStream_t stream) {
  const WideTeamPlan pl = make_plan(a);
  if (!pl.ok) return SP_EUNSUPPORTED;
  WideTeamDev dev = {};
  dev.B = 1; dev.N = a->N; dev.L = a->L; dev.H = a->H; dev.H_kv = a->H_kv; dev.G = a->H / a->H_kv;
  dev.lgG = wide_team_lg(a);
  dev.Gp = 1 << dev.lgG;
  dev.layer_reduce = a->layer_reduce;
  dev.scale = a->scale;
  dev.c = a->scale * 1.4426950408889634f;
  dev.ts = a->k_token_stride; dev.hs = a->k_head_stride; dev.T = a->T;
  dev.q = static_cast<const uint16_t*>(a->d_q);
  dev.cu = a->d_cu_seqlens; dev.n_valid = a->d_n_valid;
  dev.scores = a->d_scores; dev.lse_out = a->d_lse;
  dev.deal = pl.deal;
  dev.n_groups = pl.n_groups; dev.plain_groups = pl.plain_groups; dev.groups_per_layer = pl.gpl;
  dev.block_table = a->d_block_table;
  while (a->d_block_table && (1 << dev.lg_page) < a->page_size) ++dev.lg_page;
  dev.blocks_per_seq = a->blocks_per_seq;
  dev.page_stride = a->k_page_stride;
  dev.k_scale = a->d_k_scale;
  for (int l = 0; l < a->L; ++l) dev.k[l] = static_cast<const uint16_t*>(a->k_layers[l]);
  dev.lgP = pl.lgP; dev.share = pl.share;
  const bool shared = !(a->flags & SP_SCORE_EXCLUSIVE_DEVICE);
  dev.launch = shared ? kFirst : kAlone;
  dev.spin_budget = g_spin_budget.load(std::memory_order_relaxed);
  dev.patience = shared ? (uint32_t)wide_team_patience_us(pl, a) * 100u : 0u;
  char* ws = static_cast<char*>(a->d_workspace);
  dev.lines = reinterpret_cast<uint32_t*>(ws);
  dev.copy_words = copy_bytes(pl) / 4;
  dev.status = reinterpret_cast<uint32_t*>(ws + wide_team_status_offset(a));
  dev.group_scores = reinterpret_cast<float*>(ws + wide_team_status_offset(a) + 256);
  if (shared || !(a->flags & SP_SCORE_WORKSPACE_KEPT)) {
    const size_t n_vec = copy_bytes(pl) / 16;
    hipLaunchKernelGGL(wide_team_fill_kernel, dim3((unsigned)std::min<size_t>((n_vec + 255) / 256, 1024)), dim3(256), 0, stream,
                       reinterpret_cast<uint4*>(ws), n_vec, dev.status);
    if (hipGetLastError() != hipSuccess) return SP_ELAUNCH;
  }
  sp_status st = a->d == 64 ? wide_team_by_kind<64>(a, dev, stream) : wide_team_by_kind<128>(a, dev, stream);
  if (st == SP_OK && shared) {
    dev.launch = kSecond;
    dev.spin_budget = kDefaultSpinBudget;  // (whatever the bound: the lines are all there, one poll per look is enough)
    st = a->d == 64 ? wide_team_by_kind<64>(a, dev, stream) : wide_team_by_kind<128>(a, dev, stream);
  }
  if (st != SP_OK) return st;
  return launch_wide_finish(dev, (unsigned)wide_tiles(a), dev.status, stream);
}

}  // namespace sp

extern "C" int32_t sp_set_wait_budget(int32_t polls) {
  if (polls < 0) return sp::g_spin_budget.load(std::memory_order_relaxed);
  return sp::g_spin_budget.exchange(polls, std::memory_order_relaxed);
}
