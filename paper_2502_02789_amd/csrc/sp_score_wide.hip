// Single-pass MFMA scorer for short prompts whose KV heads carry more than a handful of query rows (the paper's
// default with look-ahead, Sec. 3.2.1): batches, or one prompt of up to about three thousand tokens.
//
// Same quantity as the other scoring kernels: row softmax of the stored queries against the prompt keys
// (Sec. 3.2 equation of arXiv 2502.02789), max over heads, max/mean over layers, mean over queries (Sec. 3.2.2).
// As in the kernel for few query rows (sp_score_seq.hip) one workgroup owns a whole sequence for a run of
// (layer, KV head) slabs, so a softmax row never leaves the compute unit, K is read once and nobody waits for
// another workgroup; but here the rows are the 32 COLUMNS of the MFMA result:
//
//   * A lane holds one query row for 16 keys of a 32-key tile: the row statistics are plain per-lane maxima and
//     sums (no shuffles inside a slab), and the 16 logits stay in the accumulator registers for the slab:
//     16 registers per tile, eight waves x MAXT tiles x 32 keys.
//   * Query row (query n, head j of the group) sits in column n + NS * j (NS = 32 / padded heads).  The maximum
//     over the heads of a group is then a maximum over lane bits 4 and 3 (and 2 with eight heads): each step
//     halves the registers instead of repeating the result in every lane (v_permlane16_swap, then v_max_f32 with
//     DPP row rotation and bank masks): a lane ends up with four consecutive keys of one query.
//   * The query tile of a slab is fetched ONCE per workgroup (the tiled and exchange kernels fetch it once per
//     wave and 64 keys, half as many bytes again as the keys) one slab ahead, and both operands are read from LDS.
//   * A wave's ring holds 16 KiB whatever the element size and head dim (two, four or eight items of 32 keys), so the
//     bytes in flight per compute unit are the same for all of them.  The loads go through a buffer descriptor per item
//     whose range ends with the sequence: no address arithmetic per lane, and keys that do not exist are not read.
//   * A wave takes its items of a slab from the last to the first, so that only one copy of the unrolled tile code
//     (the first) has to know about the ragged end of a sequence; the code has to stay small, a kernel that makes
//     one round through it per launch otherwise spends its time on instruction fetches.
//   * At the end of a slab: the waves' (max, sum) pairs meet in LDS, one bare s_barrier, every wave knows the
//     log-sum-exps; the stream of key tiles runs on underneath.
//   * Results go out as [32-key tile][slab group][query][32]: one dense 1 KiB store per tile here, one dense read
//     per tile in the merge.
//
// The running maximum over a unit's slabs takes four registers per tile.  Sequences whose tiles leave room for all of
// them (nine tiles per wave) have it there; longer ones only for a wave's first tiles, and in the unit's result
// array for the others, which writes (and reads back) up to an eighth of the key bytes: 16 prompts of 2600 keys take
// 544 us, 459 of them without those writes (writes cost the stream more than their bytes), 16 prompts of 300..3000
// keys 374 us with all running maxima in memory and 338 this way.  Both forms of the slab loop are in the kernel.
// Bound by the HBM stream of K and, beyond 2304 keys, by the result writes.  Measured (32 layers, 8 KV heads, d = 128,
// eight queries; two-pass or exchange kernels before): 16 ragged prompts of 300..3000 keys (1.73 GB) out of a paged
// cache 1005 -> 331 us, one prompt of 3001 keys 138 -> 43 us (+ merge 7 us).  Neither the matrix cores nor the
// exponentials limit it (either taken out: no change).
#include <mutex>

#include "sp_wide_core.h"

namespace sp {

constexpr int kWideTiles = 12;    // 32-key tiles per wave, and the first
constexpr int kWideRunTiles = 4;  // of them whose running maxima are in registers where not all fit

template <int D, int LG, bool FP8, bool PAGED, bool STRETCHES>
__global__ __launch_bounds__(kTiledThreads) void wide_score_kernel(const TiledDev p) {
  extern __shared__ __align__(1024) unsigned char smem[];
  using W = WideKernel<D, LG, FP8, PAGED, false>;
  constexpr int KEEP = W::KEEP;
  constexpr int kShort = 9;  // tiles per wave that fit with all their running maxima in registers
  using vkeep = typename W::vkeep;
  W w(p, smem);
  SeqUnit cur;
  if (!seq_first_unit<STRETCHES>(p, &cur)) return;

  int l = __builtin_amdgcn_readfirstlane(cur.s0 / p.H_kv), g = cur.s0 - l * p.H_kv;
  w.ah = {w.slab_keys(l, g, cur.seq0), cur.b, 0, cur.M, w.items_of(cur.M)};
  w.issue_queries(l, g, cur.b, 0);
  w.start_stream();
  w.first_queries();

  int slabs = 0;  // slabs finished so far
  bool more = true;
  SeqUnit nxt = cur;  // the unit of the slab behind the one at hand

  // all slabs of unit `cur`, tiles_c tiles per wave of which the first run_c have their running maxima in registers
  auto do_unit = [&](auto tiles_c, auto run_c) __attribute__((always_inline)) {
    constexpr int MAXT = decltype(tiles_c)::value, RUN = decltype(run_c)::value;
    f32x16 held[MAXT];
    vkeep run[RUN];
    const int M = cur.M, b = cur.b;
    const int nt = w.items_of(M);
#pragma unroll
    for (int t = 0; t < RUN; ++t)
#pragma unroll
      for (int k = 0; k < KEEP; ++k) run[t][k] = -INFINITY;
    // result array of this unit: element [tile][group][query][32 keys]
    float* const out0 = p.group_scores + ((int64_t)wide_tile_base(cur.seq0, b) * p.n_groups + cur.grp) * p.N * 32;
    const int64_t out_step = (int64_t)p.n_groups * p.N * 32;  // from tile to tile
#pragma unroll 1
    for (int s = cur.s0; s < cur.s1; ++s) {
      const int buf = slabs & 1;
      // the next slab: its query tile goes into the buffer the previous slab has just left (the barrier at its
      // end); requests move on to it when this slab's items have all been sent
      int nl = l, ng = g + 1;
      if (ng == p.H_kv) { ng = 0; ++nl; }
      w.nx.left = 0;
      // (In rounds the slab of the same unit has a way of its own, without what a next unit looks up: 128 prompts of 125..250
      // keys, eight queries, 390 us with one set-up behind both ways, 359 so; 64 of 320..400 8-bit keys 229 and 222.  In
      // stretches, where it is the other way round, one: 64 of 100..700 342 and 357.)
      if (!STRETCHES && s + 1 < cur.s1) {
        w.nx = {w.slab_keys(nl, ng, cur.seq0), b, 0, M, nt};
        w.issue_queries(nl, ng, b, buf ^ 1);
      } else {
        if (s + 1 == cur.s1) {
          more = seq_next_unit<STRETCHES>(p, &nxt);
          nl = __builtin_amdgcn_readfirstlane(nxt.s0 / p.H_kv);
          ng = nxt.s0 - nl * p.H_kv;
        }
        if (more) {
          w.nx = {w.slab_keys(nl, ng, nxt.seq0), nxt.b, 0, nxt.M, w.items_of(nxt.M)};
          w.issue_queries(nl, ng, nxt.b, buf ^ 1);
        }
      }
      w.begin_slab();
      w.slab_scale(l, g);
      float rm = -INFINITY, rs = 0.f;
      w.slab_logits(held, nt, M, buf, rm, rs);
      const float lse2 = w.workgroup_lse(rm, rs, buf);
      const float neg_lse2 = -lse2;
      ++slabs;
      if (p.lse_out && w.wave == 0) w.store_lse(l, g, b, lse2);

      // log2-probabilities; maximum over the heads of a group and over the unit's slabs
      const int first = w.fold_key(), q_n = W::lane_id() & (W::NS - 1);
      float* out = out0 + (w.wave + (nt - 1) * kTiledWaves) * out_step + q_n * 32 + first;
      auto place = [&](int t) __attribute__((always_inline)) {  // of a tile's results
        return reinterpret_cast<vkeep*>(out - t * kTiledWaves * out_step);
      };
      wide_static_for<0, RUN>([&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        if (t < nt) {
          float x[KEEP];
          w.fold_heads(held[t], neg_lse2, x);
#pragma unroll
          for (int k = 0; k < KEEP; ++k) run[t][k] = fmaxf(run[t][k], x[k]);
        }
      });
      // the other tiles two at a time: what the unit's earlier slabs left is requested for all of them before the
      // first is needed (one after the other each would wait for its own round trip to L2)
      constexpr int STEP = 2;
      wide_static_for<0, (MAXT - RUN + STEP - 1) / STEP>([&](auto bc) __attribute__((always_inline)) {
        constexpr int t0 = RUN + decltype(bc)::value * STEP, tn = t0 + STEP <= MAXT ? STEP : MAXT - t0;
        if (t0 < nt) {
          vkeep old[tn];
#pragma unroll
          for (int i = 0; i < tn; ++i)
#pragma unroll
            for (int k = 0; k < KEEP; ++k) old[i][k] = -INFINITY;
          if (s != cur.s0 && q_n < p.N) {
#pragma unroll
            for (int i = 0; i < tn; ++i)
              if (t0 + i < nt) old[i] = *place(t0 + i);
          }
#pragma unroll
          for (int i = 0; i < tn; ++i) {
            float x[KEEP];
            w.fold_heads(held[t0 + i], neg_lse2, x);
#pragma unroll
            for (int k = 0; k < KEEP; ++k) old[i][k] = fmaxf(old[i][k], x[k]);
          }
          if (q_n < p.N) {
#pragma unroll
            for (int i = 0; i < tn; ++i)
              if (t0 + i < nt) __builtin_nontemporal_store(old[i], place(t0 + i));
          }
        }
      });
      if (s + 1 == cur.s1 && q_n < p.N) {  // the unit's result
        wide_static_for<0, RUN>([&](auto tc) __attribute__((always_inline)) {
          constexpr int t = decltype(tc)::value;
          if (t < nt) __builtin_nontemporal_store(run[t], place(t));
        });
      }
      if (s + 1 == cur.s1) note_group_count<STRETCHES>(p, cur);
      w.end_slab();
      l = nl;
      g = ng;
    }
  };
#pragma unroll 1
  for (;;) {
    if (cur.M <= kShort * 32 * kTiledWaves) do_unit(std::integral_constant<int, kShort>{}, std::integral_constant<int, kShort>{});
    else do_unit(std::integral_constant<int, kWideTiles>{}, std::integral_constant<int, kWideRunTiles>{});
    if (!more) break;
    cur = nxt;
  }
  wait_vmcnt<0>();
}

// Merge of the units' results and the average over the valid queries.  One workgroup per 32-key tile (or per half
// of one: KEYS = 16): it reads one dense block, KEYS / 4 threads per (group, query) row, every thread keeps to one query, the
// threads of a query meet in LDS.  Sequences the scoring kernel left out (longer than it holds) get NaN.
// Bound by its dependent steps: the first eight rows of a thread are requested before anything else is looked at (they lie
// in the result array whatever it says), a single sequence is not looked up, and rows are divided by the number of queries
// with one reciprocal.  LAYERS: the mean over layers from parts of layers, a kernel of its own (the look at what the rows are
// would come in front of the first request of the other: 178 keys 13.6 -> 14.7 us).  Whole call, eight queries, before -> now:
// mean over layers 700 keys 21.1 -> 19.9 us, 16 layers of d = 64, 1800 keys 20.9 -> 19.8; 28 layers, 224 results a tile, 700 keys 18.9 -> 17.2.
template <int KEYS, int THREADS, bool LAYERS>
__global__ __launch_bounds__(THREADS) void wide_finish_kernel(const TiledDev p, uint32_t* status) {
  constexpr int TPR = KEYS / 4;            // threads per row
  constexpr int ROWS = THREADS / TPR;      // rows per step
  constexpr int AHEAD = 8;
  __shared__ float red[ROWS][KEYS];
  const int tile = blockIdx.x / (32 / KEYS), part = blockIdx.x % (32 / KEYS);
  const bool mean = p.layer_reduce != SP_LAYER_MAX;
  const uint32_t inverse = 65536u / (uint32_t)p.N + 1u;  // x / N = x * inverse >> 16 for x below 4096
  const int per = (int)(ROWS * inverse >> 16);           // groups (mean: layers) per step
  const int row = threadIdx.x / TPR, quad = threadIdx.x % TPR;
  const int g0 = (int)((uint32_t)row * inverse >> 16), n = row - g0 * p.N;
  const int64_t step = (int64_t)p.N * 32;
  const float* src = p.group_scores + ((int64_t)tile * p.n_groups * p.N + n) * 32 + part * KEYS + quad * 4;
  // What is requested ahead: rows of the thread's groups, or, where parts of layers are all there is, of its first layer (whole
  // layers then are rows like the others, but logarithms).
  const int gpl = LAYERS ? p.groups_per_layer : 1;
  const bool layers_only = LAYERS && p.plain_groups == 0, logs = layers_only && gpl == 1;
  // Parts of a layer are taken eight at a time: two layers (the thread's next one lies `per` behind) of up to four parts, or one.
  const bool pairs = gpl <= 4;
  auto part_row = [&](int l, int j, int i) __attribute__((always_inline)) {  // (i: which of eight; beyond the last layer or part that one again)
    const int first = min((pairs && i >= 4 ? l + per : l) * gpl, p.n_groups - p.plain_groups - gpl);
    return first + min(pairs ? i & 3 : j + i, gpl - 1);
  };
  f32x4 ahead[AHEAD];
  if (layers_only && !logs) {
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) ahead[i] = *reinterpret_cast<const f32x4*>(src + part_row(g0, 0, i) * step);
  } else {
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) ahead[i] = *reinterpret_cast<const f32x4*>(src + min(g0 + i * per, p.n_groups - 1) * step);
  }

  int lo = 0, seq0 = 0, M = (int)p.T;
  if (p.B > 1) {                           // the sequence: the largest b whose first tile is <= tile
    int hi = p.B;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (wide_tile_base(p.cu[mid], mid) <= tile) lo = mid; else hi = mid;
    }
    seq0 = p.cu[lo];
    M = p.cu[lo + 1] - seq0;
  }
  const int key0 = (tile - wide_tile_base(seq0, lo)) * 32 + part * KEYS;
  // (exchange kernels: words 0 and 1 say whether a wait of this call expired -- the other parity's word is clear --,
  // word 2 counts the calls)
  const bool expired = status != nullptr && (status[0] | status[1]) != 0;
  if (status != nullptr && blockIdx.x == 0 && threadIdx.x == 0) status[2] += 1;
  if (key0 >= M) return;
  if (expired || (p.seq_limit > 0 && M > p.seq_limit)) {
    if (threadIdx.x < KEYS && key0 + (int)threadIdx.x < M) p.scores[seq0 + key0 + threadIdx.x] = __uint_as_float(0x7FC00000u);
    return;
  }
  const int n_groups = p.group_count ? p.group_count[lo] : p.n_groups;
  f32x4 v = mean ? f32x4{0.f, 0.f, 0.f, 0.f} : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  if (g0 < per) {
    auto take = [&](const f32x4& x) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        v[k] = mean ? v[k] + (logs ? fast_exp2(x[k]) : x[k]) : fmaxf(v[k], x[k]);  // (mean: sums over a group's layers)
    };
    const int plain = LAYERS && !logs ? p.plain_groups : n_groups;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
      if (g0 + i * per < plain) take(ahead[i]);
    int g = g0 + AHEAD * per;
    for (; g + (AHEAD - 1) * per < plain; g += AHEAD * per) {
      f32x4 x[AHEAD];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) x[i] = *reinterpret_cast<const f32x4*>(src + (g + i * per) * step);
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) take(x[i]);
    }
    if (g < plain) {  // (what is left, all at once: of 192 or 224 groups four or six rows, which a loop waits for one by one)
      f32x4 x[AHEAD - 1];
#pragma unroll
      for (int i = 0; i < AHEAD - 1; ++i) x[i] = *reinterpret_cast<const f32x4*>(src + min(g + i * per, plain - 1) * step);
#pragma unroll
      for (int i = 0; i < AHEAD - 1; ++i)
        if (g + i * per < plain) take(x[i]);
    }
    if (LAYERS && !logs) {  // the groups of a layer hold the log2 of its maxima over their KV heads; the layers' maxima add up
      src += p.plain_groups * step;
      const int layers = (p.n_groups - p.plain_groups) / gpl;
      for (int l = g0; l < layers; l += pairs ? 2 * per : per) {
        f32x4 m[2] = {{-INFINITY, -INFINITY, -INFINITY, -INFINITY}, {-INFINITY, -INFINITY, -INFINITY, -INFINITY}};
        for (int j = 0; j < gpl; j += AHEAD) {
          f32x4 x[AHEAD];
          if (layers_only && l == g0 && j == 0) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) x[i] = ahead[i];
          } else {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) x[i] = *reinterpret_cast<const f32x4*>(src + part_row(l, j, i) * step);
          }
#pragma unroll
          for (int i = 0; i < AHEAD; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) m[i / 4][k] = fmaxf(m[i / 4][k], x[i][k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (!pairs) v[k] += fast_exp2(fmaxf(m[0][k], m[1][k]));
          else v[k] += fast_exp2(m[0][k]) + (l + per < layers ? fast_exp2(m[1][k]) : 0.f);
        }
      }
    }
  }
  *reinterpret_cast<f32x4*>(&red[row][quad * 4]) = v;
  __syncthreads();
  // all threads fold the rows of a (query, key), then KEYS * N of them the THREADS / (KEYS * N) results of each
  const int fk = threadIdx.x % KEYS, fr = threadIdx.x / KEYS, sub = (int)((uint32_t)fr * inverse >> 16), fn = fr - sub * p.N;
  const int subs = max(1, (int)((uint32_t)(THREADS / KEYS) * inverse >> 16));
  float x = mean ? 0.f : -INFINITY;
  if (sub < subs) {
#pragma unroll 4
    for (int q = sub; q < per; q += subs) {
      const float y = red[q * p.N + fn][fk];
      x = mean ? x + y : fmaxf(x, y);
    }
  }
  __syncthreads();
  if (subs > 1) {
    if (sub < subs) red[sub * p.N + fn][fk] = x;
    __syncthreads();
    if (sub == 0) {
#pragma unroll 4
      for (int q = 1; q < min(subs, per); ++q) {
        const float y = red[q * p.N + fn][fk];
        x = mean ? x + y : fmaxf(x, y);
      }
    }
  }
  if (sub == 0) red[fn][fk] = mean ? x : fast_exp2(x);  // (rows 0..N-1 are read by their own threads only)
  __syncthreads();
  if (threadIdx.x >= KEYS || key0 + fk >= M) return;
  int nv = p.n_valid ? p.n_valid[lo] : p.N;
  nv = max(1, min(nv, p.N));
  float sum = 0.f;
#pragma unroll 8
  for (int q = 0; q < nv; ++q) sum += red[q][fk];
  p.scores[seq0 + key0 + fk] = sum / (mean ? (float)nv * (float)p.L : (float)nv);
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
int wide_max_keys(const sp_score_args*) { return kWideTiles * 32 * kTiledWaves; }
static int64_t wide_stated_max(const sp_score_args* a) { return a->B == 1 ? a->T : a->max_seqlen; }

bool wide_supported(const sp_score_args* a) {
  if (a->rope_theta > 0.f || wide_stated_max(a) <= 0 || a->T < 1) return false;
  if (a->H / a->H_kv > 8 || (a->N << wide_lg(a)) > 32) return false;
  if (a->k_dtype == SP_K_FP8_E4M3 && a->d_block_table && a->page_size < (a->d == 64 ? 16 : 8)) return false;
  if (wide_stated_max(a) > wide_max_keys(a)) return false;
  if (a->k_token_stride > (INT32_MAX / 256)) return false;  // (a ring slot's keys must span less than 2 GiB)
  if (a->B > 8192) return false;
  // Units: a workgroup owns a whole sequence, so one prompt of a small draft leaves compute units idle.  Against the two
  // passes (which cut it over the whole device) it is ahead from 64 units on (8 layers, 8 KV heads, d = 128, eight
  // queries: 500 keys 15 us against 23, 3000 keys 32 against 33; d = 64 13 against 18, 26 against 27).  The teams of
  // workgroups that the promise of an idle device allows would be ahead of both for 64 units beyond some 1000 keys too (3000
  // keys: 22 us); there they are not taken, so that one short prompt has the same scores, bit for bit, with and without the
  // promise (from 128 units and 2048 keys on they may be, two_to_a_slab in sp_score.hip).
  if ((int64_t)a->B * a->L * a->H_kv < 64) return false;
  return true;
}

// Units: runs of slabs; with the mean over layers parts of one layer (the merge adds the layers up).
static UnitDeal wide_deal(const sp_score_args* a, int* n_groups) {
  *n_groups = 0;
  return a->layer_reduce == SP_LAYER_MEAN ? UnitDeal{} : make_unit_deal(a, seq_cu_count(), wide_max_keys(a), false, n_groups);
}
void wide_grouping(const sp_score_args* a, int* slabs_per_group, int* n_groups, int* groups_per_layer) {
  *groups_per_layer = 0;
  *slabs_per_group = 1;
  if (wide_deal(a, n_groups).stretch != 0) return;
  if (a->layer_reduce == SP_LAYER_MEAN) {
    int per = 1;
    for (int cand = a->H_kv; cand >= 1; --cand)
      if (a->H_kv % cand == 0 && (int64_t)a->B * a->L * (a->H_kv / cand) >= 512) { per = cand; break; }
    *slabs_per_group = per;
    *groups_per_layer = a->H_kv / per;
    *n_groups = a->L * *groups_per_layer;
    return;
  }
  *n_groups = round_groups(a, 1, slabs_per_group);
}

static size_t wide_scores_bytes(const sp_score_args* a) {
  int per, groups, gpl;
  wide_grouping(a, &per, &groups, &gpl);
  return align_up(sizeof(float) * 32 * (size_t)groups * a->N * wide_tiles(a), 256);
}
size_t wide_workspace_bytes(const sp_score_args* a) {
  if (!wide_supported(a)) return 0;
  return wide_scores_bytes(a) + align_up(sizeof(int32_t) * (size_t)a->B, 256);
}

template <int D, int LG, bool FP8, bool PAGED, bool STRETCHES>
static sp_status launch_wide(const TiledDev& dev, hipStream_t stream) {
  auto kernel = wide_score_kernel<D, LG, FP8, PAGED, STRETCHES>;
  const size_t smem = WideKernel<D, LG, FP8, PAGED>::kSmem;
  static std::mutex mu;  // once per kernel and device
  static bool prepared[kMaxDevices] = {};
  {
    std::lock_guard<std::mutex> lock(mu);
    const int slot = current_device();
    if (!prepared[slot]) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)smem) != hipSuccess)
        return SP_ELAUNCH;
      prepared[slot] = true;
    }
  }
  const int wgs = STRETCHES ? seq_cu_count() : std::min(dev.B * dev.n_groups, seq_cu_count());
  hipLaunchKernelGGL(kernel, dim3(wgs), dim3(kTiledThreads), smem, stream, dev);
  return launch_status();
}
template <int D, int LG, bool FP8, bool PAGED>
static sp_status wide_by_deal(const TiledDev& dev, hipStream_t stream) {
  return dev.deal.stretch != 0 ? launch_wide<D, LG, FP8, PAGED, true>(dev, stream) : launch_wide<D, LG, FP8, PAGED, false>(dev, stream);
}
template <int D, int LG, bool FP8>
static sp_status wide_by_pages(const TiledDev& dev, hipStream_t stream) {
  return dev.block_table ? wide_by_deal<D, LG, FP8, true>(dev, stream) : wide_by_deal<D, LG, FP8, false>(dev, stream);
}
template <int D>
static sp_status wide_by_kind(const sp_score_args* a, const TiledDev& dev, hipStream_t stream) {
  if (a->k_dtype == SP_K_FP8_E4M3)
    return dev.lgG == 2 ? wide_by_pages<D, 2, true>(dev, stream) : wide_by_pages<D, 3, true>(dev, stream);
  return dev.lgG == 2 ? wide_by_pages<D, 2, false>(dev, stream) : wide_by_pages<D, 3, false>(dev, stream);
}

sp_status wide_score(const sp_score_args* a, const TiledDev& dev_, hipStream_t stream) {
  TiledDev dev = dev_;
  wide_grouping(a, &dev.slabs_per_group, &dev.n_groups, &dev.groups_per_layer);
  dev.lgG = wide_lg(a);
  dev.Gp = 1 << dev.lgG;
  dev.seq_limit = wide_max_keys(a);
  int n_groups;
  dev.deal = wide_deal(a, &n_groups);
  prepare_units(a, &dev, reinterpret_cast<int32_t*>(reinterpret_cast<char*>(dev.group_scores) + wide_scores_bytes(a)), dev.seq_limit, stream);
  const sp_status st = a->d == 64 ? wide_by_kind<64>(a, dev, stream) : wide_by_kind<128>(a, dev, stream);
  if (st != SP_OK) return st;
  return launch_wide_finish(dev, (unsigned)wide_tiles(a), nullptr, stream);
}

template <bool LAYERS>
static sp_status launch_finish(const TiledDev& dev, unsigned tiles, uint32_t* status, hipStream_t stream) {
  // A tile of many rows by 512 threads: 256 leave too little in flight, 1024 too few workgroups on a compute unit (whole
  // call with 256, 512 and 1024 threads, in us: 16 layers of d = 64, eight queries, 4096 keys 28.8, 27.8, 28.0, 12000 keys 51.5,
  // 51.3, 52.5; 32 layers of d = 128, 3001 keys 51.6, 50.2, 50.7, 8192 keys 101.2, 100.2, 100.8; with halves of tiles by 1024,
  // as up to 512 tiles before, 30.0, 54.8, 51.7, 103.5).  Of few rows by 256: 32K keys 340.7, 342.6, 352.8, one query on 12000 keys
  // 134.6, 135.4, 137.3.  Halves of tiles where there are so few that compute units would have none: 700 keys 20.5 against 21.2;
  // of 1792 rows a tile (28 layers of d = 64, eight queries) 1900 keys 26.1 and 28.3, 2200 28.1 and 31.4, level at 2600, 82 tiles; of 1024 rows
  // (32 layers of d = 128, four queries) level at 1300, 2200 35.8 and 35.2.
  if (dev.n_groups * dev.N <= 256 && dev.N <= 8) hipLaunchKernelGGL((wide_finish_kernel<32, 256, LAYERS>), dim3(tiles), dim3(256), 0, stream, dev, status);
  else if (tiles < (dev.n_groups * dev.N > 1024 ? 77 : 48)) hipLaunchKernelGGL((wide_finish_kernel<16, 512, LAYERS>), dim3(2 * tiles), dim3(512), 0, stream, dev, status);
  else hipLaunchKernelGGL((wide_finish_kernel<32, 512, LAYERS>), dim3(tiles), dim3(512), 0, stream, dev, status);
  return launch_status();
}

sp_status launch_wide_finish(const TiledDev& dev, unsigned tiles, uint32_t* status, hipStream_t stream) {
  return dev.layer_reduce != SP_LAYER_MAX && dev.groups_per_layer > 0 ? launch_finish<true>(dev, tiles, status, stream)
                                                                      : launch_finish<false>(dev, tiles, status, stream);
}

}  // namespace sp
