// Two-pass MFMA scorer for many query rows per KV head where no single pass is possible: batches with sequences longer
// than one workgroup holds, prompts longer than the teams of sp_score_wide_team.hip hold, and short prompts of few slabs
// (fewer than 64, up to 3072 keys) without the promise of an idle device.
//
// Same quantity as the other scoring kernels: row softmax of the stored queries against the prompt keys
// (Sec. 3.2 equation of arXiv 2502.02789), max over heads, max/mean over layers, mean over queries (Sec. 3.2.2).
// Stream, products, statistics and the fold over heads are those of sp_score_wide.hip (sp_wide_core.h); a workgroup
// owns a piece of a sequence (up to 4096 keys) for a run of (layer, KV head) slabs.  What the teams of
// sp_score_wide_team.hip exchange while they run, goes through memory between two launches here:
//
//   pass 0   per slab and piece one line of 32 base-2 log-sum-exps (nothing is held: any number of keys would do);
//   combine  the lines of a sequence's pieces -> its rows' log-sum-exps;
//   pass 1   the same products again; the rows' log-sum-exps arrive with the query tile, every tile is folded at once
//            into the running maxima (registers, four per tile);
//   merge    of the units' results as for the single-pass kernels.
//
// Against the kernels of sp_score_tiled.hip (which keep un-rotated caches, batches of unstated lengths and more than
// eight queries) the query tile is fetched once per workgroup and slab instead of once per 64 keys.
// Bound by the HBM stream of K, read twice.
#include <mutex>

#include "sp_wide_core.h"
#include "sp_wide_pass_plan.h"

namespace sp {

static_assert(kPassWaves == kTiledWaves, "the plan counts in items of the stream");

struct WidePassDev : TiledDev {
  int chunk, slots;     // keys of a piece; places for pieces: sequence b's pieces start at place pass_first_place
  float* lines;         // [slab][place][32]
  float* row_lse;       // [slab][sequence][32]
};

// piece of place `slot`: its sequence, first token, first key in it, keys (<= 0: there is no such piece)
struct Piece { int b, seq0, key0, M; };
__device__ __forceinline__ Piece piece_at(const WidePassDev& p, int slot) {
  const ScalarTable cu = scalar_table(p.cu);
  int lo = 0, hi = p.B;  // the largest b whose first place is <= slot
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pass_first_place(cu[mid], mid, p.chunk) <= slot) lo = mid; else hi = mid;
  }
  Piece u;
  u.b = lo;
  u.seq0 = cu[lo];
  u.key0 = (slot - pass_first_place(u.seq0, lo, p.chunk)) * p.chunk;
  u.M = min(p.chunk, cu[lo + 1] - u.seq0 - u.key0);
  return u;
}

struct PassUnit { int k, grp, slot, s0, s1; Piece u; };
__device__ __forceinline__ bool next_pass_unit(const WidePassDev& p, int k, PassUnit* out) {
  const int W = gridDim.x, n_units = p.slots * p.n_groups;
  for (;; ++k) {
    const int idx = k * W + (int)blockIdx.x;
    if (idx >= n_units) return false;
    const int grp = idx % p.n_groups, slot = idx / p.n_groups;
    const Piece u = piece_at(p, slot);
    const int s0 = grp * p.slabs_per_group, s1 = min(p.L * p.H_kv, s0 + p.slabs_per_group);
    if (u.M <= 0 || s0 >= s1) continue;
    *out = {k, grp, slot, s0, s1, u};
    return true;
  }
}

template <int D, int LG, bool FP8, bool PAGED, int PASS>
__global__ __launch_bounds__(kTiledThreads) void wide_pass_kernel(const WidePassDev p) {
  extern __shared__ __align__(1024) unsigned char smem[];
  using W = WideKernel<D, LG, FP8, PAGED>;
  constexpr int KEEP = W::KEEP, MAXT = kPassTiles;
  using vkeep = typename W::vkeep;
  W w(p, smem);
  const uint32_t lse_lds = (uint32_t)reinterpret_cast<uintptr_t>(smem) + W::kSmem;  // PASS 1: two lines of 64 words
  PassUnit cur;
  if (!next_pass_unit(p, 0, &cur)) return;

  // the query tile of a slab, and in pass 1 its rows' log-sum-exps behind it (by the first wave)
  auto issue_rows = [&](int l, int g, int b, int buf) __attribute__((always_inline)) {
    w.issue_queries(l, g, b, buf);
    if (PASS == 1 && w.wave == 0)
      w.load_line(p.row_lse + ((int64_t)(l * p.H_kv + g) * p.B + b) * 32, lse_lds + buf * 256);
  };
  int l = cur.s0 / p.H_kv, g = cur.s0 - l * p.H_kv;
  w.ah = {w.slab_keys(l, g, cur.u.seq0), cur.u.b, cur.u.key0, cur.u.M, w.items_of(cur.u.M)};
  issue_rows(l, g, cur.u.b, 0);
  w.start_stream();
  w.first_queries();

  int buf = 0;
  bool more = true;
  PassUnit nxt = cur;
#pragma unroll 1
  for (;;) {
    const int M = cur.u.M, b = cur.u.b, nt = w.items_of(M);
    vkeep run[PASS == 1 ? MAXT : 1];
#pragma unroll
    for (int t = 0; t < (PASS == 1 ? MAXT : 1); ++t)
#pragma unroll
      for (int k = 0; k < KEEP; ++k) run[t][k] = -INFINITY;
#pragma unroll 1
    for (int s = cur.s0; s < cur.s1; ++s) {
      int nl = l, ng = g + 1;
      if (ng == p.H_kv) { ng = 0; ++nl; }
      w.nx.left = 0;
      if (s + 1 < cur.s1) {
        w.nx = {w.slab_keys(nl, ng, cur.u.seq0), b, cur.u.key0, M, nt};
        issue_rows(nl, ng, b, buf ^ 1);
      } else {
        more = next_pass_unit(p, cur.k + 1, &nxt);
        if (more) {
          nl = nxt.s0 / p.H_kv;
          ng = nxt.s0 - nl * p.H_kv;
          w.nx = {w.slab_keys(nl, ng, nxt.u.seq0), nxt.u.b, nxt.u.key0, nxt.u.M, w.items_of(nxt.u.M)};
          issue_rows(nl, ng, nxt.u.b, buf ^ 1);
        }
      }
      w.begin_slab();
      w.slab_scale(l, g);
      if constexpr (PASS == 0) {
        float rm = -INFINITY, rs = 0.f;
        if (nt > 0) w.template item_logits<0>(nt, M, buf, rm, rs);
#pragma unroll 1
        for (int it = 1; it < nt; ++it) w.template item_logits<1>(nt, M, buf, rm, rs);
        const float own = w.workgroup_lse(rm, rs, buf);
        const int ln = W::lane_id();
        if (w.wave == 0 && ln < 32) p.lines[((int64_t)(l * p.H_kv + g) * p.slots + cur.slot) * 32 + ln] = own;
      } else {
        const float lse2 = __uint_as_float(lds_peek(lse_lds + buf * 256 + (W::lane_id() & 31) * 4));
        wide_static_for<0, MAXT>([&](auto ic) __attribute__((always_inline)) {
          constexpr int it = decltype(ic)::value;
          if (it < nt) {
            float y[KEEP];
            w.fold_heads(w.item_products(buf), -lse2, y);
            vkeep& r = run[PASS == 1 ? it : 0];
#pragma unroll
            for (int k = 0; k < KEEP; ++k) r[k] = fmaxf(r[k], y[k]);  // (keys beyond the sequence: never read back)
          }
        });
        w.slab_barrier();
      }
      w.end_slab();
      l = nl;
      g = ng;
      buf ^= 1;
    }
    if constexpr (PASS == 1) {  // the unit's result
      const int q_n = W::lane_id() & (W::NS - 1);
      const int64_t step = (int64_t)p.n_groups * p.N * 32;  // from tile to tile
      float* const out = p.group_scores +
          ((int64_t)(wide_tile_base(cur.u.seq0, b) + (cur.u.key0 >> 5) + w.wave + (nt - 1) * kTiledWaves) * p.n_groups + cur.grp) * p.N * 32 +
          q_n * 32 + w.fold_key();
      wide_static_for<0, MAXT>([&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        if (q_n < p.N && t < nt) __builtin_nontemporal_store(run[PASS == 1 ? t : 0], reinterpret_cast<vkeep*>(out - t * kTiledWaves * step));
      });
    }
    if (!more) break;
    cur = nxt;
  }
  wait_vmcnt<0>();
}

// The lines of a sequence's pieces -> its rows' log-sum-exps; a wave per (slab, sequence), a half-wave every other line.
template <int LG>
__global__ __launch_bounds__(64) void wide_pass_combine_kernel(const WidePassDev p) {
  const int slab = blockIdx.x / p.B, b = blockIdx.x % p.B;
  const int ln = threadIdx.x, row = ln & 31;
  const int first = pass_first_place(p.cu[b], b, p.chunk), pieces = (p.cu[b + 1] - p.cu[b] + p.chunk - 1) / p.chunk;
  const float* src = p.lines + ((int64_t)slab * p.slots + first) * 32 + row;
  float m = -INFINITY, z = 0.f;
#pragma unroll 4
  for (int i = ln >> 5; i < pieces; i += 2) {
    const float v = src[(int64_t)i * 32];
    const float mn = fmaxf(m, v);
    const float ref = mn == -INFINITY ? 0.f : mn;  // (a piece whose logits of this row all overflowed)
    z = z * fast_exp2(m - ref) + fast_exp2(v - ref);
    m = mn;
  }
  const float pm = __shfl_xor(m, 32, kWave), pz = __shfl_xor(z, 32, kWave);
  const float mn = fmaxf(m, pm), ref = mn == -INFINITY ? 0.f : mn;
  const float lse2 = mn + __builtin_amdgcn_logf(z * fast_exp2(m - ref) + pz * fast_exp2(pm - ref));
  if (ln >= 32) return;
  p.row_lse[((int64_t)slab * p.B + b) * 32 + row] = lse2;
  const int n = row & ((32 >> LG) - 1), j = row >> (5 - LG);
  if (p.lse_out && n < p.N && j < p.G)
    p.lse_out[(((int64_t)(slab / p.H_kv) * p.B + b) * p.N + n) * p.H + (slab % p.H_kv) * p.G + j] =
        pieces > 0 ? lse2 * 0.6931471805599453f : 0.f;
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
bool wide_passes_supported(const sp_score_args* a) {
  if (a->rope_theta > 0.f || a->T < 1) return false;
  // A batch whose longest sequence is not stated stays on the kernels that also take un-rotated caches: its scores are
  // then bit for bit those of the same cache stored un-rotated.
  if (a->B > 1 && a->max_seqlen <= 0) return false;
  if (a->H / a->H_kv > 8 || (a->N << wide_lg(a)) > 32) return false;
  if (a->k_dtype == SP_K_FP8_E4M3 && a->d_block_table && a->page_size < (a->d == 64 ? 16 : 8)) return false;
  if (a->k_token_stride > INT32_MAX / 256) return false;  // (a ring slot's keys must span less than 2 GiB)
  // results of at most 16 GiB, as for kept logits; the tiled kernels beyond (the plan is made only where it matters)
  constexpr size_t kMostBytes = (size_t)16 << 30;
  return (size_t)a->L * a->H_kv * a->N * 128 * wide_tiles(a) <= kMostBytes / 2 || wide_passes_workspace_bytes(a) <= kMostBytes;
}

static size_t pass_lines_bytes(const sp_score_args* a, const WidePassPlan& pl) { return align_up((size_t)a->L * a->H_kv * pl.slots * 128, 256); }
static size_t pass_lse_bytes(const sp_score_args* a) { return align_up((size_t)a->L * a->H_kv * a->B * 128, 256); }
size_t wide_passes_workspace_bytes(const sp_score_args* a) {
  const WidePassPlan pl = make_wide_pass_plan(a);
  return pass_lines_bytes(a, pl) + pass_lse_bytes(a) + align_up(sizeof(float) * 32 * (size_t)pl.n_groups * a->N * wide_tiles(a), 256);
}

template <int D, int LG, bool FP8, bool PAGED, int PASS>
static sp_status launch_wide_pass(const WidePassDev& dev, hipStream_t stream) {
  auto kernel = wide_pass_kernel<D, LG, FP8, PAGED, PASS>;
  constexpr int smem = WideKernel<D, LG, FP8, PAGED>::kSmem + 512;
  static std::mutex mu;  // once per kernel and device
  static bool prepared[kMaxDevices] = {};
  {
    std::lock_guard<std::mutex> lock(mu);
    const int slot = current_device();
    if (!prepared[slot]) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
        return SP_ELAUNCH;
      prepared[slot] = true;
    }
  }
  const int64_t units = (int64_t)dev.slots * dev.n_groups;
  hipLaunchKernelGGL(kernel, dim3((unsigned)std::min<int64_t>(units, seq_cu_count())), dim3(kTiledThreads), smem, stream, dev);
  return launch_status();
}
template <int D, int LG, bool FP8, bool PAGED>
static sp_status wide_both_passes(const WidePassDev& dev, hipStream_t stream) {
  const sp_status st = launch_wide_pass<D, LG, FP8, PAGED, 0>(dev, stream);
  if (st != SP_OK) return st;
  hipLaunchKernelGGL(wide_pass_combine_kernel<LG>, dim3((unsigned)(dev.L * dev.H_kv * dev.B)), dim3(64), 0, stream, dev);
  return launch_wide_pass<D, LG, FP8, PAGED, 1>(dev, stream);
}
template <int D, bool FP8>
static sp_status wide_passes_by_kind(const WidePassDev& dev, hipStream_t stream) {
  if (dev.block_table) return dev.lgG == 2 ? wide_both_passes<D, 2, FP8, true>(dev, stream) : wide_both_passes<D, 3, FP8, true>(dev, stream);
  return dev.lgG == 2 ? wide_both_passes<D, 2, FP8, false>(dev, stream) : wide_both_passes<D, 3, FP8, false>(dev, stream);
}

sp_status wide_passes_score(const sp_score_args* a, const TiledDev& dev_, void* extra, hipStream_t stream) {
  const WidePassPlan pl = make_wide_pass_plan(a);
  WidePassDev dev;
  static_cast<TiledDev&>(dev) = dev_;
  dev.lgG = wide_lg(a);
  dev.Gp = 1 << dev.lgG;
  dev.seq_limit = 0;
  dev.chunk = pl.chunk;
  dev.slots = pl.slots;
  dev.slabs_per_group = pl.per;
  dev.n_groups = pl.n_groups;
  dev.groups_per_layer = pl.gpl;
  char* ws = static_cast<char*>(extra);
  dev.lines = reinterpret_cast<float*>(ws);
  dev.row_lse = reinterpret_cast<float*>(ws + pass_lines_bytes(a, pl));
  dev.group_scores = reinterpret_cast<float*>(ws + pass_lines_bytes(a, pl) + pass_lse_bytes(a));
  sp_status st;
  if (a->k_dtype == SP_K_FP8_E4M3) st = a->d == 64 ? wide_passes_by_kind<64, true>(dev, stream) : wide_passes_by_kind<128, true>(dev, stream);
  else st = a->d == 64 ? wide_passes_by_kind<64, false>(dev, stream) : wide_passes_by_kind<128, false>(dev, stream);
  if (st != SP_OK) return st;
  return launch_wide_finish(dev, (unsigned)wide_tiles(a), nullptr, stream);
}

}  // namespace sp
