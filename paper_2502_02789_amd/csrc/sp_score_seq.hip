// Single-pass MFMA scorer for batches of short prompts whose KV heads carry few query rows (the
// paper's variants without look-ahead, Sec. 4.3): many prompts at a time, or one prompt of a few thousand tokens.
//
// Same quantity as the other scoring kernels: row softmax of the stored queries against the
// prompt keys (Sec. 3.2 equation of arXiv 2502.02789), max over heads, max/mean over layers,
// mean over queries (Sec. 3.2.2).  The K cache is read ONCE and no logit ever leaves the chip:
//
//   * The work is cut into units (one whole sequence, one run of (layer, KV head) slabs) for one workgroup per compute unit:
//     in stretches of equal cost (sp_unit_deal.h), or, where a workgroup has too few slabs for that, numbered with
//     the longest sequences first and dealt out in rounds whose direction alternates.  Every workgroup gets nearly the
//     same number of keys without any shared counter, and nobody ever waits for another workgroup.
//   * A workgroup walks over the (layer, KV head) slabs of its unit.  Inside a slab its eight waves take the sequence's
//     32-key items in turn out of the ring of the wide kernels (sp_wide_core.h: loads through a buffer descriptor per
//     item, the query rows once per workgroup and slab) and multiply them with the KV head's query rows on the matrix
//     cores -- with the QUERY rows as the rows of the result, so that a lane ends up with all R <= 8 logits of one key
//     (one v_permlane32_swap per register joins two items to 64 keys).
//   * Those R logits per key stay in registers for the whole slab (R registers per pair of items), each
//     lane keeps a running (max, sum exp2) per row, and at the end of the slab the lanes' and the
//     eight waves' statistics are merged (DPP, one small LDS table, ONE workgroup barrier):
//     every wave then knows the rows' log-sum-exps and turns its held logits into
//     log2-probabilities, folds the heads of a group and keeps the running maximum over KV heads
//     and layers (or the sum over layers of the per-layer maxima) per key in registers.
//   * The loop over the pairs is a loop: the pair's logits go to registers indexed by its number.  (Unrolled sixteen
//     times, with 64-bit address arithmetic for every load, the kernel had 192 KB of code, three times what the instruction
//     cache holds, for each slab anew; now 14.  Whole call, one query, 32 layers, 8 KV heads, d = 128, before -> now in us: one
//     prompt of 700 keys 18.9 -> 15.4, 2048 33.1 -> 29.6, 5003 68.3 -> 62.1, 8000 106 -> 93; 12 prompts of 400 to 2400 keys,
//     8-bit 156 -> 121, out of pages of 16 286 -> 198; 64 of 1024 to 4096 1622 -> 1600, which the HBM stream of K bounds.)
//   * The stream of items never stops, neither at a slab's end nor between units: the loads run a ringful
//     ahead of the arithmetic straight into the next slab or unit, and the barrier is a bare
//     s_barrier (no vector-memory wait in front of it but for the next query rows).
//   * Each unit writes its [N][M] partial result; units_finish_kernel merges the units of a sequence and
//     averages over the valid queries.
//
// Bound by the HBM stream of K where workgroups have several slabs (64 prompts of 1024..4096 keys 1600 us = 6.9 TB/s), by
// the start (5 us until the first keys are there) and end of the one slab of a workgroup for one short prompt.
//
// A sequence must fit the registers: 64 * 8 * SeqLimits<R>::kMaxPairs keys.  The host cannot see the
// sequence lengths of a batch (they live on the device), so for B > 1 this path is taken only on the caller's
// promise sp_score_args.max_seqlen; a sequence that breaks the promise gets NaN scores (units_finish_kernel).
#include <mutex>

#include "sp_wide_core.h"

namespace sp {

template <int R> struct SeqLimits { static constexpr int kMaxPairs = (R == 4) ? 16 : 8; };  // pairs of items per wave

// maximum / sum over the wave's lanes, in every lane: inside a row of sixteen by DPP (lane ^ 1, lane ^ 2, the mirrored half
// row and row), then across rows and halves
template <typename Op>
__device__ __forceinline__ float wave_join(float v, Op op) {
  v = op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true)));
  v = op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true)));
  v = op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true)));
  v = op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true)));
  const auto rows = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(__uint_as_float(rows[0]), __uint_as_float(rows[1]));
  const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
}

// The stream of the wide kernels with R query rows in LDS instead of 32, and the products turned round.
template <int D, int R, int LG, bool FP8, bool PAGED>
struct SeqKernel : WideKernel<D, 2, FP8, PAGED> {
  using W = WideKernel<D, 2, FP8, PAGED>;
  static constexpr int KS = W::KS;
  static constexpr int QB = R * W::QROW_B;         // bytes of the query rows: 512 to 2048
  static constexpr int QWAVES = (QB + 1023) / 1024;  // waves that fetch them
  bf16x8 qf[KS];

  __device__ __forceinline__ SeqKernel(const TiledDev& p_, unsigned char* smem) : W(p_, smem) {}

  // the query rows of (l, g, b) -> query buffer `buf`: row n * 2^LG + j holds Q[l, b, n, g*G + j, :] (rows of queries
  // beyond N and padding heads repeat query 0 / head 0: the former are never used, the latter change no maximum)
  __device__ __forceinline__ void issue_queries(int l, int g, int b, int buf) {
    if (this->wave >= QWAVES) return;
    const int at = this->wave * 1024 + W::lane_id() * 16;
    const int r = (at / W::QROW_B) & (R - 1);  // (lanes beyond the last row repeat rows)
    const int n = (r >> LG) < this->p.N ? r >> LG : 0, j = (r & ((1 << LG) - 1)) < this->p.G ? r & ((1 << LG) - 1) : 0;
    const int64_t row0 = (((int64_t)l * this->p.B + b) * this->p.N) * this->p.H + g * this->p.G;
    const unsigned char* base = reinterpret_cast<const unsigned char*>(this->p.q) + row0 * W::QROW_B;
    const uint32_t off = (uint32_t)((n * this->p.H + j) * W::QROW_B + at % W::QROW_B);
    W::load16(base + off, this->qbuf + buf * W::QTILE_B + this->wave * 1024);
  }
  // the slab's query operand: lane column c holds row c mod R (rows of the result beyond R are never looked at)
  __device__ __forceinline__ void read_queries(int buf) {
    const int ln = W::lane_id();
    const uint32_t row = this->qbuf + buf * W::QTILE_B + (ln & (R - 1)) * W::QROW_B, half = ln >> 5;
#pragma unroll
    for (int t = 0; t < KS; ++t) qf[t] = this->read16(row + (FP8 ? 4 * (t >> 1) + (t & 1) + 2 * half : 2 * t + half) * 16);
  }
  // As in the wide kernels, but with the key scale's sign (every logit is scaled before anything is compared with it), a zero
  // being the least number of either sign.
  __device__ __forceinline__ void slab_scale(int l, int g) {
    this->c2 = this->p.c;
    if constexpr (FP8) {
      if (this->p.k_scale) {
        const float ks = __int_as_float(scalar_table(reinterpret_cast<const int32_t*>(this->p.k_scale))[l * this->p.H_kv + g]);
        this->c2 = copysignf(positive_scale(this->p.c, ks), ks);
      }
    }
  }
  // the unscaled logit of a key that does not exist
  __device__ __forceinline__ float none() const { return FP8 ? -copysignf(INFINITY, this->c2) : -INFINITY; }
  // The next item's logits: rows 0..3 of key `col` in registers 0..3 of the lower half-wave, rows 4..7 in the upper one.
  __device__ __forceinline__ f32x16 item_rows() {
    const int later = this->sent - this->pos - 1;
    if (later == W::SLOTS - 1) wait_vmcnt<(W::SLOTS - 1) * W::LOADS>(); else W::wait_items(later);
    f32x16 a = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    uint32_t k0 = this->krd0;
    asm volatile("" : "+v"(k0));
    const uint32_t kadd = (this->pos & (W::SLOTS - 1)) * W::ITEM_B;
    if constexpr (FP8) {
      u32x4 raw[KS / 2];
#pragma unroll
      for (int j = 0; j < KS / 2; ++j) raw[j] = __builtin_bit_cast(u32x4, this->read16((k0 ^ (uint32_t)((2 * j) << 4)) + kadd));
#pragma unroll
      for (int t = 0; t < KS; ++t) {
        u32x4 o;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          o[2 * x] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[t >> 1][2 * (t & 1) + x], 1.0f, false));
          o[2 * x + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[t >> 1][2 * (t & 1) + x], 1.0f, true));
        }
        a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[t], __builtin_bit_cast(bf16x8, o), a, 0, 0, 0);
      }
    } else {
      bf16x8 kf[KS];
#pragma unroll
      for (int t = 0; t < KS; ++t) kf[t] = this->read16((k0 ^ (uint32_t)(t << 5)) + kadd);
#pragma unroll
      for (int t = 0; t < KS; ++t) a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[t], kf[t], a, 0, 0, 0);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot's reads are done: it may be overwritten
    ++this->pos;
    this->refill();
    return a;
  }
};

template <int D, int R, int LG, bool MEAN, bool FP8, bool PAGED, bool STRETCHES>
__global__ __launch_bounds__(kTiledThreads) void seq_score_kernel(const TiledDev p) {
  extern __shared__ __align__(1024) unsigned char smem[];
  using W = SeqKernel<D, R, LG, FP8, PAGED>;
  constexpr int MAXP = SeqLimits<R>::kMaxPairs;
  constexpr int GP = 1 << LG;   // heads of a KV group, padded to a power of two
  constexpr int NQ = R >> LG;   // queries whose rows fit the R held rows
  typedef float vpair __attribute__((ext_vector_type(MAXP)));
  W w(p, smem);
  SeqUnit cur;
  if (!seq_first_unit<STRETCHES>(p, &cur)) return;

  int l = __builtin_amdgcn_readfirstlane(cur.s0 / p.H_kv), g = cur.s0 - l * p.H_kv;
  w.ah = {w.slab_keys(l, g, cur.seq0), cur.b, 0, cur.M, w.items_of(cur.M)};
  w.issue_queries(l, g, cur.b, 0);
  w.start_stream();

  int slabs = 0;  // slabs finished so far (the query and exchange buffers have two halves used in turn)
  bool more = true;
  SeqUnit nxt = cur;  // the unit of the slab behind the one at hand
  vpair held[R];  // row r of the lane's key of pair t, not yet scaled
  float smax[MAXP][NQ], tot[MEAN ? MAXP : 1][NQ];

#pragma unroll 1
  for (;;) {
    const int M = cur.M, b = cur.b, nt = w.items_of(M);
#pragma unroll
    for (int t = 0; t < MAXP; ++t)
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        smax[t][n] = -INFINITY;
        if constexpr (MEAN) tot[t][n] = 0.f;
      }
#pragma unroll 1
    for (int s = cur.s0; s < cur.s1; ++s) {
      const int buf = slabs & 1;
      // the next slab: its query rows go into the buffer the previous slab has just left (the barrier at its end);
      // requests move on to it when this slab's items have all been sent
      int nl = l, ng = g + 1;
      if (ng == p.H_kv) { ng = 0; ++nl; }
      if (s + 1 == cur.s1) {
        more = seq_next_unit<STRETCHES>(p, &nxt);
        nl = __builtin_amdgcn_readfirstlane(nxt.s0 / p.H_kv);
        ng = nxt.s0 - nl * p.H_kv;
      }
      w.nx.left = 0;
      if (more) {
        w.nx = {w.slab_keys(nl, ng, nxt.seq0), nxt.b, 0, nxt.M, w.items_of(nxt.M)};
        w.issue_queries(nl, ng, nxt.b, buf ^ 1);
      }
      w.begin_slab();
      if (slabs == 0) w.first_queries();
      w.read_queries(buf);
      w.slab_scale(l, g);
      float rm[R], rs[R];  // this lane's running max and sum of exp2 per row, base-2 logits
#pragma unroll
      for (int r = 0; r < R; ++r) { rm[r] = -INFINITY; rs[r] = 0.f; }

      // Items come from the last to the first, so the ragged end of the keys is in some wave's first item; of an odd number
      // the last pair has only one (the upper half-wave then has no keys).
#pragma unroll 1
      for (int t = 0; 2 * t < nt; ++t) {
        f32x16 a = w.item_rows(), c;
        if (t == 0) {
          const int left = M - (w.wave + (nt - 1) * kTiledWaves) * 32 - (W::lane_id() & 31);  // > 0: the lane's key exists
#pragma unroll
          for (int i = 0; i < 4; ++i) a[i] = left > 0 ? a[i] : w.none();
        }
        if (2 * t + 1 < nt) {
          c = w.item_rows();
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) c[i] = w.none();
        }
        float x[R];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i]), __float_as_uint(c[i]), false, false);
          x[i] = __uint_as_float(sw[0]);
          if (R == 8) x[4 + i] = __uint_as_float(sw[1]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float m_new = fmaxf(rm[r], x[r] * w.c2);
          const float off = (m_new == -INFINITY) ? 0.f : -m_new;
          rs[r] = rs[r] * fast_exp2(rm[r] + off) + fast_exp2(fmaf(x[r], w.c2, off));
          rm[r] = m_new;
          held[r][t] = x[r];
        }
      }

      // the rows' statistics over the wave's keys, then over the workgroup's
      ++slabs;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float mw = wave_join(rm[r], [](float x, float y) { return fmaxf(x, y); });
        const float ref = (mw == -INFINITY) ? 0.f : mw;
        const float sw = wave_join(rs[r] * fast_exp2(rm[r] - ref), [](float x, float y) { return x + y; });
        if (W::lane_id() == 0)
          lds_poke64<0>(w.xchg + ((buf * kTiledWaves + w.wave) * R + r) * 8, ((uint64_t)__float_as_uint(sw) << 32) | __float_as_uint(mw));
      }
      w.slab_barrier();
      float lse2[R];
      {
        const int ln = W::lane_id();  // every lane folds the eight waves' pairs of row ln mod R
        const uint32_t at = w.xchg + (buf * kTiledWaves * R + (ln & (R - 1))) * 8;
        const u64x4 lo = lds_peek64x4<R * 8>(at), hi = lds_peek64x4<R * 8>(at + 4 * R * 8);
        float m = -INFINITY, z = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) m = fmaxf(m, fmaxf(__uint_as_float((uint32_t)lo.v[i]), __uint_as_float((uint32_t)hi.v[i])));
        const float ref = (m == -INFINITY) ? 0.f : m;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          z += __uint_as_float((uint32_t)(lo.v[i] >> 32)) * fast_exp2(__uint_as_float((uint32_t)lo.v[i]) - ref);
          z += __uint_as_float((uint32_t)(hi.v[i] >> 32)) * fast_exp2(__uint_as_float((uint32_t)hi.v[i]) - ref);
        }
        const float lse = m + __builtin_amdgcn_logf(z);  // base 2
#pragma unroll
        for (int r = 0; r < R; ++r) lse2[r] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lse), r));
        if (p.lse_out && w.wave == 0) {
          const int n = ln >> LG, j = ln & (GP - 1);
          if (ln < R && n < p.N && j < p.G)
            p.lse_out[(((int64_t)l * p.B + b) * p.N + n) * p.H + g * p.G + j] = lse * 0.6931471805599453f;
        }
      }

      // log2-probabilities; max over the heads of a group, over KV heads and layers
      wide_static_for<0, MAXP>([&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        if (2 * t < nt) {
#pragma unroll
          for (int n = 0; n < NQ; ++n) {
            float v = fmaf(held[n * GP][t], w.c2, -lse2[n * GP]);
#pragma unroll
            for (int j = 1; j < GP; ++j) v = fmaxf(v, fmaf(held[n * GP + j][t], w.c2, -lse2[n * GP + j]));
            smax[t][n] = fmaxf(smax[t][n], v);
          }
        }
      });
      if constexpr (MEAN) {
        if (g == p.H_kv - 1) {  // the layer is complete: its max probability joins the sum
#pragma unroll
          for (int t = 0; t < MAXP; ++t)
#pragma unroll
            for (int n = 0; n < NQ; ++n) {
              tot[t][n] += fast_exp2(smax[t][n]);
              smax[t][n] = -INFINITY;
            }
        }
      }
      w.end_slab();
      l = nl;
      g = ng;
    }

    // the unit's result (stores only make the next items' waits stricter than they need be)
    const int ln = W::lane_id(), in_tile = ln & 31, half = ln >> 5;
    wide_static_for<0, MAXP>([&](auto tc) __attribute__((always_inline)) {
      constexpr int t = decltype(tc)::value;
      if (2 * t < nt) {
        const int key = (w.wave + (nt - 1 - 2 * t - half) * kTiledWaves) * 32 + in_tile;
        if (2 * t + half < nt && key < M) {
#pragma unroll
          for (int n = 0; n < NQ; ++n)
            if (n < p.N) {
              float v = smax[t][n];
              if constexpr (MEAN) v = tot[t][n];
              p.group_scores[((int64_t)cur.grp * p.N + n) * p.T + cur.seq0 + key] = v;
            }
        }
      }
    });
    note_group_count<STRETCHES>(p, cur);
    if (!more) break;
    cur = nxt;
  }
  wait_vmcnt<0>();
}

// order[r] = the sequence with the r-th most keys (equal lengths: lower index first); one workgroup,
// every thread ranks its sequences by counting those ahead of them
// (and the log-sum-exp rows of the sequences the scoring kernel leaves out: 0 by convention where there are no
// keys, NaN where there are more than `limit`; order = null: only these)
__global__ __launch_bounds__(1024) void seq_order_kernel(int B, const int32_t* __restrict__ cu, int32_t* __restrict__ order,
                                                         float* __restrict__ lse_out, int limit, int L, int rows) {
  constexpr int kChunk = 4096;
  __shared__ int32_t len[kChunk];
  for (int b0 = 0; b0 < B; b0 += 1024) {  // (all threads take part in every round: barriers inside)
    const int b = b0 + threadIdx.x;
    const int mine = b < B ? cu[b + 1] - cu[b] : 0;
    int rank = 0;
    for (int c0 = 0; order && c0 < B; c0 += kChunk) {
      const int n = min(kChunk, B - c0);
      __syncthreads();
      for (int i = threadIdx.x; i < n; i += 1024) len[i] = cu[c0 + i + 1] - cu[c0 + i];
      __syncthreads();
      for (int i = 0; i < n; ++i) rank += (len[i] > mine || (len[i] == mine && c0 + i < b)) ? 1 : 0;
    }
    if (order && b < B) order[rank] = b;
    if (b < B && lse_out && (mine <= 0 || mine > limit))
      for (int i = 0; i < L * rows; ++i)
        lse_out[((int64_t)(i / rows) * B + b) * rows + i % rows] = mine <= 0 ? 0.f : __uint_as_float(0x7FC00000u);
  }
}

// Merge of the units' (or the two-pass kernels' layer groups') partial results and the average over the valid queries
// (Sec. 3.2.2).  A workgroup takes TOK
// tokens; its 64 * WAVES / TOK groups of TOK threads take every so-many-th slab group (one TOK * 4 byte read per group and
// query), the lanes of a wave fold by shuffles, the waves' results meet in LDS.  Sequences the scoring
// kernel left out (longer than it holds) get NaN.  Bound by the latency of the reads for one short prompt, whose
// few tokens make few workgroups of 64 (2K tokens, 256 groups of one query: 7.6 us): narrower workgroups there.
template <int NQ, int TOK, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void units_finish_kernel(const TiledDev p) {
  __shared__ float red[WAVES][NQ][TOK];
  __shared__ float prob[NQ][TOK];
  __shared__ int32_t cu_lds[kStagedOffsets];
  const int32_t* const cu = p.B > 1 ? staged_offsets(p.cu, p.B, cu_lds) : p.cu;
  constexpr int kParts = 64 * WAVES / TOK;
  const int k = threadIdx.x % TOK, part = threadIdx.x / TOK;
  const int64_t tok = (int64_t)blockIdx.x * TOK + k;
  const bool inside = tok < p.T;
  const bool mean = p.layer_reduce != SP_LAYER_MAX;
  int n_groups = p.n_groups;
  if (inside && p.group_count) {  // (none for a sequence that was left out)
    const int b = upper_segment(cu, p.B, (int)tok);
    n_groups = cu[b + 1] - cu[b] > p.seq_limit ? 0 : p.group_count[b];
  }
  float v[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) v[n] = mean ? 0.f : -INFINITY;
  if (inside && mean && p.groups_per_layer > 0) {
    // mean over layers from units that are parts of a layer: the groups of a layer hold the log2 of its maxima over
    // their KV heads; the layer's maximum over all heads is their maximum, and the layers' maxima add up
    for (int l = part; l < p.L; l += kParts) {
      float m[NQ];
#pragma unroll
      for (int n = 0; n < NQ; ++n) m[n] = -INFINITY;
      for (int j = 0; j < p.groups_per_layer; ++j)
#pragma unroll
        for (int n = 0; n < NQ; ++n)
          if (n < p.N) m[n] = fmaxf(m[n], p.group_scores[((int64_t)(l * p.groups_per_layer + j) * p.N + n) * p.T + tok]);
#pragma unroll
      for (int n = 0; n < NQ; ++n) v[n] += fast_exp2(m[n]);
    }
  } else if (inside) {
#pragma unroll 4
    for (int g = part; g < n_groups; g += kParts)
#pragma unroll
      for (int n = 0; n < NQ; ++n)
        if (n < p.N) {
          const float x = p.group_scores[((int64_t)g * p.N + n) * p.T + tok];
          v[n] = mean ? v[n] + x : fmaxf(v[n], x);
        }
  }
#pragma unroll
  for (int off = TOK; off < 64; off <<= 1)
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const float x = __shfl_xor(v[n], off, kWave);
      v[n] = mean ? v[n] + x : fmaxf(v[n], x);
    }
  if ((threadIdx.x & 63) < TOK)
#pragma unroll
    for (int n = 0; n < NQ; ++n) red[threadIdx.x >> 6][n][k] = v[n];
  __syncthreads();
  for (int i = threadIdx.x; i < NQ * TOK; i += 64 * WAVES) {
    const int n = i / TOK;
    float x = red[0][n][k];
#pragma unroll
    for (int q = 1; q < WAVES; ++q) x = mean ? x + red[q][n][k] : fmaxf(x, red[q][n][k]);
    prob[n][k] = mean ? x : fast_exp2(x);
  }
  __syncthreads();
  if (threadIdx.x >= TOK || !inside) return;
  const int b = upper_segment(cu, p.B, (int)tok);
  if (p.seq_limit > 0 && cu[b + 1] - cu[b] > p.seq_limit) {
    p.scores[tok] = __uint_as_float(0x7FC00000u);
    return;
  }
  int nv = p.n_valid ? p.n_valid[b] : p.N;
  nv = max(1, min(nv, p.N));
  float sum = 0.f;
#pragma unroll
  for (int n = 0; n < NQ; ++n)
    if (n < nv) sum += prob[n][k];
  p.scores[tok] = sum / (mean ? (float)nv * (float)p.L : (float)nv);
}

template <int NQ>
static sp_status finish_by_tokens(const TiledDev& dev, hipStream_t stream) {
  // Tokens per workgroup: 64 where that makes at least two workgroups per compute unit, else 16; waves: sixteen where
  // there are that many groups for each, else four (64 prompts, 168K tokens in eight groups: 12 us with sixteen).
  if (dev.T < 64 * 512) hipLaunchKernelGGL((units_finish_kernel<NQ, 16, 16>), dim3((unsigned)((dev.T + 15) / 16)), dim3(1024), 0, stream, dev);
  else if (dev.n_groups > 64 && NQ <= 8) hipLaunchKernelGGL((units_finish_kernel<NQ, 64, NQ <= 8 ? 16 : 4>), dim3((unsigned)((dev.T + 63) / 64)), dim3(NQ <= 8 ? 1024 : 256), 0, stream, dev);
  else hipLaunchKernelGGL((units_finish_kernel<NQ, 64, 4>), dim3((unsigned)((dev.T + 63) / 64)), dim3(256), 0, stream, dev);
  return launch_status();
}
sp_status launch_units_finish(const TiledDev& dev, hipStream_t stream) {
  return dev.N == 1 ? finish_by_tokens<1>(dev, stream) : dev.N == 2 ? finish_by_tokens<2>(dev, stream)
       : dev.N <= 4 ? finish_by_tokens<4>(dev, stream) : dev.N <= 8 ? finish_by_tokens<8>(dev, stream) : finish_by_tokens<16>(dev, stream);
}

void prepare_units(const sp_score_args* a, TiledDev* dev, int32_t* words, int limit, hipStream_t stream) {
  const bool rounds = dev->deal.stretch == 0;
  dev->group_count = rounds ? nullptr : words;
  dev->seq_order = rounds && a->B > 1 ? words : nullptr;
  if (a->B > 1 && (rounds || a->d_lse))  // (one sequence: nothing to order, and the host has seen that its length fits)
    hipLaunchKernelGGL(seq_order_kernel, dim3(1), dim3(1024), 0, stream, a->B, a->d_cu_seqlens, rounds ? words : nullptr, a->d_lse,
                       limit, a->L, a->N * a->H);
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
// heads per KV head as this path lays them out: padded to four or eight (columns of padding heads repeat head
// 0, which changes neither a maximum nor a row's own statistics; one or two heads per KV head are padded to four
// as well, so that the same kernel variants serve them)
static int seq_padded_group(const sp_score_args* a) {
  const int G = a->H / a->H_kv;
  return G <= 4 ? 4 : 8;
}
static int seq_rows(const sp_score_args* a) {  // held rows per key: 4 or 8 (0: too many)
  const int rows = seq_padded_group(a) * a->N;
  return rows <= 4 ? 4 : rows <= 8 ? 8 : 0;
}
int seq_max_keys(const sp_score_args* a) {
  const int R = seq_rows(a);
  return R == 0 ? 0 : kWaveKeys * kTiledWaves * (R == 4 ? SeqLimits<4>::kMaxPairs : SeqLimits<8>::kMaxPairs);
}

// The cut along the (layer, KV head) slabs into units.  With the maximum over layers a
// group may be any run of slabs (a maximum can be completed in any order); with the mean over layers a group
// holds whole layers (a layer's maximum over heads must be complete before it joins the sum).
static UnitDeal seq_deal(const sp_score_args* a, int* n_groups) {
  return make_unit_deal(a, seq_cu_count(), seq_max_keys(a), a->layer_reduce == SP_LAYER_MEAN, n_groups);
}
void seq_grouping(const sp_score_args* a, int* slabs_per_group, int* n_groups, int* groups_per_layer) {
  *groups_per_layer = 0;
  *slabs_per_group = 1;
  if (seq_deal(a, n_groups).stretch != 0) return;
  if (a->layer_reduce == SP_LAYER_MEAN && (int64_t)a->B * a->L < 256) {
    // too few whole layers to fill the device: units of a part of a layer's KV heads (the scoring kernel then
    // hands on maxima, as for the maximum over layers, and the merge adds the layers up)
    int per = 1;
    for (int cand = a->H_kv; cand >= 1; --cand)
      if (a->H_kv % cand == 0 && (int64_t)a->B * a->L * (a->H_kv / cand) >= 256) { per = cand; break; }
    if (per < a->H_kv) {
      *slabs_per_group = per;
      *groups_per_layer = a->H_kv / per;
      *n_groups = a->L * *groups_per_layer;
      return;
    }
  }
  *n_groups = round_groups(a, a->layer_reduce == SP_LAYER_MEAN ? a->H_kv : 1, slabs_per_group);
}
// the longest sequence the caller vouches for (one sequence: its length is the host's to see)
static int64_t seq_stated_max(const sp_score_args* a) { return a->B == 1 ? a->T : a->max_seqlen; }

bool seq_supported(const sp_score_args* a) {
  if (a->rope_theta > 0.f || seq_stated_max(a) <= 0) return false;
  if (a->k_dtype == SP_K_FP8_E4M3 && a->d_block_table && a->page_size < (a->d == 64 ? 16 : 8)) return false;
  const int R = seq_rows(a);
  if (R == 0 || seq_stated_max(a) > seq_max_keys(a)) return false;
  if (a->k_token_stride > (INT32_MAX / 256)) return false;  // (a ring slot's keys must span less than 2 GiB)
  if (a->B > 8192) return false;                            // (the sequences are ranked by counting: quadratic in B)
  // too few units to fill the device?
  if ((int64_t)a->B * a->L * a->H_kv < 256) return false;
  return true;
}

static size_t seq_scores_bytes(const sp_score_args* a) {
  int lpg, groups, gpl;
  seq_grouping(a, &lpg, &groups, &gpl);
  return align_up(sizeof(float) * (size_t)groups * a->N * (size_t)a->T, 256);
}

size_t seq_workspace_bytes(const sp_score_args* a) {
  if (!seq_supported(a)) return 0;
  return seq_scores_bytes(a) + align_up(sizeof(int32_t) * (size_t)a->B, 256);  // partial results, then the sequence order or group counts
}

int seq_cu_count() {  // compute units of the current device
  static std::mutex mu;
  static int cached[kMaxDevices] = {};
  std::lock_guard<std::mutex> lock(mu);
  const int slot = current_device();
  if (cached[slot] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, slot) != hipSuccess || n < 1) {
      (void)hipGetLastError();
      n = 256;
    }
    cached[slot] = n;
  }
  return cached[slot];
}

template <int D, int R, int LG, bool MEAN, bool FP8, bool PAGED, bool STRETCHES>
static sp_status launch_seq(const TiledDev& dev, hipStream_t stream) {
  auto kernel = seq_score_kernel<D, R, LG, MEAN, FP8, PAGED, STRETCHES>;
  const size_t smem = SeqKernel<D, R, LG, FP8, PAGED>::kSmem;
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
  // one workgroup per compute unit walks over its share of the (sequence, layer group) units
  const int wgs = STRETCHES ? seq_cu_count() : std::min(dev.B * dev.n_groups, seq_cu_count());
  hipLaunchKernelGGL(kernel, dim3(wgs), dim3(kTiledThreads), smem, stream, dev);
  return launch_status();
}

template <int D, int R, int LG, bool MEAN, bool FP8, bool PAGED>
static sp_status seq_by_deal(const TiledDev& dev, hipStream_t stream) {
  return dev.deal.stretch != 0 ? launch_seq<D, R, LG, MEAN, FP8, PAGED, true>(dev, stream) : launch_seq<D, R, LG, MEAN, FP8, PAGED, false>(dev, stream);
}
template <int D, int R, int LG, bool MEAN, bool FP8>
static sp_status seq_by_pages(const TiledDev& dev, hipStream_t stream) {
  return dev.block_table ? seq_by_deal<D, R, LG, MEAN, FP8, true>(dev, stream) : seq_by_deal<D, R, LG, MEAN, FP8, false>(dev, stream);
}
template <int D, bool MEAN, bool FP8>
static sp_status seq_by_rows(const TiledDev& dev, int R, hipStream_t stream) {
  if (dev.lgG == 2) return R == 4 ? seq_by_pages<D, 4, 2, MEAN, FP8>(dev, stream) : seq_by_pages<D, 8, 2, MEAN, FP8>(dev, stream);
  return seq_by_pages<D, 8, 3, MEAN, FP8>(dev, stream);
}
template <int D, bool FP8>
static sp_status seq_by_mode(const TiledDev& dev, int R, bool mean, hipStream_t stream) {
  return mean ? seq_by_rows<D, true, FP8>(dev, R, stream) : seq_by_rows<D, false, FP8>(dev, R, stream);
}

// `dev` as the tiled kernels fill it in, with group_scores, slabs_per_group, n_groups and
// seq_limit set for this path
sp_status seq_score(const sp_score_args* a, const TiledDev& dev_, hipStream_t stream) {
  TiledDev dev = dev_;
  int n_groups;
  dev.deal = seq_deal(a, &n_groups);
  prepare_units(a, &dev, reinterpret_cast<int32_t*>(reinterpret_cast<char*>(dev.group_scores) + seq_scores_bytes(a)), seq_max_keys(a), stream);
  const int R = seq_rows(a);
  // (units smaller than a layer: the kernel variant that hands on maxima, whatever the layer reduction)
  const bool mean = a->layer_reduce == SP_LAYER_MEAN && dev.groups_per_layer == 0;
  const bool fp8 = a->k_dtype == SP_K_FP8_E4M3;
  const sp_status st = a->d == 64 ? (fp8 ? seq_by_mode<64, true>(dev, R, mean, stream) : seq_by_mode<64, false>(dev, R, mean, stream))
                                  : (fp8 ? seq_by_mode<128, true>(dev, R, mean, stream) : seq_by_mode<128, false>(dev, R, mean, stream));
  if (st != SP_OK) return st;
  return launch_units_finish(dev, stream);
}

}  // namespace sp
