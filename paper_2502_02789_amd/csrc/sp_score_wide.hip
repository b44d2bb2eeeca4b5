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
//   * A ring slot is 8 KiB whatever the element size and head dim (32, 64 or 128 keys), so the bytes in flight per
//     compute unit are the same 64..128 KiB for all of them.  The loads go through a buffer descriptor per slot
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
// cache 1005 -> 340 us, one prompt of 3001 keys 138 -> 43 us (+ merge 9 us).  Neither the matrix cores nor the
// exponentials limit it (either taken out: no change).
#include <mutex>

#include "sp_tile_walker.h"

namespace sp {

constexpr int kItemBytes = 8192;  // a ring slot
constexpr int kItemLoads = kItemBytes / 1024;
constexpr int kWideTiles = 12;    // 32-key tiles per wave (whole ring slots of one, two or four tiles), and the first
constexpr int kWideRunTiles = 4;  // of them whose running maxima are in registers

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

template <int I, int N, typename F>
__device__ __forceinline__ void wide_static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    wide_static_for<I + 1, N>(f);
  }
}

// first 32-key tile of sequence b in the result array (a tile never spans two sequences: at most one tile more
// per sequence than the keys need, (T >> 5) + B in all)
__device__ __forceinline__ int wide_tile_base(int seq0, int b) { return (seq0 >> 5) + b; }

template <int D, int LG, bool FP8, bool PAGED>
struct WideKernel {
  static constexpr int ESZ = FP8 ? 1 : 2;
  static constexpr int KS = D / 16;               // MFMA k-steps
  static constexpr int KROW_B = D * ESZ;          // bytes of a key
  static constexpr int KU = KROW_B / 16;          // its 16-byte units: 16, 8 or 4
  static constexpr int KSH = KU == 16 ? 0 : KU == 8 ? 1 : 2;
  static constexpr int RPI = 64 / KU;             // keys per wave-wide load
  static constexpr int KPI = kItemBytes / KROW_B; // keys per ring slot: 32, 64 or 128
  static constexpr int SUB = KPI / 32;            // 32-key tiles per ring slot
  static constexpr int QROW_B = D * 2;
  static constexpr int QU = QROW_B / 16;
  static constexpr int QTILE_B = 32 * QROW_B;
  static constexpr int QLOADS = QTILE_B / 1024;   // one load each by the first QLOADS waves
  static constexpr int NS = 32 >> LG;             // query slots
  static constexpr int KEEP = 16 >> LG;           // keys per lane and tile after the fold over heads: 4 or 2
  static constexpr int kShort = SUB == 1 ? 9 : 8;  // tiles per wave that fit with all their running maxima
  static constexpr int kRingB = kTiledWaves * 2 * kItemBytes;
  static constexpr int kSmem = kRingB + 2 * QTILE_B + 2 * kTiledWaves * 32 * 8;

  const TiledDev& p;
  int wave;
  uint32_t ring, qbuf, xchg;  // LDS addresses: this wave's two slots, the two query tiles, the exchange table
  uint32_t ld_row, ld_unit, krd0, qrd0;  // this lane's key and 16-byte unit in a load; where it reads its operands
  uint32_t ts_b;              // bytes from key to key (the host checks that a slot's keys span less than 2 GiB)
  float c2;

  __device__ __forceinline__ WideKernel(const TiledDev& p_, unsigned char* smem) : p(p_) {
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    const uint32_t base = (uint32_t)reinterpret_cast<uintptr_t>(smem);
    ring = base + wave * 2 * kItemBytes;
    qbuf = base + kRingB;
    xchg = qbuf + 2 * QTILE_B;
    ts_b = (uint32_t)p.ts * ESZ;
    // LDS layout of a slot: key r at r * KROW_B; its 16-byte unit u at position u ^ ((r >> KSH) & (KU - 1)): the
    // 16 lanes of an operand read hit 16 distinct bank groups, and a wave-wide load still fills 1 KiB in a row
    const int i = lane / KU;
    ld_row = i * ts_b;
    ld_unit = (uint32_t)((lane % KU) ^ (i >> KSH)) << 4;
    const int kkey = (col >> KSH) & (KU - 1);
    krd0 = ring + col * KROW_B + ((half ^ kkey) << 4);
    const int qkey = (QU == 16) ? (col & 15) : ((col >> 1) & 7);
    qrd0 = qbuf + col * QROW_B + (((FP8 ? 2 * half : half) ^ qkey) << 4);
    c2 = p.c;
  }
  // the lane number where it is needed (two instructions; kept in a register it would cost a held logit its place)
  __device__ __forceinline__ static int lane_id() {
    int x = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(x));
    return x;
  }
  // byte offset of this lane in load j of a slot, from the load's first key
  __device__ __forceinline__ uint32_t lane_offset(int j) const {
    uint32_t row = ld_row, unit = ld_unit;
    asm volatile("" : "+v"(row), "+v"(unit));
    return row + (unit ^ (uint32_t)(((4 * j) & (KU - 1)) << 4));
  }
  __device__ __forceinline__ static __attribute__((address_space(3))) void* lds_ptr(uint32_t addr) {
    return reinterpret_cast<__attribute__((address_space(3))) void*>(addr);
  }
  // 1 KiB, 16 bytes per lane; lanes at or beyond `bytes` read nothing and put zeros
  __device__ __forceinline__ static void load1k(const unsigned char* base, uint32_t bytes, uint32_t lane_off, uint32_t dst) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0, bytes, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, lds_ptr(dst), 16, lane_off, 0, 0, kKeyLoadPolicy);
  }

  // where the keys of (l, g) start: of token seq0 (contiguous cache) or of the pool's first page
  __device__ __forceinline__ const unsigned char* slab_keys(int l, int g, int seq0) const {
    return reinterpret_cast<const unsigned char*>(p.k[l]) + ESZ * ((int64_t)g * p.hs + (PAGED ? 0 : (int64_t)seq0 * p.ts));
  }
  // keys [key_first, key_first + KPI) of sequence b, of which the first `rows` (>= 1) exist -> ring slot
  __device__ __forceinline__ void issue_keys(const unsigned char* slab, int b, int key_first, int rows, int slot) {
    const uint32_t dst = ring + slot * kItemBytes;
    if constexpr (PAGED) {
      // (the RPI keys of one load lie in one page: pages hold a power of two >= 8 keys, >= RPI where the host checks)
      // Two loops that stay loops, the next page's entry fetched while a page's loads go out: unrolled, this is most
      // of the kernel's code, more than the instruction cache holds.
      const ScalarTable table = scalar_table(p.block_table + (int64_t)b * p.blocks_per_seq);
      const int page = 1 << p.lg_page, last = (key_first + min(rows, KPI) - 1) >> p.lg_page;
      int pg = key_first >> p.lg_page, entry = table[pg];
      int in_page = key_first & (page - 1);
      const uint32_t lane_row = ld_row;
      int j = 0;
#pragma unroll 1
      for (;;) {
        const unsigned char* base = slab + ESZ * ((int64_t)entry * p.page_stride) + (int64_t)in_page * (int64_t)ts_b;
        entry = table[min(pg + 1, last)];
        const int j_end = min(kItemLoads, j + ((page - in_page) / RPI));
#pragma unroll 1
        for (; j < j_end; ++j) {
          const int left = min(rows - j * RPI, RPI);
          const uint32_t bytes = left <= 0 ? 0u : (uint32_t)(left - 1) * ts_b + KROW_B;
          load1k(base, bytes, lane_row + (ld_unit ^ (uint32_t)(((4 * j) & (KU - 1)) << 4)), dst + j * 1024);
          base += (int64_t)RPI * (int64_t)ts_b;
        }
        if (j == kItemLoads) break;
        ++pg;
        in_page = 0;
      }
    } else {
      const unsigned char* base = slab + (int64_t)key_first * (int64_t)ts_b;
      const uint32_t bytes = (uint32_t)(min(rows, KPI) - 1) * ts_b + KROW_B;
#pragma unroll
      for (int j = 0; j < kItemLoads; ++j) {
        load1k(base, bytes, lane_offset(j) + (uint32_t)(j * RPI) * ts_b, dst + j * 1024);
      }
    }
  }

  // this wave's share of the query tile of (l, g, b) -> query buffer `buf`: row n + NS * j holds Q[l, b, n, g*G + j, :]
  // (rows of queries beyond N and padding heads repeat query 0 / head 0: the former are never used, the latter
  // change no maximum)
  __device__ __forceinline__ void issue_queries(int l, int g, int b, int buf) {
    if (wave < QLOADS) {
      const int ln = lane_id();
      const int r = wave * (64 / QU) + ln / QU;
      const int qkey = (QU == 16) ? (r & 15) : ((r >> 1) & 7);
      const int unit = (ln % QU) ^ qkey;
      const int n = (r & (NS - 1)) < p.N ? (r & (NS - 1)) : 0;
      const int j = (r >> (5 - LG)) < p.G ? (r >> (5 - LG)) : 0;
      const int64_t row0 = (((int64_t)l * p.B + b) * p.N) * p.H + g * p.G;
      const unsigned char* base = reinterpret_cast<const unsigned char*>(p.q) + row0 * QROW_B;
      const uint32_t off = (uint32_t)((n * p.H + j) * QROW_B + unit * 16);
      __builtin_amdgcn_global_load_lds(base + off, lds_ptr(qbuf + buf * QTILE_B + wave * 1024), 16, 0, 0);
    }
  }

  __device__ __forceinline__ void slab_scale(int l, int g) {
    if constexpr (FP8) {
      if (p.k_scale) c2 = p.c * p.k_scale[l * p.H_kv + g];
    }
  }

  __device__ __forceinline__ bf16x8 read16(uint32_t addr) const {
    return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(lds_ptr(addr));
  }
  // logits of 32-key tile `sub` of the slot against the 32 query rows of buffer `buf`
  __device__ __forceinline__ f32x16 mfma_tile(int slot, int sub, int buf) {
    f32x16 a = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    uint32_t kb = krd0, qb = qrd0;
    asm volatile("" : "+v"(kb), "+v"(qb));
    const uint32_t kadd = slot * kItemBytes + sub * 32 * KROW_B, qadd = buf * QTILE_B;
    bf16x8 kf[KS], qf[KS];
    if constexpr (FP8) {
      u32x4 raw[KS / 2];
#pragma unroll
      for (int j = 0; j < KS / 2; ++j)
        raw[j] = __builtin_bit_cast(u32x4, read16((kb ^ (uint32_t)((2 * j) << 4)) + kadd));
#pragma unroll
      for (int t = 0; t < KS; ++t) qf[t] = read16((qb ^ (uint32_t)((4 * (t >> 1) + (t & 1)) << 4)) + qadd);
#pragma unroll
      for (int t = 0; t < KS; ++t) {
        u32x4 o;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          o[2 * x] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[t >> 1][2 * (t & 1) + x], 1.0f, false));
          o[2 * x + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[t >> 1][2 * (t & 1) + x], 1.0f, true));
        }
        a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, o), qf[t], a, 0, 0, 0);
      }
      return a;
    }
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      kf[t] = read16((kb ^ (uint32_t)(t << 5)) + kadd);
      qf[t] = read16((qb ^ (uint32_t)(t << 5)) + qadd);
    }
#pragma unroll
    for (int t = 0; t < KS; ++t) a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t], qf[t], a, 0, 0, 0);
    constexpr int kAhead = KS < 2 ? KS : 2;
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * kAhead, 0);
#pragma unroll
    for (int t = 0; t < KS - kAhead; ++t) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kAhead, 0);
    return a;
  }

  // log2-probabilities of a held tile, maximum over the heads of a group: the lane's KEEP consecutive keys, the
  // first of which is fold_key() of the tile, of query col & (NS - 1)
  __device__ __forceinline__ int fold_key() const {
    const int ln = lane_id(), c = ln & 31, h = ln >> 5;
    return (((c >> 4) << 1) | ((c >> 3) & 1)) * 8 + h * 4 + (LG == 3 ? ((c >> 2) & 1) * 2 : 0);
  }
  __device__ __forceinline__ void fold_heads(const f32x16& a, float neg_lse2, float (&out)[KEEP]) const {
    float y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // lanes with col bit 4 clear keep keys 0..15's registers, the others 16..31's
      const float lo = fmaf(a[i], c2, neg_lse2), hi = fmaf(a[i + 8], c2, neg_lse2);
      const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
      y[i] = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    // bit 3: lanes 0..7 of a row take y[0..3], lanes 8..15 y[4..7].  (s_nop: a DPP operand must not have been
    // written by the two instructions before)
    float z[4];
    asm("s_nop 1\n\t"
        "v_max_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_max_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_max_f32_dpp %2, %6, %6 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_max_f32_dpp %3, %7, %7 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_max_f32_dpp %0, %8, %8 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_max_f32_dpp %1, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_max_f32_dpp %2, %10, %10 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_max_f32_dpp %3, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc"
        : "=&v"(z[0]), "=&v"(z[1]), "=&v"(z[2]), "=&v"(z[3])
        : "v"(y[0]), "v"(y[1]), "v"(y[2]), "v"(y[3]), "v"(y[4]), "v"(y[5]), "v"(y[6]), "v"(y[7]));
    if constexpr (LG == 3) {  // bit 2: banks 0 and 2 take z[0..1] (partner four lanes up), banks 1 and 3 z[2..3]
      asm("s_nop 1\n\t"
          "v_max_f32_dpp %0, %2, %2 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
          "v_max_f32_dpp %1, %3, %3 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
          "v_max_f32_dpp %0, %4, %4 row_ror:4 row_mask:0xf bank_mask:0xa\n\t"
          "v_max_f32_dpp %1, %5, %5 row_ror:4 row_mask:0xf bank_mask:0xa"
          : "=&v"(out[0]), "=&v"(out[1])
          : "v"(z[0]), "v"(z[1]), "v"(z[2]), "v"(z[3]));
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) out[k] = z[k];
    }
  }
};

template <int D, int LG, bool FP8, bool PAGED>
__global__ __launch_bounds__(kTiledThreads) void wide_score_kernel(const TiledDev p) {
  extern __shared__ __align__(1024) unsigned char smem[];
  using W = WideKernel<D, LG, FP8, PAGED>;
  constexpr int KEEP = W::KEEP, SUB = W::SUB;
  typedef float vkeep __attribute__((ext_vector_type(KEEP)));
  W w(p, smem);
  SeqUnit cur;
  if (!seq_next_unit(p, 0, &cur)) return;

  // The stream of key items runs up to two items ahead of the arithmetic, on into the next slab (of this unit or the
  // next one): `ah` is where the next request comes from, `nx` the slab behind the one being computed.
  // A wave takes items wave, wave + 8, ... of a sequence, the last one first.
  auto items_of = [&](int M) __attribute__((always_inline)) {
    return __builtin_amdgcn_readfirstlane(((M + W::KPI - 1) / W::KPI - w.wave + kTiledWaves - 1) / kTiledWaves);
  };
  struct Stream { const unsigned char* slab; int b, M, left; };  // left: items of the slab not yet requested
  Stream ah, nx;
  int sent = 0, pos = 0;  // items requested / consumed so far; item number x sits in ring slot x & 1
  auto issue_one = [&]() __attribute__((always_inline)) {
    --ah.left;
    const int key_first = (w.wave + ah.left * kTiledWaves) * W::KPI;
    w.issue_keys(ah.slab, ah.b, key_first, ah.M - key_first, sent & 1);
    ++sent;
  };
  int l = cur.s0 / p.H_kv, g = cur.s0 - l * p.H_kv;
  ah = Stream{w.slab_keys(l, g, cur.seq0), cur.b, cur.M, items_of(cur.M)};
  w.issue_queries(l, g, cur.b, 0);
  if (ah.left > 0) issue_one();
  if (ah.left > 0) issue_one();
  if (sent == 2) wait_vmcnt<2 * kItemLoads>(); else wait_vmcnt<0>();  // the query tile
  __builtin_amdgcn_s_barrier();

  int slabs = 0;  // slabs finished so far
  bool more = true;
  SeqUnit nxt = cur;

  // all slabs of unit `cur`, tiles_c tiles per wave of which the first run_c have their running maxima in registers
  auto do_unit = [&](auto tiles_c, auto run_c) __attribute__((always_inline)) {
    constexpr int MAXT = decltype(tiles_c)::value, RUN = decltype(run_c)::value, MAXI = MAXT / SUB;
    static_assert(MAXT % SUB == 0, "whole items");
    f32x16 held[MAXT];
    vkeep run[RUN];
    const int M = cur.M, b = cur.b;
    const int nt = items_of(M);
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
      nx.left = 0;
      if (s + 1 < cur.s1) {
        nx = Stream{w.slab_keys(nl, ng, cur.seq0), b, M, nt};
        w.issue_queries(nl, ng, b, buf ^ 1);
      } else {
        more = seq_next_unit(p, cur.k + 1, &nxt);
        if (more) {
          nl = nxt.s0 / p.H_kv;
          ng = nxt.s0 - nl * p.H_kv;
          nx = Stream{w.slab_keys(nl, ng, nxt.seq0), nxt.b, nxt.M, items_of(nxt.M)};
          w.issue_queries(nl, ng, nxt.b, buf ^ 1);
        }
      }
      bool fresh = true;  // nx has not been moved to yet
      auto refill = [&]() __attribute__((always_inline)) {
        if (ah.left == 0 && fresh) { ah = nx; fresh = false; }
        if (ah.left > 0) issue_one();
      };
      while (sent - pos < 2 && (ah.left > 0 || (fresh && nx.left > 0))) refill();  // (waves with less than two items per slab)
      w.slab_scale(l, g);
      float rm = -INFINITY, rs = 0.f;  // the lane's row over this wave's keys: max of the base-2 logits (as rounded), sum of exp2
      wide_static_for<0, MAXI>([&](auto ic) __attribute__((always_inline)) {
        constexpr int it = decltype(ic)::value;
        if (it < nt) {
          const int slot = pos & 1;
          // (vector-memory instructions of a wave complete in order; those of the next item are the only key loads
          // behind this one's; result stores there only make the wait stricter)
          if (sent - pos == 2) wait_vmcnt<kItemLoads>(); else wait_vmcnt<0>();
#pragma unroll
          for (int sub = 0; sub < SUB; ++sub) held[it * SUB + sub] = w.mfma_tile(slot, sub, buf);
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot's reads are done: it may be overwritten
          ++pos;
          refill();
#pragma unroll
          for (int sub = 0; sub < SUB; ++sub) {
            f32x16& a = held[it * SUB + sub];
            if constexpr (it == 0) {  // the sequence's ragged end is in some wave's last item
              const int left_wave = M - (w.wave + (nt - 1) * kTiledWaves) * W::KPI - sub * 32;
              if (left_wave < 32) {
                const int left = left_wave - (W::lane_id() >> 5) * 4;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                  if ((i >> 2) * 8 + (i & 3) >= left) a[i] = -INFINITY;
              }
            }
            float tm = a[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) tm = fmaxf(tm, a[i]);
            const float m_new = fmaxf(rm, tm * w.c2);
            const float off = (it == 0 && m_new == -INFINITY) ? 0.f : -m_new;
            float s0 = rs * fast_exp2(rm + off), s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
            for (int i = 0; i < 16; i += 4) {
              s0 += fast_exp2(fmaf(a[i], w.c2, off));
              s1 += fast_exp2(fmaf(a[i + 1], w.c2, off));
              s2 += fast_exp2(fmaf(a[i + 2], w.c2, off));
              s3 += fast_exp2(fmaf(a[i + 3], w.c2, off));
            }
            rm = m_new;
            rs = (s0 + s1) + (s2 + s3);
          }
        }
      });

      // the rows' statistics over the wave's keys (two half-waves), then over the workgroup's
      {
        const auto sm = __builtin_amdgcn_permlane32_swap(__float_as_uint(rm), __float_as_uint(rm), false, false);
        const auto ss = __builtin_amdgcn_permlane32_swap(__float_as_uint(rs), __float_as_uint(rs), false, false);
        const float ma = __uint_as_float(sm[0]), mb = __uint_as_float(sm[1]);
        const float mn = fmaxf(ma, mb);
        const float ref = (mn == -INFINITY) ? 0.f : mn;
        const float z = __uint_as_float(ss[0]) * fast_exp2(ma - ref) + __uint_as_float(ss[1]) * fast_exp2(mb - ref);
        const int ln = W::lane_id(), c = ln & 31, h = ln >> 5;
        if (h == 0)
          lds_poke64<0>(w.xchg + ((buf * kTiledWaves + w.wave) * 32 + c) * 8, ((uint64_t)__float_as_uint(z) << 32) | __float_as_uint(mn));
      }
      // this wave's share of the next slab's query tile has landed (it was sent before this slab's refills; a wave
      // whose items in flight are older than that waits for them too)
      if (sent - pos == 2) wait_vmcnt<2 * kItemLoads>(); else if (sent - pos == 1) wait_vmcnt<kItemLoads>(); else wait_vmcnt<0>();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      ++slabs;
      float neg_lse2;
      {
        const int ln = W::lane_id(), c = ln & 31, h = ln >> 5;
        // a half-wave folds four of the eight waves' pairs, then the halves meet
        const u64x4 v = lds_peek64x4<256>(w.xchg + ((buf * kTiledWaves + 4 * h) * 32 + c) * 8);
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) m = fmaxf(m, __uint_as_float((uint32_t)v.v[i]));
        const float ref = (m == -INFINITY) ? 0.f : m;
        float z = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          z += __uint_as_float((uint32_t)(v.v[i] >> 32)) * fast_exp2(__uint_as_float((uint32_t)v.v[i]) - ref);
        const auto sm = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
        const auto ss = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
        const float ma = __uint_as_float(sm[0]), mb = __uint_as_float(sm[1]);
        m = fmaxf(ma, mb);  // (finite: the sequence has a key)
        z = __uint_as_float(ss[0]) * fast_exp2(ma - m) + __uint_as_float(ss[1]) * fast_exp2(mb - m);
        const float lse2 = m + __builtin_amdgcn_logf(z);
        neg_lse2 = -lse2;
        if (p.lse_out && w.wave == 0) {
          const int n = c & (W::NS - 1), j = c >> (5 - LG);
          if (h == 0 && n < p.N && j < p.G)
            p.lse_out[(((int64_t)l * p.B + b) * p.N + n) * p.H + g * p.G + j] = lse2 * 0.6931471805599453f;
        }
      }

      // log2-probabilities; maximum over the heads of a group and over the unit's slabs
      const int first = w.fold_key(), q_n = W::lane_id() & (W::NS - 1);
      float* out = out0 + (SUB * (w.wave + (nt - 1) * kTiledWaves)) * out_step + q_n * 32 + first;
      auto place = [&](int it, int sub) __attribute__((always_inline)) {  // of a tile's results
        return reinterpret_cast<vkeep*>(out + (sub - it * (SUB * kTiledWaves)) * out_step);
      };
      auto live = [&](int it, int sub) __attribute__((always_inline)) {
        // (sub-tiles of the ragged item that lie beyond the sequence have no place in the result array)
        return it < nt && (SUB == 1 || it > 0 || (w.wave + (nt - 1) * kTiledWaves) * W::KPI + sub * 32 < M);
      };
      wide_static_for<0, RUN>([&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        if (t / SUB < nt) {
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
        if (t0 / SUB < nt) {
          vkeep old[tn];
#pragma unroll
          for (int i = 0; i < tn; ++i)
#pragma unroll
            for (int k = 0; k < KEEP; ++k) old[i][k] = -INFINITY;
          if (s != cur.s0 && q_n < p.N) {
#pragma unroll
            for (int i = 0; i < tn; ++i)
              if (live((t0 + i) / SUB, (t0 + i) % SUB)) old[i] = *place((t0 + i) / SUB, (t0 + i) % SUB);
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
              if (live((t0 + i) / SUB, (t0 + i) % SUB)) __builtin_nontemporal_store(old[i], place((t0 + i) / SUB, (t0 + i) % SUB));
          }
        }
      });
      if (s + 1 == cur.s1 && q_n < p.N) {  // the unit's result
        wide_static_for<0, RUN>([&](auto tc) __attribute__((always_inline)) {
          constexpr int t = decltype(tc)::value;
          if (live(t / SUB, t % SUB)) __builtin_nontemporal_store(run[t], place(t / SUB, t % SUB));
        });
      }
      // on to the next slab (its first unrequested items may have been sent already)
      if (fresh && ah.left == 0) ah = nx;
      l = nl;
      g = ng;
    }
  };
#pragma unroll 1
  for (;;) {
    if (cur.M <= W::kShort * 32 * kTiledWaves) do_unit(std::integral_constant<int, W::kShort>{}, std::integral_constant<int, W::kShort>{});
    else do_unit(std::integral_constant<int, kWideTiles>{}, std::integral_constant<int, kWideRunTiles>{});
    if (!more) break;
    cur = nxt;
  }
  wait_vmcnt<0>();
}

// Merge of the units' results and the average over the valid queries.  One workgroup per 32-key tile (or per half
// of one: KEYS = 16, where a short prompt has too few tiles to fill the device): it reads one dense block,
// KEYS / 4 threads per (group, query) row, every thread keeps to one query, the threads of a query meet in LDS.
// Sequences the scoring kernel left out (longer than it holds) get NaN.
template <int KEYS>
__global__ __launch_bounds__(1024) void wide_finish_kernel(const TiledDev p) {
  constexpr int TPR = KEYS / 4;            // threads per row
  constexpr int ROWS = 1024 / TPR;         // rows per step
  __shared__ float red[ROWS][KEYS];
  const int tile = blockIdx.x / (32 / KEYS), part = blockIdx.x % (32 / KEYS);
  int lo = 0, hi = p.B;                    // the sequence: the largest b whose first tile is <= tile
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (wide_tile_base(p.cu[mid], mid) <= tile) lo = mid; else hi = mid;
  }
  const int seq0 = p.cu[lo], M = p.cu[lo + 1] - seq0;
  const int key0 = (tile - wide_tile_base(seq0, lo)) * 32 + part * KEYS;
  if (key0 >= M) return;
  if (M > p.seq_limit) {
    if (threadIdx.x < KEYS && key0 + (int)threadIdx.x < M) p.scores[seq0 + key0 + threadIdx.x] = __uint_as_float(0x7FC00000u);
    return;
  }
  const bool mean = p.layer_reduce != SP_LAYER_MAX;
  const int per = ROWS / p.N;              // groups (mean: layers) per step
  const int row = threadIdx.x / TPR, quad = threadIdx.x % TPR;
  const int n = row % p.N, g0 = row / p.N;
  f32x4 v = mean ? f32x4{0.f, 0.f, 0.f, 0.f} : f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  if (g0 < per) {
    const float* src = p.group_scores + ((int64_t)tile * p.n_groups * p.N + n) * 32 + part * KEYS + quad * 4;
    const int64_t step = (int64_t)p.N * 32;
    if (mean) {  // the groups of a layer hold the log2 of its maxima over their KV heads; the layers' maxima add up
      for (int l = g0; l < p.L; l += per) {
        f32x4 m = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll 4
        for (int j = 0; j < p.groups_per_layer; ++j) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(src + (int64_t)(l * p.groups_per_layer + j) * step);
#pragma unroll
          for (int k = 0; k < 4; ++k) m[k] = fmaxf(m[k], x[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += fast_exp2(m[k]);
      }
    } else {
#pragma unroll 8
      for (int g = g0; g < p.n_groups; g += per) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(src + g * step);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], x[k]);
      }
    }
  }
  *reinterpret_cast<f32x4*>(&red[row][quad * 4]) = v;
  __syncthreads();
  // all threads fold the rows of a (query, key), then KEYS * N of them the 1024 / (KEYS * N) results of each
  const int fk = threadIdx.x % KEYS, fn = threadIdx.x / KEYS % p.N, sub = threadIdx.x / KEYS / p.N;
  const int subs = 1024 / KEYS / p.N;
  float x = mean ? 0.f : -INFINITY;
  if (sub < subs)
    for (int q = sub; q < per; q += subs) {
      const float y = red[q * p.N + fn][fk];
      x = mean ? x + y : fmaxf(x, y);
    }
  __syncthreads();
  if (sub < subs) red[sub * p.N + fn][fk] = x;
  __syncthreads();
  if (sub == 0) {
    for (int q = 1; q < min(subs, per); ++q) {
      const float y = red[q * p.N + fn][fk];
      x = mean ? x + y : fmaxf(x, y);
    }
    red[fn][fk] = mean ? x : fast_exp2(x);  // (rows 0..N-1 are read by their own threads only)
  }
  __syncthreads();
  if (threadIdx.x >= KEYS || key0 + fk >= M) return;
  int nv = p.n_valid ? p.n_valid[lo] : p.N;
  nv = max(1, min(nv, p.N));
  float sum = 0.f;
  for (int q = 0; q < nv; ++q) sum += red[q][fk];
  p.scores[seq0 + key0 + fk] = sum / (mean ? (float)nv * (float)p.L : (float)nv);
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
static int wide_lg(const sp_score_args* a) { return a->H / a->H_kv <= 4 ? 2 : 3; }
int wide_max_keys(const sp_score_args*) { return kWideTiles * 32 * kTiledWaves; }
static int64_t wide_stated_max(const sp_score_args* a) { return a->B == 1 ? a->T : a->max_seqlen; }

bool wide_supported(const sp_score_args* a) {
  if (a->rope_theta > 0.f || wide_stated_max(a) <= 0 || a->T < 1) return false;
  if (a->H / a->H_kv > 8 || (a->N << wide_lg(a)) > 32) return false;
  if (a->k_dtype == SP_K_FP8_E4M3 && a->d_block_table && a->page_size < (a->d == 64 ? 16 : 8)) return false;
  if (wide_stated_max(a) > wide_max_keys(a)) return false;
  if (a->k_token_stride > (INT32_MAX / 256)) return false;  // (a ring slot's keys must span less than 2 GiB)
  if (a->B > 8192) return false;
  if ((int64_t)a->B * a->L * a->H_kv < 64) return false;
  return true;
}

// Units: runs of slabs; with the mean over layers parts of one layer (the merge adds the layers up).
void wide_grouping(const sp_score_args* a, int* slabs_per_group, int* n_groups, int* groups_per_layer) {
  if (a->layer_reduce == SP_LAYER_MEAN) {
    int per = 1;
    for (int cand = a->H_kv; cand >= 1; --cand)
      if (a->H_kv % cand == 0 && (int64_t)a->B * a->L * (a->H_kv / cand) >= 512) { per = cand; break; }
    *slabs_per_group = per;
    *groups_per_layer = a->H_kv / per;
    *n_groups = a->L * *groups_per_layer;
    return;
  }
  *groups_per_layer = 0;
  const int slabs = a->L * a->H_kv;
  const int per_wg = std::min(8, std::max(2, a->B / 32));
  int groups = std::max(1, std::min(slabs, (256 * per_wg + a->B - 1) / a->B));
  const int per = (slabs + groups - 1) / groups;
  *slabs_per_group = per;
  *n_groups = (slabs + per - 1) / per;
}

static size_t wide_tiles(const sp_score_args* a) { return (size_t)(a->T >> 5) + a->B; }  // of the result array
static size_t wide_scores_bytes(const sp_score_args* a) {
  int per, groups, gpl;
  wide_grouping(a, &per, &groups, &gpl);
  return align_up(sizeof(float) * 32 * (size_t)groups * a->N * wide_tiles(a), 256);
}
size_t wide_workspace_bytes(const sp_score_args* a) {
  if (!wide_supported(a)) return 0;
  return wide_scores_bytes(a) + align_up(sizeof(int32_t) * (size_t)a->B, 256);
}

template <int D, int LG, bool FP8, bool PAGED>
static sp_status launch_wide(const TiledDev& dev, hipStream_t stream) {
  auto kernel = wide_score_kernel<D, LG, FP8, PAGED>;
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
  const int wgs = std::min(dev.B * dev.n_groups, seq_cu_count());
  hipLaunchKernelGGL(kernel, dim3(wgs), dim3(kTiledThreads), smem, stream, dev);
  return launch_status();
}
template <int D, int LG, bool FP8>
static sp_status wide_by_pages(const TiledDev& dev, hipStream_t stream) {
  return dev.block_table ? launch_wide<D, LG, FP8, true>(dev, stream) : launch_wide<D, LG, FP8, false>(dev, stream);
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
  dev.seq_order = nullptr;
  if (a->B > 1) {
    int32_t* order = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(dev.group_scores) + wide_scores_bytes(a));
    launch_seq_order(a, order, dev.seq_limit, stream);
    dev.seq_order = order;
  }
  const sp_status st = a->d == 64 ? wide_by_kind<64>(a, dev, stream) : wide_by_kind<128>(a, dev, stream);
  if (st != SP_OK) return st;
  // two workgroups per 32-key tile where the tiles alone would not give every compute unit two
  const unsigned tiles = (unsigned)wide_tiles(a);
  if (tiles < 512) hipLaunchKernelGGL(wide_finish_kernel<16>, dim3(2 * tiles), dim3(1024), 0, stream, dev);
  else hipLaunchKernelGGL(wide_finish_kernel<32>, dim3(tiles), dim3(1024), 0, stream, dev);
  return launch_status();
}

}  // namespace sp
