// What the single-pass kernels that hold a KV head's 32 query rows as the columns of the MFMA result share
// (sp_score_wide.hip: a workgroup owns whole sequences; sp_score_wide_team.hip: a few workgroups share one long
// prompt): the stream of key items through the LDS ring, the products, the row statistics, the fold over heads, and
// the merge of the results (Sec. 3.2 equation and Sec. 3.2.2 of arXiv 2502.02789).
#pragma once

#include "sp_tile_walker.h"

namespace sp {

// A wave's ring of key items, whatever their size.  An item is one 32-key tile: with items of 8 KiB (two or four tiles of
// 8-bit keys or d = 64) a slot was held while all its tiles were multiplied, and the first of the next slab could not be
// computed early by the teams.  (Whole call, 32 layers, 8 KV heads, eight queries: 8-bit keys, d = 128, 32K keys 238 -> 232 us,
// 70000 605 -> 565; 16 layers of d = 64, 33000 keys 144 -> 134, 128K 423 -> 405; nothing beyond the noise where an item was
// one tile before.)
constexpr int kWaveRingBytes = 16384;

typedef float f32x4 __attribute__((ext_vector_type(4)));

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

// READ_AHEAD: of 8-bit keys' operands (below); it takes registers that the kernel with twelve held tiles has not got
template <int D, int LG, bool FP8, bool PAGED, bool READ_AHEAD = true>
struct WideKernel {
  static constexpr int ESZ = FP8 ? 1 : 2;
  static constexpr int KS = D / 16;               // MFMA k-steps
  static constexpr int KROW_B = D * ESZ;          // bytes of a key
  static constexpr int KU = KROW_B / 16;          // its 16-byte units: 16, 8 or 4
  static constexpr int KSH = KU == 16 ? 0 : KU == 8 ? 1 : 2;
  static constexpr int RPI = 64 / KU;             // keys per wave-wide load
  static constexpr int ITEM_B = 32 * KROW_B;      // an item: the 32 keys of a tile, 8, 4 or 2 KiB
  static constexpr int LOADS = ITEM_B / 1024;     // wave-wide loads of an item
  static constexpr int SLOTS = kWaveRingBytes / ITEM_B;  // items in the ring: 2, 4 or 8
  static constexpr int QROW_B = D * 2;
  static constexpr int QU = QROW_B / 16;
  static constexpr int QTILE_B = 32 * QROW_B;
  static constexpr int QLOADS = QTILE_B / 1024;   // one load each by the first QLOADS waves
  static constexpr int NS = 32 >> LG;             // query slots
  static constexpr int KEEP = 16 >> LG;           // keys per lane and tile after the fold over heads: 8, 4 or 2
  typedef float vkeep __attribute__((ext_vector_type(KEEP)));
  static constexpr int kRingB = kTiledWaves * kWaveRingBytes;
  static constexpr int kSmem = kRingB + 2 * QTILE_B + 2 * kTiledWaves * 32 * 8;

  const TiledDev& p;
  int wave;
  uint32_t ring, qbuf, xchg;  // LDS addresses: this wave's slots, the two query tiles, the exchange table
  uint32_t ld_row, ld_unit, krd0, qrd0;  // this lane's key and 16-byte unit in a load; where it reads its operands
  uint32_t ts_b;              // bytes from key to key (the host checks that a slot's keys span less than 2 GiB)
  float c2;
  int scale_bits;             // FP8: of the key scale of the slab at hand

  // The stream of key items runs up to a ringful ahead of the arithmetic, on into the next slab: `ah` is where the
  // next request comes from, `nx` the slab behind the one being computed (`fresh`: not moved to yet).  A wave takes
  // items wave, wave + 8, ... of the M keys its workgroup owns of a sequence, the last one first.
  struct Slab { const unsigned char* keys; int b, first, M, left; };  // first: of the owned keys; left: items not yet requested
  Slab ah, nx;
  bool fresh;
  int sent, pos;  // items requested / consumed so far; item number x sits in ring slot x mod SLOTS

  __device__ __forceinline__ WideKernel(const TiledDev& p_, unsigned char* smem) : p(p_) {
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, half = lane >> 5, col = lane & 31;
    const uint32_t base = (uint32_t)reinterpret_cast<uintptr_t>(smem);
    ring = base + wave * kWaveRingBytes;
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
    scale_bits = 1;
    sent = pos = 0;
    fresh = false;
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

  // 16 bytes per lane from where the lane says; `dst`: of the wave's first lane
  __device__ __forceinline__ static void load16(const unsigned char* from, uint32_t dst) {
    __builtin_amdgcn_global_load_lds(from, lds_ptr(dst), 16, 0, 0);
  }

  // where the keys of (l, g) start: those of token seq0 (contiguous cache) or of the pool's first page
  __device__ __forceinline__ const unsigned char* slab_keys(int l, int g, int seq0) const {
    return reinterpret_cast<const unsigned char*>(p.k[l]) + ESZ * ((int64_t)g * p.hs + (PAGED ? 0 : (int64_t)seq0 * p.ts));
  }
  // keys [key_first, key_first + 32) of sequence b, of which the first `rows` (>= 1) exist -> ring slot
  __device__ __forceinline__ void issue_keys(const unsigned char* slab, int b, int key_first, int rows, int slot) {
    const uint32_t dst = ring + slot * ITEM_B;
    if constexpr (PAGED) {
      // (the RPI keys of one load lie in one page: pages hold a power of two >= 8 keys, >= RPI where the host checks)
      // Two loops that stay loops, the next page's entry fetched while a page's loads go out: unrolled, this is most
      // of the kernel's code, more than the instruction cache holds.
      const ScalarTable table = scalar_table(p.block_table + (int64_t)b * p.blocks_per_seq);
      const int page = 1 << p.lg_page, last = (key_first + min(rows, 32) - 1) >> p.lg_page;
      int pg = key_first >> p.lg_page, entry = table[pg];
      int in_page = key_first & (page - 1);
      // A page's descriptor starts where the item's first key would be if all of it lay in that page, so that offsets and
      // range are the item's, as for a contiguous cache, and a load is left with little scalar work.
      const uint32_t bytes = (uint32_t)(min(rows, 32) - 1) * ts_b + KROW_B;
      const uint32_t lane_row = ld_row;
      uint32_t row_off = 0;
      int j = 0;
#pragma unroll 1
      for (;;) {
        const unsigned char* base = slab + ESZ * ((int64_t)entry * p.page_stride) + (int64_t)(in_page - j * RPI) * (int64_t)ts_b;
        entry = table[min(pg + 1, last)];
        const int j_end = min(LOADS, j + ((page - in_page) / RPI));
#pragma unroll 1
        for (; j < j_end; ++j) {
          load1k(base, bytes, lane_row + (ld_unit ^ (uint32_t)(((4 * j) & (KU - 1)) << 4)) + row_off, dst + j * 1024);
          row_off += (uint32_t)RPI * ts_b;
        }
        if (j == LOADS) break;
        ++pg;
        in_page = 0;
      }
    } else {
      const unsigned char* base = slab + (int64_t)key_first * (int64_t)ts_b;
      const uint32_t bytes = (uint32_t)(min(rows, 32) - 1) * ts_b + KROW_B;
#pragma unroll
      for (int j = 0; j < LOADS; ++j) {
        load1k(base, bytes, lane_offset(j) + (uint32_t)(j * RPI) * ts_b, dst + j * 1024);
      }
    }
  }

  // "At most n items still in flight" (wait_vmcnt_upto has no steps of two below eight loads: 64 prompts of 200..1000 8-bit
  // keys, 16 layers of d = 64, eight queries, 75.1 -> 71.9 us; longer sequences, whose ring is full, the same).
  __device__ __forceinline__ static void wait_items(int n) {
    if (LOADS != 2 || n >= 4) wait_vmcnt_upto(n * LOADS);
    else if (n >= 2) { if (n == 3) wait_vmcnt<6>(); else wait_vmcnt<4>(); }
    else { if (n == 1) wait_vmcnt<2>(); else wait_vmcnt<0>(); }
  }

  __device__ __forceinline__ int items_of(int M) const {
    return __builtin_amdgcn_readfirstlane(((M + 31) / 32 - wave + kTiledWaves - 1) / kTiledWaves);
  }
  __device__ __forceinline__ void issue_one() {
    --ah.left;
    const int key = (wave + ah.left * kTiledWaves) * 32;
    issue_keys(ah.keys, ah.b, ah.first + key, ah.M - key, sent & (SLOTS - 1));
    ++sent;
  }
  __device__ __forceinline__ void refill() {
    if (ah.left == 0 && fresh) { ah = nx; fresh = false; }
    if (ah.left > 0) issue_one();
  }
  // a slab begins: `nx` has been set to the one behind it (left = 0: there is none)
  __device__ __forceinline__ void begin_slab() {
    fresh = true;
    while (sent - pos < SLOTS && (ah.left > 0 || (fresh && nx.left > 0))) refill();  // (waves with less than a ringful per slab)
  }
  // a workgroup's first slab: the first items on their way ...
  __device__ __forceinline__ void start_stream() {
    while (sent < SLOTS && ah.left > 0) issue_one();
  }
  // ... and, in front of its products, the query tile (requested before them) here.  (What the kernel for few rows puts between the
  // two, the set-up of its loop and the next slab's requests, waits for instructions while the first loads travel; the kernel for 32
  // rows is faster without: one prompt of 300 keys 15.3 -> 14.8 us.)
  __device__ __forceinline__ void first_queries() {
    wait_items(sent);
    __builtin_amdgcn_s_barrier();
  }
  __device__ __forceinline__ void end_slab() {
    if (fresh && ah.left == 0) ah = nx;
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
      load16(base + off, qbuf + buf * QTILE_B + wave * 1024);
    }
  }

  // logits -> base-2 domain for (l, g), an 8-bit cache's key scale included (through the scalar cache, as a block table)
  __device__ __forceinline__ void slab_scale(int l, int g) {
    if constexpr (FP8) {
      if (p.k_scale) {
        scale_bits = scalar_table(reinterpret_cast<const int32_t*>(p.k_scale))[l * p.H_kv + g];
        c2 = positive_scale(p.c, __int_as_float(scale_bits));
        return;
      }
    }
    c2 = p.c;
  }

  __device__ __forceinline__ bf16x8 read16(uint32_t addr) const {
    return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(lds_ptr(addr));
  }
  // logits of the slot's keys against the 32 query rows of buffer `buf`
  __device__ __forceinline__ f32x16 mfma_tile(int slot, int buf) {
    f32x16 a = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    uint32_t kb = krd0, qb = qrd0;
    asm volatile("" : "+v"(kb), "+v"(qb));
    const uint32_t kadd = slot * ITEM_B, qadd = buf * QTILE_B;
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
      // All key units and two query units are read ahead: left to itself the compiler waits for every read in front of
      // the product it is for, eight LDS round trips a tile (whole call, 32K keys, 8B shape 232 -> 224 us; three ahead 227,
      // four spill: 294).  (The 8-bit matrix instructions, which would take the stored bytes with the queries split into
      // two terms each, are no faster than that, 223 us, and round sums to 2^-17 of their terms; the bf16 ones to 2^-24.)
      if constexpr (READ_AHEAD) {
        constexpr int kAhead = 2;
        __builtin_amdgcn_sched_group_barrier(0x100, KS / 2 + kAhead, 0);
#pragma unroll
        for (int t = 0; t < KS; ++t) {
          __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (t < KS - kAhead) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
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

  // log2-probabilities of a held tile, maximum over the heads of a group: the lane's KEEP keys, of query col & (NS - 1).
  // The first is fold_key() of the tile, the others follow it (with two heads per group: four, and four from eight on).
  __device__ __forceinline__ int fold_key() const {
    const int ln = lane_id(), c = ln & 31, h = ln >> 5;
    if constexpr (LG == 1) return (c >> 4) * 16 + h * 4;
    return (((c >> 4) << 1) | ((c >> 3) & 1)) * 8 + h * 4 + (LG == 3 ? ((c >> 2) & 1) * 2 : 0);
  }
  // a lane's keys of a tile in the result array, `at` being fold_key()'s
  __device__ __forceinline__ static void store_keep(float* at, const vkeep& v) {
    if constexpr (LG == 1) {
      __builtin_nontemporal_store(f32x4{v[0], v[1], v[2], v[3]}, reinterpret_cast<f32x4*>(at));
      __builtin_nontemporal_store(f32x4{v[4], v[5], v[6], v[7]}, reinterpret_cast<f32x4*>(at + 8));
    } else {
      __builtin_nontemporal_store(v, reinterpret_cast<vkeep*>(at));
    }
  }
  __device__ __forceinline__ static vkeep load_keep(const float* at) {
    if constexpr (LG == 1) {
      const f32x4 lo = *reinterpret_cast<const f32x4*>(at), hi = *reinterpret_cast<const f32x4*>(at + 8);
      return vkeep{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    } else {
      return *reinterpret_cast<const vkeep*>(at);
    }
  }
  __device__ __forceinline__ void fold_heads(const f32x16& a, float neg_lse2, float (&out)[KEEP]) const { fold_heads(a, c2, neg_lse2, out); }
  __device__ __forceinline__ static void fold_heads(const f32x16& a, float c2, float neg_lse2, float (&out)[KEEP]) {
    float y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // lanes with col bit 4 clear keep keys 0..15's registers, the others 16..31's
      const float lo = fmaf(a[i], c2, neg_lse2), hi = fmaf(a[i + 8], c2, neg_lse2);
      const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
      y[i] = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
    if constexpr (LG == 1) {
#pragma unroll
      for (int k = 0; k < 8; ++k) out[k] = y[k];
      return;
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
    } else if constexpr (LG == 2) {
#pragma unroll
      for (int k = 0; k < 4; ++k) out[k] = z[k];
    }
  }

  // 64 words (the 32 of a line, twice) straight into LDS
  __device__ __forceinline__ void load_line(const float* line, uint32_t dst) const {
    __builtin_amdgcn_global_load_lds(line + (lane_id() & 31), lds_ptr(dst), 4, 0, 0);
  }

  // the next item's products with the query rows of buffer `buf`
  __device__ __forceinline__ f32x16 item_products(int buf) {
    // (vector-memory instructions of a wave complete in order; those of later items are the only key loads behind
    // this one's; result stores there only make the wait stricter)
    const int later = sent - pos - 1;
    if (later == SLOTS - 1) wait_vmcnt<(SLOTS - 1) * LOADS>(); else wait_items(later);
    f32x16 a = mfma_tile(pos & (SLOTS - 1), buf);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slot's reads are done: it may be overwritten
    ++pos;
    refill();
    if constexpr (FP8) odd_products(a, scale_bits);
    return a;
  }
  // Item IT of the wave's nt items of a slab: its logits, and the lane's row's statistics over the wave's keys so far:
  // (rm, rs) = maximum of the base-2 logits (as rounded) and sum of exp2 relative to it
  template <int IT>
  __device__ __forceinline__ f32x16 item_logits(int nt, int M, int buf, float& rm, float& rs) {
    f32x16 a = item_products(buf);
    if constexpr (IT == 0) {  // the ragged end of the keys is in some wave's last item
      const int left_wave = M - (wave + (nt - 1) * kTiledWaves) * 32;
      if (left_wave < 32) {
        const int left = left_wave - (lane_id() >> 5) * 4;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if ((i >> 2) * 8 + (i & 3) >= left) a[i] = -INFINITY;
      }
    }
    float tm = a[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) tm = fmaxf(tm, a[i]);
    const float m_new = fmaxf(rm, tm * c2);
    // (-inf: no key of the lane so far, or none whose logit fits fp32)
    const float off = (m_new == -INFINITY) ? 0.f : -m_new;
    float s0 = rs * fast_exp2(rm + off), s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll
    for (int i = 0; i < 16; i += 4) {
      s0 += fast_exp2(fmaf(a[i], c2, off));
      s1 += fast_exp2(fmaf(a[i + 1], c2, off));
      s2 += fast_exp2(fmaf(a[i + 2], c2, off));
      s3 += fast_exp2(fmaf(a[i + 3], c2, off));
    }
    rm = m_new;
    rs = (s0 + s1) + (s2 + s3);
    return a;
  }
  // items FIRST and up into held[]
  template <int MAXT, int FIRST = 0>
  __device__ __forceinline__ void slab_logits(f32x16 (&held)[MAXT], int nt, int M, int buf, float& rm, float& rs) {
    wide_static_for<FIRST, MAXT>([&](auto ic) __attribute__((always_inline)) {
      constexpr int it = decltype(ic)::value;
      if (it < nt) held[it] = item_logits<it>(nt, M, buf, rm, rs);
    });
  }
  // (max, sum) pairs a and b -> one
  __device__ __forceinline__ static void join_halves(float& m, float& z) {
    const auto sm = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    const auto sz = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    const float ma = __uint_as_float(sm[0]), mb = __uint_as_float(sm[1]);
    m = fmaxf(ma, mb);
    const float ref = (m == -INFINITY) ? 0.f : m;
    z = __uint_as_float(sz[0]) * fast_exp2(ma - ref) + __uint_as_float(sz[1]) * fast_exp2(mb - ref);
  }
  // the barrier at the end of a slab
  __device__ __forceinline__ void slab_barrier() const {
    // this wave's share of the next slab's query tile has landed (it was sent before this slab's refills; a wave
    // whose items in flight are older than that waits for them too)
    wait_items(sent - pos);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
  }
  // The rows' statistics over the wave's keys (two half-waves), then over the workgroup's: the lane's row's base-2
  // log-sum-exp (-inf where the workgroup has no keys).  One barrier; on the way the next slab's query tile lands.
  __device__ __forceinline__ float workgroup_lse(float rm, float rs, int buf) {
    join_halves(rm, rs);
    int ln = lane_id();
    if (ln < 32)
      lds_poke64<0>(xchg + ((buf * kTiledWaves + wave) * 32 + ln) * 8, ((uint64_t)__float_as_uint(rs) << 32) | __float_as_uint(rm));
    slab_barrier();
    // a half-wave folds four of the eight waves' pairs, then the halves meet
    const u64x4 v = lds_peek64x4<256>(xchg + ((buf * kTiledWaves + 4 * (ln >> 5)) * 32 + (ln & 31)) * 8);
    float m = -INFINITY, z = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) m = fmaxf(m, __uint_as_float((uint32_t)v.v[i]));
    const float ref = (m == -INFINITY) ? 0.f : m;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      z += __uint_as_float((uint32_t)(v.v[i] >> 32)) * fast_exp2(__uint_as_float((uint32_t)v.v[i]) - ref);
    join_halves(m, z);
    return m == -INFINITY ? -INFINITY : m + __builtin_amdgcn_logf(z);
  }
  // row log-sum-exps of (l, g, b) -> d_lse, by one wave
  __device__ __forceinline__ void store_lse(int l, int g, int b, float lse2) const {
    const int ln = lane_id(), n = ln & (NS - 1), j = (ln & 31) >> (5 - LG);
    if (ln < 32 && n < p.N && j < p.G)
      p.lse_out[(((int64_t)l * p.B + b) * p.N + n) * p.H + g * p.G + j] = lse2 * 0.6931471805599453f;
  }
};

// result array [32-key tile][group][query][32]: tiles of a call, and the merge (sp_score_wide.hip)
inline size_t wide_tiles(const sp_score_args* a) { return (size_t)(a->T >> 5) + a->B; }
inline int wide_lg(const sp_score_args* a) { return a->H / a->H_kv <= 4 ? 2 : 3; }
// `status`: null, or the status words of the exchange (then any score is NaN if a wait expired, and the epoch turns)
sp_status launch_wide_finish(const TiledDev& dev, unsigned tiles, uint32_t* status, hipStream_t stream);

}  // namespace sp
