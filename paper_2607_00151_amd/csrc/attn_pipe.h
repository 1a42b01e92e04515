// Software-pipelined form of the paged prefill attention (same work items,
// same LDS tiles and operand layouts as attn_kernel<P, 1, 4>).
//
// A CDNA4 SIMD overlaps matrix-core and VALU work only when both come from
// the same wave: an MFMA-only wave next to a VALU-only wave on one SIMD runs
// no faster than the two back to back, while a few VALU ops placed after each
// 32x32x16 MFMA of one wave cost little beyond the MFMA time (measured on
// MI355X).  So each wave splits key tile t into two interleaved phases,
//   phase 1:  S(t+1)^T = K(t+1) Q^T   16 MFMAs
//             P(t) = exp2(x(t)), keys 0-31     VALU (16 exp, 8 cvt, 16 add per
//                                               lane; the adds form l)
//   phase 2:  O^T += V(t)^T P(t)^T    16 MFMAs
//             P(t), keys 32-63        during the first 8 (the PV MFMAs of
//                                       keys 0-31), the same VALU work
//             row max of x(t+1)       during the last 8 (16 max3), then the
//                                       lazy rescale test
// with K one tile ahead of V.  The VALU work of each phase depends only on
// results of the previous phase or of earlier MFMAs, so it issues between the
// MFMAs; splitting the exponentials between the phases measured ~1% faster
// than making all of P(t) in phase 1.  Steps whose next tile needs the causal
// mask, and the last step, run the same sequence without the interleaving.
//
// Two ways to apply the softmax scale.  The default (kExact) keeps q as
// given, starts the S accumulations from zero and computes each exponent as
// fma(s, c, -m) in fp32 (c = softmax scale times log2 e, m the row's offset),
// with the offset moved whenever a row's max grows.  The fast mode folds the
// scale into the MFMA instead: the query rows are scaled by c once, when they
// are loaded, and every S accumulation starts from -m, which takes the 32 fma
// per lane and tile off the VALU; its offset moves only when the max grows by
// 2^kRescaleLog2.  Its price is one more bf16 rounding, of c q (each x moves
// by at most 2^-8 sum_d |c q_d k_d|, so the log-sum-exp by at most ln 2 times
// that), plus the rounding of a row's largest probability.
#pragma once

#include "attn_kernel.h"

namespace sa {


template <int N>
struct IntC {
  static constexpr int value = N;
};

// The phase-2 exponentials of the interleaved step go to PV slots
// ((e - 8 kG1) w2) / (32 - 8 kG1) - 1 and each pair is packed one slot after
// its second element; the PV MFMAs of 16-key group g are slots 4g .. 4g + 3.
// True if every group of phase 2 is packed before slot 4g - 1.
constexpr bool phase2_in_time(int kg1, int w2) {
  for (int g = kg1; g < 4; ++g) {
    const int e = 8 * g + 7;                                 // last element of the group
    const int pack = ((e - 8 * kg1) * w2) / (32 - 8 * kg1);
    if (pack >= 4 * g - 1) return false;
  }
  return true;
}

constexpr int kPipeWaves = 4;                              // waves per group, 32 rows each
constexpr int kPipeRows = 32 * kPipeWaves;                 // query rows per work item
constexpr int kTileBytes = kKT * kHD * 2;                  // one K or V tile, 16 KB

// LDS of one group: its double-buffered K and V tiles.  A second group also
// names the first group's partial-result area (four 16 KB arrays and a 2 KB
// array of row statistics), which the other group fills at the end.
struct PipeLds {
  lds_u8 *k0, *k1, *v0, *v1;
  lds_u8 *x0, *x1, *x2, *x3;
  __attribute__((address_space(3))) float* ml;
};

// Page slots of an item are checked once: true if every page its keys need is
// present and in range.  The first round of reads (four per thread, enough
// for an item of up to 4 x nthreads pages) is issued early and evaluated
// later, so its latency overlaps the first tile loads; every thread of the
// block takes part in the evaluation (one barrier).
struct TableCheck {
  int32_t v[4];
  int pg, pg_end;
  bool bad;
};

template <int P>
__device__ __forceinline__ TableCheck table_check_issue(const AttnArgs& a, const AttnItem& it, int32_t pt_base,
                                                        int32_t pt_count, int nthreads) {
  constexpr int kPagesPerTile = kKT / P;
  const int t0 = it.kv_begin / kKT;
  const int t1 = (it.kv_end + kKT - 1) / kKT;
  TableCheck c;
  c.bad = pt_count < (it.kv_end + P - 1) / P;
  c.pg = t0 * kPagesPerTile + (int)threadIdx.x;
  c.pg_end = min(t1 * kPagesPerTile, pt_count);
#pragma unroll
  for (int u = 0; u < 4; ++u) c.v[u] = c.pg + u * nthreads < c.pg_end ? a.indices[pt_base + c.pg + u * nthreads] : 0;
  return c;
}

__device__ __forceinline__ bool table_check_finish(const AttnArgs& a, TableCheck& c, int32_t pt_base, int nthreads) {
  bool bad = c.bad;
#pragma unroll
  for (int u = 0; u < 4; ++u) bad |= !(c.v[u] >= 0 && c.v[u] < a.num_slots);
  for (int pg = c.pg + 4 * nthreads; pg < c.pg_end; pg += nthreads) {
    const int32_t s = a.indices[pt_base + pg];
    bad |= !(s >= 0 && s < a.num_slots);
  }
  return !__syncthreads_or(bad);
}

// ---- the segment's rows, written by the launch that attends over them
//
// With kRead every block takes the segment's keys (positions kv_len - q_len
// on) from the token-major k_new / v_new and never from their pages, so no
// block depends on another block's writes.  The first key-range part of each
// row tile (kv_begin == 0; of a decode item's, those with keys of the segment)
// stores to the pages the rows of the tokens whose first query row lies in its
// tile: the row tiles partition the rows, so every token's row is written, and
// by one block (or, where a decode item's segment crosses a part's edge, with
// the same bytes by both).  A row whose page is missing or lies
// outside the pool is not written and raises error flag 2, as the append
// kernel does.  Four chunks per thread are loaded before any is stored, so the
// block waits for one round trip per 1024 chunks (64 tokens).
template <int P>
__device__ __forceinline__ void write_own_rows(const AttnArgs& a, const AttnItem& it) {
  const int G = a.G;
  const int tb = (it.row0 + G - 1) / G;
  const int te = min((it.row0 + kPipeRows + G - 1) / G, it.q_len);
  const int n = (te - tb) * 16;                             // 16-byte chunks of K (and of V)
  const int pre = it.kv_len - it.q_len;
  const int32_t pt_base = ld_uniform(a.indptr + it.seq);
  const int32_t pt_count = ld_uniform(a.indptr + it.seq + 1) - pt_base;
  uint16_t* const kp = const_cast<uint16_t*>(a.k);
  uint16_t* const vp = const_cast<uint16_t*>(a.v);
  constexpr int kDepth = 4;
  for (int c0 = (int)threadIdx.x; c0 < n; c0 += kDepth * (int)blockDim.x) {
    int64_t dst[kDepth];
    u32x4 kx[kDepth], vx[kDepth];
#pragma unroll
    for (int u = 0; u < kDepth; ++u) {
      const int c = c0 + u * (int)blockDim.x;
      dst[u] = -1;
      if (c >= n) continue;
      const int tok = tb + (c >> 4), ch = c & 15;
      const int x = pre + tok;
      const int page = x / P, row = x - page * P;
      const int32_t slot = page < pt_count ? a.indices[pt_base + page] : -1;
      if (slot < 0 || slot >= a.num_slots) {
        atomicOr(a.err, 2);
        continue;
      }
      const int64_t src = ((int64_t)(it.q_start + tok) * a.Hkv + it.kvh) * kHD + ch * 8;
      kx[u] = ld_u32x4(a.k_new + src);
      vx[u] = ld_u32x4(a.v_new + src);
      dst[u] = (((int64_t)slot * a.Hkv + it.kvh) * P + row) * kHD + ch * 8;
    }
#pragma unroll
    for (int u = 0; u < kDepth; ++u)
      if (dst[u] >= 0) {
        st_u32x4(kp + dst[u], kx[u]);
        st_u32x4(vp + dst[u], vx[u]);
      }
  }
}

// ---- split items: partial results and their merge inside the launch
//
// Every key-range part of a split item leaves its normalised partial O and
// log2 LSE in memory; the part that arrives last at the item's counter reads
// all of them back and writes the item's output, so a split launch needs no
// second kernel.  Nothing waits: each arrival is one fetch-add, and only the
// one that completes the count goes on.
//
// The parts of an item run on different XCDs, whose L2s do not see each
// other's ordinary stores before the kernel ends.  A release fence at device
// scope would write back the whole L2 once per part (measured 2-3x on small
// launches); instead the partials alone are stored and loaded at device scope
// (the cache-policy bit sc1, as relaxed device-scope atomics are: written
// through, and not served from a stale line), and a part counts itself only
// after its own stores have been acknowledged (vmcnt 0).  Against the separate
// merge launch: a 256-token chunk over a 4K prefix 36 -> 31 us of kernels.
constexpr int kDeviceScope = 16;                           // sc1 of a buffer access
constexpr int kPartCounters = 4;                           // counters per part: one per wave (prefill items)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t part_rsrc(const AttnArgs& a) {
  return __builtin_amdgcn_make_buffer_rsrc(a.part_o, (short)0, (int)a.part_bytes, 0x00020000);
}
// The whole offset goes in the vector operand: with a register as the scalar
// offset of a 16-byte buffer store the compiler leaves out the wait state
// between the store and a VALU write of its data registers, and the store was
// seen (in this code, on MI355X) to pick up the new value of the first one.
__device__ __forceinline__ void part_st4(const __amdgpu_buffer_rsrc_t& r, uint32_t off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, off, 0, kDeviceScope);
}
__device__ __forceinline__ f32x4 part_ld4(const __amdgpu_buffer_rsrc_t& r, uint32_t off, uint32_t base) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, base, kDeviceScope));
}
__device__ __forceinline__ void part_st1(const __amdgpu_buffer_rsrc_t& r, uint32_t off, uint32_t base, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, base, kDeviceScope);
}
__device__ __forceinline__ float part_ld1(const __amdgpu_buffer_rsrc_t& r, uint32_t off, uint32_t base) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, base, kDeviceScope));
}

// This wave's stores are at device scope once acknowledged; then one arrival
// at counter c of the item.  True for the last of its nsplit arrivals, which
// also puts the counter back to zero for the next launch.
__device__ __forceinline__ bool part_arrive(const AttnArgs& a, const PartInfo& pi, int c) {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070);
  asm volatile("" ::: "memory");
  int32_t* const cnt = a.part_count + (int64_t)pi.part0 * kPartCounters + c;
  int last = 0;
  if (__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)) == 0) {
    last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == pi.nsplit - 1;
    if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  last = __builtin_amdgcn_readfirstlane(last);
  asm volatile("" ::: "memory");
  return last != 0;
}

// One group of four waves runs the item's rows over the keys
// [g_lo, g_hi): the whole item when kGroups == 1; with two groups, group 0
// takes the first half of the item's key tiles and group 1 the rest, and the
// two meet at the end to merge their partial results.  With two groups every
// step holds two barriers (one before each phase) and group 1 runs one
// barrier behind group 0, so on each SIMD one group's phase 1 overlaps the
// other's phase 2.
//
// kPoolRsrc: a layer's K (and V) pool spans < 2^31 bytes, so one buffer
// resource per pool reaches every page through the 32-bit scalar offset;
// otherwise each page load builds a resource for its page.
//
// kRead: keys from kv_len - q_len on (the segment's) are loaded from k_new /
// v_new instead of from their pages (write_own_rows).  Within a tile the
// source is chosen per group of four keys; a group holding keys of both kinds
// (prefix lengths that are not a multiple of 4) takes the checked load, so the
// steps that load its tile are plain steps.
template <int P, bool kPoolRsrc, int kGroups, int GRP, bool kRead = false, bool kExact = false>
__device__ __attribute__((always_inline)) inline void pipe_group(const AttnArgs& a, const AttnItem& it,
                                                                 const SeqDesc& sd, const PipeLds& L) {
  static_assert(P == 16 || P == 32, "page size");
  static_assert(!kRead || (kPoolRsrc && kGroups == 1), "segment reads: one group, pool-wide resources");
  constexpr int WAVES = kPipeWaves;
  constexpr int kRows = kPipeRows;
  constexpr int kPagesPerTile = kKT / P;
  constexpr int kNJ = 16 / WAVES;                          // loads per wave per tile and operand
  constexpr int kAhead = 2;                                // operand reads issued this many steps ahead
  constexpr int kG1 = 2;                                   // 16-key groups of P(t) made in phase 1

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & (WAVES - 1);
  const int hh = lane >> 5;
  const int G = a.G;
  const int rows_total = sd.q_len * G;
  const int pre = sd.kv_len - sd.q_len;

  const int r_row = it.row0 + wave * 32 + (lane & 31);
  const bool row_valid = r_row < rows_total;
  const int rr = row_valid ? r_row : rows_total - 1;
  const int tok = rr / G;
  const int head = it.kvh * G + (rr - tok * G);
  const int qpos = pre + tok;

  // this group's keys [g_lo, g_hi) and tiles [t0, t1)
  const int ti0 = it.kv_begin / kKT;
  const int ti1 = (it.kv_end + kKT - 1) / kKT;
  const int tmid = ti0 + (ti1 - ti0 + 1) / 2;
  const int g_lo = (kGroups == 2 && GRP == 1) ? tmid * kKT : it.kv_begin;
  const int g_hi = (kGroups == 2 && GRP == 0) ? min(it.kv_end, tmid * kKT) : it.kv_end;
  const int t0 = g_lo / kKT;
  const int t1 = g_lo < g_hi ? (g_hi + kKT - 1) / kKT : t0;

  const int wrow0 = it.row0 + wave * 32;
  const bool wave_active = wrow0 < rows_total;
  const int w_full = min(g_hi, pre + wrow0 / G + 1);         // keys below are visible to all rows

  // the query row; it is scaled by c (below) only once the first tiles and
  // the page-table check are under way, so its load latency overlaps theirs
  bf16x8 qop[8];             // c q, rounded to bf16
  {
    const uint16_t* qrow = a.q + ((int64_t)(sd.q_start + tok) * a.Hq + head) * kHD;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qop[ks] = ld_bf16x8(qrow + (2 * ks + hh) * 8);
  }

  const int32_t pt_base = ld_uniform(a.indptr + it.seq);
  const int32_t pt_count = ld_uniform(a.indptr + it.seq + 1) - pt_base;
  TableCheck tcheck = table_check_issue<P>(a, it, pt_base, pt_count, 64 * WAVES * kGroups);
  const int64_t slot_bytes = (int64_t)a.Hkv * P * kHD * 2;
  const char* kbase = (const char*)a.k;
  const char* vbase = (const char*)a.v;
  int koff[kNJ], voff[kNJ];
#pragma unroll
  for (int j = 0; j < kNJ; ++j) {
    const int key = 4 * (j * WAVES + wave) + (lane >> 4);
    const int row_bytes = (it.kvh * P + key % P) * (kHD * 2);
    koff[j] = row_bytes + (((lane & 15) ^ swz_k(key)) << 4);
    voff[j] = row_bytes + (((lane & 15) ^ swz_v(key)) << 4);
  }

  struct Slots {
    int32_t s[kPagesPerTile];
    int32_t ts;              // the tile's first key
  };
  auto fetch = [&](int t) __attribute__((always_inline)) {
    Slots S;
#pragma unroll
    for (int j = 0; j < kPagesPerTile; ++j) {
      const int pg = t * kPagesPerTile + j;
      S.s[j] = (pg >= 0 && pg < pt_count) ? ld_uniform(a.indices + pt_base + pg) : -1;
    }
    S.ts = t * kKT;
    return S;
  };
  auto slot_ok = [&](int32_t s) __attribute__((always_inline)) { return s >= 0 && s < a.num_slots; };

  // A block whose table is intact (table_ok) loads tiles without per-page
  // tests; otherwise every tile takes the checked path, which zero-fills
  // what it cannot load and raises the error flag.  The check itself runs
  // while the first tiles load, which take the checked path.
  bool table_ok = false;
  const uint32_t pool_bytes = kPoolRsrc ? (uint32_t)(a.num_slots * slot_bytes) : 0u;
  const __amdgpu_buffer_rsrc_t rsrc_k =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.k), (short)0, (int)pool_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_v =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.v), (short)0, (int)pool_bytes, 0x00020000);

  // kRead: the segment's rows.  Key 4 gb + (lane >> 4) of the tile starting
  // at key ts is token q_start + ts + 4 gb + (lane >> 4) - pre of k_new; a
  // lane's offset within its group of four keys (the row within the group
  // and the swizzled chunk, which depends only on key % 16 for K and key % 4
  // for V, and key = 16 j + 4 wave + (lane >> 4)) is the same for every j,
  // and the group's start goes in the scalar offset.
  const __amdgpu_buffer_rsrc_t rsrc_nk =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.k_new), (short)0, kRead ? (int)a.new_bytes : 0,
                                        0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_nv =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.v_new), (short)0, kRead ? (int)a.new_bytes : 0,
                                        0x00020000);
  const int nk_off = (koff[0] & 255) + (lane >> 4) * a.Hkv * (kHD * 2);
  const int nv_off = (voff[0] & 255) + (lane >> 4) * a.Hkv * (kHD * 2);
  auto new_soff = [&](int ts, int gb) __attribute__((always_inline)) {
    return ((uint32_t)(sd.q_start + ts + 4 * gb - pre) * (uint32_t)a.Hkv + (uint32_t)it.kvh) * (uint32_t)(kHD * 2);
  };
  // the tile holding a group of four keys of both kinds, or -1
  const int t_mixed = (kRead && (pre & 3) != 0) ? pre / kKT : -1;

  // global -> LDS loads of one operand (K or V) of tile t into dst
  auto load_op = [&](int t, const Slots& S, const char* base, const __amdgpu_buffer_rsrc_t& rsrc, const int* off,
                     const __amdgpu_buffer_rsrc_t& nrsrc, int noff, lds_u8* dst) __attribute__((always_inline)) {
    const int ts = t * kKT;
    if (table_ok && ts + kKT <= g_hi && t != t_mixed) {
#pragma unroll
      for (int j = 0; j < kNJ; ++j) {
        const int gb = j * WAVES + wave;
        const int32_t slot = S.s[(4 * gb) / P];
        __attribute__((address_space(3))) void* d = (__attribute__((address_space(3))) void*)(dst + gb * 1024);
        if (kRead && ts + 4 * gb >= pre)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(nrsrc, d, 16, noff, new_soff(ts, gb), 0, 0);
        else if constexpr (kPoolRsrc)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, d, 16, off[j], (uint32_t)slot * (uint32_t)slot_bytes, 0, 0);
        else
          lds_dma16(base + (int64_t)slot * slot_bytes, (uint32_t)slot_bytes, off[j], d);
      }
    } else {
      bool bad = false;
#pragma unroll
      for (int j = 0; j < kNJ; ++j) {
        const int gb = j * WAVES + wave;
        const int32_t s = S.s[(4 * gb) / P];
        const int key = ts + 4 * gb + (lane >> 4);
        // the group's page is read when it holds keys of the item taken from pages
        const bool page_needed = ts + 4 * gb < g_hi && (!kRead || ts + 4 * gb < pre);
        bad |= page_needed && !slot_ok(s);
        const bool ld = page_needed && slot_ok(s) && key < g_hi && (!kRead || key < pre);
        const bool ldn = kRead && key < g_hi && key >= pre;
        __attribute__((address_space(3))) void* d = (__attribute__((address_space(3))) void*)(dst + gb * 1024);
        if (ld) lds_dma16(base + (int64_t)s * slot_bytes, (uint32_t)slot_bytes, off[j], d);
        if constexpr (kRead) {
          if (ldn)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                nrsrc, d, 16, (off[j] & 255) + ((sd.q_start + key - pre) * a.Hkv + it.kvh) * (kHD * 2), 0, 0, 0);
        }
        if (!ld && !ldn) {
          // absent keys: zero rows keep the masked products finite
          const u32x4 z = {0u, 0u, 0u, 0u};
          *(__attribute__((address_space(3))) u32x4*)(dst + gb * 1024 + lane * 16) = z;
        }
      }
      if (bad && lane == 0) atomicOr(a.err, 1);
    }
  };

  f32x16 oacc[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) oacc[dt] = f32x16{};
  float m_used = -INFINITY;  // exponent offset in use (log2 domain)
  float msub = 0.f;          // m_used, or 0 while it is -inf
  float m_seen = -INFINITY;  // (exact scale) c times the row's largest score so far
  float l = 0.f;             // this lane's share of the denominator
  float corr = 0.f;          // (exact scale) bf16 roundings of its rows' largest probabilities
  f32x16 negm = f32x16{};    // -msub in every element: where each S accumulation starts
  f32x16 sc[2][2];           // [buffer][32-key block] scores of tiles t and t + 1
  bf16x8 pop[4];             // [16-key group] probabilities of tile t

  const int krow = lane & 31;
  const int tr_g = lane >> 4, tr_s = lane & 15;
  const int tr_key = 4 * (tr_g >> 1) + (tr_s >> 2);
  const int tr_d = 16 * (tr_g & 1) + 4 * (tr_s & 3);

  // MFMA operands from LDS.  S step i: 32-key block i & 1, d-chunk pair
  // i >> 1 (the two accumulation chains alternate).  PV step i: 16-key group
  // i >> 2, 32-wide d block i & 3.
  auto read_k = [&](const lds_u8* kb, int i) __attribute__((always_inline)) {
    const int key = 32 * (i & 1) + krow;
    return *(const __attribute__((address_space(3))) bf16x8*)(
        kb + key * 256 + (((2 * (i >> 1) + hh) ^ swz_k(key)) << 4));
  };
  auto read_v = [&](const lds_u8* vb, int i) __attribute__((always_inline)) {
    bf16x8 vop;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int vkey = 16 * (i >> 2) + 8 * r + tr_key;
      const int d = 32 * (i & 3) + tr_d;
      const bf16x4 x = lds_read_tr(vb + vkey * 256 + ((((d >> 3) ^ swz_v(vkey)) << 4) | ((d & 7) << 1)));
#pragma unroll
      for (int e = 0; e < 4; ++e) vop[4 * r + e] = x[e];
    }
    return vop;
  };
  auto s_step = [&](f32x16* S, bf16x8 kop, int i) __attribute__((always_inline)) {
    S[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop, qop[i >> 1], i < 2 ? negm : S[i & 1], 0, 0, 0);
  };
  auto pv_step = [&](bf16x8 vop, int i) __attribute__((always_inline)) {
    oacc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop, pop[i >> 2], oacc[i & 3], 0, 0, 0);
  };
  // probabilities of pair j (elements 2j, 2j + 1 of the tile, in P^T slot
  // order: group j >> 2, slots 2 (j & 3) and 2 (j & 3) + 1)
  auto xpair = [&](const f32x16* X, int j, int h) __attribute__((always_inline)) {
    const int g = j >> 2;
    return X[g >> 1][8 * (g & 1) + 2 * (j & 3) + h];
  };
  // probability of one score: the accumulator holds x - m already, or (exact
  // scale) the raw q.k, which is scaled and offset here in fp32
  auto xexp = [&](float v) __attribute__((always_inline)) {
    if constexpr (kExact) return exp2f_fast(__builtin_fmaf(v, a.c, -msub));
    else return exp2f_fast(v);
  };
  auto exp_pair = [&](const f32x16* X, int j) __attribute__((always_inline)) {
    const int g = j >> 2, e = 2 * (j & 3);
    const float p0 = xexp(xpair(X, j, 0));
    const float p1 = xexp(xpair(X, j, 1));
    pop[g][e] = (__bf16)p0;
    pop[g][e + 1] = (__bf16)p1;
    return p0 + p1;
  };
  auto mask_tile = [&](int t, f32x16* S) __attribute__((always_inline)) {
    const int ts = t * kKT;
    const int lim = min(qpos, g_hi - 1);
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = ts + 32 * kt + 8 * (e >> 2) + 4 * hh + (e & 3);
        if (key > lim) S[kt][e] = -INFINITY;
      }
  };
  // rescale test, given this lane's max mx of a tile's x values (raw scores
  // with exact scale): move the offset when c (row max) outgrows it by
  // 2^kRescaleLog2, rescale O and l, and shift the tile's x values to the new
  // offset.
  // With exact scale the offset lags the row's max, so the largest
  // probability of a row is 2^x for some x in [0, kRescaleLog2], which the
  // bf16 packing of P rounds; the numerator then carries that rounding and
  // the fp32 denominator would not.  Whenever a row's max grows, the lane
  // holding the new largest score therefore adds its key's rounding,
  // bf16(p) - p, to corr (rescaled with l): p is formed exactly as the tile's
  // exponentials will form it (same fma, same offset), so the output, divided
  // by l + corr, carries in numerator and denominator the same value for
  // every key that was its row's largest when it arrived, as when the offset
  // tracks every growth of the max (largest probability exactly 1), without
  // the rescale of O that this would take at each growth.  The log-sum-exp
  // takes l alone, the fp32 sum.
  auto rescale_test = [&](float mx, f32x16* X) __attribute__((always_inline)) {
    const float mine = mx;
    mx = pair_max(mx);
    const float cand = kExact ? mx * a.c : mx + msub;       // c * row max
    bool grew = false;
    if constexpr (kExact) grew = __ballot(cand > m_seen) != 0;
    if ((!kExact || grew) && __ballot(cand > m_used + kRescaleLog2)) {
      const float m_new = fmaxf(m_used, cand);
      const float alpha = (m_new == -INFINITY) ? 1.f : exp2f_fast(m_used - m_new);
      m_used = m_new;
      const float msub_new = (m_used == -INFINITY) ? 0.f : m_used;
      const float shift = msub_new - msub;
      msub = msub_new;
      // the accumulators start from the new offset (x values only; exact-scale
      // scores carry no offset)
      if constexpr (!kExact) {
#pragma unroll
        for (int e = 0; e < 16; ++e) negm[e] = -msub;
      }
      l *= alpha;
      if constexpr (kExact) corr *= alpha;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[dt][e] *= alpha;
      if constexpr (!kExact) {
        // and the tile's x values move to it
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int e = 0; e < 16; ++e) X[kt][e] -= shift;
      } else {
        (void)shift;
        (void)X;
      }
    }
    if constexpr (kExact) {
      if (grew) {
        const float p = exp2f_fast(__builtin_fmaf(mx, a.c, -msub));
        const float d = (float)(__bf16)p - p;
        corr += (cand > m_seen && mine == mx) ? d : 0.f;
        m_seen = fmaxf(m_seen, cand);
      }
    }
  };
  auto row_max = [&](const f32x16* S) __attribute__((always_inline)) {
    float mx = S[0][0];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = vmax(mx, S[kt][e]);
    return mx;
  };

  // plain step, S(t) in sc[0]: S(t+1) into sc[1] if there is a next tile;
  // P(t); O += V(t) P(t); sum; mask and rescale test of tile t+1, which then
  // moves to sc[0]
  auto plain_step = [&](int t, const lds_u8* kb, const lds_u8* vb) __attribute__((always_inline)) {
    const bool has_next = t + 1 < t1;
    float ls = 0.f;
    if (wave_active) {
      if (has_next) {
        // operand reads two MFMAs ahead, P(t) between the MFMAs
        bf16x8 kop[16];
#pragma unroll
        for (int i = 0; i < 2; ++i) kop[i] = read_k(kb, i);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          if (i + 2 < 16) kop[i + 2] = read_k(kb, i + 2);
          s_step(sc[1], kop[i], i);
          ls += exp_pair(sc[0], i);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) ls += exp_pair(sc[0], j);
      }
    }
    if constexpr (kGroups == 2) lds_barrier();
    if (wave_active) {
      bf16x8 vop[16];
#pragma unroll
      for (int i = 0; i < 2; ++i) vop[i] = read_v(vb, i);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i + 2 < 16) vop[i + 2] = read_v(vb, i + 2);
        pv_step(vop[i], i);
      }
      l += ls;
      if (has_next) {
        if ((t + 2) * kKT > w_full) mask_tile(t + 1, sc[1]);
        rescale_test(row_max(sc[1]), sc[1]);
        sc[0][0] = sc[1][0];
        sc[0][1] = sc[1][1];
      }
    }
  };

  // interleaved step (next tile exists and needs no mask)
  Slots s_a, s_b;          // pages of tiles t + 1 and t + 2 in step t

  // one 16-byte-per-lane load of a full tile with an intact table: from the
  // group's page, or (kRead) from the segment's rows, chosen without a branch
  auto tile_load = [&](const Slots& S, const char* base, const __amdgpu_buffer_rsrc_t& rsrc, const int* off,
                       const __amdgpu_buffer_rsrc_t& nrsrc, int noff, lds_u8* dst, int j) __attribute__((always_inline)) {
    const int gb = j * WAVES + wave;
    const int32_t slot = S.s[(4 * gb) / P];
    __attribute__((address_space(3))) void* d = (__attribute__((address_space(3))) void*)(dst + gb * 1024);
    if constexpr (kRead) {
      const bool seg = S.ts + 4 * gb >= pre;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(seg ? nrsrc : rsrc, d, 16, seg ? noff : off[j],
                                               seg ? new_soff(S.ts, gb) : (uint32_t)slot * (uint32_t)slot_bytes, 0, 0);
    } else if constexpr (kPoolRsrc) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, d, 16, off[j], (uint32_t)slot * (uint32_t)slot_bytes, 0, 0);
    } else {
      lds_dma16(base + (int64_t)slot * slot_bytes, (uint32_t)slot_bytes, off[j], d);
    }
  };

  // interleaved step; also issues this step's loads, K(t+2) into kn and
  // V(t+1) into vn (full tiles, intact table), one per MFMA of phase 1.
  // The exponentials of P(t) are split between the phases: the first
  // 4 kG1 pairs (16-key groups 0 .. kG1 - 1) between the S(t+1) MFMAs of
  // phase 1, the rest between the PV MFMAs of phase 2, each group finished
  // at least one MFMA before the PV MFMA that reads it.  Every VALU op waits on one
  // issued a step earlier, never on its neighbour, so the next MFMA issues on
  // time.
  auto fast_step = [&](auto bc, const lds_u8* kb, const lds_u8* vb, lds_u8* kn, lds_u8* vn) __attribute__((always_inline)) {
    constexpr int B = decltype(bc)::value, N = 1 - B;
    constexpr int E1 = 8 * kG1;              // exponentials in phase 1 (of 32)
    constexpr int E2 = 32 - E1;              // in phase 2
    // phase-2 steps that take them: spread up to the step before the PV MFMA
    // of the last group (slot 4 kG1 + 4 ... 12 with two groups per phase) needs
    // it, rather than packed into the first 4 kG1 slots (measured ~1% faster at
    // c2 with kG1 = 2)
    constexpr int W2 = kG1 == 2 ? 11 : (kG1 < 4 ? 4 * kG1 : 1);
    // step of element e (pair e / 2, half e % 2); -1: before the first MFMA
    auto p1_step = [](int e) constexpr { return (e * 16) / E1 - 1; };
    auto p2_step = [](int e) constexpr { return ((e - E1) * W2) / (E2 > 0 ? E2 : 1) - 1; };
    // a pair is packed and summed one step after its second element
    auto p1_pack = [&](int j) constexpr { return p1_step(2 * j + 1) + 1; };
    auto p2_pack = [&](int j) constexpr { return p2_step(2 * j + 1) + 1; };
    // row max of x(t+1), 16 three-way maxes: in the phase-2 steps past the exponentials
    auto mx_step = [](int k) constexpr { return kG1 <= 2 ? 8 + k / 2 : k; };
    static_assert(phase2_in_time(kG1, W2), "a 16-key group of P packed after the PV MFMA that reads it");
    bf16x8 kop[16], vop[16];
    float ex[16][2];
    // two accumulation chains for the denominator; -0 + y is y, so the first
    // add of each chain folds away
    float ls[2] = {-0.f, -0.f};
    // (exact scale) exponents c s - m, each made one MFMA slot before its
    // exponential, so the exponential never waits on the fma beside it
    float xv[32];
    auto do_x = [&](int e) __attribute__((always_inline)) {
      if constexpr (kExact) xv[e] = __builtin_fmaf(xpair(sc[B], e >> 1, e & 1), a.c, -msub);
    };
    auto do_exp = [&](int e) __attribute__((always_inline)) {
      if constexpr (kExact) ex[e >> 1][e & 1] = exp2f_fast(xv[e]);
      else ex[e >> 1][e & 1] = exp2f_fast(xpair(sc[B], e >> 1, e & 1));
    };
    auto do_pack = [&](int j) __attribute__((always_inline)) {
      ls[j & 1] += ex[j][0] + ex[j][1];
      pop[j >> 2][2 * (j & 3)] = (__bf16)ex[j][0];
      pop[j >> 2][2 * (j & 3) + 1] = (__bf16)ex[j][1];
    };
    // phase 1: S(t+1) MFMAs
#pragma unroll
    for (int i = 0; i < kAhead; ++i) kop[i] = read_k(kb, i);
#pragma unroll
    for (int e = 0; e < E1; ++e)
      if (p1_step(e) <= 0) do_x(e);
#pragma unroll
    for (int e = 0; e < E1; ++e)
      if (p1_step(e) < 0) do_exp(e);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i + kAhead < 16) kop[i + kAhead] = read_k(kb, i + kAhead);
      if (i < kNJ) tile_load(s_b, kbase, rsrc_k, koff, rsrc_nk, nk_off, kn, i);
      else if (i < 2 * kNJ) tile_load(s_a, vbase, rsrc_v, voff, rsrc_nv, nv_off, vn, i - kNJ);
      s_step(sc[N], kop[i], i);
      int nv = 0;
#pragma unroll
      for (int e = 0; e < E1; ++e)
        if (p1_step(e) == i) { do_exp(e); ++nv; }
      if constexpr (kExact) {
#pragma unroll
        for (int e = 0; e < E1; ++e)
          if (p1_step(e) == i + 1) { do_x(e); ++nv; }
        // the exponents of the first elements of phase 2
#pragma unroll
        for (int e = E1; e < 32; ++e)
          if (i == 15 && p2_step(e) < 0) { do_x(e); ++nv; }
      }
#pragma unroll
      for (int j = 0; j < E1 / 2; ++j)
        if (p1_pack(j) == i) { do_pack(j); nv += 3; }
      // pin each step's operand read, tile load, MFMA and VALU work to this step
      if (i + kAhead < 16) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (i < 2 * kNJ) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (nv > 0) __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the pairs of phase 1 packed after its last MFMA
#pragma unroll
    for (int j = 0; j < E1 / 2; ++j)
      if (p1_pack(j) >= 16) do_pack(j);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kGroups == 2) lds_barrier();
    // phase 2: PV MFMAs; the rest of P(t) and the row max of x(t+1) between them
#pragma unroll
    for (int i = 0; i < kAhead; ++i) vop[i] = read_v(vb, i);
#pragma unroll
    for (int e = E1; e < 32; ++e)
      if (p2_step(e) < 0) do_exp(e);
#pragma unroll
    for (int e = E1; e < 32; ++e)
      if (p2_step(e) == 0) do_x(e);
    float mx[2] = {-INFINITY, -INFINITY};   // two accumulation chains
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i + kAhead < 16) vop[i + kAhead] = read_v(vb, i + kAhead);
      pv_step(vop[i], i);
      int nv = 0;
#pragma unroll
      for (int e = E1; e < 32; ++e)
        if (p2_step(e) == i) { do_exp(e); ++nv; }
      if constexpr (kExact) {
#pragma unroll
        for (int e = E1; e < 32; ++e)
          if (p2_step(e) == i + 1) { do_x(e); ++nv; }
      }
#pragma unroll
      for (int j = E1 / 2; j < 16; ++j)
        if (p2_pack(j) == i) { do_pack(j); nv += 3; }
#pragma unroll
      for (int k = 0; k < 16; ++k)
        if (mx_step(k) == i) {
          mx[k & 1] = vmax(vmax(mx[k & 1], sc[N][k & 1][2 * (k >> 1)]), sc[N][k & 1][2 * (k >> 1) + 1]);
          ++nv;
        }
      if (i + kAhead < 16) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (nv > 0) __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    l += ls[0] + ls[1];
    rescale_test(vmax(mx[0], mx[1]), sc[N]);
  };

  lds_u8* const K0 = L.k0;
  lds_u8* const K1 = L.k1;
  lds_u8* const V0 = L.v0;
  lds_u8* const V1 = L.v1;

  // ---- prologue: K(t0), V(t0), K(t0 + 1); S(t0) and its rescale test
  if (t0 < t1) {
    const Slots s0 = fetch(t0);
    load_op(t0, s0, kbase, rsrc_k, koff, rsrc_nk, nk_off, K0);
    load_op(t0, s0, vbase, rsrc_v, voff, rsrc_nv, nv_off, V0);
  }
  s_b = fetch(t0 + 1);
  if (t0 + 1 < t1) load_op(t0 + 1, s_b, kbase, rsrc_k, koff, rsrc_nk, nk_off, K1);
  // Interleaved steps take the page slots of their loads from a vector load
  // issued a step ahead: it is counted with the tile loads and has a whole
  // step to land, where a scalar load would be waited for at the next barrier.
  const __amdgpu_buffer_rsrc_t rsrc_pt = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int32_t*>(a.indices + pt_base), (short)0, pt_count * 4, 0x00020000);
  typedef uint32_t slot_vec __attribute__((ext_vector_type(kPagesPerTile)));
  auto fetch_vec = [&](int t) __attribute__((always_inline)) {
    if constexpr (kPagesPerTile == 4)
      return __builtin_bit_cast(slot_vec, __builtin_amdgcn_raw_buffer_load_b128(rsrc_pt, t * 16, 0, 0));
    else
      return __builtin_bit_cast(slot_vec, __builtin_amdgcn_raw_buffer_load_b64(rsrc_pt, t * 8, 0, 0));
  };
  slot_vec v_next = fetch_vec(t0 + 2);                      // pages of tile t + 2, in flight
  table_ok = table_check_finish(a, tcheck, pt_base, 64 * WAVES * kGroups);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if constexpr (!kExact) qop[ks][e] = (__bf16)((float)qop[ks][e] * a.c);
  __builtin_amdgcn_s_waitcnt(0x0070);
  lds_barrier();
  if (kGroups == 2 && GRP == 1) lds_barrier();             // group 1 runs a barrier behind
  if (wave_active && t0 < t1) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s_step(sc[0], read_k(K0, i), i);
    if ((t0 + 1) * kKT > w_full) mask_tile(t0, sc[0]);
    rescale_test(row_max(sc[0]), sc[0]);
  }

  // ---- step t reads K(t+1) and V(t) and loads K(t+2), V(t+1).  K(t) and
  // V(t) sit in buffer (t - t0) & 1.
  auto wait_tiles = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x0070);                     // my loads of K(t+1), V(t) landed
    lds_barrier();                                          // everyone's; the next buffers are free
  };
  // the item's first `boost` steps run at raised wave priority
  const int t_boost = t0 + (kGroups == 1 ? it.boost : 0);
  auto priority = [&](int t) __attribute__((always_inline)) {
    if (t == t_boost) __builtin_amdgcn_s_setprio(0);
  };
  if (t_boost > t0) __builtin_amdgcn_s_setprio(1);
  auto top = [&](int t, lds_u8* kn, lds_u8* vn) __attribute__((always_inline)) {
    wait_tiles();
    if (t + 2 < t1) load_op(t + 2, s_b, kbase, rsrc_k, koff, rsrc_nk, nk_off, kn);
    if (t + 1 < t1) load_op(t + 1, s_a, vbase, rsrc_v, voff, rsrc_nv, nv_off, vn);
  };
  auto advance = [&](int t) __attribute__((always_inline)) {
    s_a = s_b;
    s_b = fetch(t + 3);
  };
  // start of interleaved step t: s_a <- pages of t + 1, s_b <- pages of t + 2
  // (landed with the last tile loads), pages of t + 3 requested
  auto advance_fast = [&](int t) __attribute__((always_inline)) {
    s_a = s_b;
#pragma unroll
    for (int j = 0; j < kPagesPerTile; ++j) s_b.s[j] = (int32_t)__builtin_amdgcn_readfirstlane(v_next[j]);
    s_b.ts = (t + 2) * kKT;
    v_next = fetch_vec(t + 3);
  };
  // Steps t < t_fast interleave: their next tile needs no mask, V(t+1) is a
  // full tile and K(t+2) a tile of the item (the last one may be partial: its
  // rows past the end are whatever the page holds, and the step that scores
  // them masks them), all covered by an intact table.  Waves run different
  // numbers of each kind of step but the same number of steps, each with one
  // barrier and its share of the tile loads.
  int t_fast = (wave_active && table_ok) ? max(t0, min(w_full / kKT - 1, t1 - 2)) : t0;
  // (kRead) no interleaved step loads the tile with a mixed group of keys
  if (t_mixed >= 0) t_fast = max(t0, min(t_fast, t_mixed - 2));
  int t = t0;
  for (; t + 1 < t_fast; t += 2) {
    priority(t);
    wait_tiles();
    advance_fast(t);
    fast_step(IntC<0>{}, K1, V0, K0, V1);
    priority(t + 1);
    wait_tiles();
    advance_fast(t + 1);
    fast_step(IntC<1>{}, K0, V1, K1, V0);
  }
  if (t < t_fast) {
    priority(t);
    wait_tiles();
    advance_fast(t);
    fast_step(IntC<0>{}, K1, V0, K0, V1);
    ++t;
  }
  // plain steps: scalar page reads (-1 for pages the table lacks)
  s_a = fetch(t + 1);
  s_b = fetch(t + 2);
  if ((t - t0) & 1) {                                       // S(t) is in sc[1]
    sc[0][0] = sc[1][0];
    sc[0][1] = sc[1][1];
  }
  for (; t < t1; ++t) {
    const bool odd = (t - t0) & 1;
    priority(t);
    top(t, odd ? K1 : K0, odd ? V0 : V1);
    plain_step(t, odd ? K0 : K1, odd ? V1 : V0);
    advance(t);
  }

  // (two groups) the partial results merge through l alone
  if constexpr (kExact && kGroups == 2) {
    l += corr;
    corr = 0.f;
  }
  if constexpr (kGroups == 2) {
    // Both groups pass the same number of barriers: group g has passed
    // 1 + g + 2 (its steps) so far; pad to the larger count, then one more
    // barrier frees the tile buffers for group 1's partial results and
    // another publishes them.
    const int n0 = tmid - ti0, n1 = ti1 - tmid;              // steps of each group
    const int passed = 1 + GRP + 2 * (GRP == 0 ? n0 : n1);
    const int total = max(1 + 2 * n0, 2 + 2 * n1);
    for (int k = passed; k < total; ++k) lds_barrier();
    __builtin_amdgcn_s_waitcnt(0x0070);                     // no tile load of mine in flight
    lds_barrier();
    auto slot = [&](int k) __attribute__((always_inline)) {
      lds_u8* const x[4] = {L.x0, L.x1, L.x2, L.x3};
      return (__attribute__((address_space(3))) f32x4*)(x[k >> 2] + ((k & 3) * WAVES + wave) * 1024 + lane * 16);
    };
    if (GRP == 1) {
      if (wave_active) {
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const int dt = k >> 2, i = k & 3;
          *slot(k) = f32x4{oacc[dt][4 * i], oacc[dt][4 * i + 1], oacc[dt][4 * i + 2], oacc[dt][4 * i + 3]};
        }
        L.ml[wave * 64 + lane] = m_used;
        L.ml[kRows * 2 + wave * 64 + lane] = l;
      }
      lds_barrier();
      return;
    }
    lds_barrier();
    if (!wave_active) return;
    // merge: both partials are sums against their own exponent offsets
    const float m_b = L.ml[wave * 64 + lane];
    const float l_b = L.ml[kRows * 2 + wave * 64 + lane];
    const float m_new = fmaxf(m_used, m_b);
    const float alpha = (m_used == -INFINITY) ? 0.f : exp2f_fast(m_used - m_new);
    const float beta = (m_b == -INFINITY) ? 0.f : exp2f_fast(m_b - m_new);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int dt = k >> 2, i = k & 3;
      const f32x4 ob = *slot(k);
#pragma unroll
      for (int e = 0; e < 4; ++e) oacc[dt][4 * i + e] = oacc[dt][4 * i + e] * alpha + ob[e] * beta;
    }
    l = l * alpha + l_b * beta;
    m_used = m_new;
  }

  if (!wave_active) return;
  const float l_tot = pair_sum(l);
  const float l_out = kExact ? pair_sum(l + corr) : l_tot;
  const float inv = l_out > 0.f ? 1.f / l_out : 0.f;
  const float lse2 = l_tot > 0.f ? m_used + __builtin_amdgcn_logf(l_tot) : -INFINITY;
  // The output row is worked out again from the lane index here rather than
  // kept from the start: values live across the loops beyond its registers
  // are spilled to scratch memory.
  const int lane_o = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int hh_o = lane_o >> 5;
  const int o_row = it.row0 + wave * 32 + (lane_o & 31);
  const int o_tok = o_row / G;
  const int o_head = it.kvh * G + (o_row - o_tok * G);
  if (it.part < 0) {
    if (o_row < rows_total) {
      uint16_t* orow = a.o + ((int64_t)(sd.q_start + o_tok) * a.Hq + o_head) * kHD;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d = 32 * dt + 8 * i + 4 * hh_o;
          st_bf16x4(orow + d, oacc[dt][4 * i] * inv, oacc[dt][4 * i + 1] * inv,
                    oacc[dt][4 * i + 2] * inv, oacc[dt][4 * i + 3] * inv);
        }
      if (a.lse != nullptr && hh_o == 0)
        a.lse[(int64_t)(sd.q_start + o_tok) * a.Hq + o_head] = lse2 * 0.69314718055994531f;
    }
  } else if constexpr (kGroups == 1) {
    // A part's partial: this wave's 32 rows in accumulator order (16-byte
    // piece k of lane l at k KiB + 16 l), so stores and loads are whole lines.
    // Each wave counts and merges its own rows: no barrier.
    const __amdgpu_buffer_rsrc_t rp = part_rsrc(a);
    const PartInfo pi = ld_uniform(a.part_info + it.part);
    const uint32_t o_off = (uint32_t)(wave * 16 * 64 + lane_o) * 16;      // + k KiB
    const uint32_t l_off = (uint32_t)a.n_parts * (kRows * kHD * 4) + (uint32_t)(wave * 32 + (lane_o & 31)) * 4;
    {
      const uint32_t base = (uint32_t)it.part * (kRows * kHD * 4);
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int dt = k >> 2, i = k & 3;
        part_st4(rp, base + o_off + k * 1024,
                 f32x4{oacc[dt][4 * i] * inv, oacc[dt][4 * i + 1] * inv, oacc[dt][4 * i + 2] * inv,
                       oacc[dt][4 * i + 3] * inv});
      }
      if (hh_o == 0) part_st1(rp, l_off, (uint32_t)it.part * (kRows * 4), lse2);
    }
    if (!part_arrive(a, pi, wave)) return;
    float mx = -INFINITY;
#pragma unroll 4
    for (int s = 0; s < pi.nsplit; ++s) mx = fmaxf(mx, part_ld1(rp, l_off, (uint32_t)(pi.part0 + s) * (kRows * 4)));
    f32x4 num[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) num[k] = f32x4{};
    float den = 0.f;
    const float sub = mx == -INFINITY ? 0.f : mx;
#pragma unroll 2
    for (int s = 0; s < pi.nsplit; ++s) {
      const uint32_t base = (uint32_t)(pi.part0 + s) * (kRows * kHD * 4);
      f32x4 x[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = part_ld4(rp, o_off + k * 1024, base);
      const float w = exp2f_fast(part_ld1(rp, l_off, (uint32_t)(pi.part0 + s) * (kRows * 4)) - sub);
      den += w;
#pragma unroll
      for (int k = 0; k < 16; ++k) num[k] += w * x[k];
    }
    if (o_row < rows_total) {
      const float dinv = den > 0.f ? 1.f / den : 0.f;
      uint16_t* orow = a.o + ((int64_t)(sd.q_start + o_tok) * a.Hq + o_head) * kHD;
#pragma unroll
      for (int k = 0; k < 16; ++k)
        st_bf16x4(orow + 32 * (k >> 2) + 8 * (k & 3) + 4 * hh_o, num[k][0] * dinv, num[k][1] * dinv,
                  num[k][2] * dinv, num[k][3] * dinv);
      if (a.lse != nullptr && hh_o == 0)
        a.lse[(int64_t)(sd.q_start + o_tok) * a.Hq + o_head] =
            den > 0.f ? (mx + __builtin_amdgcn_logf(den)) * 0.69314718055994531f : -INFINITY;
    }
  } else {
    // two groups: plain rows, merged by merge_kernel
    const int lrow = wave * 32 + (lane_o & 31);
    float* po = a.part_o + ((int64_t)it.part * kRows + lrow) * kHD;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int d = 32 * dt + 8 * i + 4 * hh_o;
        f32x4 w = {oacc[dt][4 * i] * inv, oacc[dt][4 * i + 1] * inv, oacc[dt][4 * i + 2] * inv,
                   oacc[dt][4 * i + 3] * inv};
        *(f32x4*)(po + d) = w;
      }
    if (hh_o == 0) a.part_lse[(int64_t)it.part * kRows + lrow] = lse2;
  }
}

// ---- work items of at most 32 packed rows (decode requests)
//
// A decode request has one query token, so its item holds the G query heads
// of one KV head over the whole cached context.  Run like a prefill item, one
// wave would carry every matrix instruction of the item on one SIMD while the
// other three only load tiles, and a prefill block sharing the CU, whose waves
// wait on each other at every barrier, would run at the pace of its wave on
// that SIMD.  Here the four waves split the item's keys instead: wave w takes
// the 32-key tiles u0 + w, u0 + w + 4, ..., keeps its own online-softmax state
// over the same rows, and needs no barrier.  The item is bound by HBM when the
// batch is large and by latency when it is small, so a wave keeps two tiles
// (32 KB) in flight: K in two register sets (K is the A operand of
// S^T = K Q^T, so no LDS round trip is needed), V in two 8 KB LDS slices of its
// own (the PV product reads it transposed); page slots come 64 at a time in
// one vector load, so no load waits for its page id.
//
// 16x16x32 MFMAs, kNB 16-row blocks: a request with G <= 16 query heads pads
// its rows to 16, not 32 (half the exponentials, matrix time and accumulators
// of a 32x32 block), and a K load covers 64 contiguous bytes of each of 16
// rows.  Key 4 g + j (j < 4) and 16 + 4 g + j of a tile sit in the S^T
// accumulators of lane group g = lane / 16, which makes them the k-slots
// 8 g + j and 8 g + 4 + j of the PV product's P^T operand; two transposed
// 4-key reads give V^T in the same order.
//
// Each page is reached through a buffer resource of its own, so the pool may
// be of any size (a layer of a pool of a 288 GB card is easily past 2 GiB).
//
// Measured (MI355X, 32/8 heads, page 16, one stream of calls; before: 32-row
// blocks, one K and two V tiles in flight, 1024-key parts, a merge launch):
// 4 requests of 1K-4K keys 24.3 -> 13.0 us, 1 of 4K 22.0 -> 9.9 us, 8 of 6K-8K
// 59.7 -> 48.5 us, 32 of 2K-8K 142 -> 111 us (5.9 TB/s), 64 of 4K-16K 451 -> 448
// us (6.0 TB/s); 64/8 heads, page 32, 1 request of 73729 keys 93.0 -> 58.8 us
// (5.1 TB/s; the merge kernel's 8 busy blocks had taken 28 us of it).
typedef __attribute__((address_space(3))) float lds_f32;
constexpr int kDecRows = kDecodeRows;        // rows of an item this path takes
constexpr int kDecKeys = 32;                 // keys per tile of one wave

__device__ __forceinline__ int swz_dec(int key) { return (key & 7) << 1; }

// over the four lanes that share lane % 16
__device__ __forceinline__ float quad_max(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return pair_max(vmax(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float quad_sum(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return pair_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

template <int P, bool kExact, int kNB>
__device__ __attribute__((always_inline)) inline void decode_group(const AttnArgs& a, const AttnItem& it,
                                                                   lds_u8* k0, lds_u8* k1, lds_u8* v0, lds_u8* v1,
                                                                   lds_f32* stats) {
  // k0 .. v1: the prefill path's tile buffers; stats: [4 waves][32 rows] m, then l, and a flag behind
  static_assert(P == 16 || P == 32, "page size");
  constexpr int kWaves = 4;
  constexpr int kPagesPerTile = kDecKeys / P;                // 2 or 1
  constexpr int kSliceBytes = kDecKeys * kHD * 2;            // 8 KB: one V tile of one wave
  constexpr int kSlotTiles = 64 / kPagesPerTile;             // tiles of one vector load of page slots
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & (kWaves - 1);
  const int g = lane >> 4, r16 = lane & 15;
  const int G = a.G;
  const int rows = it.q_len * G - it.row0;                   // 1 .. 16 kNB
  const int pre = it.kv_len - it.q_len;
  const int g_lo = it.kv_begin, g_hi = it.kv_end;
  const int w_full = min(g_hi, pre + it.row0 / G + 1);      // keys below are visible to all rows
  const int32_t pt_base = ld_uniform(a.indptr + it.seq);
  const int32_t pt_count = ld_uniform(a.indptr + it.seq + 1) - pt_base;

  // page slots of this wave's tiles u, u + 4, ... from tile u0 + wave + 4 j0 on:
  // lane i holds page i % kPagesPerTile of the (i / kPagesPerTile)-th of them.  A
  // page the table lacks or a slot outside the pool is -1: it is not read, its
  // rows are zeros, and it raises the error flag if the item has keys in it.
  const int u0 = g_lo / kDecKeys;
  const int u1 = (g_hi + kDecKeys - 1) / kDecKeys;
  bool bad = false;
  auto load_slots = [&](int u) __attribute__((always_inline)) {
    const int pg = (u + kWaves * (lane / kPagesPerTile)) * kPagesPerTile + lane % kPagesPerTile;
    const bool need = pg * P < g_hi;
    int32_t s = need && pg < pt_count ? a.indices[pt_base + pg] : -1;
    s = (s >= 0 && s < a.num_slots) ? s : -1;
    bad |= need && s < 0;
    return s;
  };
  int u = u0 + wave;                                         // tile of the current step
  int32_t slots = load_slots(u);
  int u_slots = u;                                           // first tile the slots are of

  // every wave holds the same rows: row r16 of each 16-row block
  int qpos[kNB];
  bf16x8 qop[kNB][4];
#pragma unroll
  for (int nb = 0; nb < kNB; ++nb) {
    const int rr = it.row0 + min(16 * nb + r16, rows - 1);
    const int tok = rr / G;
    const int head = it.kvh * G + (rr - tok * G);
    qpos[nb] = pre + tok;
    const uint16_t* qrow = a.q + ((int64_t)(it.q_start + tok) * a.Hq + head) * kHD;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      qop[nb][ks] = ld_bf16x8(qrow + 32 * ks + 8 * g);
      if constexpr (!kExact) {
#pragma unroll
        for (int e = 0; e < 8; ++e) qop[nb][ks][e] = (__bf16)((float)qop[nb][ks][e] * a.c);
      }
    }
  }

  auto slice = [&](int w, int b) __attribute__((always_inline)) {          // slice b of wave w
    return (b ? (w & 2 ? v1 : v0) : (w & 2 ? k1 : k0)) + (w & 1) * kSliceBytes;
  };
  lds_u8* const vslice[2] = {slice(wave, 0), slice(wave, 1)};
  const int64_t slot_bytes = (int64_t)a.Hkv * P * kHD * 2;
  // a page's resource: nothing in it when the page is not to be read
  auto page_rsrc = [&](const uint16_t* pool, int32_t s) __attribute__((always_inline)) {
    return __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void*>((const void*)((const char*)pool + (int64_t)max(s, 0) * slot_bytes)), (short)0,
        s >= 0 ? (int)slot_bytes : 0, 0x00020000);
  };
  auto slot_of = [&](int t, int p) __attribute__((always_inline)) {
    return __builtin_amdgcn_readlane(slots, (t - u_slots) / kWaves * kPagesPerTile + p);
  };
  // Every tile issues exactly 8 K loads and 8 V loads, so that "at most the
  // next tile's loads may still be outstanding" is an exact wait: a row that
  // must not be read gets an offset past its page's resource, which returns
  // zeros -- into registers or into LDS alike.
  constexpr uint32_t kOutside = 0x80000000u;
  // K of tile t: [16-key block][32-d step], lane l holds key l % 16, d 8 (l / 16) on
  auto load_k = [&](int t, bf16x8 (&kr)[2][4]) __attribute__((always_inline)) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const int key = 16 * kb + r16;
      const __amdgpu_buffer_rsrc_t r = page_rsrc(a.k, slot_of(t, kb * kPagesPerTile / 2));
      const uint32_t off = t * kDecKeys + key < g_hi ? (uint32_t)((it.kvh * P + key % P) * (kHD * 2) + g * 16) : kOutside;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        kr[kb][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off + ks * 64, 0, 0));
    }
  };
  // V of tile t into an LDS slice: load j fills rows 4j .. 4j + 3, lane i one
  // 16-byte chunk of row 4j + i / 16, XOR-swizzled so that the transposed
  // reads of 8 keys x 32 bytes touch every bank once.  Keys past the item's end
  // and absent pages are zero rows, which keep the masked products finite.
  auto load_v = [&](int t, lds_u8* dst) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int key = 4 * j + g;
      const __amdgpu_buffer_rsrc_t r = page_rsrc(a.v, slot_of(t, (4 * j) / P));
      const uint32_t off = (uint32_t)((it.kvh * P + key % P) * (kHD * 2) + ((r16 ^ swz_dec(key)) << 4));
      __attribute__((address_space(3))) void* d = (__attribute__((address_space(3))) void*)(dst + j * 1024);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, d, 16, t * kDecKeys + key < g_hi ? off : kOutside, 0, 0, 0);
    }
  };
  // the slots of tile t are at hand (wave-uniform; every 32nd or 64th tile of the wave loads the next ones)
  auto need_slots = [&](int t) __attribute__((always_inline)) {
    if (t - u_slots >= kWaves * kSlotTiles) {
      u_slots = t;
      slots = load_slots(t);
    }
  };

  f32x4 oacc[kNB][8];                                        // [16-d block]: d 16 db + 4 g + r of row r16
#pragma unroll
  for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
    for (int db = 0; db < 8; ++db) oacc[nb][db] = f32x4{};
  float m_used[kNB], msub[kNB], l[kNB];
#pragma unroll
  for (int nb = 0; nb < kNB; ++nb) {
    m_used[nb] = -INFINITY;
    msub[nb] = 0.f;
    l[nb] = 0.f;
  }
  bf16x8 kr[2][2][4];

  // Issue order: K(u), V(u), K(u + 4), V(u + 4); then in the step of tile u,
  // K(u + 8) once S(u) has read K(u) out of its registers, and V(u + 8) once the
  // PV product has read V(u) out of its slice.  So at the top of a step at most
  // V(u), K(u + 4) and V(u + 4) may be outstanding, and before the PV product
  // K(u + 4), V(u + 4) and K(u + 8).  The compiler waits for the K registers by
  // itself; the waits for V in LDS are the ones below.
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int t = u + b * kWaves;
    if (t < u1) {
      load_k(t, kr[b]);
      load_v(t, vslice[b]);
    }
  }
  const int tr_key = 4 * g + (r16 >> 2), tr_d = 4 * (r16 & 3);
  auto step = [&](auto bc) __attribute__((always_inline)) {
    constexpr int b = decltype(bc)::value;
    // S^T = K Q^T: two 16-key blocks
    f32x4 S[kNB][2];
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const float init = kExact ? 0.f : -msub[nb];
        S[nb][kb] = f32x4{init, init, init, init};
      }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          S[nb][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kr[b][kb][ks], qop[nb][ks], S[nb][kb], 0, 0, 0);
    const int t2 = u + 2 * kWaves;
    if (t2 < u1) {
      need_slots(t2);
      load_k(t2, kr[b]);
    }
    const int ts = u * kDecKeys;
    bf16x8 pop[kNB];
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) {
      f32x4* const X = S[nb];
      // mask keys past the row's own position or the item's end
      if (ts + kDecKeys > w_full) {
        const int lim = min(qpos[nb], g_hi - 1);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (ts + 16 * kb + 4 * g + e > lim) X[kb][e] = -INFINITY;
      }
      // offset test (exact scale: whenever the row max grows; folded: past 2^kRescaleLog2)
      float mx = X[0][0];
#pragma unroll
      for (int e = 1; e < 8; ++e) mx = vmax(mx, X[e >> 2][e & 3]);
      mx = quad_max(mx);
      const float cand = kExact ? mx * a.c : mx + msub[nb];
      if (__ballot(cand > m_used[nb] + (kExact ? kRescaleLog2Exact : kRescaleLog2))) {
        const float m_new = fmaxf(m_used[nb], cand);
        const float alpha = (m_new == -INFINITY) ? 1.f : exp2f_fast(m_used[nb] - m_new);
        m_used[nb] = m_new;
        const float msub_new = (m_new == -INFINITY) ? 0.f : m_new;
        const float shift = msub_new - msub[nb];
        msub[nb] = msub_new;
        l[nb] *= alpha;
#pragma unroll
        for (int db = 0; db < 8; ++db) oacc[nb][db] *= alpha;
        if constexpr (!kExact) {
#pragma unroll
          for (int e = 0; e < 8; ++e) X[e >> 2][e & 3] -= shift;
        } else {
          (void)shift;
        }
      }
      float ls[2] = {0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = X[e >> 2][e & 3];
        const float p = kExact ? exp2f_fast(__builtin_fmaf(x, a.c, -msub[nb])) : exp2f_fast(x);
        pop[nb][e] = (__bf16)p;
        ls[e & 1] += p;
      }
      l[nb] += ls[0] + ls[1];
    }
    // O^T += V^T P^T: 8 blocks of 16 d, all 32 keys in one k-step
    if (t2 < u1) __builtin_amdgcn_s_waitcnt(0x4F78);         // vmcnt(24): V(u) landed
    else if (u + kWaves < u1) __builtin_amdgcn_s_waitcnt(0x4F70);   // vmcnt(16)
    else __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0)
    asm volatile("" ::: "memory");
    const lds_u8* const vb = vslice[b];
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      bf16x8 vop;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int vkey = 16 * h + tr_key;
        const int d = 16 * db + tr_d;
        const bf16x4 x = lds_read_tr(vb + vkey * 256 + ((((d >> 3) ^ swz_dec(vkey)) << 4) | ((d & 7) << 1)));
#pragma unroll
        for (int e = 0; e < 4; ++e) vop[4 * h + e] = x[e];
      }
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb)
        oacc[nb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, pop[nb], oacc[nb][db], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);                    // lgkmcnt(0): V operands read out of LDS
    asm volatile("" ::: "memory");
    if (t2 < u1) load_v(t2, vslice[b]);
    u += kWaves;
  };
  while (u < u1) {
    step(IntC<0>{});
    if (u >= u1) break;
    step(IntC<1>{});
  }
  if (__ballot(bad) != 0 && lane == 0) atomicOr(a.err, 1);

  // ---- merge the four waves' partial results through LDS (their slices are
  // free): every wave leaves the rows it has, and all 256 threads combine,
  // thread by (row, four d), straight to the output or the part's partial
  __attribute__((address_space(3))) float* const sm = stats;
  __attribute__((address_space(3))) float* const sl = stats + kWaves * kDecRows;
  __attribute__((address_space(3))) int* const flag = (__attribute__((address_space(3))) int*)(stats + 2 * kWaves * kDecRows);
  auto piece = [&](int w, int row, int c) __attribute__((always_inline)) {   // 16-byte piece c of a row, spread over the banks
    return (__attribute__((address_space(3))) f32x4*)((row < 16 ? slice(w, 0) : slice(w, 1)) + (row & 15) * (kHD * 4) +
                                                     ((c ^ (row & 7)) << 4));
  };
#pragma unroll
  for (int nb = 0; nb < kNB; ++nb) {
    const int row = 16 * nb + r16;
    const float lt = quad_sum(l[nb]);
    if (row < rows) {
#pragma unroll
      for (int db = 0; db < 8; ++db) *piece(wave, row, 4 * db + g) = oacc[nb][db];
      if (g == 0) {
        sm[wave * kDecRows + row] = m_used[nb];
        sl[wave * kDecRows + row] = lt;
      }
    }
  }
  __syncthreads();
  const bool whole = it.part < 0;
  const __amdgpu_buffer_rsrc_t rp = part_rsrc(a);
  const uint32_t l_base = whole ? 0u : (uint32_t)a.n_parts * (kPipeRows * kHD * 4);
  const int per = rows * (kHD / 4);                         // 16-byte pieces of the item's rows
  for (int e = tid; e < per; e += 256) {
    const int row = e >> 5, c = e & 31;
    float m = sm[row];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, sm[w * kDecRows + row]);
    const float sub = m == -INFINITY ? 0.f : m;
    f32x4 o = f32x4{};
    float lsum = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float f = exp2f_fast(sm[w * kDecRows + row] - sub);
      lsum += f * sl[w * kDecRows + row];
      o += f * *piece(w, row, c);
    }
    const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
    const float lse2 = lsum > 0.f ? m + __builtin_amdgcn_logf(lsum) : -INFINITY;
    o *= inv;
    if (whole) {
      const int r = it.row0 + row, tok = r / G;
      const int64_t orow = (int64_t)(it.q_start + tok) * a.Hq + it.kvh * G + (r - tok * G);
      st_bf16x4(a.o + orow * kHD + 4 * c, o[0], o[1], o[2], o[3]);
      if (a.lse != nullptr && c == 0) a.lse[orow] = lse2 * 0.69314718055994531f;
    } else {
      part_st4(rp, (uint32_t)it.part * (kPipeRows * kHD * 4) + (uint32_t)e * 16, o);
      if (c == 0) part_st1(rp, l_base + (uint32_t)it.part * (kPipeRows * 4) + row * 4, 0, lse2);
    }
  }
  if (whole) return;
  // A key-range part: counted once all of its stores are acknowledged; the
  // block of the last part merges the item's parts, its threads spread over
  // (row, four d, every nsub-th part).
  const PartInfo pi = ld_uniform(a.part_info + it.part);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0070);
  __syncthreads();
  if (wave == 0) {
    const bool last = part_arrive(a, pi, 0);
    if (lane == 0) *flag = last;
  }
  __syncthreads();
  if (*flag == 0) return;
  // every part's LSE into LDS: nsplit x rows words, in the room of one K tile
  static_assert(kMaxDecodeParts * kDecRows * sizeof(float) <= kTileBytes, "the LSEs of an item's parts fit k0");
  __attribute__((address_space(3))) float* const ls = (__attribute__((address_space(3))) float*)k0;
  const int nsub = max(1, 256 / per);                       // thread groups, each over every nsub-th part
  const int sub = nsub > 1 ? tid / per : 0;
  for (int i = tid; i < pi.nsplit * rows; i += 256) {
    const int s = i / rows;
    ls[i] = part_ld1(rp, l_base + (uint32_t)(pi.part0 + s) * (kPipeRows * 4) + (i - s * rows) * 4, 0);
  }
  __syncthreads();
  for (int e0 = 0; e0 < per; e0 += 256) {                   // several passes only past 8 rows (then nsub is 1)
    const int e = e0 + tid - sub * per;
    const bool mine = nsub > 1 ? sub < nsub : e < per;
    const int row = mine ? e >> 5 : 0, c = e & 31;
    float mx = -INFINITY;
    for (int s = 0; s < pi.nsplit; ++s) mx = fmaxf(mx, ls[s * rows + row]);
    const float msub2 = mx == -INFINITY ? 0.f : mx;
    f32x4 num = f32x4{};
    float den = 0.f;
    if (mine) {
      const uint32_t off = (uint32_t)pi.part0 * (kPipeRows * kHD * 4) + (uint32_t)e * 16;
      constexpr int kBatch = 8;                             // partial rows in flight per thread
      for (int s0 = sub; s0 < pi.nsplit; s0 += kBatch * nsub) {
        f32x4 x[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          const int s = s0 + k * nsub;
          x[k] = part_ld4(rp, s < pi.nsplit ? off + (uint32_t)s * (kPipeRows * kHD * 4) : kOutside, 0);
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          const int s = s0 + k * nsub;
          const float w = s < pi.nsplit ? exp2f_fast(ls[s * rows + row] - msub2) : 0.f;
          den += w;
          num += w * x[k];
        }
      }
    }
    if (nsub > 1) {                                         // one pass: the thread groups meet in LDS
      __attribute__((address_space(3))) f32x4* const red = (__attribute__((address_space(3))) f32x4*)v0;
      __attribute__((address_space(3))) float* const red_den = (__attribute__((address_space(3))) float*)v1;
      if (mine) {
        red[tid] = num;
        red_den[tid] = den;
      }
      __syncthreads();
      if (tid >= per) return;
      for (int k = 1; k < nsub; ++k) {
        num += red[k * per + tid];
        den += red_den[k * per + tid];
      }
    }
    if (mine) {
      const float dinv = den > 0.f ? 1.f / den : 0.f;
      const int r = it.row0 + row, tok = r / G;
      const int64_t orow = (int64_t)(it.q_start + tok) * a.Hq + it.kvh * G + (r - tok * G);
      st_bf16x4(a.o + orow * kHD + 4 * c, num[0] * dinv, num[1] * dinv, num[2] * dinv, num[3] * dinv);
      if (a.lse != nullptr && c == 0)
        a.lse[orow] = den > 0.f ? (mx + __builtin_amdgcn_logf(den)) * 0.69314718055994531f : -INFINITY;
    }
  }
}

// One group of four waves per block, two blocks per CU.
// kRead: the launch also writes the segment's new K/V rows (write_own_rows)
// and reads the segment's keys from them, not from their pages.  A decode item
// reads its keys through the pages, whole or split: a part with keys of the
// segment writes all of the item's rows itself first and reads them back after a
// barrier, so it depends on no other block (one part has them all unless the
// segment's up to 32 keys cross a part's edge; then both write the same bytes).
// One 16570-key request, 8 heads over two KV heads, append included: 52.3 us with
// its parts on the general path, 13.3 on this one.
// kExact: the softmax scale is applied in fp32 to each score instead of to
// the query rows in bf16 (one fma per score; no rounding of c q).
template <int P, bool kPoolRsrc, bool kRead, bool kExact = false>
__global__ __launch_bounds__(256, 2) void attn_pipe_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) uint8_t k_lds0[kTileBytes], k_lds1[kTileBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t v_lds0[kTileBytes], v_lds1[kTileBytes];
  __shared__ float dec_stats[2 * 4 * kDecRows + 1];
  const AttnItem it = ld_uniform(a.items + blockIdx.x);
  if (a.blk_clock != nullptr && threadIdx.x == 0) {
    uint64_t* r = a.blk_clock + 4 * (int64_t)blockIdx.x;
    r[0] = __builtin_amdgcn_s_memrealtime();
    // {sequence, KV head, first key tile mod 2^16}, {q_len, first row}
    r[2] = (uint64_t)(uint32_t)it.seq | ((uint64_t)(uint16_t)it.kvh << 32) |
           ((uint64_t)(uint16_t)(it.kv_begin / kKT) << 48);
    r[3] = (uint64_t)(uint32_t)it.q_len | ((uint64_t)(uint32_t)it.row0 << 32);
  }
  if (it.kv_begin < it.kv_end) {                            // else a padding item
    const SeqDesc sd{it.q_start, it.q_len, it.kv_len, 0};
    const PipeLds L{(lds_u8*)k_lds0, (lds_u8*)k_lds1, (lds_u8*)v_lds0, (lds_u8*)v_lds1,
                    nullptr, nullptr, nullptr, nullptr, nullptr};
    // the parts of a split item all take one path, since they share its partials' layout
    const bool decode = it.q_len * a.G <= kDecRows;
    if constexpr (kRead) {
      if (decode ? it.kv_end > it.kv_len - it.q_len : it.kv_begin == 0) {
        write_own_rows<P>(a, it);
        if (decode) __syncthreads();                         // its own rows, read back below
      }
    }
    if (decode && it.q_len * a.G <= 16)
      decode_group<P, kExact, 1>(a, it, (lds_u8*)k_lds0, (lds_u8*)k_lds1, (lds_u8*)v_lds0, (lds_u8*)v_lds1, (lds_f32*)dec_stats);
    else if (decode)
      decode_group<P, kExact, 2>(a, it, (lds_u8*)k_lds0, (lds_u8*)k_lds1, (lds_u8*)v_lds0, (lds_u8*)v_lds1, (lds_f32*)dec_stats);
    else
      pipe_group<P, kPoolRsrc, 1, 0, kRead, kExact>(a, it, sd, L);
  }
  if (a.blk_clock != nullptr) {
    // every wave's stores are done once the barrier is passed
    __syncthreads();
    if (threadIdx.x == 0) a.blk_clock[4 * (int64_t)blockIdx.x + 1] = __builtin_amdgcn_s_memrealtime();
  }
}

// Two groups of four waves per block on the same rows, each over half of the
// item's key tiles, one block per CU; the halves merge in LDS.
template <int P, bool kPoolRsrc>
__global__ __launch_bounds__(512, 1) void attn_pp_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(1024))) uint8_t k_a0[kTileBytes], k_a1[kTileBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t v_a0[kTileBytes], v_a1[kTileBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t k_b0[kTileBytes], k_b1[kTileBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t v_b0[kTileBytes], v_b1[kTileBytes];
  __shared__ float ml[4 * kPipeRows];
  const AttnItem it = ld_uniform(a.items + blockIdx.x);
  if (it.kv_begin >= it.kv_end) return;                     // padding item
  const SeqDesc sd{it.q_start, it.q_len, it.kv_len, 0};
  lds_u8* const xb0 = (lds_u8*)k_b0;
  lds_u8* const xb1 = (lds_u8*)k_b1;
  lds_u8* const xb2 = (lds_u8*)v_b0;
  lds_u8* const xb3 = (lds_u8*)v_b1;
  __attribute__((address_space(3))) float* const mlp = (__attribute__((address_space(3))) float*)ml;
  if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) < kPipeWaves) {
    const PipeLds L{(lds_u8*)k_a0, (lds_u8*)k_a1, (lds_u8*)v_a0, (lds_u8*)v_a1, xb0, xb1, xb2, xb3, mlp};
    pipe_group<P, kPoolRsrc, 2, 0>(a, it, sd, L);
  } else {
    const PipeLds L{xb0, xb1, xb2, xb3, xb0, xb1, xb2, xb3, mlp};
    pipe_group<P, kPoolRsrc, 2, 1>(a, it, sd, L);
  }
}

}  // namespace sa
