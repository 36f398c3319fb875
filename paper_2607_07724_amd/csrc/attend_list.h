// What the attention kernels share before their block loops: the parameters,
// the order of the units, and the unit's list of kept blocks (from a kv_idx
// row, a bitmap row, or the selection over the tile scores).
#pragma once
#include <atomic>
#include <type_traits>

#include "attend_common.h"

namespace ugbs {

// Work order: two kv heads at a time across the whole device (XCDs 0-3 on
// one, 4-7 on the other, so the memory-side cache holds the working set),
// one kv head at a time when the (batch, kv head) count is odd; within a
// kv head the XCDs of its group take its tiles in turn, heaviest first, the
// sibling query heads of a tile one after another on the same XCD, whose L2
// then serves the blocks they share.  Workgroup j runs on XCD j mod 8.
// - Above 64 tiles the turns go back and forth over the XCDs, so that no XCD
//   always gets the heavier tile (d 256, 64K: 4.52 -> 4.39 ms; at 64 tiles,
//   two rounds of units, it was 1% slower).
// - When the tiles don't divide over the XCDs of a group, an XCD has one
//   fewer in the last turn and the workgroups of the missing one leave at
//   once.  Dealing such lengths unit by unit over all XCDs put sibling heads
//   on different ones: 0.70 -> 0.66 ms at 141 blocks (28/4 heads, batch 2),
//   0.205 -> 0.188 ms at 253 blocks (16/4 heads, d 64, with the turns).
//   Below 64 tiles that order stays: a kv head's K and V fit an L2 whole, and
//   the padding could double the grid.
struct AttendOrder {
  int hpp, lg;   // kv heads in flight, log2 of the XCDs per kv head
  int per;       // workgroups of one XCD per kv head; 0: units round-robin
  int snake;     // the tiles change direction every turn
  int grid;
};


struct AttnParams {
  Shape s;
  const uint16_t* Q;
  const uint16_t* K;
  const uint16_t* V;
  const int32_t* kv_idx;
  uint16_t* O;
  int kv_width;
  double expected;   // kept blocks of a unit, as the budget has it
  double longest;    // and the most a unit keeps
  AttendOrder order;
  int conc;          // units resident at once on one XCD (rotation period)
  float scale_log2;
  // in-kernel selection (ugbs_attend_select)
  const float* sel_scores;    // [B, H, T, N_B] tile scores, or nullptr: packed rows
  const float* sel_packed;    // packed candidate rows (workspace)
  const uint8_t* sel_trigger; // [B, T] trigger flags
  // block bitmaps (ugbs_attend_bitmap)
  const uint32_t* bitmap;     // [B, H, T, nw]
  int nw;
};

// Attention at d 64 and 128, the keys of a unit split over its waves
// (attend_keys.hip); mode: a Mode.
hipError_t launch_attend_keys(const AttnParams& P, int mode, hipStream_t stream);

namespace {

// The running maximum of a row before its first finite score.  A number, not
// -inf: the first keys a wave sees may all have scores of -inf for a row (keys
// after the row, or products that overflow) where later ones, or another wave's,
// are finite, and -inf - -inf would make the row NaN; so their probabilities are 0.
constexpr float kNoMax = -3.402823466e38f;

// Where a tile's blocks come from.  kSelectWide: kSelect for rows of more
// than 2048 candidate blocks (64 instead of 32 candidates per lane).
enum Mode { kLists = 0, kSelect = 1, kBitmap = 2, kSelectWide = 3 };

inline AttendOrder attend_order(const Shape& s) {
  AttendOrder o;
  const int nbh = s.B * s.Hkv;
  o.hpp = nbh % 2 == 0 ? 2 : 1;
  o.lg = nbh % 2 == 0 ? 2 : 3;
  o.snake = s.T > 64 ? 1 : 0;
  const int stride = 1 << o.lg;
  if (s.T < 64 && s.T % stride != 0) {
    o.per = 0;
    o.grid = nbh * s.G * s.T;
  } else {
    o.per = (s.T + stride - 1) / stride * s.G;
    o.grid = 8 * ((nbh + o.hpp - 1) / o.hpp) * o.per;
  }
  return o;
}

// This workgroup's unit; false: it has none.
__device__ __forceinline__ bool attend_unit(const Shape& s, const AttendOrder& o, Unit* u) {
  if (o.per == 0) {
    *u = unit_of(blockIdx.x, s);
    return true;
  }
  const int n_x = blockIdx.x >> 3, x = blockIdx.x & 7;
  const int phase = n_x / o.per;
  const int within = n_x - phase * o.per;
  const int hh = o.hpp * phase + (x >> o.lg);                // (batch, kv head) index
  // tile rank, heaviest first, in a snake over the XCDs of the group
  const int turn = within / s.G, last = (1 << o.lg) - 1;
  const int tr = (turn << o.lg) + ((x ^ ((o.snake & (turn + phase)) ? last : 0)) & last);
  if (hh >= s.B * s.Hkv || tr >= s.T) return false;
  u->b = hh / s.Hkv;
  u->h = (hh % s.Hkv) * s.G + (within - turn * s.G);
  u->t = s.T - 1 - tr;
  return true;
}

// The tile's kept blocks, ascending, into s_list (called by all NWV waves of
// the unit; a workgroup barrier follows): kv_idx entries outside 0..t are
// dropped and repeated entries count once (set semantics, as in Eq. (Attn)),
// so the diagonal block t, the only one needing the causal mask, is the last
// entry when present.  *s_n: their number; *s_below: those below start_blk.
// surv (2 KiB) and top (NWV x (768 + 4) bytes) are LDS scratch.
template <int MODE, int NWV>
__device__ __forceinline__ void build_list(const AttnParams& P, const Unit& u, size_t rowid, int start_blk, int w,
                                           int lane, uint64_t* surv, uint32_t* top, uint32_t* s_bits,
                                           uint16_t* s_list, int* s_n, int* s_below) {
  const Shape& s = P.s;
  // Selection modes, shared part: the unit's waves split the candidate
  // loads, the keys, each lane's top-3 pre-filter and the survivor
  // compaction (wave v takes the v-th contiguous slice of the slots, so the
  // survivors land in position order, as one wave would write them); the
  // exact threshold among the survivors stays with wave 0 below.  A lane's
  // top 3 over the waves' slices is its top 3 over every slot, so the bound
  // t0, the survivors and the kept set are those of the one-wave form.
  int staged = -1;                                     // survivors staged in surv, or -1
  if constexpr (MODE == kSelect || MODE == kSelectWide) {
    const int t = u.t;
    const int nf = (t == 0) ? 1 : 2;
    const int nc = (t >= 1) ? t - 1 : 0;
    const int flag = __builtin_amdgcn_readfirstlane((int)P.sel_trigger[(size_t)u.b * s.T + t]);
    const int R = min((flag != 0 ? s.W : s.k) - nf, nc);
    if (R < nc && R <= 192) {
      constexpr int kSlots = MODE == kSelectWide ? UGBS_MAX_BLOCKS / 64 : 32;
      static_assert(kSlots % NWV == 0, "slots split evenly over the waves");
      constexpr int kPer = kSlots / NWV;
      const int nslots = (nc + 63) / 64;
      const float* src = P.sel_scores ? P.sel_scores + rowid * s.NB + 1
                                      : P.sel_packed + packed_row(u.b * s.H + u.h, t, s.T);
      uint32_t keys[kPer];
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const int sl = w * kPer + j;
        const int p = 64 * sl + lane;
        keys[j] = (sl < nslots && p < nc) ? order_key(src[p]) : 0u;
      }
      uint32_t top3[3] = {0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const uint32_t x = keys[j];
        top3[2] = max(top3[2], min(top3[1], x));
        top3[1] = max(top3[1], min(top3[0], x));
        top3[0] = max(top3[0], x);
      }
      uint32_t* s_t3 = top;                                          // [NWV][3][64]
      int* s_cnt = reinterpret_cast<int*>(s_t3 + NWV * 3 * 64);      // [NWV]
#pragma unroll
      for (int i = 0; i < 3; ++i) s_t3[(w * 3 + i) * 64 + lane] = top3[i];
      __syncthreads();
      uint32_t m3[3] = {0u, 0u, 0u};
#pragma unroll
      for (int v = 0; v < NWV * 3; ++v) {
        const uint32_t x = s_t3[v * 64 + lane];
        m3[2] = max(m3[2], min(m3[1], x));
        m3[1] = max(m3[1], min(m3[0], x));
        m3[0] = max(m3[0], x);
      }
      bool exact0;
      const uint32_t t0 = kth_largest<3>(m3, 3, R, &exact0);
      int mine = 0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) mine += __popcll(__ballot(t0 > 0u && keys[j] >= t0));
      if (lane == 0) s_cnt[w] = mine;
      __syncthreads();
      int off = 0, ns = 0;
#pragma unroll
      for (int v = 0; v < NWV; ++v) {
        const int c = s_cnt[v];
        off += (v < w) ? c : 0;
        ns += c;
      }
      constexpr int kSurv = 256;
      if (t0 > 0u && ns <= kSurv) {
        uint64_t* s_surv = surv;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          const bool tk = keys[j] >= t0;
          const uint64_t mk = __ballot(tk);
          if (tk) s_surv[off + lanes_below(mk)] = ((uint64_t)keys[j] << 32) | (uint32_t)(64 * (w * kPer + j) + lane);
          off += __popcll(mk);
        }
        staged = ns;
      }
      __syncthreads();
    }
  }
  if (w == 0) {
    const int nwords = (u.t >> 5) + 1;                 // bitmap words covering blocks 0..t
    for (int i = lane; i < nwords; i += 64) s_bits[i] = 0u;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    if constexpr (MODE == kBitmap) {
      // the caller's bitmap row; bits of blocks after t are dropped
      const uint32_t* br = P.bitmap + rowid * P.nw;
      for (int i = lane; i < nwords; i += 64) {
        uint32_t v = br[i];
        if (i == (u.t >> 5)) v &= (u.t & 31) == 31 ? 0xffffffffu : ((2u << (u.t & 31)) - 1u);
        s_bits[i] = v;
      }
    } else if constexpr (MODE == kLists) {
      const int32_t* kr = P.kv_idx + rowid * P.kv_width;
      for (int base = 0; base < P.kv_width; base += 64) {
        const int sl = base + lane;
        const int blk = (sl < P.kv_width) ? kr[sl] : -1;
        if (blk >= 0 && blk <= u.t) atomicOr(&s_bits[blk >> 5], 1u << (blk & 31));
      }
    } else {
      // selection (A.4-A.5, A.9) from the tile scores: the forced sink and
      // self blocks, then the R best candidates of C(t) = {1..t-1} by (score
      // descending, block ascending), R = (trigger ? rho k : k) - |F|, all
      // of them when fewer: the same set as the kept prefix of kv_idx
      const int t = u.t;
      const int nf = (t == 0) ? 1 : 2;
      const int nc = (t >= 1) ? t - 1 : 0;
      // The flag is loaded unconditionally (every (b, t) has one) and moved
      // to a scalar register: written as a load guarded by nc > 0, the
      // branch around the load and the k / rho k phi after it came out of
      // this compiler with the phi's rho k copy executed unconditionally.
      // With nc == 0, R is 0 whatever the flag.
      const int flag = __builtin_amdgcn_readfirstlane((int)P.sel_trigger[(size_t)u.b * s.T + t]);
      const int R = min((flag != 0 ? s.W : s.k) - nf, nc);
      if (lane == 0) {
        atomicOr(&s_bits[0], 1u);
        if (t > 0) atomicOr(&s_bits[t >> 5], 1u << (t & 31));
      }
      if (R >= nc) {
        for (int blk = 1 + lane; blk <= nc; blk += 64) atomicOr(&s_bits[blk >> 5], 1u << (blk & 31));
      } else if (staged >= 0) {
        // the survivors the waves staged: the exact R largest among them
        constexpr int kSurv = 256;
        const uint64_t* s_surv = surv;
        uint32_t k2[kSurv / 64], p2[kSurv / 64];
#pragma unroll
        for (int sl = 0; sl < kSurv / 64; ++sl) {
          const int i = 64 * sl + lane;
          const uint64_t v = (i < staged) ? s_surv[i] : 0ull;
          k2[sl] = (uint32_t)(v >> 32);
          p2[sl] = (uint32_t)v;
        }
        select_top_each<kSurv / 64>(k2, (staged + 63) / 64, R, lane, [&](int sl) {
          const int blk = 1 + (int)p2[sl];
          atomicOr(&s_bits[blk >> 5], 1u << (blk & 31));
        });
      } else {
        const float* src = P.sel_scores ? P.sel_scores + rowid * s.NB + 1
                                        : P.sel_packed + packed_row(u.b * s.H + u.h, t, s.T);
        constexpr int kSlots = MODE == kSelectWide ? UGBS_MAX_BLOCKS / 64 : 32;
        static_assert(UGBS_MAX_BLOCKS <= 64 * 64, "at most 64 slots per lane");
        const int nslots = (nc + 63) / 64;
        uint32_t keys[kSlots];
#pragma unroll
        for (int sl = 0; sl < kSlots; ++sl) {
          const int p = 64 * sl + lane;
          keys[sl] = (sl < nslots && p < nc) ? order_key(src[p]) : 0u;
        }
        // Pre-filter as in the selection kernel: the R-th largest of the
        // lanes' three largest keys bounds the R-th largest key from below;
        // the survivors (keys at or above it, in position order) go through
        // the exact threshold on 4 slots per lane instead of 32.
        bool done = false;
        if (R <= 192) {
          uint32_t top3[3] = {0u, 0u, 0u};
#pragma unroll
          for (int sl = 0; sl < kSlots; ++sl) {
            if (sl < nslots) {
              const uint32_t x = keys[sl];
              top3[2] = max(top3[2], min(top3[1], x));
              top3[1] = max(top3[1], min(top3[0], x));
              top3[0] = max(top3[0], x);
            }
          }
          bool exact0;
          const uint32_t t0 = kth_largest<3>(top3, 3, R, &exact0);
          constexpr int kSurv = 256;
          uint64_t* s_surv = surv;
          int ns = 0;
#pragma unroll
          for (int sl = 0; sl < kSlots; ++sl) {
            if (sl < nslots) {
              const bool tk = t0 > 0u && keys[sl] >= t0;
              const uint64_t mk = __ballot(tk);
              const int at = ns + lanes_below(mk);
              if (tk && at < kSurv) s_surv[at] = ((uint64_t)keys[sl] << 32) | (uint32_t)(64 * sl + lane);
              ns += __popcll(mk);
            }
          }
          if (t0 > 0u && ns <= kSurv) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_wave_barrier();
            uint32_t k2[kSurv / 64], p2[kSurv / 64];
#pragma unroll
            for (int sl = 0; sl < kSurv / 64; ++sl) {
              const int i = 64 * sl + lane;
              const uint64_t v = (i < ns) ? s_surv[i] : 0ull;
              k2[sl] = (uint32_t)(v >> 32);
              p2[sl] = (uint32_t)v;
            }
            select_top_each<kSurv / 64>(k2, (ns + 63) / 64, R, lane, [&](int sl) {
              const int blk = 1 + (int)p2[sl];
              atomicOr(&s_bits[blk >> 5], 1u << (blk & 31));
            });
            done = true;
          }
        }
        if (!done)
          select_top_each<kSlots>(keys, nslots, R, lane, [&](int sl) {
            const int blk = 1 + 64 * sl + lane;
            atomicOr(&s_bits[blk >> 5], 1u << (blk & 31));
          });
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    int n = 0, below = 0;
    for (int base = 0; base <= u.t; base += 64) {
      const int blk = base + lane;
      const bool on = blk <= u.t && ((s_bits[blk >> 5] >> (blk & 31)) & 1u);
      const uint64_t m = __ballot(on);
      if (on) s_list[n + lanes_below(m)] = (uint16_t)blk;
      n += __popcll(m);
      below += __popcll(__ballot(on && blk < start_blk));
    }
    if (lane == 0) {
      *s_n = n;
      *s_below = below;
    }
  }
}

// Kept blocks of a unit that sees many: k, or W on the share q of the tiles
// that trigger, for the pipeline's lists of W slots; all slots of other lists.
inline double expected_blocks(const Shape& s, int width) {
  const double e = width == s.W ? s.k + s.q * (s.W - s.k) : width;
  return e < s.NB ? e : s.NB;
}

inline double longest_list(const Shape& s, int width) {
  const double m = width == s.W && s.q == 0.0 ? s.k : width;   // q 0: no tile triggers
  return m < s.NB ? m : s.NB;
}

// Mean of the kept blocks over the tiles of a sequence: tile t sees t + 1.
inline double mean_blocks(const AttnParams& P) {
  return P.expected - P.expected * (P.expected - 1.0) / (2.0 * P.s.T);
}

// LDS of a unit's list: at most kv_width distinct blocks, and at most N_B, 16 bits
// each (long lists cost resident units).  The same for lists of 2k slots and for
// the in-kernel selection, so both run at the same occupancy and visit the
// blocks in the same order.
static_assert(UGBS_MAX_BLOCKS <= 65536, "16-bit list entries");
inline size_t list_bytes(const AttnParams& P) {
  return sizeof(uint16_t) * (size_t)(P.kv_width < P.s.NB ? P.kv_width : P.s.NB);
}

// Workgroups of an attention kernel resident at once on one XCD, for the given
// dynamic LDS size (occupancy per CU x CUs per XCD).  Cached per kernel and
// device as one packed word (smem << 32 | value); a stale or missing entry only
// costs a recomputation.  The value steers the visiting order, never the result.
// RAISE: the static LDS alone reaches 64 KiB, so the kernel's dynamic limit is
// raised first (to the widest list, the same value whoever calls).
constexpr int kMaxDevices = 64;
template <auto KERNEL, bool RAISE = false>
hipError_t xcd_concurrency(int threads, size_t smem, int* conc) {
  static std::atomic<uint64_t> cache[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev >= kMaxDevices) dev = -1;
  if (dev >= 0) {
    const uint64_t e = cache[dev].load(std::memory_order_relaxed);
    if (e != 0 && (e >> 32) == (uint64_t)smem) {
      *conc = (int)(uint32_t)e;
      return hipSuccess;
    }
  }
  if (RAISE) {
    const hipError_t e = hipFuncSetAttribute((const void*)KERNEL, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)sizeof(uint16_t) * UGBS_MAX_KV_WIDTH);
    if (e != hipSuccess) return e;
  }
  int per_cu = 0, n_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, KERNEL, threads, smem) != hipSuccess) per_cu = 1;
  if (dev < 0 || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) n_cu = 8;
  *conc = per_cu * n_cu / 8 > 0 ? per_cu * n_cu / 8 : 1;
  if (dev >= 0) cache[dev].store(((uint64_t)smem << 32) | (uint32_t)*conc, std::memory_order_relaxed);
  return hipSuccess;
}

}  // namespace
}  // namespace ugbs
