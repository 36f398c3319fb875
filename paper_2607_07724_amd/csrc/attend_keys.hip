// Stage 5 at d 64 and 128: block-sparse causal attention with the keys of a
// unit split over its waves.
//
// One workgroup per (batch, query head, Q-tile) unit.  Wave w owns key half
// w & 1 (32 of a block's 64 keys) of every NP-th listed block (NP = waves / 2,
// entries w >> 1, w >> 1 + NP, ...), for all 64 query rows of the tile, with
// its own running softmax; the waves' results are merged once at the end of
// the unit.  So nothing in the block loop is shared between waves: each wave
// stages its own 32-key half tiles of K and V (8 KiB each at d 128) with
// direct-to-LDS loads and waits only for its own loads, there is no barrier
// until the merge, and the two waves of a SIMD drift against each other, one
// on the matrix cores while the other is in its softmax.
//
// Per listed half block and wave (v_mfma_f32_16x16x32_bf16):
//   S^T = K Q^T   [32 keys x 64 rows]: K rows from LDS (ds_read_b128) are the
//                 A operand, read once for all 64 rows; the query rows stay in
//                 registers as the B operand (at d 128 the last 16 of them in
//                 LDS: 252 registers with two waves, 256 with four, no spills;
//                 the in-kernel selection spills up to 8); a lane ends up with
//                 8 keys of one row per 16-row tile;
//   softmax       fp32, base 2; whether a reference maximum has to move is asked
//                 per lane first, the cross-lane maximum only taken when one does;
//   O^T += V^T P^T  a lane's probabilities, packed to bf16, already are the B
//                 operand; V^T comes from the natural-layout LDS tile through
//                 the transposing read ds_read_b64_tr_b16.
//
// Loads.  Issuing a direct load stalls the wave until the texture unit takes
// it, so a half tile's eight loads are never issued in a row: V's go out one by
// one between the matrix instructions of S, the next K's four at a time between
// the exponentials.  Each half tile is refilled once it has been read, and has
// the other two phases to land.  With PV at a raised priority the two waves of
// a SIMD settle on opposite phases.
//
// What bounds it: at d 128 the power limit and, right behind it, the loads.  128K,
// 32/8 heads, k 64: 10.1 ms at 1.64 GHz, the matrix cores 53% busy, the vector ALU
// issuing 52% of the time, the texture unit 69% busy; zeros in all inputs run at 2.39
// GHz and take 9.4 ms.  (The 64-byte-per-clock staging path is as long as the matrix
// work, 64 FLOP per staged byte, and 53 GB of it come from beyond the L2.)  At d 64 the vector ALU (exponentials).  Measured against the
// form it replaced (both waves of a unit on all 64 keys and 32 rows each, two
// workgroup barriers per block, twice the LDS reads): lists at d 128, 128K
// (32/8 heads, k 64) 10.4 -> 9.8 ms, 64K (28/4) 4.34 -> 4.10, 32K (k 32) 1.13 ->
// 1.07; d 64, 128K 6.6 -> 5.6 ms; bitmaps (28/4 heads, 32K) 6.5 -> 6.0 ms.
// Steps on the way, 64K: all loads of a tile at once 1.02x, V spread 1.00x, K
// spread too 0.97x, priority of PV alone 0.95x; 32x32x16 matrix instructions
// drew more power (clock 1.77 GHz for 1.85) and were 1% slower.
#include "attend_list.h"

namespace ugbs {
namespace {

// A wave's half tile: 32 keys x D in natural [key][channel] layout, the
// 16-byte columns of a row permuted by an XOR so that both the K-operand reads
// (16 consecutive lanes read one column of 16 consecutive rows) and the
// transposing V reads (32 lanes read four columns of four consecutive rows)
// touch every bank once.
template <int D>
struct Half {
  static constexpr int CPR = D / 8;               // 16-byte columns per row
  static constexpr int kRow = 2 * D;              // bytes per row
  static constexpr int kBytes = 32 * kRow;
  static constexpr int kLoads = kBytes / 1024;    // direct loads, 1 KiB each
  static constexpr int kRows = 1024 / kRow;       // rows per load
  // distinct lane offsets over the loads: load i's are an XOR of step bytes x (i mod period)
  static constexpr int kPeriodK = D == 128 ? 4 : 2, kStepK = 64;
  static constexpr int kPeriodV = D == 128 ? 2 : 1, kStepV = 128;
  __device__ static __forceinline__ int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  __device__ static __forceinline__ int swz_v(int r) { return D == 128 ? 2 * (r & 7) : 2 * ((r >> 1) & 3); }
};

// sum over the four 16-lane rows holding one query row
__device__ __forceinline__ float rows_sum(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// c ? a : b on values (a conditional on the array elements themselves would
// take their addresses and move the accumulators to memory)
__device__ __forceinline__ f32x4 pick(bool c, f32x4 a, f32x4 b) {
  return f32x4{c ? a[0] : b[0], c ? a[1] : b[1], c ? a[2] : b[2], c ? a[3] : b[3]};
}

// x, opaque to the compiler: values derived from it are recomputed where they
// are used instead of being held in registers over the block loop.
__device__ __forceinline__ uint32_t here(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Waves per SIMD: what the registers allow (O alone takes D of them).
template <int D>
constexpr int kWaves = D == 64 ? 3 : 2;

template <int D, int MODE, int NWV>
__global__ void __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(kWaves<D>, kWaves<D>)))
attend_keys_kernel(AttnParams P) {
  using L = Half<D>;
  constexpr int KS = D / 32;      // k-steps of QK^T
  constexpr int DT = D / 16;      // 16-channel tiles of O^T
  constexpr int NP = NWV / 2;     // waves per key half
  constexpr int QR = D == 128 ? 3 : 4;   // 16-row query tiles held in registers, the others in LDS
  constexpr int AHEAD = 2;        // K operands read ahead of the matrix instructions (3 spills at d 128)
  __shared__ __align__(16) unsigned char s_tile[NWV][2][L::kBytes];   // K and V half tile of each wave
  // the prologue's block bitmap; after the loop the running (max, sum) of each wave and row
  __shared__ __align__(16) float2 s_ml[NWV][kBlock];
  static_assert(sizeof(float2) * 2 * kBlock >= UGBS_MAX_BLOCKS / 8, "the bitmap fits");
  uint32_t* const s_bits = reinterpret_cast<uint32_t*>(s_ml);
  __shared__ __align__(16) unsigned char s_q[QR < 4 ? (4 - QR) * 16 * L::kRow : 16];   // query tiles QR..3
  extern __shared__ uint16_t s_list[];              // list_bytes
  __shared__ int s_n, s_below;

  const Shape& s = P.s;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform per wave
  const int g = lane >> 4, c16 = lane & 15;
  Unit u;
  if (!attend_unit(s, P.order, &u)) return;
  const int kvh = u.h / s.G;
  const size_t rowid = ((size_t)u.b * s.H + u.h) * s.T + u.t;

  // Visiting order.  The j-th workgroup an XCD receives starts its walk at
  // the first listed block >= (j mod 2 conc) / (2 conc) of its key range and
  // wraps around (the diagonal block stays last).  Workgroups follow each
  // other on an XCD in the order of j, conc of them at a time, so the ones
  // resident together sweep the key range in step and blocks they share
  // stay in that XCD's L2.  Bitmaps with four waves: a period of 1 conc (1600
  // blocks, 16/4 heads: 34.6 ms for 36.4); with two, 2 conc as for lists (512
  // blocks, 28/4 heads: 5.6 ms for 6.2).
  const int j_xcd = blockIdx.x >> 3;
  const int period = (MODE == kBitmap && NWV == 4 ? 1 : 2) * P.conc;
  const int start_blk = (int)(((long long)(j_xcd % period) * u.t) / period);
  const size_t qo_base = ((size_t)u.b * s.H + u.h) * s.N + (size_t)u.t * kBlock;
  build_list<MODE, NWV>(P, u, rowid, start_blk, w, lane, reinterpret_cast<uint64_t*>(s_tile),
                        reinterpret_cast<uint32_t*>(&s_tile[0][0][2048]), s_bits, s_list, &s_n, &s_below);
  __syncthreads();
  const int n = __builtin_amdgcn_readfirstlane(s_n);
  const bool diag_last = n > 0 && s_list[n - 1] == u.t;
  // entries 0..n_rot-1 are visited from position rot0 on, cyclically
  const int n_rot = __builtin_amdgcn_readfirstlane(diag_last ? n - 1 : n);
  const int rot0 = __builtin_amdgcn_readfirstlane(s_below < n_rot ? s_below : 0);
  // the i-th block to visit, as a per-lane LDS value (every lane the same)
  auto listed_raw = [&](int i) {
    int p = i;
    if (i < n_rot) {
      p = i + rot0;
      if (p >= n_rot) p -= n_rot;
    }
    return s_list[p];
  };

  if (n == 0) {  // no attended key: O = 0
    for (int i = tid; i < kBlock * D / 8; i += 64 * NWV)
      reinterpret_cast<uint4*>(P.O + qo_base * D)[i] = make_uint4(0, 0, 0, 0);
    return;
  }

  // ---- this wave's loads ------------------------------------------------------
  const int kh = w & 1;
  const uint16_t* Kh = P.K + (((size_t)u.b * s.Hkv + kvh) * s.N + 32 * kh) * D;
  const uint16_t* Vh = P.V + (((size_t)u.b * s.Hkv + kvh) * s.N + 32 * kh) * D;
  const unsigned char* tk = s_tile[w][0];
  const unsigned char* tv = s_tile[w][1];
  const uint32_t k_lds = __builtin_amdgcn_readfirstlane(lds_addr(tk));
  const uint32_t v_lds = __builtin_amdgcn_readfirstlane(lds_addr(tv));
  // lane offsets of the loads; load i moves rows kRows i .. + kRows - 1
  uint32_t koff, voff;
  {
    const int r = lane / L::CPR, c = lane % L::CPR;
    koff = (uint32_t)(r * L::kRow + 16 * (c ^ L::swz_k(r)));
    voff = (uint32_t)(r * L::kRow + 16 * (c ^ L::swz_v(r)));
  }
  auto load_k = [&](const uint16_t* src, uint32_t o, int i) {
    dma16(src + i * 512, o ^ (uint32_t)(L::kStepK * (i % L::kPeriodK)), k_lds + (uint32_t)(i * 1024));
  };
  auto load_v = [&](const uint16_t* src, uint32_t o, int i) {
    dma16(src + i * 512, o ^ (uint32_t)(L::kStepV * (i % L::kPeriodV)), v_lds + (uint32_t)(i * 1024));
  };
  auto fetch_k = [&](int b) {
    const uint16_t* src = Kh + (size_t)b * kBlock * D;
    const uint32_t o = here(koff);
#pragma unroll
    for (int i = 0; i < L::kLoads; ++i) load_k(src, o, i);
  };
  // the first K and V half tiles and the query rows are in flight together
  int e = w >> 1;
  int cur = 0, raw = 0;
  if (e < n) {
    cur = __builtin_amdgcn_readfirstlane(listed_raw(e));
    raw = (e + NP < n) ? listed_raw(e + NP) : 0;
    fetch_k(cur);
    const uint16_t* vsrc = Vh + (size_t)cur * kBlock * D;
#pragma unroll
    for (int i = 0; i < L::kLoads; ++i) load_v(vsrc, voff, i);
  }

  // ---- query rows as the B operand: row 16 rt + c16, channels 32 ks + 8 g .. + 7
  // operand read address within a K half tile or an LDS query tile
  const uint32_t ka = (uint32_t)(c16 * L::kRow + 16 * (g ^ L::swz_k(c16)));
  bf16x8 bq[QR][KS];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    const uint16_t* qr = P.Q + (qo_base + 16 * rt + c16) * D + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (rt < QR) {
        bq[rt < QR ? rt : 0][ks] = as_bf16x8(*reinterpret_cast<const uint4*>(qr + 32 * ks));
      } else if (w == rt % NWV) {
        *reinterpret_cast<uint4*>(s_q + (rt - QR) * 16 * L::kRow + (ka ^ (uint32_t)(64 * ks))) =
            *reinterpret_cast<const uint4*>(qr + 32 * ks);
      }
    }
  }
  wait_vmcnt<0>();
  if constexpr (QR < 4) __syncthreads();

  // transposing read address within a V half tile
  const int tr_row = 4 * g + (c16 >> 2);
  const uint32_t va = (uint32_t)(tr_row * L::kRow + 16 * (((c16 & 3) >> 1) ^ L::swz_v(tr_row)) + 8 * (c16 & 1));

  f32x4 acc_o[DT][4];
  float m_run[4], l_run[4];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc_o[dt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run[rt] = kNoMax;
    l_run[rt] = 0.f;
  }

  // S^T of the half block whose K half tile has landed; LOAD_V: the loads of
  // its V half tile (block cur) go out between the matrix instructions
  f32x4 sc[2][4];
  auto compute_s = [&](int cur, auto load_tag) {
    constexpr bool LOAD_V = decltype(load_tag)::value;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) sc[kt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t* vsrc = Vh + (size_t)cur * kBlock * D;
    const uint32_t kr = here(ka), vo = here(voff);
    constexpr int NR = 2 * KS;
    bf16x8 ak[NR], lq[KS][4];
    auto k_op = [&](int j) {
      if ((j & 1) == 0) {
#pragma unroll
        for (int rt = QR; rt < 4; ++rt)
          lq[j >> 1][rt] = as_bf16x8(*reinterpret_cast<const uint4*>(s_q + (kr ^ (uint32_t)(64 * (j >> 1))) +
                                                                     (rt - QR) * 16 * L::kRow));
      }
      ak[j] = as_bf16x8(*reinterpret_cast<const uint4*>(tk + (kr ^ (uint32_t)(64 * (j >> 1))) + (j & 1) * 16 * L::kRow));
    };
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) k_op(j);
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      if (j + AHEAD < NR) k_op(j + AHEAD);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int rt = 0; rt < 4; ++rt)
        sc[j & 1][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak[j], rt < QR ? bq[rt < QR ? rt : 0][j >> 1] : lq[j >> 1][rt],
                                                                sc[j & 1][rt], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (LOAD_V) load_v(vsrc, vo, j);
    }
    static_assert(NR == L::kLoads, "one V load per K operand");
  };

  // One half block.  On entry its K half tile is in flight or landed, and for
  // the wave's first one its V half tile too.  MASK: the diagonal block, whose
  // keys after the query row are masked.
  auto step = [&](bool first, int cur, bool has_next, int nxt, auto mask_tag) {
    constexpr bool MASK = decltype(mask_tag)::value;
    wait_vmcnt<0>();                                     // K landed
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_setprio(0);
    if (first) compute_s(cur, std::false_type{});
    else compute_s(cur, std::true_type{});
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the K half tile is read: it may be refilled

    // online softmax (base 2): lane holds row 16 rt + c16, keys 16 kt + 4 g + i
    // of the half.  The reference max m_run only moves when a row max exceeds
    // it by more than 2^8, so p <= 256 and O is rescaled rarely; whether one
    // does is first asked per lane, so the common case needs no cross-lane max.
    if constexpr (MASK) {
#pragma unroll
      for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (32 * kh + 16 * kt + 4 * g + i > 16 * rt + c16) sc[kt][rt][i] = -__builtin_huge_valf();
    }
    float mx[4], over = -__builtin_huge_valf();
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      const f32x4 a = sc[0][rt], b = sc[1][rt];
      float m = fmaxf(fmaxf(a[0], a[1]), a[2]);
      m = fmaxf(fmaxf(m, a[3]), b[0]);
      m = fmaxf(fmaxf(m, b[1]), b[2]);
      mx[rt] = fmaxf(m, b[3]);
      over = fmaxf(over, __builtin_fmaf(mx[rt], P.scale_log2, -m_run[rt]));
    }
    if (__ballot(over > 8.0f)) {
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) {
        const float r = rows_max(mx[rt]) * P.scale_log2;
        const float m_new = r > m_run[rt] + 8.0f ? r : m_run[rt];
        const float alpha = r > m_run[rt] + 8.0f ? __builtin_amdgcn_exp2f(m_run[rt] - m_new) : 1.0f;
        m_run[rt] = m_new;
        l_run[rt] *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc_o[dt][rt][i] *= alpha;
      }
    }
    uint32_t pb[4][4];
    const uint16_t* ksrc = Kh + (size_t)nxt * kBlock * D;
    const uint32_t ko = here(koff);
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      // the next K half tile's loads, four at a time (see the top of the file)
      if (4 * rt < L::kLoads) {
        __builtin_amdgcn_sched_barrier(0);
        if (has_next) {
#pragma unroll
          for (int i = 4 * rt; i < 4 * rt + 4; ++i) load_k(ksrc, ko, i);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      float p[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i >> 2][rt][i & 3], P.scale_log2, -m_run[rt]));
        l_run[rt] += p[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) pb[rt][i] = pack_bf16(p[2 * i], p[2 * i + 1]);
      // the softmax is complete here: left alone, the compiler sinks its sums
      // and packs past the wait and holds all 32 probabilities over PV
      asm volatile("" : "+v"(l_run[rt]), "+v"(pb[rt][0]), "+v"(pb[rt][1]), "+v"(pb[rt][2]), "+v"(pb[rt][3]));
    }
    __builtin_amdgcn_sched_barrier(0);
    // V landed; the kLoads younger loads (the next K) may be in flight
    if (has_next) wait_vmcnt<L::kLoads>();
    else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    // O^T += V^T P^T; lane (channel 16 dt + c16, group g) takes keys 4 g + 0..3
    // and 16 + 4 g + 0..3 through two transposing reads
    const uint32_t vr = here(va);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const unsigned char* at = tv + (vr ^ (uint32_t)(32 * dt));
      const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS v4i16*)(at));
      const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS v4i16*)(at + 16 * L::kRow));
      const bf16x8 av = __builtin_bit_cast(
          bf16x8, (short __attribute__((ext_vector_type(8)))){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
#pragma unroll
      for (int rt = 0; rt < 4; ++rt) {
        const bf16x8 bp = as_bf16x8(make_uint4(pb[rt][0], pb[rt][1], pb[rt][2], pb[rt][3]));
        acc_o[dt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bp, acc_o[dt][rt], 0, 0, 0);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the V half tile is read
  };

  // this wave's entries: e = w >> 1, + NP, ...; the diagonal, if listed, is entry n - 1
  {
    if (e < n) {
      bool first = true;
      for (; e < n_rot; e += NP) {
        const int nxt = __builtin_amdgcn_readfirstlane(raw);
        if (e + 2 * NP < n) raw = listed_raw(e + 2 * NP);
        step(first, cur, e + NP < n, nxt, std::false_type{});
        cur = nxt;
        first = false;
      }
      if (e < n) step(first, cur, false, 0, std::true_type{});   // e == n - 1, the diagonal
    }
  }

  // ---- merge the waves and normalise -----------------------------------------
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    const float l = rows_sum(l_run[rt]);
    if (g == 0) s_ml[w][16 * rt + c16] = make_float2(m_run[rt], l);
  }
  __syncthreads();
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    float2 ml[NWV];
    float M = kNoMax;
#pragma unroll
    for (int v = 0; v < NWV; ++v) {
      ml[v] = s_ml[v][16 * rt + c16];
      M = fmaxf(M, ml[v].x);
    }
    float l = 0.f;
#pragma unroll
    for (int v = 0; v < NWV; ++v) l += ml[v].y * __builtin_amdgcn_exp2f(ml[v].x - M);
    // (l is 0 for a row whose every score is -inf: NaN, as its softmax is)
    const float f = __builtin_amdgcn_exp2f(m_run[rt] - M) * (l != 0.f ? 1.0f / l : __builtin_nanf(""));
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc_o[dt][rt][i] *= f;
  }
  // Sums over the waves.  First exchange, partner w ^ 1: the wave keeps rows
  // 32 (w & 1) .. + 31 and hands over the others.  A wave's tile area is its
  // own until the first barrier.
  f32x4* mine = reinterpret_cast<f32x4*>(s_tile[w]);
  const bool odd = (w & 1) != 0;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r2 = 0; r2 < 2; ++r2) mine[(dt * 2 + r2) * 64 + lane] = pick(odd, acc_o[dt][r2], acc_o[dt][2 + r2]);
  __syncthreads();
  const f32x4* other = reinterpret_cast<const f32x4*>(s_tile[w ^ 1]);
  f32x4 o[DT][2];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r2 = 0; r2 < 2; ++r2)
      o[dt][r2] = pick(odd, acc_o[dt][2 + r2], acc_o[dt][r2]) + other[(dt * 2 + r2) * 64 + lane];
  // second exchange with four waves, partner w ^ 2: half of the channels
  constexpr int DH = NWV == 4 ? DT / 2 : DT;   // channel tiles stored per wave
  const bool up = NWV == 4 && (w >> 1) != 0;
  if constexpr (NWV == 4) {
    __syncthreads();
#pragma unroll
    for (int d0 = 0; d0 < DH; ++d0)
#pragma unroll
      for (int r2 = 0; r2 < 2; ++r2) mine[(d0 * 2 + r2) * 64 + lane] = pick(up, o[d0][r2], o[DH + d0][r2]);
    __syncthreads();
    const f32x4* far = reinterpret_cast<const f32x4*>(s_tile[w ^ 2]);
#pragma unroll
    for (int d0 = 0; d0 < DH; ++d0)
#pragma unroll
      for (int r2 = 0; r2 < 2; ++r2)
        o[d0][r2] = pick(up, o[DH + d0][r2], o[d0][r2]) + far[(d0 * 2 + r2) * 64 + lane];
  }
  // 16-byte stores: a swap between 16-lane rows gathers 8 consecutive channels
  // on a lane (of tile d0 on the even rows, of tile d0 + 1 on the odd ones)
#pragma unroll
  for (int r2 = 0; r2 < 2; ++r2) {
    uint16_t* orow = P.O + (qo_base + 32 * (w & 1) + 16 * r2 + c16) * D + (up ? DH * 16 : 0);
#pragma unroll
    for (int d0 = 0; d0 < DH; d0 += 2) {
      const f32x4 a = o[d0][r2], b = o[d0 + 1][r2];
      const auto x = __builtin_amdgcn_permlane16_swap(pack_bf16(a[0], a[1]), pack_bf16(b[0], b[1]), false, false);
      const auto y = __builtin_amdgcn_permlane16_swap(pack_bf16(a[2], a[3]), pack_bf16(b[2], b[3]), false, false);
      *reinterpret_cast<uint4*>(orow + 16 * (d0 + (g & 1)) + 4 * (g & 2)) = make_uint4(x[0], y[0], x[1], y[1]);
    }
  }
}

template <int D, int MODE, int NWV>
hipError_t launch_w(AttnParams P, hipStream_t stream) {
  const size_t smem = list_bytes(P);
  constexpr auto kernel = attend_keys_kernel<D, MODE, NWV>;
  const hipError_t e = xcd_concurrency<kernel, NWV * 2 * Half<D>::kBytes >= 65536>(64 * NWV, smem, &P.conc);
  if (e != hipSuccess) return e;
  kernel<<<P.order.grid, 64 * NWV, smem, stream>>>(P);
  return hipGetLastError();
}

// Waves of a CU that the LDS of the units leaves resident (at most what the
// registers do): static part of the kernel (half tiles, (max, sum) pairs, query
// tiles, two counters) and the list, in granules of 1280 bytes out of 160 KiB.
template <int D, int NWV>
int lds_waves(const AttnParams& P) {
  constexpr size_t fixed = NWV * (2 * Half<D>::kBytes + kBlock * sizeof(float2)) + (D == 128 ? 16 * Half<D>::kRow : 0) + 8;
  const size_t granules = (fixed + list_bytes(P) + 1279) / 1280;
  const int units = (int)(163840 / 1280 / granules);
  return units * NWV < 4 * kWaves<D> ? units * NWV : 4 * kWaves<D>;
}

// Waves per unit.  Two fill the chip with the most units at once (d 128: 1024
// on 256 CUs, d 64: 1536); four halve a unit's serial chain at half as many,
// for a second merge round and the query rows read by two more waves.  So four
// where they still hold every unit at once, and, up to a few rounds of units,
// where a unit visits enough blocks to pay for the longer ends; the expected
// blocks come from the budget.  A short list that is as long as most others (few
// tiles expand) leaves no long chain to halve: two there, unless they would leave
// most of a second round empty.  Measured with two / four waves (us):
//   d 128   256 units of 16 blocks      39.1 / 26.3     928 units of 7       24.6 / 32.3
//           912 units of 26             89.2 / 71.8    2048 units of 35       188 / 162
//           900 of 10 (32 at most)     60.0 / 53.0
//          2048 of 17.6 (32)            93.9 / 96.8    2048 of 13            77.0 / 83.1
//          1792 of 17.6 (32)            86.5 / 85.9    3584 of 25             187 / 198
//          3568 of 46 (66)               351 / 357     5200 of 53 (96)        715 / 689
//     no tile expands (rho 1, or few):
//          1024 of 11 (16)              37.5 / 43.0    1024 of 24            48.4 / 52.7
//           892 of 24                   51.0 / 59.9    2240 of 24             104 / 121
//          1200 of 24, 600 tiles        91.2 / 82.3    1120 of 24, 40 tiles  52.4 / 60.6
//   d 64    448 units of 10             28.3 / 18.7    4368 units of 5       42.1 / 57.8
//          4048 units of 28              178 / 161    65536 units of 70      5690 / 5840
//          1024 of 11 (16)              24.6 / 28.3     892 of 24             33.6 / 38.0
//           640 of 4 (6)                13.4 / 14.4
// The choice depends on the problem alone, so ugbs_attend and
// ugbs_attend_select take the same kernel and agree bit for bit.
//
// Bitmaps don't say how many blocks they hold, and their list is as long as the
// sequence.  Four waves where the LDS leaves two-wave units short (at d 128 above
// 1532 blocks: 1600 blocks, 16/4 heads, 37.2 / 34.6 ms).  Else two from about
// where the units outnumber what is resident, as for lists; later at d 64, and
// for the short sequences at d 128 whose unions hold most of what is visible.
// Unions of per-row selections, two / four waves (us):
//   d 128   2048 units, 64 blocks (k 4)       127 / 120     3200, 100 (k 4)     222 / 221
//           2400 units, 300 blocks (k 16)     693 / 733    14336, 512 (k 32)   5620 / 6090
//   d 64    6400 units, 200 blocks (k 16)     658 / 612     8400, 300 (k 16)   1343 / 1345
//          14336 units, 512 blocks (k 32)    3940 / 4050
// and with random bitmaps of few blocks, d 128: 3200 units of 3, 54 / 81.
template <int D, int MODE>
bool four_waves(const AttnParams& P) {
  const int n_units = P.s.B * P.s.H * P.s.T;
  if (lds_waves<D, 4>(P) > lds_waves<D, 2>(P)) return true;
  if (MODE == kBitmap) return n_units <= (D == 64 ? 7680 : P.s.NB < 96 ? 2560 : 1024);
  if (n_units <= (D == 64 && P.longest > 6.0 ? 768 : 512)) return true;
  const double mean = mean_blocks(P);
  if (P.expected < 32.0 && P.longest < 1.3 * (mean + 4.0)) {
    const bool second_round_short = n_units > 1024 && n_units <= 1536 && mean > 0.9 * P.expected;
    if (D == 64 ? n_units <= 1152 : !second_round_short) return false;
  }
  return n_units <= 6144 && n_units <= (D == 64 ? 200.0 : n_units <= 1536 || P.s.G < 4 ? 160.0 : 140.0) * (P.expected - 4.0);
}

template <int D, int MODE>
hipError_t launch_d(const AttnParams& P, hipStream_t stream) {
  return four_waves<D, MODE>(P) ? launch_w<D, MODE, 4>(P, stream) : launch_w<D, MODE, 2>(P, stream);
}

}  // namespace

hipError_t launch_attend_keys(const AttnParams& P, int mode, hipStream_t stream) {
  if (P.s.d == 128) {
    switch (mode) {
      case kLists: return launch_d<128, kLists>(P, stream);
      case kSelect: return launch_d<128, kSelect>(P, stream);
      case kSelectWide: return launch_d<128, kSelectWide>(P, stream);
      default: return launch_d<128, kBitmap>(P, stream);
    }
  }
  switch (mode) {
    case kLists: return launch_d<64, kLists>(P, stream);
    case kSelect: return launch_d<64, kSelect>(P, stream);
    case kSelectWide: return launch_d<64, kSelectWide>(P, stream);
    default: return launch_d<64, kBitmap>(P, stream);
  }
}

}  // namespace ugbs
