// Stage 5 at d 256, at d 128 where the walk is bound beyond the L2 (coupled_walk),
// and at d 64 and 128 for few short lists (few_short_lists); attend_keys.hip: the
// rest of d 64 and 128.  Block-sparse causal attention over kv_idx, a bitmap, or an in-kernel selection (A.10; Eq. (Attn)).
//
// One workgroup per (batch, query head, Q-tile) unit: four waves of 16 query
// rows (d 64 and 128: two of 32); a wave owns its rows for every key of a block.  The
// tile's kept blocks are first turned into an ascending list of distinct blocks
// in 0..t (so the diagonal block comes last), then visited one by one.
// (Splitting the keys over the waves instead, as attend_keys.hip does, needs all
// 64 rows' accumulators in every wave: 256 registers at d 256.)
//
// Staging.  K and V blocks (64 keys x d, bf16) go global -> LDS with
// direct-to-LDS loads (global_load_lds_dwordx4: no registers, no VALU).
// Both live unpadded in natural [key][d] layout with the 16-byte columns of
// each row permuted by an XOR swizzle (column c of row r of K at c ^ (r mod
// d/8), of V at c ^ (2r mod d/8)), chosen so that the K-operand reads and the
// transposing V reads below are free of LDS bank conflicts.  K and V have one
// buffer each and are refilled in a split ping-pong: K(i+1) is fetched as
// soon as all waves have finished S(i), V(i+1) as soon as all have
// finished PV(i), so the fetches overlap the softmax and the other matrix
// product.
//
// Compute, per block and wave (v_mfma_f32_16x16x32_bf16):
//   S^T = K Q^T   K rows from LDS (ds_read_b128) are the A operand; the
//                 wave's query rows stay in registers as the B operand;
//                 each lane ends up holding 16 keys of one query row.  S of
//                 the next block is issued together with the softmax of the
//                 current one, so the matrix cores and the VALU overlap.
//   softmax       fp32 online softmax in base 2 (log2 e folded into the
//                 scale); only the diagonal block t is masked (key > row);
//                 the reference max is raised only when a row max exceeds
//                 it by more than 2^8, so O is rarely rescaled.
//   O^T += V^T P^T  the lane's probabilities, packed to bf16, already are
//                 the B operand; V^T comes straight from the natural-layout
//                 LDS tile through the transposing read ds_read_b64_tr_b16
//                 (16 lanes fetch a 4-key x 16-channel patch and each lane
//                 receives the 4 keys of one channel).
// Per listed block and unit: 4*64*64*d FLOP on 2*64*d*2 bytes of K/V.
#include "attend_list.h"

namespace ugbs {
namespace {

// Waves per unit and 16-row tiles per wave: d 64 and 128 run two waves of 32
// query rows, d 256 four waves of 16 (half the accumulators per wave).  Two waves
// per SIMD at each.
template <int D>
struct Geo {
  static constexpr int RT = D > 128 ? 1 : 2;   // 16-row tiles per wave
  static constexpr int NWV = 4 / RT;           // waves per unit (64 rows)
  static constexpr int kThreads = 64 * NWV;
};

template <int D, int MODE>
__global__ void __launch_bounds__(Geo<D>::kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
attend_kernel(AttnParams P) {
  using L = TileGeom<D>;
  constexpr int NWV = Geo<D>::NWV, kThreads = Geo<D>::kThreads;
  constexpr int RT = Geo<D>::RT;
  constexpr int RPW = 16 * RT;    // query rows per wave
  constexpr int KS = D / 32;      // k-steps of QK^T
  constexpr int DT = D / 16;      // 16-channel tiles of O^T
  __shared__ __align__(16) uint16_t s_k[L::kElems];
  __shared__ __align__(16) uint16_t s_v[L::kElems];
  extern __shared__ uint16_t s_list[];              // list_bytes
  __shared__ uint32_t s_bits[UGBS_MAX_BLOCKS / 32];
  __shared__ int s_n, s_below;

  const Shape& s = P.s;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, uniform per wave
  const int g = lane >> 4, c16 = lane & 15;
  Unit u;
  if (!attend_unit(s, P.order, &u)) return;
  const int kvh = u.h / s.G;
  const size_t rowid = ((size_t)u.b * s.H + u.h) * s.T + u.t;

  // ---- the tile's kept blocks, ascending (wave 0): kv_idx entries outside
  // 0..t are dropped and repeated entries count once (set semantics, as in
  // Eq. (Attn)), so the diagonal block t, the only one needing the causal
  // mask, is the last entry when present.
  //
  // Visiting order.  The j-th workgroup an XCD receives starts its walk at
  // the first listed block >= (j mod 2 conc) / (2 conc) of its key range and
  // wraps around (the diagonal block stays last).  Workgroups follow each
  // other on an XCD in the order of j, conc of them at a time, so the ones
  // resident together sweep the key range in step and blocks they share
  // stay in that XCD's L2.  Measured at 128K: with kv_idx lists (about 70
  // blocks per tile, or every visible block) a period of 2 conc is best (1
  // and 4 conc slower); with the per-row bitmaps (hundreds of blocks per
  // tile) 1 conc is 9% faster than 2 conc.  The order changes only the
  // summation order of the softmax.
  const int j_xcd = blockIdx.x >> 3;
  const int period = (MODE == kBitmap ? 1 : 2) * P.conc;
  const int start_blk = (int)(((long long)(j_xcd % period) * u.t) / period);
  build_list<MODE, NWV>(P, u, rowid, start_blk, w, lane, reinterpret_cast<uint64_t*>(s_k),
                                reinterpret_cast<uint32_t*>(s_v), s_bits, s_list, &s_n, &s_below);
  __syncthreads();
  const int n = __builtin_amdgcn_readfirstlane(s_n);
  const bool diag_last = n > 0 && s_list[n - 1] == u.t;
  // entries 0..n_rot-1 are visited from position rot0 on, cyclically
  const int n_rot = __builtin_amdgcn_readfirstlane(diag_last ? n - 1 : n);
  const int rot0 = __builtin_amdgcn_readfirstlane(s_below < n_rot ? s_below : 0);
  // listed_raw: the i-th block to visit as a per-lane LDS value (every lane
  // the same); listed: the same, moved to a scalar register
  auto listed_raw = [&](int i) {
    int p = i;
    if (i < n_rot) {
      p = i + rot0;
      if (p >= n_rot) p -= n_rot;
    }
    return s_list[p];
  };
  auto listed = [&](int i) { return __builtin_amdgcn_readfirstlane(listed_raw(i)); };

  const size_t qo_base = ((size_t)u.b * s.H + u.h) * s.N + (size_t)u.t * kBlock;
  if (n == 0) {  // no attended key: O = 0
    for (int i = tid; i < kBlock * D / 8; i += kThreads)
      reinterpret_cast<uint4*>(P.O + qo_base * D)[i] = make_uint4(0, 0, 0, 0);
    return;
  }

  // ---- query rows as the B operand --------------------------------------
  bf16x8 bq[RT][KS];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const uint16_t* qr = P.Q + (qo_base + RPW * w + 16 * rt + c16) * D + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) bq[rt][ks] = as_bf16x8(*reinterpret_cast<const uint4*>(qr + 32 * ks));
  }
  wait_vmcnt<0>();

  const uint16_t* Kh = P.K + ((size_t)u.b * s.Hkv + kvh) * s.N * D;
  const uint16_t* Vh = P.V + ((size_t)u.b * s.Hkv + kvh) * s.N * D;
  const uint32_t k_lds = __builtin_amdgcn_readfirstlane(lds_addr(s_k));
  const uint32_t v_lds = __builtin_amdgcn_readfirstlane(lds_addr(s_v));
  // Who issues a tile's 1 KiB loads.  At d 128 the first wave issues all of a K
  // tile and the last wave all of a V tile, so while one wave waits for the
  // texture unit to accept its loads the other keeps computing (1-2% faster at
  // 32K-128K than each wave issuing half of every tile, same output bits).  At
  // d 256 each wave issues its share: one issuer would need more offset
  // registers than that kernel has.
  constexpr bool kSplitIssue = D <= 128;
  constexpr int kIssuers = kSplitIssue ? 1 : NWV;
  FetchPlanT<D, false, kIssuers> kplan;
  FetchPlanT<D, true, kIssuers> vplan;
  const int iw = kSplitIssue ? 0 : w;             // index within the issuing waves
  kplan.init(lane, iw);
  vplan.init(lane, iw);
  auto fetch_k = [&](int b) {
    if (!kSplitIssue || w == 0) kplan.fetch(Kh + (size_t)b * L::kElems, k_lds, iw);
  };
  auto fetch_v = [&](int b) {
    if (!kSplitIssue || w == NWV - 1) vplan.fetch(Vh + (size_t)b * L::kElems, v_lds, iw);
  };

  f32x4 acc_o[DT][RT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) acc_o[dt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run[RT], l_run[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m_run[rt] = kNoMax;
    l_run[rt] = 0.f;
  }

  // S^T = K Q^T : [64 keys x 16 RT rows] per wave, K from LDS
  auto compute_s = [&](f32x4 (&sc)[4][RT]) {
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) sc[kt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        const int r = 16 * kt + c16;
        const bf16x8 ak = as_bf16x8(*reinterpret_cast<const uint4*>(s_k + L::off(r, 4 * ks + g, false)));
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          sc[kt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak, bq[rt][ks], sc[kt][rt], 0, 0, 0);
      }
    }
  };

  // Pipeline per listed block i (K and V have one LDS buffer each):
  //   S(i+1) on the matrix cores overlaps the softmax of S(i) on the VALU,
  //   then O += P(i) V(i).  K(i+2) is fetched once S(i+1) is done, V(i+1)
  //   once PV(i) is done.  Fetch order per wave: K0 V0 K1 | K2 V1 | K3 V2 ...
  //   Two barriers per block: each one both frees a buffer (all waves done
  //   reading it) and publishes the one load then in flight (V(i) before
  //   PV(i), K(i+2) before the next S), so every wait is for all loads.
  int blk = listed(0);
  fetch_k(blk);
  fetch_v(blk);
  f32x4 sc[4][RT];
  // K0 landed (V0 may still be in flight)
  if constexpr (kSplitIssue) {
    if (w == 0) wait_vmcnt<0>();
  } else {
    wait_vmcnt<L::kLoads / NWV>();
  }
  lds_barrier();
  compute_s(sc);
  wait_lgkm0();
  lds_barrier();                         // all waves are done reading s_k
  // The indices of the next two blocks travel one step ahead: the LDS read
  // of block it + 3 goes out at the end of step it, and its scalar copy is
  // taken where step it + 1 needs it, so no list read waits on the LDS
  // right after a barrier.
  int nb1 = (n > 1) ? listed(1) : 0;     // block it + 1
  int raw2 = (n > 2) ? listed_raw(2) : 0;  // block it + 2, per-lane copy
  if (n > 1) {
    fetch_k(nb1);
    wait_vmcnt<0>();                     // K1 (and V0) landed
    lds_barrier();
  }

  // One pipeline step for listed block `it`; MASK: it is the diagonal block
  // (always the last one), whose keys after the query row are masked.
  auto step = [&](int it, auto mask_tag) {
    constexpr bool MASK = decltype(mask_tag)::value;
    const bool has_next = it + 1 < n;
    const bool has_next2 = it + 2 < n;
    const int nblk = has_next ? nb1 : 0;

    // S(it+1): on the last block this re-reads s_k (no fetch is pending) and is discarded
    f32x4 sn[4][RT];
    __builtin_amdgcn_s_setprio(1);       // matrix-core phases issue ahead of other waves' fetch phases
    compute_s(sn);

    // online softmax of S(it) (base 2); lane holds row (RPW w + 16rt + c16),
    // keys 16kt + 4g + i.  The reference max m_run only moves when a row max
    // exceeds it by more than 2^8, so p <= 256 and O is rescaled rarely.
    if constexpr (MASK) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int r = RPW * w + 16 * rt + c16;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((16 * kt + 4 * g + i) > r) sc[kt][rt][i] = -__builtin_huge_valf();
      }
    }
    float alpha[RT];
    uint32_t pb[RT][2][4];
    bool moved = false;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float mx = fmaxf(fmaxf(sc[0][rt][0], sc[0][rt][1]), fmaxf(sc[0][rt][2], sc[0][rt][3]));
#pragma unroll
      for (int kt = 1; kt < 4; ++kt)
        mx = fmaxf(mx, fmaxf(fmaxf(sc[kt][rt][0], sc[kt][rt][1]), fmaxf(sc[kt][rt][2], sc[kt][rt][3])));
      mx = rows_max(mx) * P.scale_log2;
      const bool up = mx > m_run[rt] + 8.0f;
      const float m_new = up ? mx : m_run[rt];
      alpha[rt] = up ? __builtin_amdgcn_exp2f(m_run[rt] - m_new) : 1.0f;
      moved |= up;
      m_run[rt] = m_new;
      float ls = 0.f;
      float p[4][4];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          p[kt][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[kt][rt][i], P.scale_log2, -m_new));
          ls += p[kt][i];
        }
      l_run[rt] = l_run[rt] * alpha[rt] + ls;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        pb[rt][j][0] = pack_bf16(p[2 * j][0], p[2 * j][1]);
        pb[rt][j][1] = pack_bf16(p[2 * j][2], p[2 * j][3]);
        pb[rt][j][2] = pack_bf16(p[2 * j + 1][0], p[2 * j + 1][1]);
        pb[rt][j][3] = pack_bf16(p[2 * j + 1][2], p[2 * j + 1][3]);
      }
    }
    // interleave, in two halves: the K-operand reads, then one MFMA of
    // S(it+1) per few softmax VALU instructions (8 reads, 16 x (1 + 5) at d 128)
    constexpr int kHalfReads = 2 * KS, kHalfMfma = 2 * KS * RT, kVpm = RT == 2 ? 5 : 2;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      __builtin_amdgcn_sched_group_barrier(0x100, kHalfReads, 0);
#pragma unroll
      for (int i = 0; i < kHalfMfma; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, kVpm, 0);
      }
    }

    // the whole softmax stays above the barrier, where it overlaps the
    // landing of V(it)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    // one barrier: every wave is done reading s_k, and V(it), the only load
    // in flight, has landed
    wait_lgkm0();
    wait_vmcnt<0>();
    lds_barrier();
    if (has_next2) fetch_k(__builtin_amdgcn_readfirstlane(raw2));

    __builtin_amdgcn_s_setprio(1);
    if (__ballot(moved)) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int i = 0; i < 4; ++i) acc_o[dt][rt][i] *= alpha[rt];
    }

    // O^T += V^T P^T ; lane (channel 16dt + c16, group g) takes keys
    // 32j + 4g + 0..3 and 32j + 16 + 4g + 0..3 through two transposing reads
    const int tr_row = 4 * g + (c16 >> 2);
    const int tr_col = (c16 & 3) >> 1, tr_half = (c16 & 1) * 4;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const int r0 = 32 * j + tr_row, r1 = r0 + 16;
        const int c = 2 * dt + tr_col;
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (LDS_AS v4i16*)(s_v + L::off(r0, c, true) + tr_half));
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (LDS_AS v4i16*)(s_v + L::off(r1, c, true) + tr_half));
        const bf16x8 av = __builtin_bit_cast(
            bf16x8, (short __attribute__((ext_vector_type(8)))){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const bf16x8 bp = as_bf16x8(make_uint4(pb[rt][j][0], pb[rt][j][1], pb[rt][j][2], pb[rt][j][3]));
          acc_o[dt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bp, acc_o[dt][rt], 0, 0, 0);
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    if (has_next) {
      // one barrier: every wave is done reading s_v, and K(it+2), the only
      // load in flight (if any), has landed for the next step's S
      wait_lgkm0();
      wait_vmcnt<0>();
      lds_barrier();
      fetch_v(nblk);
    }
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) sc[kt][rt] = sn[kt][rt];
    nb1 = __builtin_amdgcn_readfirstlane(raw2);
    raw2 = (it + 3 < n) ? listed_raw(it + 3) : 0;
  };

  for (int it = 0; it + 1 < n; ++it) step(it, std::false_type{});
  if (diag_last) step(n - 1, std::true_type{});
  else step(n - 1, std::false_type{});

  // ---- normalise and store: lane holds O^T[16dt + 4g + i][row] ------------
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float l = l_run[rt];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    // (l is 0 for a row whose every score is -inf: NaN, as its softmax is)
    const float inv = l != 0.f ? 1.0f / l : __builtin_nanf("");
    const int r = RPW * w + 16 * rt + c16;
    uint16_t* orow = P.O + (qo_base + r) * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const f32x4 a = acc_o[dt][rt];
      *reinterpret_cast<uint2*>(orow + 16 * dt + 4 * g) =
          make_uint2(pack_bf16(a[0] * inv, a[1] * inv), pack_bf16(a[2] * inv, a[3] * inv));
    }
  }
}

template <int D, int MODE>
hipError_t launch_t(AttnParams P, hipStream_t stream) {
  const size_t smem = list_bytes(P);
  constexpr auto kernel = attend_kernel<D, MODE>;
  const hipError_t e = xcd_concurrency<kernel, (D > 128)>(Geo<D>::kThreads, smem, &P.conc);
  if (e != hipSuccess) return e;
  kernel<<<P.order.grid, Geo<D>::kThreads, smem, stream>>>(P);
  return hipGetLastError();
}

// d 128 lists: true where the units' walks are bound by what misses the L2.  The
// kernel here keeps a unit's waves on one block between barriers, so a unit that
// has to wait for a block waits whole, the units behind it on that XCD catch up,
// and the blocks they share are fetched once more often: L2 hits .59 against .45
// of attend_keys.hip's independent waves at 2048 blocks (14/2 heads, k 256, q
// 0.1), with 7 TB/s beyond the L2 either way.  Where the L2 isn't the bound those
// waves are faster.  Two things take a list there: long sequences, whose range
// of blocks is far larger than an L2 (4 MB: 128 blocks of K and V), and many
// blocks per list; K-mean scores, which spread a tile's blocks more than the
// Quest bound does, at any budget.  Measured (ms, here / attend_keys.hip):
//   Quest, q 0.1    1500 blocks   k 256, 14/2 heads   12.1 / 11.1
//                   2048          k 64, 32/8          10.6 / 10.0    k 256, 14/2   17.5 / 19.2
//                   3000          k 64, 32/8          16.3 / 16.0    k 96, 14/2    10.4 / 11.0
//                   4096          k 64, 32/8          23.5 / 23.5    k 128, 14/2   22.3 / 22.8
//   K-mean, q 0.1   1200          k 64, 14/2          2.79 / 2.68
//                   1500          k 64, 14/2          3.68 / 3.99
//                   2048          k 33, 14/2          3.06 / 3.15    k 256, 14/2   21.9 / 24.3
//   every block     1400, 32/8    75 / 75      2048   171 / 211     4096, 16/4   391 / 476
// The choice depends on the problem and the list's width alone, so ugbs_attend
// and ugbs_attend_select take the same kernel and agree bit for bit.
inline bool coupled_walk(const AttnParams& P) {
  return P.s.NB >= 1408 && (P.s.backbone == UGBS_KMEAN || P.expected * P.s.NB >= 300000.0);
}

// d 64 and 128 lists of three or four blocks where the units are few: the merge of
// attend_keys.hip's waves is longer than the half blocks they save.  Measured (us,
// here / two / four waves there):
//   d 128   64 units of 3 blocks    9.1 / 9.7 / 10.9    512 of 3    12.2 / 13.3 / 15.5
//           64 of 4.2, 6 at most   12.8 / 13.1 / 12.2  1024 of 3    17.4 / 17.9 / 27.8
//   d 64    64 of 3                 7.1 / 7.2 / 7.9     512 of 3     8.9 / 9.6 / 10.7
//           1024 of 3              10.8 / 11.4 / 17.6  1120 of 3    15.8 / 13.2 / 18.8
inline bool few_short_lists(const AttnParams& P) {
  return P.longest <= 4.0 && P.s.B * P.s.H * P.s.T <= 1024;
}

template <int MODE>
hipError_t launch_mode(const AttnParams& P, hipStream_t stream) {
  if (P.s.d == 256) return launch_t<256, MODE>(P, stream);
  if constexpr (MODE != kBitmap)
    if (P.s.d == 128 && (coupled_walk(P) || few_short_lists(P))) return launch_t<128, MODE>(P, stream);
  if constexpr (MODE == kLists || MODE == kSelect)
    if (P.s.d == 64 && few_short_lists(P)) return launch_t<64, MODE>(P, stream);
  return launch_attend_keys(P, MODE, stream);
}

}  // namespace

hipError_t launch_attend(const Shape& s, const uint16_t* Q, const uint16_t* K,
                         const uint16_t* V, const int32_t* kv_idx, int kv_width,
                         uint16_t* O, hipStream_t stream) {
  AttnParams P{};
  P.s = s;
  P.order = attend_order(s);
  P.Q = Q;
  P.K = K;
  P.V = V;
  P.kv_idx = kv_idx;
  P.O = O;
  P.kv_width = kv_width;
  P.expected = expected_blocks(s, kv_width);
  P.longest = longest_list(s, kv_width);
  P.scale_log2 = s.scale * 1.4426950408889634f;
  return launch_mode<kLists>(P, stream);
}

hipError_t launch_attend_select(const Shape& s, const uint16_t* Q, const uint16_t* K,
                                const uint16_t* V, const float* scores, const uint8_t* trigger,
                                const void* workspace, uint16_t* O, hipStream_t stream) {
  AttnParams P{};
  P.s = s;
  P.order = attend_order(s);
  P.Q = Q;
  P.K = K;
  P.V = V;
  P.O = O;
  // at most |F| + (rho k - |F|) distinct blocks per tile, and never more than t + 1
  P.kv_width = s.W < s.NB ? s.W : s.NB;
  P.expected = expected_blocks(s, s.W);
  P.longest = longest_list(s, s.W);
  P.scale_log2 = s.scale * 1.4426950408889634f;
  const unsigned char* ws = static_cast<const unsigned char*>(workspace);
  P.sel_scores = scores;
  P.sel_packed = ws ? reinterpret_cast<const float*>(ws + ws_scores_off(s)) : nullptr;
  P.sel_trigger = trigger ? trigger : ws + ws_trigger_off(s);
  return s.NB > 32 * 64 ? launch_mode<kSelectWide>(P, stream) : launch_mode<kSelect>(P, stream);
}

hipError_t launch_attend_bitmap(const Shape& s, const uint16_t* Q, const uint16_t* K,
                                const uint16_t* V, const uint32_t* bitmap, uint16_t* O,
                                hipStream_t stream) {
  AttnParams P{};
  P.s = s;
  P.order = attend_order(s);
  P.Q = Q;
  P.K = K;
  P.V = V;
  P.O = O;
  P.kv_width = s.NB;  // a row may list every visible block
  P.expected = P.longest = s.NB;
  P.scale_log2 = s.scale * 1.4426950408889634f;
  P.bitmap = bitmap;
  P.nw = (s.NB + 31) / 32;
  return launch_mode<kBitmap>(P, stream);
}

}  // namespace ugbs
