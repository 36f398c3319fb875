// Stage 4: head mean of sigma, per-layer quantile trigger and padded
// expansion (A.7-A.9; Eq. (trigger)).
//
// The quantile couples every tile of a sequence, so this is the pipeline's
// one device-wide step.  sigma_bar[t] is the fp32 sum over heads in head order,
// divided by H; the n_trig-th smallest sigma_bar of the population is found by
// a radix descent on its bit pattern (sigma_bar >= 0, so that is order
// preserving); trigger[t] is (t in P) and sigma_bar[t] <= tau; slots k..W-1 of
// the kv_idx rows of tiles that do not trigger become the sentinel N_B.
// n_pop and n_trig = ceil(q n_pop) depend only on N, k and q and are
// computed on the host, so no device-to-host synchronisation is needed.
#include <mutex>
#include <type_traits>

#include "select_common.h"

namespace ugbs {
namespace {

constexpr int kStatsThreads = 1024;

__device__ __forceinline__ bool in_population(int t, int k) {
  const int nf = (t == 0) ? 1 : 2;
  const int nc = (t >= 1) ? t - 1 : 0;
  return nc > k - nf;
}

struct RouteParams {
  Shape s;
  int n_trig;
  const float* sigma;
  const int32_t* idx_sorted;
  int32_t* kv_idx;
  float* sigma_bar;   // optional user copy
  float* tau;         // optional user copy
  uint8_t* trigger;   // optional user copy
  float* ws_sigma_bar;
  float* ws_tau;
  uint8_t* ws_trigger;
};

template <int V>
__device__ __forceinline__ void load_slots(const int32_t* p, int32_t (&v)[V]) {
  if constexpr (V == 4) {
    const int4 x = *reinterpret_cast<const int4*>(p);
    v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
  } else {
    v[0] = *p;
  }
}
template <int V>
__device__ __forceinline__ void store_slots(int32_t* p, const int32_t (&v)[V]) {
  if constexpr (V == 4)
    *reinterpret_cast<int4*>(p) = make_int4(v[0], v[1], v[2], v[3]);
  else
    *p = v[0];
}

// The n-th smallest (1 <= n <= T) of the T keys in s_key by the whole workgroup,
// the same value as nth_smallest: a radix descent by digits of four bits, one
// barrier each.  A wave counts its threads' keys with ballots (LDS atomics took 15
// us longer where all sigmas are equal, as at k 3).  Every thread reads only keys
// that it wrote (tid, tid + kStatsThreads, ..).
__device__ __forceinline__ uint32_t nth_smallest_wide(const uint32_t* s_key, int T, int n,
                                                      uint32_t (*s_hist)[kStatsThreads / 64][16]) {
  constexpr int kPer = UGBS_MAX_BLOCKS / kStatsThreads, kWaves = kStatsThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  uint32_t key[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) key[j] = tid + j * kStatsThreads < T ? s_key[tid + j * kStatsThreads] : 0xffffffffu;
  uint32_t ans = 0;
  int need = n, buf = 0;
  for (int shift = 28; shift >= 0; shift -= 4, buf ^= 1) {
    int mine = 0;   // this wave's keys in play whose digit is lane & 15
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const uint32_t x = (key[j] ^ ans) >> shift;   // below 16: in play, and its digit
      const uint64_t in = __ballot(x < 16u);
      if (in == 0) continue;
      uint64_t m = in;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint64_t one = __ballot((x >> i) & 1u);
        m &= (lane >> i) & 1 ? one : ~one;
      }
      mine += __popcll(m);
    }
    if (lane < 16) s_hist[buf][wv][lane] = (uint32_t)mine;
    __syncthreads();
    int c = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c += (int)s_hist[buf][w][lane & 15];
    int sum = c;   // inclusive, over the digits 0..15
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int y = __shfl_up(sum, o, 16);
      if ((lane & 15) >= o) sum += y;
    }
    const int digit = __ffsll((unsigned long long)__ballot(sum >= need)) - 1;   // the lowest lane is in 0..15
    need -= __shfl(sum - c, digit);
    ans |= (uint32_t)digit << shift;
    if (shift > 0 && need == __shfl(c, digit)) {   // all of this digit: its largest key
      uint32_t m = 0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) m = max(m, ((key[j] ^ ans) >> shift) == 0u ? key[j] : 0u);
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o));
      if (lane == 0) s_hist[buf ^ 1][wv][0] = m;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kWaves; ++w) m = max(m, s_hist[buf ^ 1][w][0]);
      return m;
    }
  }
  return ans;
}

// One launch.  Every workgroup of a sequence (n_wg of them) computes the
// sequence's sigma_bar, tau and flags for itself, out of the L2 and through no
// more than two barriers; the first one stores them, and all of them share the
// kv_idx rows to patch.  Two launches, statistics then patch with 32 barriered
// radix steps, took 12.7 + 3.6 us at 16 tiles, 17.3 + 6.1 us at 512 tiles and 28
// heads, 21.5 + 17.8 us at 2048 tiles and 32 heads. Launches back to back, two
// launches / this one: 14.7 / 7.8, 18.3 / 11.4, 36.3 / 23.6, at 4096 tiles 56 / 37 us.
template <int V>
__global__ void __launch_bounds__(kStatsThreads) route_kernel(RouteParams P, int n_wg, int lg_row, int from, int in_place) {
  __shared__ uint32_t s_key[UGBS_MAX_BLOCKS];
  __shared__ uint32_t s_hist[2][kStatsThreads / 64][16];
  __shared__ float s_tau;
  const Shape& s = P.s;
  const int b = blockIdx.x / n_wg, part = blockIdx.x - b * n_wg;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;

  for (int t = tid; t < s.T; t += kStatsThreads) {
    float sb = -1.0f;
    uint32_t key = 0xffffffffu;
    if (in_population(t, s.k)) {
#pragma clang fp contract(off)
      // fp32 sum in head order; the loads of 16 heads (of 4 where that is all
      // that is left: 2 heads, 4096 tiles, flags: 9.0 -> 7.5 us) are issued together
      // before their adds (the order of the adds is unchanged)
      const float* col = P.sigma + (size_t)b * s.H * s.T + t;
      float acc = 0.0f;
      auto add = [&](auto n_tag, int h0) {
        constexpr int n = decltype(n_tag)::value;
        float v[n];
#pragma unroll
        for (int j = 0; j < n; ++j) v[j] = (h0 + j < s.H) ? col[(size_t)(h0 + j) * s.T] : 0.0f;
#pragma unroll
        for (int j = 0; j < n; ++j)
          if (h0 + j < s.H) acc += v[j];
      };
      int h0 = 0;
      for (; s.H - h0 > 4; h0 += 16) add(std::integral_constant<int, 16>{}, h0);
      if (h0 < s.H) add(std::integral_constant<int, 4>{}, h0);
      sb = __fdiv_rn(acc, (float)s.H);
      if (sb == 0.0f) sb = 0.0f;
      key = __float_as_uint(sb);
    }
    s_key[t] = key;
    if (part == 0) {
      P.ws_sigma_bar[(size_t)b * s.T + t] = sb;
      if (P.sigma_bar) P.sigma_bar[(size_t)b * s.T + t] = sb;
    }
  }
  // The descent by one wave takes steps of T / 64 ballots; above 1024 tiles that is
  // longer than the barriers between 16 waves.  Flags alone, one wave / 16 / the 32
  // barriered steps of one bit of before (us): 512 tiles 7.6 / 8.7 / 12.5, 1024 9.4 /
  // 9.1 / 14.8, 1500 12.6 / 10.5 / 15.5, 2048 15.3 / 11.2 / 17.1, 3000 22.5 / 14.7 /
  // 19.4; where all sigmas are equal 1024 13.3 / 12.2 / 14.6, 2048 20.9 / 14.1 / 17.1.
  const bool wide = s.T > 1024 && P.n_trig > 0;
  const uint32_t nth = wide ? nth_smallest_wide(s_key, s.T, P.n_trig, s_hist) : 0u;
  __syncthreads();
  if (wv == 0) {
    float tau = -1.0f;
    if (wide)
      tau = __uint_as_float(nth);
    else if (P.n_trig > 0)
      tau = __uint_as_float(nth_smallest<1024 / 64>([&](int i) { return s_key[i]; }, s.T, P.n_trig, lane));
    if (lane == 0) s_tau = tau;
  }
  __syncthreads();
  const float tau = s_tau;
  auto triggered = [&](int t) {
    return P.n_trig > 0 && s_key[t] != 0xffffffffu && __uint_as_float(s_key[t]) <= tau;
  };
  if (part == 0) {
    if (tid == 0) {
      P.ws_tau[b] = tau;
      if (P.tau) P.tau[b] = tau;
    }
    for (int t = tid; t < s.T; t += kStatsThreads) {
      const uint8_t trig = triggered(t) ? 1 : 0;
      P.ws_trigger[(size_t)b * s.T + t] = trig;
      if (P.trigger) P.trigger[(size_t)b * s.T + t] = trig;
    }
  }
  if (!P.kv_idx) return;

  // Slots k..W-1 of the rows whose tile does not trigger become the sentinel
  // N_B.  V slots a lane (16-byte accesses), 2^lg_row lanes a row (short rows
  // share a wave), and kBatch rows of every lane in flight together: the copy
  // is bound by the bytes in flight, one workgroup per CU.
  const int per = 64 >> lg_row, sub = lane >> lg_row, first = (lane & ((1 << lg_row) - 1)) * V + from;
  const int n_rows = s.H * s.T;
  const int step = n_wg * (kStatsThreads / 64) * per;
  const size_t base = (size_t)b * n_rows * s.W;
  constexpr int kBatch = 4;
  for (int r0 = (part * (kStatsThreads / 64) + wv) * per + sub; r0 < n_rows; r0 += kBatch * step) {
    for (int slot = first; slot < s.W; slot += V << lg_row) {
      int32_t v[kBatch][V];
      bool trig[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int r = r0 + i * step;
        if (r >= n_rows) break;
        trig[i] = triggered(r % s.T);
        if (in_place || (slot >= s.k && !trig[i])) continue;
        load_slots<V>(P.idx_sorted + base + (size_t)r * s.W + slot, v[i]);
      }
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        const int r = r0 + i * step;
        if (r >= n_rows) break;
        int32_t* dst = P.kv_idx + base + (size_t)r * s.W + slot;
        if (in_place) {
          if (trig[i] || slot + V <= s.k) continue;
          if (slot >= s.k) {   // whole accesses (32 heads, 128 tiles, batch 8, k 128, W 384: 16.3 -> 10.8 us, with no lanes on the kept slots)
#pragma unroll
            for (int e = 0; e < V; ++e) v[i][e] = s.NB;
            store_slots<V>(dst, v[i]);
          } else {
#pragma unroll
            for (int e = 0; e < V; ++e)
              if (slot + e >= s.k) dst[e] = s.NB;
          }
        } else {
#pragma unroll
          for (int e = 0; e < V; ++e)
            if (slot + e >= s.k && !trig[i]) v[i][e] = s.NB;
          store_slots<V>(dst, v[i]);
        }
      }
    }
  }
}

// Route sections (sigma_bar | tau | trigger) of ugbs_route_noalloc, in device
// memory the library owns: one copy of this array per GPU, held until the
// process ends.  Host code must not pass `scratch` itself to a kernel (on the
// host it names a stand-in, not a device address); the per-device address
// comes from hipGetSymbolAddress below.
static __device__ __align__(256) unsigned char scratch[kRouteScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch`, per device

}  // namespace

// Device address of the current device's `scratch`, looked up once per
// device with that device current.
hipError_t route_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_route(const Shape& s, int n_pop, int n_trig, const float* sigma,
                        const int32_t* idx_sorted, int32_t* kv_idx, float* sigma_bar,
                        float* tau, uint8_t* trigger, void* workspace, hipStream_t stream) {
  (void)n_pop;
  RouteParams P;
  P.s = s;
  P.n_trig = n_trig;
  P.sigma = sigma;
  P.idx_sorted = idx_sorted;
  P.kv_idx = kv_idx;
  P.sigma_bar = sigma_bar;
  P.tau = tau;
  P.trigger = trigger;
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  P.ws_sigma_bar = reinterpret_cast<float*>(ws + ws_sigma_bar_off(s));
  P.ws_tau = reinterpret_cast<float*>(ws + ws_tau_off(s));
  P.ws_trigger = ws + ws_trigger_off(s);
  // four slots a lane where rows and pointers are 16-byte aligned
  const bool quad = s.W % 4 == 0 && ((reinterpret_cast<uintptr_t>(idx_sorted) | reinterpret_cast<uintptr_t>(kv_idx)) & 15) == 0;
  const int in_place = idx_sorted == kv_idx ? 1 : 0;
  const int from = !in_place ? 0 : quad ? s.k & ~3 : s.k;   // first slot a lane takes
  const int lanes = (s.W - from) / (quad ? 4 : 1);
  int lg_row = 0;
  while (lg_row < 6 && (1 << lg_row) < lanes) ++lg_row;
  // at least four rows per lane, and no more workgroups than CUs
  const long per_wg = 4l * (kStatsThreads >> lg_row);
  const long rounds = kv_idx ? ((long)s.H * s.T + per_wg - 1) / per_wg : 1;
  const long most = s.B < 256 ? 256 / s.B : 1;
  const int n_wg = (int)(rounds < most ? rounds : most);
  if (quad)
    route_kernel<4><<<(unsigned)(s.B * n_wg), kStatsThreads, 0, stream>>>(P, n_wg, lg_row, from, in_place);
  else
    route_kernel<1><<<(unsigned)(s.B * n_wg), kStatsThreads, 0, stream>>>(P, n_wg, lg_row, from, in_place);
  return hipGetLastError();
}

}  // namespace ugbs
