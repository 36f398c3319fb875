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

// One launch.  Every workgroup of a sequence (n_wg of them) computes the
// sequence's sigma_bar, tau and flags for itself, out of the L2 and through no
// more than two barriers; the first one stores them, and all of them share the
// kv_idx rows to patch.  Two launches, statistics then patch with 32 barriered
// radix steps, took 12.7 + 3.6 us at 16 tiles, 17.3 + 6.1 us at 512 tiles and 28
// heads, 21.5 + 17.8 us at 2048 tiles and 32 heads. Launches back to back, two
// launches / this one: 14.3 / 7.0, 18.0 / 12.7, 37.1 / 32.3, at 4096 tiles 57 / 50 us.
template <int V>
__global__ void __launch_bounds__(kStatsThreads) route_kernel(RouteParams P, int n_wg, int lg_row, int in_place) {
  __shared__ uint32_t s_key[UGBS_MAX_BLOCKS];
  __shared__ float s_tau;
  const Shape& s = P.s;
  const int b = blockIdx.x / n_wg, part = blockIdx.x - b * n_wg;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;

  for (int t = tid; t < s.T; t += kStatsThreads) {
    float sb = -1.0f;
    uint32_t key = 0xffffffffu;
    if (in_population(t, s.k)) {
#pragma clang fp contract(off)
      // fp32 sum in head order; the loads of 16 heads are issued together
      // before their adds (the order of the adds is unchanged)
      const float* col = P.sigma + (size_t)b * s.H * s.T + t;
      float acc = 0.0f;
      for (int h0 = 0; h0 < s.H; h0 += 16) {
        float v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = (h0 + j < s.H) ? col[(size_t)(h0 + j) * s.T] : 0.0f;
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (h0 + j < s.H) acc += v[j];
      }
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
  __syncthreads();
  if (wv == 0) {
    const float tau = P.n_trig > 0 ? __uint_as_float(nth_smallest<UGBS_MAX_BLOCKS / 64>([&](int i) { return s_key[i]; }, s.T, P.n_trig, lane)) : -1.0f;
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
  const int per = 64 >> lg_row, sub = lane >> lg_row, first = (lane & ((1 << lg_row) - 1)) * V;
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
#pragma unroll
          for (int e = 0; e < V; ++e)
            if (slot + e >= s.k) dst[e] = s.NB;
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
  const int lanes = quad ? s.W / 4 : s.W;
  int lg_row = 0;
  while (lg_row < 6 && (1 << lg_row) < lanes) ++lg_row;
  // at least four rows per lane, and no more workgroups than CUs
  const long per_wg = 4l * (kStatsThreads >> lg_row);
  const long rounds = kv_idx ? ((long)s.H * s.T + per_wg - 1) / per_wg : 1;
  const long most = s.B < 256 ? 256 / s.B : 1;
  const int n_wg = (int)(rounds < most ? rounds : most);
  const int in_place = idx_sorted == kv_idx ? 1 : 0;
  if (quad)
    route_kernel<4><<<(unsigned)(s.B * n_wg), kStatsThreads, 0, stream>>>(P, n_wg, lg_row, in_place);
  else
    route_kernel<1><<<(unsigned)(s.B * n_wg), kStatsThreads, 0, stream>>>(P, n_wg, lg_row, in_place);
  return hipGetLastError();
}

}  // namespace ugbs
