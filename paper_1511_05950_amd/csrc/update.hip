// Fused sumGradients + applyUpdate kernel (Section 2.1 server steps; n-softsync rule of
// Section 2.2 with the per-gradient learning rate of Section 2.4).
//
// One streaming pass over the parameter vector:
//     s      = sum_{l=0}^{c-1} coef_l * g_l            (arrival order, fp32 FMA chain)
//     v'     = m * v + s + decay * theta_i              decay = (sum_l coef_l) * wd
//     theta' = theta_i - v'
// Reads c gradients, theta_i and v once, writes theta_{i+1} and v once (plus an optional bf16
// copy of theta_{i+1}): 4 (c + 4) bytes per parameter, nothing else touches HBM.  The kernel is
// bandwidth bound (latency bound below a million parameters); each lane moves 16-byte vectors,
// gradients are read with non-temporal loads because they are never read again.
//
// Long windows over long vectors (two_pass_update) take the same arithmetic in two launches per stretch of kSumStretch parameters:
// sum_gradients_kernel writes s for the stretch to a small buffer, apply_update_kernel then runs on the stretch with
// that buffer as its one "gradient" of coefficient 1 (fma(1, s, 0) = s: the result is bit-identical).  A pass that
// only reads streams c gradients at the rate of a pure read (7.07 TB/s measured); in the single pass the two written
// streams are interleaved with the c read ones all the time.  The
// buffer is 8 MiB and is read back right after it was written (it passes the L2s' memory interface both ways, 8 bytes
// per parameter of counted traffic, and fits the memory-side cache many times over).  The line, from one pass against two over
// P = 4 M .. 62 M: from 48 gradients on two passes are the faster form everywhere (P = 62 M with a bf16 copy c = 48 2 055 against
// 2 212 us, c = 54 2 266 against 2 431; P = 10 M c = 54 365 against 380; P = 4 M c = 48 133 against 134), up to 32 one pass is
// (P = 17 M, c = 32: 399 against 433), and between them they differ by up to 4 % either way: two passes win beyond 32 M
// parameters (P = 62 M, c = 40: 1 804 against 1 859), one pass below (17 M: by 3 %).
// The second pass keeps the shape of the first, blocks of 256 lanes with four pieces each, and reads the sums with ordinary loads:
// c = 54 behind c = 1 updates of 60 M parameters 2 175 us, against 2 228 with one-wavefront workgroups of two pieces, 2 226 with
// four pieces, 2 224 with two pieces a lane in blocks of 256, and 2 265 with ordinary loads of theta and v.
#include "ctx.hpp"
#include "dev_common.hpp"

#include <string.h>

#include <algorithm>
#include <mutex>

namespace sasgd {

// Buffer of partial sums for callers that may not allocate (sasgd_applyUpdateNoAlloc): one stretch of the two-pass
// form, 8 MiB per device, held from the library's load until the process ends.  Host code never passes this name to a
// kernel: it is a host-side stand-in, the device address comes from hipGetSymbolAddress (static_sum_buffer below).
static __device__ __align__(256) float scratch[kSumStretch];

constexpr int kMaxDevices = 64;
static float* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;

hipError_t static_sum_buffer(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // this device's copy of the array (the current device's)
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

struct GradTable {
  const float* g[kMaxLearners];
  float coef[kMaxLearners];
};

typedef float float4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 ldg_nt(const float4* p) {
  const float4v r = __builtin_nontemporal_load(reinterpret_cast<const float4v*>(p));
  return make_float4(r.x, r.y, r.z, r.w);
}
__device__ __forceinline__ void stg_nt(float4* p, float4 v) {
  const float4v r = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(r, reinterpret_cast<float4v*>(p));
}
__device__ __forceinline__ uint2 pack_bf4(float4 a) {
  uint2 o;
  o.x = pack2bf(a.x, a.y);
  o.y = pack2bf(a.z, a.w);
  return o;
}
__device__ __forceinline__ void fma4(float4& s, float cf, const float4& g) {
  s.x = fmaf(cf, g.x, s.x);
  s.y = fmaf(cf, g.y, s.y);
  s.z = fmaf(cf, g.z, s.z);
  s.w = fmaf(cf, g.w, s.w);
}
// v' = m v + s + decay theta, theta' = theta - v': the one place the four-wide update is written down
__device__ __forceinline__ void update4(float4& a, float4& b, const float4& s, float m, float decay) {
  b.x = fmaf(m, b.x, s.x) + decay * a.x;
  b.y = fmaf(m, b.y, s.y) + decay * a.y;
  b.z = fmaf(m, b.z, s.z) + decay * a.z;
  b.w = fmaf(m, b.w, s.w) + decay * a.w;
  a.x -= b.x;
  a.y -= b.y;
  a.z -= b.z;
  a.w -= b.w;
}

// sum_l coef_l g_l of one element over gradients [begin, end), U loads in flight: the chain of fma4 in the same order.
template <int U>
__device__ __forceinline__ float sum_element(const GradTable& t, int begin, int end, int64_t k) {
  float s = 0.f;
  for (int l = begin; l < end; l += U) {
    float g[U];
#pragma unroll
    for (int u = 0; u < U; u++)
      if (l + u < end) g[u] = t.g[l + u][k];
#pragma unroll
    for (int u = 0; u < U; u++)
      if (l + u < end) s = fmaf(t.coef[l + u], g[u], s);
  }
  return s;
}

// One-wavefront workgroups, ILP pieces of 16 bytes per lane and stream, U gradients in flight.  Two things decide the rate:
// the loads a lane has outstanding (a window's gradients are requested U at a time, the rest of the window in one go as
// well), and how many lanes are resident at once.  Fewer resident wavefronts with more loads each keep the c + 2 streams
// more sequential in DRAM: the launcher bounds the residency by giving a workgroup LDS that it never touches (10 wavefronts
// per compute unit at 16 KiB, 8 at 20 KiB).  Measured at P = 62 M with the bf16 copy against blocks of 256 lanes with four
// pieces and three gradients each: c = 18 1 046 -> 875 us (5.4 -> 6.4 TB/s), c = 8 574 -> 459 us, c = 1 249 -> 193 us; at
// P = 89 578, c = 30 18 -> 6 us (350 wavefronts instead of 22 blocks and a second launch for the last elements).
// reverse: workgroups take the pieces from the far end first.  A server that applies updates back to back
// alternates the direction, so each pass starts on the theta and v lines the previous pass touched last, which
// the 256 MB last-level cache still holds (P = 40 M, c = 1: 136 -> 108 us per update).
// MODE: kCached  theta and v by ordinary loads and stores (vectors that stay in the caches from call to call);
//       kReuse   ordinary loads, non-temporal stores (the last-level cache serves part of the next pass);
//       kStream  non-temporal both ways: nothing of theta and v survives until the next pass.
// A vector length that is no multiple of 4 leaves at most 3 elements to a workgroup of their own, one lane each (left to a
// lane of the last whole workgroup, their loads come after that wavefront's own: 11.3 instead of 6 us at P = 89 578, c = 30).
enum { kCached = 0, kReuse = 1, kStream = 2 };
constexpr int kUpdThreads = 64;
// TH: lanes of a workgroup.  GPLAIN: the gradients are read with ordinary loads (the second pass of a long window).
template <int ILP, int U, bool SHADOW, int MODE, int TH = kUpdThreads, bool GPLAIN = false>
__global__ __launch_bounds__(TH) void apply_update_kernel(const float* theta_in, float* theta_out, float* v,
                                                                   bf16_t* __restrict__ shadow, int64_t P, int c, GradTable t, float m,
                                                                   float decay, int reverse) {
  const int64_t n4 = P >> 2, whole = (n4 + TH * ILP - 1) / (TH * ILP);
  if (blockIdx.x >= whole) {
    const int64_t k = n4 * 4 + threadIdx.x;
    if (k >= P) return;
    const float s = sum_element<U>(t, 0, c, k);
    const float a = theta_in[k], b = fmaf(m, v[k], s) + decay * a;
    v[k] = b;
    theta_out[k] = a - b;
    if (SHADOW) shadow[k] = f2bf(a - b);
    return;
  }
  const int64_t blk = reverse ? whole - 1 - blockIdx.x : blockIdx.x;
  const int64_t base = blk * (TH * ILP) + threadIdx.x;
  const float4* th4 = reinterpret_cast<const float4*>(theta_in);
  float4* v4 = reinterpret_cast<float4*>(v);
  float4 s[ILP], th[ILP], vv[ILP];
  bool in[ILP];
#pragma unroll
  for (int e = 0; e < ILP; e++) {
    const int64_t i = base + e * TH;
    in[e] = i < n4;
    s[e] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (in[e]) {
      th[e] = MODE == kStream ? ldg_nt(th4 + i) : th4[i];
      vv[e] = MODE == kStream ? ldg_nt(v4 + i) : v4[i];
    }
  }
  int l = 0;
  for (; l + U <= c; l += U) {
    float4 g[U][ILP];
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int e = 0; e < ILP; e++)
        if (in[e]) g[u][e] = GPLAIN ? reinterpret_cast<const float4*>(t.g[l + u])[base + e * TH] : ldg_nt(reinterpret_cast<const float4*>(t.g[l + u]) + base + e * TH);
#pragma unroll
    for (int u = 0; u < U; u++)             // arrival order l, l+1, ... within every element
#pragma unroll
      for (int e = 0; e < ILP; e++) fma4(s[e], t.coef[l + u], g[u][e]);
  }
  if (l < c) {
    float4 g[U][ILP];
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int e = 0; e < ILP; e++)
        if (in[e] && l + u < c) g[u][e] = GPLAIN ? reinterpret_cast<const float4*>(t.g[l + u])[base + e * TH] : ldg_nt(reinterpret_cast<const float4*>(t.g[l + u]) + base + e * TH);
#pragma unroll
    for (int u = 0; u < U; u++)
      if (l + u < c) {
#pragma unroll
        for (int e = 0; e < ILP; e++) fma4(s[e], t.coef[l + u], g[u][e]);
      }
  }
#pragma unroll
  for (int e = 0; e < ILP; e++) {
    const int64_t i = base + e * TH;
    if (in[e]) {
      update4(th[e], vv[e], s[e], m, decay);
      float4* to = reinterpret_cast<float4*>(theta_out) + i;
      if (MODE == kCached) { v4[i] = vv[e]; *to = th[e]; } else { stg_nt(v4 + i, vv[e]); stg_nt(to, th[e]); }
      if (SHADOW) {
        const uint2 o = pack_bf4(th[e]);
        if (MODE == kReuse) __builtin_nontemporal_store(((uint64_t)o.y << 32) | o.x, reinterpret_cast<uint64_t*>(shadow) + i);
        else reinterpret_cast<uint2*>(shadow)[i] = o;
      }
    }
  }
}

// First pass of a long window: s = sum_l coef_l g_l for one stretch, the FMA chain of apply_update_kernel, written
// with ordinary stores.  Blocks of 256 lanes, ILP pieces each (a pass that only reads is at 7.07 TB/s this way).
template <int ILP, int U>
__global__ __launch_bounds__(256) void sum_gradients_kernel(float* __restrict__ out, int64_t len, int c, GradTable t) {
  const int64_t base = (int64_t)blockIdx.x * (256 * ILP) + threadIdx.x, n4 = len >> 2;
  if (blockIdx.x >= (n4 + 256 * ILP - 1) / (256 * ILP)) {
    const int64_t k = n4 * 4 + threadIdx.x;
    if (k < len) out[k] = sum_element<16>(t, 0, c, k);
    return;
  }
  float4 s[ILP];
#pragma unroll
  for (int e = 0; e < ILP; e++) s[e] = make_float4(0.f, 0.f, 0.f, 0.f);
  int l = 0;
  for (; l + U <= c; l += U) {
    float4 g[U][ILP];
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int e = 0; e < ILP; e++) {
        const int64_t i = base + e * 256;
        if (i < n4) g[u][e] = ldg_nt(reinterpret_cast<const float4*>(t.g[l + u]) + i);
      }
#pragma unroll
    for (int u = 0; u < U; u++)             // arrival order l, l+1, ... within every element
#pragma unroll
      for (int e = 0; e < ILP; e++) fma4(s[e], t.coef[l + u], g[u][e]);
  }
  for (; l < c; l++)
#pragma unroll
    for (int e = 0; e < ILP; e++) {
      const int64_t i = base + e * 256;
      if (i < n4) fma4(s[e], t.coef[l], ldg_nt(reinterpret_cast<const float4*>(t.g[l]) + i));
    }
#pragma unroll
  for (int e = 0; e < ILP; e++) {
    const int64_t i = base + e * 256;
    if (i < n4) reinterpret_cast<float4*>(out)[i] = s[e];
  }
}

// Fused steps over a flat stretch (see StepTable): per element the operations of apply_update_kernel, step after step.
// The gradients of all steps are one list, requested U at a time whatever step they belong to: the chain of steps waits
// for memory once per U gradients instead of once per step (P = 89 578, 8 steps of one gradient: 13.7 + 6.5 us for the
// pass and its scalar tail with one dependent read per step -> 5 us).
template <int U, bool NT>
__global__ __launch_bounds__(kUpdThreads) void apply_updates_fused_kernel(const float* theta_in, float* theta_final, float* v, int64_t P, int c,
                                                                          GradTable t, StepTable st, float m) {
  const int64_t i = (int64_t)blockIdx.x * kUpdThreads + threadIdx.x, n4 = P >> 2, whole = (n4 + kUpdThreads - 1) / kUpdThreads;
  if (i < n4) {
    const float4* th4 = reinterpret_cast<const float4*>(theta_in) + i;
    float4* v4 = reinterpret_cast<float4*>(v) + i;
    float4 a = NT ? ldg_nt(th4) : *th4, b = NT ? ldg_nt(v4) : *v4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    int step = 0, end = st.first[1];
    for (int l0 = 0; l0 < c; l0 += U) {
      float4 g[U];
#pragma unroll
      for (int u = 0; u < U; u++)
        if (l0 + u < c) g[u] = ldg_nt(reinterpret_cast<const float4*>(t.g[l0 + u]) + i);
#pragma unroll
      for (int u = 0; u < U; u++) {
        if (l0 + u >= c) continue;
        fma4(s, t.coef[l0 + u], g[u]);      // arrival order
        if (l0 + u + 1 == end) {            // the step's window is complete
          update4(a, b, s, m, st.decay[step]);
          s = make_float4(0.f, 0.f, 0.f, 0.f);
          if (st.theta_out[step]) {
            float4* to = reinterpret_cast<float4*>(st.theta_out[step]) + i;
            if (NT) stg_nt(to, a); else *to = a;
          }
          if (st.shadow_out[step]) reinterpret_cast<uint2*>(st.shadow_out[step])[i] = pack_bf4(a);
          step++;
          if (step < st.steps) end = st.first[step + 1];
        }
      }
    }
    if (NT) stg_nt(v4, b); else *v4 = b;
    if (theta_final) {
      float4* to = reinterpret_cast<float4*>(theta_final) + i;
      if (NT) stg_nt(to, a); else *to = a;
    }
  } else if (blockIdx.x >= whole) {          // at most 3 elements behind the last whole piece, one lane each
    const int64_t k = n4 * 4 + threadIdx.x;
    if (k >= P) return;
    float a = theta_in[k], b = v[k], s = 0.f;
    int step = 0, end = st.first[1];
    for (int l0 = 0; l0 < c; l0 += U) {
      float g[U];
#pragma unroll
      for (int u = 0; u < U; u++)
        if (l0 + u < c) g[u] = t.g[l0 + u][k];
#pragma unroll
      for (int u = 0; u < U; u++) {
        if (l0 + u >= c) continue;
        s = fmaf(t.coef[l0 + u], g[u], s);
        if (l0 + u + 1 == end) {
          b = fmaf(m, b, s) + st.decay[step] * a;
          a = a - b;
          s = 0.f;
          if (st.theta_out[step]) st.theta_out[step][k] = a;
          if (st.shadow_out[step]) st.shadow_out[step][k] = f2bf(a);
          step++;
          if (step < st.steps) end = st.first[step + 1];
        }
      }
    }
    v[k] = b;
    if (theta_final) theta_final[k] = a;
  }
}

// Workgroups for n4 pieces, `per` each, plus the one of the remaining elements.
static unsigned update_grid(int64_t P, int64_t per) { return (unsigned)((P / 4 + per - 1) / per + (P % 4 ? 1 : 0)); }

template <int ILP, int U, int MODE, int TH = kUpdThreads, bool GPLAIN = false>
static void launch_update(const UpdateLaunch& u, const GradTable& t, int residency_lds, hipStream_t stream) {
  const dim3 grid(update_grid(u.P, TH * ILP));
  if (u.shadow_out)
    hipLaunchKernelGGL((apply_update_kernel<ILP, U, true, MODE, TH, GPLAIN>), grid, dim3(TH), residency_lds, stream, u.theta_in, u.theta_out, u.v,
                       u.shadow_out, u.P, u.c, t, u.momentum, u.decay, u.reverse);
  else
    hipLaunchKernelGGL((apply_update_kernel<ILP, U, false, MODE, TH, GPLAIN>), grid, dim3(TH), residency_lds, stream, u.theta_in, u.theta_out, u.v,
                       u.shadow_out, u.P, u.c, t, u.momentum, u.decay, u.reverse);
}

hipError_t launch_apply_update(const UpdateLaunch& u, hipStream_t stream) {
  if (u.P <= 0) return hipSuccess;
  if (u.P / 4 > (int64_t)0x7fffff00 * kUpdThreads) return hipErrorInvalidValue;
  GradTable t;
  for (int l = 0; l < kMaxLearners; l++) {
    t.g[l] = l < u.c ? u.grads[l] : nullptr;
    t.coef[l] = l < u.c ? u.coef[l] : 0.f;
  }
  if (two_pass_update(u.P, u.c) && u.sum_buf) {
    // stretches of 512 summing workgroups (two per compute unit; 256-1024 measured within 4 %, other counts slower)
    UpdateLaunch r = u;
    r.c = 1;
    r.reverse = 0;
    GradTable tb;
    for (int l = 0; l < kMaxLearners; l++) { tb.g[l] = nullptr; tb.coef[l] = 0.f; }
    tb.g[0] = u.sum_buf;
    tb.coef[0] = 1.0f;
    for (int64_t off = 0; off < u.P; off += kSumStretch) {
      const int64_t len = std::min(kSumStretch, u.P - off);
      GradTable ta = t;
      for (int l = 0; l < u.c; l++) ta.g[l] = t.g[l] + off;
      hipLaunchKernelGGL((sum_gradients_kernel<4, 3>), dim3(update_grid(len, 1024)), dim3(256), 0, stream, u.sum_buf, len, u.c, ta);
      r.theta_in = u.theta_in + off;
      r.theta_out = u.theta_out + off;
      r.v = u.v + off;
      r.shadow_out = u.shadow_out ? u.shadow_out + off : nullptr;
      r.P = len;
      launch_update<4, 1, kStream, 256, true>(r, tb, 0, stream);
    }
    return hipGetLastError();
  }
  // The lines between the shapes are where their times crossed in sweeps over P = 20 k .. 62 M and c = 1 .. 54 (residency in
  // wavefronts per compute unit: 10 at 16 KiB of LDS each, 8 at 20 KiB, otherwise bounded by registers):
  //   up to 0.6 M parameters the chip is not full: one piece per lane and as many loads in flight as registers allow;
  //   above, short windows want two pieces per lane, long ones fewer resident wavefronts;
  //   beyond 32 M parameters theta and v (8 bytes each) no longer fit the last-level cache: unless the passes alternate in
  //   direction (u.reuse), nothing of them can be reused and the streaming hints win.
  const bool stream_mode = !u.reuse && u.P > ((int64_t)1 << 25);
  if (u.P <= 600000) launch_update<1, 16, kCached>(u, t, 0, stream);
  else if (u.P <= 1500000) launch_update<2, 8, kCached>(u, t, 0, stream);
  else if (stream_mode && u.c <= 4) launch_update<1, 16, kStream>(u, t, 0, stream);
  else if (stream_mode) launch_update<1, 8, kStream>(u, t, 20 * 1024, stream);
  else if (u.c <= 4) launch_update<2, 8, kReuse>(u, t, 0, stream);
  else if (u.P <= 6000000 || u.c > 24) launch_update<2, 4, kReuse>(u, t, 20 * 1024, stream);
  else launch_update<1, 8, kReuse>(u, t, 16 * 1024, stream);
  return hipGetLastError();
}

hipError_t launch_apply_updates_fused(const UpdateLaunch& u, const StepTable& st, float* final_theta, hipStream_t stream) {
  if (u.P <= 0) return hipSuccess;
  if (st.steps < 1 || st.steps > kMaxFusedSteps || st.first[0] != 0 || st.first[st.steps] != u.c || u.c > kMaxLearners) return hipErrorInvalidValue;
  for (int k = 0; k < st.steps; k++)
    if (st.first[k + 1] <= st.first[k]) return hipErrorInvalidValue;   // the kernel closes a step with its last gradient
  if (u.P / 4 > (int64_t)0x7fffff00 * kUpdThreads) return hipErrorInvalidValue;
  GradTable t;
  for (int l = 0; l < kMaxLearners; l++) {
    t.g[l] = l < u.c ? u.grads[l] : nullptr;
    t.coef[l] = l < u.c ? u.coef[l] : 0.f;
  }
  const dim3 grid(update_grid(u.P, kUpdThreads));
  if (u.P >= 1500000)
    hipLaunchKernelGGL((apply_updates_fused_kernel<8, true>), grid, dim3(kUpdThreads), 0, stream, u.theta_in, final_theta, u.v, u.P, u.c, t, st, u.momentum);
  else
    hipLaunchKernelGGL((apply_updates_fused_kernel<16, false>), grid, dim3(kUpdThreads), 0, stream, u.theta_in, final_theta, u.v, u.P, u.c, t, st, u.momentum);
  return hipGetLastError();
}

// ------------------------------------------------------------------ update of a fully connected layer from factors
// For a fully connected layer with a mini-batch of N images the weight gradient is the rank-N product
// dW[o][i] = sum_n dy[n][o] x[n][i].  A learner keeps the two factors transposed, dyT [out][NP] and xT [in][NP] (bf16, NP = N
// rounded up to 8, zero-filled), instead of writing dW, and this kernel forms the product while it streams theta and v:
// one bf16 MFMA (32 x 32 x 16, fp32 accumulation) yields the gradient of a 32 x 32 block of weights from two 1 KiB operand
// reads -- both factors are k-contiguous, so the fragments come straight from memory.  HBM traffic per weight drops by the
// 4 bytes of gradient, and with several steps fused theta and v pass through once for all of them.
// A wavefront owns 32 output units x 32 input units.  theta, v and the running sums live in registers in row-major order
// (8 lanes x 16 bytes cover the 128 contiguous bytes of a row); a product leaves the matrix cores in MFMA order and is
// turned around through the wavefront's own piece of LDS.  Gradients without factors (pushed from outside) are read as
// written-out vectors, in the same order.  Per element: p_l = product (or the written-out value), s = sum_l coef_l p_l in
// arrival order, then the update of apply_update_kernel.  The layer's bias follows its weights in the flat vector and is
// updated by one extra row of workgroups from the written-out bias gradients.
struct FcFactors {
  const bf16_t* base[kMaxLearners];  // the pending gradient's factors, or nullptr: gradient l is a written-out vector
};
// The layers of one launch: workgroups tile0[k] .. tile0[k + 1] - 1 belong to layer k, cols[k] of them per block of 32
// output units (plus one such row for the bias).
struct FcLayerTab {
  int count;
  int in[kMaxFactoredLayers], out[kMaxFactoredLayers], cols[kMaxFactoredLayers];
  int tile0[kMaxFactoredLayers + 1];
  int64_t w_off[kMaxFactoredLayers];
  int64_t fx_off[kMaxFactoredLayers], fdy_off[kMaxFactoredLayers];
};

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;

constexpr int kFcTileRows = 32, kFcTileCols = 32;     // per wavefront
constexpr int kFcCB = kFcTileCols / 32;               // MFMA column blocks per wavefront
constexpr int kFcLPR = kFcTileCols / 4;               // lanes per tile row in row-major order (16 bytes each)
constexpr int kFcRPI = 64 / kFcLPR;                   // tile rows one 64-lane access covers
constexpr int kFcNQ = kFcTileRows / kFcRPI;           // 16-byte pieces per lane and array
constexpr int kFcLds = kFcTileCols + 4;               // LDS row stride in floats

template <bool SHADOW>
__global__ __launch_bounds__(256) void apply_update_fc_kernel(const float* theta_in, float* theta_out, float* v, int NP, GradTable t,
                                                              FcFactors f, FcLayerTab lt, StepTable st, float m) {
  __shared__ __attribute__((aligned(16))) float lds[4 * kFcTileRows * kFcLds];
  int layer = 0;
  for (int k = 1; k < lt.count; k++) layer = (int)blockIdx.x >= lt.tile0[k] ? k : layer;
  const int local = (int)blockIdx.x - lt.tile0[layer];
  const int bx = local % lt.cols[layer], by = local / lt.cols[layer];
  const int in = lt.in[layer], out = lt.out[layer];
  const int64_t woff = lt.w_off[layer];
  theta_in += woff; theta_out += woff; v += woff;
  const int nrb = (out + kFcTileRows - 1) / kFcTileRows;
  if (by == nrb) {       // bias: elements out * in + col .. col + 3
    const int col = (bx * 256 + threadIdx.x) * 4;
    if (col >= out) return;
    const int64_t e = (int64_t)out * in + col;
    float4 a = *reinterpret_cast<const float4*>(theta_in + e), b = *reinterpret_cast<const float4*>(v + e);
    for (int step = 0; step < st.steps; step++) {
      float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int l = st.first[step]; l < st.first[step + 1]; l++) {
        const float4 g = *reinterpret_cast<const float4*>(t.g[l] + woff + e);
        s.x = fmaf(t.coef[l], g.x, s.x); s.y = fmaf(t.coef[l], g.y, s.y);
        s.z = fmaf(t.coef[l], g.z, s.z); s.w = fmaf(t.coef[l], g.w, s.w);
      }
      const float decay = st.decay[step];
      b.x = fmaf(m, b.x, s.x) + decay * a.x; b.y = fmaf(m, b.y, s.y) + decay * a.y;
      b.z = fmaf(m, b.z, s.z) + decay * a.z; b.w = fmaf(m, b.w, s.w) + decay * a.w;
      a.x -= b.x; a.y -= b.y; a.z -= b.z; a.w -= b.w;
      if (SHADOW) {
        uint2 o;
        o.x = pack2bf(a.x, a.y);
        o.y = pack2bf(a.z, a.w);
        *reinterpret_cast<uint2*>(st.shadow_out[step] + woff + e) = o;
      }
    }
    *reinterpret_cast<float4*>(v + e) = b;
    *reinterpret_cast<float4*>(theta_out + e) = a;
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int o0 = by * kFcTileRows;
  const int w0 = (bx * 4 + wave) * kFcTileCols;
  if (w0 >= in) return;               // whole wavefronts leave: no workgroup barrier below
  float* tile = lds + wave * (kFcTileRows * kFcLds);
  // row-major registers: piece q is row kFcRPI q + lane / kFcLPR, columns 4 (lane % kFcLPR) .. + 3 of the tile
  const int rr = lane / kFcLPR, cc = (lane % kFcLPR) * 4;
  const bool col_ok = w0 + cc < in;   // in is a multiple of 4
  float4 th[kFcNQ], vv[kFcNQ];
#pragma unroll
  for (int q = 0; q < kFcNQ; q++) {
    const int o = o0 + kFcRPI * q + rr;
    if (o < out && col_ok) {
      const int64_t e = (int64_t)o * in + w0 + cc;
      th[q] = ldg_nt(reinterpret_cast<const float4*>(theta_in + e));
      vv[q] = ldg_nt(reinterpret_cast<const float4*>(v + e));
    }
  }
  // MFMA operands: lane (j = lane % 32, h = lane / 32) holds k = 8 h .. 8 h + 7 of row / column j
  const int j = lane & 31, h = lane >> 5;
  const int KB = (NP + 15) >> 4;
  for (int step = 0; step < st.steps; step++) {
    float4 s[kFcNQ];
#pragma unroll
    for (int q = 0; q < kFcNQ; q++) s[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int l = st.first[step]; l < st.first[step + 1]; l++) {
      const float cf = t.coef[l];
      if (f.base[l]) {
        const bf16_t* xT = f.base[l] + lt.fx_off[layer];
        const bf16_t* dyT = f.base[l] + lt.fdy_off[layer];
        floatx16_t p[kFcCB];
#pragma unroll
        for (int b = 0; b < kFcCB; b++)
#pragma unroll
          for (int r = 0; r < 16; r++) p[b][r] = 0.f;
        for (int kb = 0; kb < KB; kb++) {
          const int n0 = 16 * kb + 8 * h;
          union { uint4 u; bf16x8_t x; } fa, fb[kFcCB];
          fa.u = make_uint4(0u, 0u, 0u, 0u);
          if (n0 < NP && o0 + j < out) fa.u = *reinterpret_cast<const uint4*>(dyT + (int64_t)(o0 + j) * NP + n0);
#pragma unroll
          for (int b = 0; b < kFcCB; b++) {
            fb[b].u = make_uint4(0u, 0u, 0u, 0u);
            if (n0 < NP && w0 + 32 * b + j < in) fb[b].u = *reinterpret_cast<const uint4*>(xT + (int64_t)(w0 + 32 * b + j) * NP + n0);
          }
#pragma unroll
          for (int b = 0; b < kFcCB; b++) p[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa.x, fb[b].x, p[b], 0, 0, 0);
        }
        // MFMA order (column 32 b + j, rows 8 (r / 4) + 4 h + r % 4) -> row-major, through this wavefront's LDS piece
#pragma unroll
        for (int b = 0; b < kFcCB; b++)
#pragma unroll
          for (int r = 0; r < 16; r++) tile[(8 * (r >> 2) + 4 * h + (r & 3)) * kFcLds + 32 * b + j] = p[b][r];
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int q = 0; q < kFcNQ; q++) {
          const float4 g = *reinterpret_cast<const float4*>(tile + (kFcRPI * q + rr) * kFcLds + cc);
          s[q].x = fmaf(cf, g.x, s[q].x); s[q].y = fmaf(cf, g.y, s[q].y);
          s[q].z = fmaf(cf, g.z, s[q].z); s[q].w = fmaf(cf, g.w, s[q].w);
        }
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
      } else {
#pragma unroll
        for (int q = 0; q < kFcNQ; q++) {
          const int o = o0 + kFcRPI * q + rr;
          if (o < out && col_ok) {
            const float4 g = ldg_nt(reinterpret_cast<const float4*>(t.g[l] + woff + (int64_t)o * in + w0 + cc));
            s[q].x = fmaf(cf, g.x, s[q].x); s[q].y = fmaf(cf, g.y, s[q].y);
            s[q].z = fmaf(cf, g.z, s[q].z); s[q].w = fmaf(cf, g.w, s[q].w);
          }
        }
      }
    }
    const float decay = st.decay[step];
#pragma unroll
    for (int q = 0; q < kFcNQ; q++) {
      const int o = o0 + kFcRPI * q + rr;
      if (o >= out || !col_ok) continue;
      float4 a = th[q], b = vv[q];
      b.x = fmaf(m, b.x, s[q].x) + decay * a.x; b.y = fmaf(m, b.y, s[q].y) + decay * a.y;
      b.z = fmaf(m, b.z, s[q].z) + decay * a.z; b.w = fmaf(m, b.w, s[q].w) + decay * a.w;
      a.x -= b.x; a.y -= b.y; a.z -= b.z; a.w -= b.w;
      th[q] = a;
      vv[q] = b;
      if (SHADOW) {
        uint2 w2;
        w2.x = pack2bf(a.x, a.y);
        w2.y = pack2bf(a.z, a.w);
        *reinterpret_cast<uint2*>(st.shadow_out[step] + woff + (int64_t)o * in + w0 + cc) = w2;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kFcNQ; q++) {
    const int o = o0 + kFcRPI * q + rr;
    if (o >= out || !col_ok) continue;
    const int64_t e = (int64_t)o * in + w0 + cc;
    stg_nt(reinterpret_cast<float4*>(v + e), vv[q]);
    stg_nt(reinterpret_cast<float4*>(theta_out + e), th[q]);
  }
}

// The same for one step of long sums (many gradients, or many images in one): what counts there are the factors' reads and the sums, so
// a wavefront owns 64 x 64 weights, each operand serves two products, the running sum stays in MFMA order and is turned around once,
// at its end.  theta and v come half a tile at a time, the first half on its way during the sums.
// Lone steps of the AlexNet-shaped net's 58.6 M weights, all layers, whose theta, v and bf16 copy alone take 175 us at the copy rate: 18
// gradients of 16 images 335 us with 32 x 32 weights a wavefront, 219 here; 8 of 32 267 and 205; one of 256 images 341 and 197 (written out
// by the weight-gradient kernel, 118 us, and read again, it took 200); 4 of 256 961 and 298.
typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
typedef unsigned v2u_t __attribute__((ext_vector_type(2)));
constexpr int kDeepTile = 128;                        // weights of a workgroup in each direction: 2 x 2 wavefronts
constexpr int kDeepStage = 2 * kDeepTile * 128;       // bytes of a stage: 64 images of both operands
constexpr int kDeepLds = 64 + 4;                      // LDS row stride in floats

// Weight elements e .. e + 3 of the flat vector from the sum of their gradients.
template <bool SHADOW>
__device__ __forceinline__ void update4(float4& a, float4& b, const float4& s, float m, float decay, uint2* shadow) {
  b.x = fmaf(m, b.x, s.x) + decay * a.x; b.y = fmaf(m, b.y, s.y) + decay * a.y;
  b.z = fmaf(m, b.z, s.z) + decay * a.z; b.w = fmaf(m, b.w, s.w) + decay * a.w;
  a.x -= b.x; a.y -= b.y; a.z -= b.z; a.w -= b.w;
  if (SHADOW) {
    uint2 o;
    o.x = pack2bf(a.x, a.y);
    o.y = pack2bf(a.z, a.w);
    *shadow = o;
  }
}

// Mini-batches of up to 16 images are one k-block, whose operands come straight from memory; larger ones pass through LDS in stages
// of 64 images, two in turn, which the four wavefronts share (laid out like fc_rows_kernel's stages).
// EXPAND: the product of one gradient's factors is written out at theta_out instead.
template <bool SHADOW, bool STAGED, bool EXPAND>
__global__ __launch_bounds__(256, 2) void apply_update_fc_deep_kernel(const float* theta_in, float* theta_out, float* v, bf16_t* shadow, int NP, int c,
                                                                      GradTable t, FcFactors f, FcLayerTab lt, float m, float decay) {
  __shared__ __attribute__((aligned(16))) float lds[STAGED ? 2 * kDeepStage / 4 : 4 * 32 * kDeepLds];
  int layer = 0;
  for (int k = 1; k < lt.count; k++) layer = (int)blockIdx.x >= lt.tile0[k] ? k : layer;
  const int in = lt.in[layer], out = lt.out[layer];
  const int64_t woff = lt.w_off[layer];
  theta_in += woff; theta_out += woff; v += woff;
  if (SHADOW) shadow += woff;
  const int rows = (out + kDeepTile - 1) / kDeepTile, cols = lt.cols[layer], tiles = rows * cols;
  int local = (int)blockIdx.x - lt.tile0[layer];
  const int tid = threadIdx.x;
  if (local >= tiles) {       // bias: elements out * in + col .. col + 3 (written out already)
    if (EXPAND) return;
    const int col = ((local - tiles) * 256 + tid) * 4;
    if (col >= out) return;
    const int64_t e = (int64_t)out * in + col;
    float4 a = *reinterpret_cast<const float4*>(theta_in + e), b = *reinterpret_cast<const float4*>(v + e);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int l = 0; l < c; l++) {
      const float4 g = *reinterpret_cast<const float4*>(t.g[l] + woff + e);
      s.x = fmaf(t.coef[l], g.x, s.x); s.y = fmaf(t.coef[l], g.y, s.y);
      s.z = fmaf(t.coef[l], g.z, s.z); s.w = fmaf(t.coef[l], g.w, s.w);
    }
    update4<SHADOW>(a, b, s, m, decay, SHADOW ? reinterpret_cast<uint2*>(shadow + e) : nullptr);
    *reinterpret_cast<float4*>(v + e) = b;
    *reinterpret_cast<float4*>(theta_out + e) = a;
    return;
  }
  // launch order is dealt round-robin to the eight XCDs (a layer's first workgroup is a multiple of eight): each takes a contiguous
  // eighth of the tiles column by column, whose input factors stay in its L2
  const int eighth = tiles >> 3;
  if (local < eighth * 8) local = (local & 7) * eighth + (local >> 3);
  const int bx = local / rows, by = local - bx * rows;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int o0 = by * kDeepTile + 64 * (wave >> 1), w0 = bx * kDeepTile + 64 * (wave & 1);
  if (!STAGED && (o0 >= out || w0 >= in)) return;   // whole wavefronts: no workgroup barrier below
  float* tile = lds + wave * (32 * kDeepLds);
  // row-major registers: piece q of a half is row 4 q + lane / 16, columns 4 (lane % 16) .. + 3
  const int rr = lane >> 4, cc = 4 * (lane & 15);
  // offsets from the tile's first weight; out of range where the layer ends: loads give zeros, stores do nothing
  const int64_t e0 = (int64_t)o0 * in + w0;
  auto offset = [&](int half, int q) {
    const int o = 32 * half + 4 * q + rr;
    return o0 + o < out && w0 + cc < in ? (o * in + cc) * 4 : (int)0x80000000u;      // in is a multiple of 4, and below 2^23
  };
  const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc((void*)(theta_in + e0), 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)(v + e0), 0, 0x7fffffff, 0x00020000);
  constexpr int kNt = 2;                              // streamed: nobody reads these lines again soon
  float4 th[2][8], vv[2][8];
  auto fetch = [&](int half) {
#pragma unroll
    for (int q = 0; q < 8; q++) {
      th[half][q] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rt, offset(half, q), 0, kNt));
      vv[half][q] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rv, offset(half, q), 0, kNt));
    }
  };
  if (!EXPAND && !STAGED) fetch(0);
  // MFMA operands: lane (j = lane % 32, h = lane / 32) holds k = 8 h .. 8 h + 7 of row / column j.  Units behind the layer's last
  // one repeat it: their products are not stored.
  const int j = lane & 31, h = lane >> 5;
  floatx16_t sm[2][2];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 16; r++) sm[i][b][r] = 0.f;
  if constexpr (!STAGED) {
    // three gradients' operands are on their way
    int ao[2], bo[2];                                 // bytes; the half behind the factors' rows is out of range and comes as zeros
#pragma unroll
    for (int i = 0; i < 2; i++) {
      ao[i] = 8 * h < NP ? (min(o0 + 32 * i + j, out - 1) * NP + 8 * h) * 2 : (int)0x80000000u;
      bo[i] = 8 * h < NP ? (min(w0 + 32 * i + j, in - 1) * NP + 8 * h) * 2 : (int)0x80000000u;
    }
    int fl = 0;                                       // the next one to be requested; behind the last one that one again, for nobody
    const bf16_t* fbase = f.base[0];
    auto request = [&](uint4 (&a)[2], uint4 (&b)[2]) {
      const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)(fbase + lt.fdy_off[layer]), 0, 0x7fffffff, 0x00020000);
      const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)(fbase + lt.fx_off[layer]), 0, 0x7fffffff, 0x00020000);
#pragma unroll
      for (int i = 0; i < 2; i++) {
        a[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rd, ao[i], 0, 0));
        b[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, bo[i], 0, 0));
      }
      fl = min(fl + 1, c - 1);
      fbase = f.base[fl];
    };
    int l = 0;
    auto multiply = [&](uint4 (&fa)[2], uint4 (&fb)[2]) {
      const floatx16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      floatx16_t p[2][2];
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int q = 0; q < 2; q++)
          p[i][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fa[i]), __builtin_bit_cast(bf16x8_t, fb[q]), zero, 0, 0, 0);
      request(fa, fb);
      const float cf = t.coef[l++];
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int q = 0; q < 2; q++)
#pragma unroll
          for (int r = 0; r < 16; r++) sm[i][q][r] = fmaf(cf, p[i][q][r], sm[i][q][r]);
    };
    uint4 a0[2], b0[2], a1[2], b1[2], a2[2], b2[2];
    request(a0, b0);
    request(a1, b1);
    request(a2, b2);
#pragma unroll 1
    for (int it = 0; it < c; it += 3) {
      multiply(a0, b0);
      if (it + 1 < c) multiply(a1, b1);
      if (it + 2 < c) multiply(a2, b2);
    }
  } else {
    // a row of a stage is the 64 images (128 bytes) of a unit, its 16-byte pieces exchanged: piece p of row r at place p ^ (r % 8)
    const int per = (NP + 63) >> 6, total = c * per;
    const int pc = (lane & 7) ^ (lane >> 3);
    int ro[4], rx[4];                                 // load q of a wavefront fetches rows 8 (4 wave + q) .. + 7 of either operand
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int r = 8 * (4 * wave + q) + (lane >> 3);
      ro[q] = (min(by * kDeepTile + r, out - 1) * NP + 8 * pc) * 2;
      rx[q] = (min(bx * kDeepTile + r, in - 1) * NP + 8 * pc) * 2;
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)lds);
    int fl = 0, fst = 0;                              // the next stage to be requested
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"       // the host pass knows no m0
    auto request = [&](uint32_t at) {                 // behind the last gradient: the last one's once more, for nobody
      const bf16_t* base = f.base[min(fl, c - 1)];
      const bool ok = 64 * fst + 8 * pc < NP;
      const uintptr_t pd = (uintptr_t)(base + lt.fdy_off[layer] + 64 * fst), px = (uintptr_t)(base + lt.fx_off[layer] + 64 * fst);
      const v4u_t rd = {(uint32_t)pd, (uint32_t)(pd >> 32) & 0xffffu, 0x7fffffffu, 0x00020000u};
      const v4u_t rxs = {(uint32_t)px, (uint32_t)(px >> 32) & 0xffffu, 0x7fffffffu, 0x00020000u};
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const uint32_t dst = lds0 + at + (4 * wave + q) * 1024;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(dst), "v"(ok ? ro[q] : (int)0x80000000u), "s"(rd) : "memory", "m0");
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(dst + kDeepTile * 128), "v"(ok ? rx[q] : (int)0x80000000u), "s"(rxs) : "memory", "m0");
      }
      if (++fst == per) { fst = 0; fl++; }
    };
#pragma clang diagnostic pop
    // (theta's and momentum's pieces in front: the waits below count the loads to LDS behind a stage and nothing that the compiler issues,
    // however many instructions it makes of a fetch)
    if (!EXPAND) fetch(0);
    request(0);
    request(kDeepStage);
    const char* L = reinterpret_cast<const char*>(lds);
    const int arow = (64 * (wave >> 1) + j) * 128, brow = kDeepTile * 128 + (64 * (wave & 1) + j) * 128;
    floatx16_t p[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int q = 0; q < 2; q++)
#pragma unroll
        for (int r = 0; r < 16; r++) p[i][q][r] = 0.f;
    int l = 0, stg = 0;
    uint32_t at = 0;
#pragma unroll 1
    for (int s = 0; s < total; s++) {
      asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");         // this stage has landed: eight loads of the next one are behind it
      const int kks = min(4, (NP - 64 * stg + 15) >> 4);
      auto read = [&](bf16x8_t (&a)[2], bf16x8_t (&b)[2], int kk) {
        const int place = ((2 * kk + h) ^ (j & 7)) * 16;
#pragma unroll
        for (int i = 0; i < 2; i++) {
          a[i] = *reinterpret_cast<const bf16x8_t*>(L + at + arow + 32 * 128 * i + place);
          b[i] = *reinterpret_cast<const bf16x8_t*>(L + at + brow + 32 * 128 * i + place);
        }
      };
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
        if (kk >= kks) break;                         // the pieces behind are zeros
        bf16x8_t a[2], b[2];
        read(a, b, kk);
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int q = 0; q < 2; q++) p[i][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[q], p[i][q], 0, 0, 0);
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // every wavefront has read it
      request(at);
      at ^= kDeepStage;
      if (++stg == per) {
        const float cf = t.coef[l];
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int q = 0; q < 2; q++)
#pragma unroll
            for (int r = 0; r < 16; r++) {
              sm[i][q][r] = fmaf(cf, p[i][q][r], sm[i][q][r]);
              p[i][q][r] = 0.f;
            }
        stg = 0;
        l++;
      }
    }
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");        // no load is on its way to LDS, which takes the sums now
  }
  if (!EXPAND) fetch(1);
  const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc((void*)(theta_out + e0), 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(shadow + e0), 0, 0x7fffffff, 0x00020000);
#pragma unroll
  for (int half = 0; half < 2; half++) {
#pragma unroll
    for (int b = 0; b < 2; b++)
#pragma unroll
      for (int r = 0; r < 16; r++) tile[(8 * (r >> 2) + 4 * h + (r & 3)) * kDeepLds + 32 * b + j] = sm[half][b][r];
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < 8; q++) {
      const int at = offset(half, q);
      const float4 s = *reinterpret_cast<const float4*>(tile + (4 * q + rr) * kDeepLds + cc);
      if (EXPAND) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u_t, s), ro, at, 0, kNt);
        continue;
      }
      float4 a = th[half][q], b = vv[half][q];
      uint2 sh;
      update4<SHADOW>(a, b, s, m, decay, &sh);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u_t, b), rv, at, 0, kNt);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u_t, a), ro, at, 0, kNt);
      if (SHADOW) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u_t, sh), rs, at < 0 ? at : at >> 1, 0, 0);
    }
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
  }
}

hipError_t launch_apply_update_fc(const FcUpdateLaunch& u, hipStream_t stream, const StepTable* steps) {
  if (u.layers < 1 || u.layers > kMaxFactoredLayers || u.c < 1 || u.c > kMaxLearners) return hipErrorInvalidValue;
  if (u.NP < 8 || u.NP > kMaxFactorRows || (u.NP & 7)) return hipErrorInvalidValue;
  GradTable t;
  FcFactors f;
  for (int l = 0; l < kMaxLearners; l++) {
    t.g[l] = l < u.c ? u.grads[l] : nullptr;
    t.coef[l] = l < u.c ? u.coef[l] : 0.f;
    f.base[l] = l < u.c ? u.factors[l] : nullptr;
  }
  FcLayerTab lt;
  memset(&lt, 0, sizeof(lt));
  lt.count = u.layers;
  // where the two kernels' times cross (one step, us, small tiles / large ones): 16 images, 6 gradients 186 / 194, 9 222 / 202; 8 images, 8
  // gradients 201 / 198; one gradient of 64 images 196 / 196, of 96 204 / 192; 4 of 32 199 / 195, 2 of 32 175 / 200.  Large tiles read no written-out gradients.
  bool deep = (steps ? steps->steps : 1) == 1 && (u.NP <= 16 ? u.c >= 8 : u.c * ((u.NP + 15) / 16) >= 5);
  for (int l = 0; l < u.c; l++) deep = deep && u.factors[l];
  for (int k = 0; k < u.layers; k++) deep = deep && u.in[k] < 1 << 23;
  int64_t tiles = 0;
  for (int k = 0; k < u.layers; k++) {
    if (u.in[k] < 4 || u.out[k] < 4 || (u.in[k] & 3) || (u.out[k] & 3)) return hipErrorInvalidValue;
    lt.in[k] = u.in[k];
    lt.out[k] = u.out[k];
    lt.w_off[k] = u.w_off[k];
    lt.fx_off[k] = (int64_t)u.fx_off[k];
    lt.fdy_off[k] = (int64_t)u.fdy_off[k];
    if (deep) {
      tiles = (tiles + 7) & ~(int64_t)7;
      lt.cols[k] = (u.in[k] + kDeepTile - 1) / kDeepTile;
      lt.tile0[k] = (int)tiles;
      tiles += (int64_t)lt.cols[k] * ((u.out[k] + kDeepTile - 1) / kDeepTile) + (u.out[k] + 1023) / 1024;
      if (tiles > 0x7fffffff) return hipErrorInvalidValue;
      continue;
    }
    // 4 kFcTileCols input units per workgroup (four wavefronts side by side), or 1024 bias elements in the extra row
    lt.cols[k] = std::max((u.in[k] + 4 * kFcTileCols - 1) / (4 * kFcTileCols), (u.out[k] + 1023) / 1024);
    lt.tile0[k] = (int)tiles;
    tiles += (int64_t)lt.cols[k] * ((u.out[k] + kFcTileRows - 1) / kFcTileRows + 1);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  }
  lt.tile0[u.layers] = (int)tiles;
  StepTable st;
  if (steps) {
    st = *steps;
    if (st.steps < 1 || st.steps > kMaxFusedSteps || st.first[0] != 0 || st.first[st.steps] != u.c) return hipErrorInvalidValue;
  } else {
    memset(&st, 0, sizeof(st));
    st.steps = 1;
    st.first[1] = u.c;
    st.decay[0] = u.decay;
    st.shadow_out[0] = u.shadow_out;
  }
  bool shadow = st.shadow_out[0] != nullptr;
  for (int k = 0; k < st.steps; k++)
    if ((st.shadow_out[k] != nullptr) != shadow) return hipErrorInvalidValue;
  const dim3 grid((unsigned)tiles);
  auto launch_deep = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, u.theta_in, u.theta_out, u.v, st.shadow_out[0], u.NP, u.c, t, f, lt, u.momentum, st.decay[0]);
  };
  if (deep && u.NP <= 16) shadow ? launch_deep(apply_update_fc_deep_kernel<true, false, false>) : launch_deep(apply_update_fc_deep_kernel<false, false, false>);
  else if (deep) shadow ? launch_deep(apply_update_fc_deep_kernel<true, true, false>) : launch_deep(apply_update_fc_deep_kernel<false, true, false>);
  else if (shadow)
    hipLaunchKernelGGL((apply_update_fc_kernel<true>), grid, dim3(256), 0, stream, u.theta_in, u.theta_out, u.v, u.NP, t, f, lt, st, u.momentum);
  else
    hipLaunchKernelGGL((apply_update_fc_kernel<false>), grid, dim3(256), 0, stream, u.theta_in, u.theta_out, u.v, u.NP, t, f, lt, st, u.momentum);
  return hipGetLastError();
}

hipError_t launch_fc_expand_factors(const void* fx, const void* fdy, float* dw, int in, int out, int NP, hipStream_t stream) {
  if (in < 4 || out < 4 || (in & 3) || (out & 3) || in >= 1 << 23 || NP < 8 || NP > kMaxFactorRows || (NP & 7)) return hipErrorInvalidValue;
  GradTable t;
  FcFactors f;
  FcLayerTab lt;
  memset(&t, 0, sizeof(t)); memset(&f, 0, sizeof(f)); memset(&lt, 0, sizeof(lt));
  t.coef[0] = 1.f;
  f.base[0] = (const bf16_t*)fx;
  lt.count = 1;
  lt.in[0] = in;
  lt.out[0] = out;
  lt.fdy_off[0] = (const bf16_t*)fdy - (const bf16_t*)fx;
  lt.cols[0] = (in + kDeepTile - 1) / kDeepTile;
  const int64_t tiles = (int64_t)lt.cols[0] * ((out + kDeepTile - 1) / kDeepTile);
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(256), 0, stream, dw, dw, dw, (bf16_t*)nullptr, NP, 1, t, f, lt, 0.f, 0.f);
  };
  if (NP <= 16) launch(apply_update_fc_deep_kernel<false, false, true>);
  else launch(apply_update_fc_deep_kernel<false, true, true>);
  return hipGetLastError();
}

__global__ void fp32_to_bf16_kernel(const float* __restrict__ src, bf16_t* __restrict__ dst, int64_t n) {
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dst[i] = f2bf(src[i]);
}
__global__ void bf16_to_fp32_kernel(const bf16_t* __restrict__ src, float* __restrict__ dst, int64_t n) {
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    dst[i] = __uint_as_float((uint32_t)src[i] << 16);
}

hipError_t launch_fp32_to_bf16(const float* src, bf16_t* dst, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  int64_t want = (n + 255) / 256;
  int blocks = (int)(want < 4096 ? want : 4096);
  hipLaunchKernelGGL(fp32_to_bf16_kernel, dim3(blocks), dim3(256), 0, stream, src, dst, n);
  return hipGetLastError();
}
hipError_t launch_bf16_to_fp32(const bf16_t* src, float* dst, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  int64_t want = (n + 255) / 256;
  int blocks = (int)(want < 4096 ? want : 4096);
  hipLaunchKernelGGL(bf16_to_fp32_kernel, dim3(blocks), dim3(256), 0, stream, src, dst, n);
  return hipGetLastError();
}

}  // namespace sasgd
