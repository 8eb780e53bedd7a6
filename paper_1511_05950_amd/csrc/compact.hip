// calcGradient of small networks and small mini-batches (Section 2.1 learner step; layer shapes of Section 4.1) in few, short
// launches.  With a handful of images per learner a layer-by-layer pass is about thirty launches of 3 - 13 us, each a latency
// chain with most of the chip idle: one CIFAR-shaped mini-batch of 4 images took 147 us for 0.3 GFLOP.  Here
//   * a pooling layer is never launched: the next layer computes the pooled values while it fills its input patch in LDS (and
//     keeps them, and the winners, for the backward pass); the backward pass of a pooling layer is evaluated where the
//     gradient under it is read;
//   * a convolution keeps the whole contraction inside the workgroup: its wavefronts share one tile of output positions x
//     channels and divide the contraction (four channels x one filter row), so no second pass is needed and the chain of
//     matrix instructions of a tile is a sixteenth as long;
//   * input gradient and weight gradient of a layer go in one launch (they only read the same gradient);
//   * the last fully connected layer, softmax, loss and that layer's input gradient are one launch, a workgroup per image;
//   * every weight gradient that was split over workgroups, the fully connected weight gradients and the mean losses are
//     finished in one launch at the end.
// Eight launches forward and backward for the CIFAR-shaped net instead of 29: 66 us instead of 147 for a mini-batch of 4 in
// fp32, 162 instead of 256 for 16 of them.
//
// What bounds such a launch is latency: a memory round trip is 2 000 cycles when another chiplet wrote the data, and code that
// runs once is fetched as it goes (unrolling the contraction into 13 KiB of straight-line code made the CIFAR-shaped conv2 take
// 14 us with 2.7 us of matrix instructions).  So loops stay rolled, independent requests are issued together in front of them,
// and small calls use workgroups of 16 wavefronts on 32 x 16 tiles: many small pieces, each loaded in one round.
//
// Arithmetic: fp32 matrix instructions on fp32 operands whatever the storage type T is (bf16 values are exact in fp32), fp32
// accumulation.  Tensors are rounded to T at the same points as in the other paths (layer outputs, pooled values, activation
// gradients), so parity does not depend on the path.  All sums have a fixed order.
//
// LDS patches hold one float per element, `CS` floats per pixel with CS = 4 (mod 8): the 16 positions x 4 channels a matrix
// operand reads lie in different banks, and four channels are one aligned 16-byte write.
#include <algorithm>
#include <type_traits>

#include "dev_common.hpp"
#include "kernels.hpp"

namespace sasgd {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v3i_t __attribute__((ext_vector_type(3)));
typedef int v2i_t __attribute__((ext_vector_type(2)));

namespace {

constexpr uint32_t kOOB = 0x80000000u;   // buffer offset beyond any tensor: the load returns zeros
constexpr int kRedFloats = 1024 + 64;    // a column block and a bias sum per lane
constexpr int kDyLd = 32;                // row stride of the weight gradient's dy tile (floats): the lane halves read neighbouring rows

// ---------------------------------------------------------------- V consecutive elements
template <typename T, int V>
__device__ __forceinline__ void ldv(const T* p, float (&f)[V]) {
  if constexpr (V == 1) {
    f[0] = ldf(p);
  } else if constexpr (sizeof(T) == 4) {
    const float4 q = *reinterpret_cast<const float4*>(p);
    f[0] = q.x; f[1] = q.y; f[2] = q.z; f[3] = q.w;
  } else {
    const uint2 q = *reinterpret_cast<const uint2*>(p);
    f[0] = __uint_as_float(q.x << 16); f[1] = __uint_as_float(q.x & 0xffff0000u);
    f[2] = __uint_as_float(q.y << 16); f[3] = __uint_as_float(q.y & 0xffff0000u);
  }
}
template <typename T, int V>
__device__ __forceinline__ void stv(T* p, const float (&f)[V]) {
  if constexpr (V == 1) {
    stf(p, f[0]);
  } else if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
  } else {
    uint2 q;
    q.x = pack2bf(f[0], f[1]);
    q.y = pack2bf(f[2], f[3]);
    *reinterpret_cast<uint2*>(p) = q;
  }
}
template <int V>
__device__ __forceinline__ void put(float* p, const float (&f)[V]) {
  if constexpr (V == 1) *p = f[0];
  else *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
}
// Channels C .. of a pixel up to a multiple of four: zeros (the contraction walks four channels at a time).
template <int NTH>
__device__ __forceinline__ void zero_channels(float* lds, int pixels, int C, int CS) {
  const int pad = (4 - (C & 3)) & 3;
  for (int i = threadIdx.x; i < pixels * pad; i += NTH) {
    const int pix = pad == 3 ? i / 3 : i >> (pad - 1);
    lds[pix * CS + C + (i - pix * pad)] = 0.f;
  }
}
// a value as it comes back after being stored as T
__device__ __forceinline__ float stored(float f, const float*) { return f; }
__device__ __forceinline__ float stored(float f, const bf16_t*) { return bf2f(f2bf(f)); }

// ---------------------------------------------------------------- pooling while reading
// V channels from c of the pooled pixel (ph, pw): clipped windows, first maximum in row-major order, average over the
// in-bounds elements, optional ReLU behind it, rounded to T.
template <typename T, int V>
__device__ __forceinline__ void pooled_at(const T* y, const CompactSrc& s, int n, int ph, int pw, int c, float (&val)[V], uint32_t (&best)[V]) {
  const int h0 = ph * s.pst, w0 = pw * s.pst;
  const int nh = min(s.pks, s.YH - h0), nw = min(s.pks, s.YW - w0);
  const uint32_t b = ((uint32_t)(n * s.YH + h0) * s.YW + w0) * s.C + c;   // a tensor has fewer than 2^29 elements
  const bool is_max = s.kind == CSRC_MAXPOOL;
  if (s.pks == 3) {                       // all nine reads requested before the first is used; outside ones repeat the first
    float f[9][V];
#pragma unroll
    for (int t = 0; t < 9; t++) {
      const bool in = t / 3 < nh && t % 3 < nw;
      ldv<T, V>(y + (b + (in ? (uint32_t)((t / 3) * s.YW + t % 3) * s.C : 0u)), f[t]);
    }
#pragma unroll
    for (int v = 0; v < V; v++) { val[v] = f[0][v]; best[v] = 0; }
#pragma unroll
    for (int t = 1; t < 9; t++) {
      const bool in = t / 3 < nh && t % 3 < nw;
#pragma unroll
      for (int v = 0; v < V; v++) {
        if (is_max) {
          if (in && f[t][v] > val[v]) { val[v] = f[t][v]; best[v] = t; }
        } else if (in) {
          val[v] += f[t][v];
        }
      }
    }
  } else {
#pragma unroll
    for (int v = 0; v < V; v++) { val[v] = 0.f; best[v] = 0; }
    for (int kh = 0; kh < nh; kh++)
      for (int kw = 0; kw < nw; kw++) {
        float f[V];
        ldv<T, V>(y + (b + (uint32_t)(kh * s.YW + kw) * s.C), f);
#pragma unroll
        for (int v = 0; v < V; v++) {
          if (is_max) {
            if (kh + kw == 0 || f[v] > val[v]) { val[v] = f[v]; best[v] = (uint32_t)(kh * s.pks + kw); }
          } else {
            val[v] += f[v];
          }
        }
      }
  }
  const float cnt = (float)(nh * nw);
#pragma unroll
  for (int v = 0; v < V; v++) {
    if (!is_max) val[v] /= cnt;
    if (s.relu) val[v] = fmaxf(val[v], 0.f);
    val[v] = stored(val[v], (const T*)nullptr);
  }
}

template <int V>
__device__ __forceinline__ void store_winners(uint8_t* p, const uint32_t (&best)[V]) {
  if constexpr (V == 1) *p = (uint8_t)best[0];
  else *reinterpret_cast<uint32_t*>(p) = best[0] | (best[1] << 8) | (best[2] << 16) | (best[3] << 24);
}

// Input rows ih0 .. ih0 + rows - 1, columns iw0 .. iw0 + cols - 1 of image n into LDS, zero outside the image.  Pooled rows in
// [own_lo, own_hi) are also written to the workspace (every row belongs to exactly one workgroup).  POOL = false: the source
// is never a pooled one (the backward pass reads what the forward pass kept).
template <typename T, int V, bool POOL, int NTH>
__device__ __forceinline__ void load_patch_v(float* lds, const CompactSrc& s, char* wsb, int n, int ih0, int rows, int iw0, int cols, FastDiv by_cols,
                                             int CS, int own_lo, int own_hi) {
  const int cg = s.C / V, total = rows * cols * cg;
  const FastDiv by_cg = V == 4 ? s.by_c4 : s.by_c;
  const T* t = (const T*)wsb + s.off;
  for (int idx = threadIdx.x; idx < total; idx += NTH) {
    const int pix = by_cg(idx), c = (idx - pix * cg) * V;
    const int r = by_cols(pix), q = pix - r * cols;
    const int ih = ih0 + r, iw = iw0 + q;
    float val[V];
#pragma unroll
    for (int v = 0; v < V; v++) val[v] = 0.f;
    if ((unsigned)ih < (unsigned)s.H && (unsigned)iw < (unsigned)s.W) {
      const uint32_t e = ((uint32_t)(n * s.H + ih) * s.W + iw) * s.C + c;
      if (!POOL || s.kind == CSRC_TENSOR) {
        ldv<T, V>(t + e, val);
      } else {
        uint32_t best[V];
        pooled_at<T, V>(t, s, n, ih, iw, c, val, best);
        if (ih >= own_lo && ih < own_hi) {
          stv<T, V>((T*)wsb + s.out_off + e, val);
          if (s.kind == CSRC_MAXPOOL) store_winners<V>((uint8_t*)wsb + s.arg_off + e, best);
        }
      }
    }
    put<V>(lds + pix * CS + c, val);
  }
}

template <typename T, bool POOL, int NTH>
__device__ __forceinline__ void load_patch(float* lds, const CompactSrc& s, char* wsb, const float* img, const float* mean, int n, int ih0,
                                           int rows, int iw0, int cols, FastDiv by_cols, int CS, int own_lo, int own_hi) {
  if (s.kind == CSRC_IMAGES) {            // the caller's NCHW images: neighbouring lanes on neighbouring columns
    const int total = rows * cols;
    for (int idx = threadIdx.x; idx < total; idx += NTH) {
      const int r = by_cols(idx), q = idx - r * cols;
      const int ih = ih0 + r, iw = iw0 + q;
      const bool in = (unsigned)ih < (unsigned)s.H && (unsigned)iw < (unsigned)s.W;
      const uint32_t pixel = in ? (uint32_t)(ih * s.W + iw) : 0u, plane = (uint32_t)(s.H * s.W);
      const float* im = img + (uint32_t)n * s.C * plane;
      for (int c0 = 0; c0 < s.C; c0 += 4) {            // the channels of a pixel four at a time
        float f[4];
#pragma unroll
        for (int e = 0; e < 4; e++) f[e] = c0 + e < s.C ? im[pixel + (c0 + e) * plane] : 0.f;
        if (mean)
#pragma unroll
          for (int e = 0; e < 4; e++) f[e] -= c0 + e < s.C ? mean[pixel + (c0 + e) * plane] : 0.f;
#pragma unroll
        for (int e = 0; e < 4; e++)
          if (c0 + e < s.C) lds[idx * CS + c0 + e] = in ? stored(f[e], (const T*)nullptr) : 0.f;
      }
    }
  } else if (s.C % 4 == 0) {
    load_patch_v<T, 4, POOL, NTH>(lds, s, wsb, n, ih0, rows, iw0, cols, by_cols, CS, own_lo, own_hi);
  } else {
    load_patch_v<T, 1, POOL, NTH>(lds, s, wsb, n, ih0, rows, iw0, cols, by_cols, CS, own_lo, own_hi);
  }
  if (s.C & 3) zero_channels<NTH>(lds, rows * cols, s.C, CS);
}

// ---------------------------------------------------------------- gradient of a convolution's output
// V channels from c at output position (oh, ow): as stored, or through the pooling layer behind the convolution (at most two
// windows per direction reach a position), masked by the convolution's ReLU, rounded to T.  In two steps, so that a caller can
// put other loads between the requests and their use.
template <typename T, int V>
struct GradAt {
  float d[4][V], mk[V];                  // windows' gradients, the ReLU's output
  uint32_t won[4];
  // Where a gradient that is read as stored goes.  Four channels: to mk's place (two arrays, read in two branches, were merged into
  // one read with a selected destination, and both went to scratch memory: 68 -> 61 us of a 5 x 5 layer of 64 channels).  One
  // channel of bf16: to d's (13 channels, 18 learners x 32 images: 222 us in mk's place, 206 here; fp32 is level, 201 and 202).
  __device__ __forceinline__ const float (&plain() const)[V] {
    if constexpr (V == 1 && sizeof(T) == 2) return d[0];
    else return mk;
  }

  __device__ __forceinline__ void request(const char* wsb, const CompactGrad& g, int n, int oh, int ow, int c) {
    const T* dp = (const T*)wsb + g.off;
    const uint32_t e = ((uint32_t)(n * g.OH + oh) * g.OW + ow) * g.K + c;
    if (g.kind == CGRAD_PLAIN) {
      ldv<T, V>(dp + e, const_cast<float (&)[V]>(plain()));
      return;
    }
    const uint8_t* arg = (const uint8_t*)wsb + g.arg_off;
    const int ph_hi = g.by_pst(oh), pw_hi = g.by_pst(ow);
#pragma unroll
    for (int q = 0; q < 4; q++) {         // windows in ascending order; absent ones read a clamped address and are not used
      const int ph = min(max(ph_hi - 1 + q / 2, 0), g.PH - 1), pw = min(max(pw_hi - 1 + q % 2, 0), g.PW - 1);
      const uint32_t o = ((uint32_t)(n * g.PH + ph) * g.PW + pw) * g.K + c;
      ldv<T, V>(dp + o, d[q]);
      if (g.kind == CGRAD_MAXPOOL) {
        if constexpr (V == 1) won[q] = arg[o];
        else won[q] = *reinterpret_cast<const uint32_t*>(arg + o);
      }
    }
    if (g.use_mask) ldv<T, V>((const T*)wsb + g.mask_off + e, mk);
  }

  __device__ __forceinline__ void value(const CompactGrad& g, int oh, int ow, float (&val)[V]) const {
    if (g.kind == CGRAD_PLAIN) {
#pragma unroll
      for (int v = 0; v < V; v++) val[v] = plain()[v];
      return;
    }
    const int ph_hi = g.by_pst(oh), pw_hi = g.by_pst(ow);
#pragma unroll
    for (int v = 0; v < V; v++) val[v] = 0.f;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int ph = ph_hi - 1 + q / 2, pw = pw_hi - 1 + q % 2, h0 = ph * g.pst, w0 = pw * g.pst;
      const bool ok = ph >= 0 && ph < g.PH && pw >= 0 && pw < g.PW && oh - h0 < g.pks && ow - w0 < g.pks;
      const uint32_t pos = (uint32_t)((oh - h0) * g.pks + (ow - w0));
      const float inv = g.kind == CGRAD_MAXPOOL ? 1.f : 1.f / (float)((min(h0 + g.pks, g.OH) - h0) * (min(w0 + g.pks, g.OW) - w0));
#pragma unroll
      for (int v = 0; v < V; v++) {
        if (g.kind == CGRAD_MAXPOOL) {
          if (ok && ((won[q] >> (8 * v)) & 0xffu) == pos) val[v] += d[q][v];
        } else if (ok) {
          val[v] += d[q][v] * inv;
        }
      }
    }
#pragma unroll
    for (int v = 0; v < V; v++) {
      if (g.use_mask && !(mk[v] > 0.f)) val[v] = 0.f;
      val[v] = stored(val[v], (const T*)nullptr);
    }
  }
};

template <typename T, int V, int NTH>
__device__ __forceinline__ void load_grad_patch_v(float* lds, const CompactGrad& g, const char* wsb, int n, int oh0, int rows, int ow0, int cols,
                                                  FastDiv by_cols, int CS) {
  const int cg = g.K / V, total = rows * cols * cg;
  const FastDiv by_cg = V == 4 ? g.by_k4 : g.by_k;
  for (int idx = threadIdx.x; idx < total; idx += NTH) {
    const int pix = by_cg(idx), c = (idx - pix * cg) * V;
    const int r = by_cols(pix), q = pix - r * cols;
    const int oh = oh0 + r, ow = ow0 + q;
    float val[V];
#pragma unroll
    for (int v = 0; v < V; v++) val[v] = 0.f;
    if ((unsigned)oh < (unsigned)g.OH && (unsigned)ow < (unsigned)g.OW) {
      GradAt<T, V> ga;
      ga.request(wsb, g, n, oh, ow, c);
      ga.value(g, oh, ow, val);
    }
    put<V>(lds + pix * CS + c, val);
  }
}
template <typename T, int NTH>
__device__ __forceinline__ void load_grad_patch(float* lds, const CompactGrad& g, const char* wsb, int n, int oh0, int rows, int ow0, int cols,
                                                FastDiv by_cols, int CS) {
  if (g.K % 4 == 0) load_grad_patch_v<T, 4, NTH>(lds, g, wsb, n, oh0, rows, ow0, cols, by_cols, CS);
  else load_grad_patch_v<T, 1, NTH>(lds, g, wsb, n, oh0, rows, ow0, cols, by_cols, CS);
  if (g.K & 3) zero_channels<NTH>(lds, rows * cols, g.K, CS);
}

// ---------------------------------------------------------------- one filter row of the B operand
// KS consecutive values of the flat filter at byte offset `off` of the resource (out of range: zeros).
template <int KS>
__device__ __forceinline__ void fetch_row(__amdgpu_buffer_rsrc_t r, int off, float (&b)[KS], const float*) {
  int k = 0;
#pragma unroll
  for (; k + 4 <= KS; k += 4) {
    const v4i_t q = __builtin_amdgcn_raw_buffer_load_b128(r, off, k * 4, 0);
    b[k] = __int_as_float(q.x); b[k + 1] = __int_as_float(q.y); b[k + 2] = __int_as_float(q.z); b[k + 3] = __int_as_float(q.w);
  }
  if constexpr (KS % 4 == 3) {
    const v3i_t q = __builtin_amdgcn_raw_buffer_load_b96(r, off, k * 4, 0);
    b[KS - 3] = __int_as_float(q.x); b[KS - 2] = __int_as_float(q.y); b[KS - 1] = __int_as_float(q.z);
  } else if constexpr (KS % 4 == 2) {
    const v2i_t q = __builtin_amdgcn_raw_buffer_load_b64(r, off, k * 4, 0);
    b[KS - 2] = __int_as_float(q.x); b[KS - 1] = __int_as_float(q.y);
  } else if constexpr (KS % 4 == 1) {
    b[KS - 1] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, k * 4, 0));
  }
}
template <int KS>
__device__ __forceinline__ void fetch_row(__amdgpu_buffer_rsrc_t r, int off, float (&b)[KS], const bf16_t*) {
#pragma unroll
  for (int k = 0; k < KS; k++) b[k] = bf2f((bf16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, k * 2, 0));
}

// ---------------------------------------------------------------- a tile of convolution output
// 16 MT output positions of one image x 16 NT output channels per group of KW wavefronts, NW / KW such groups along the
// positions.  The wavefronts of a group take the contraction's units (four channels, one filter row) in turn: lane quarter q
// multiplies channel 4 quad + q, KS matrix instructions per unit and 16 x 16 block.  B
// comes straight from the flat filter, one contiguous filter row per lane, requested one unit ahead (the first one before the
// patch is loaded).
struct TileGeom {
  int C;                 // contraction channels
  int K;                 // output channels
  int OH, OW;            // output positions
  int cols;              // patch columns
  int CS;                // floats per patch pixel
  int stride;
  int sn, sc;            // filter strides (elements) of an output channel and of a contraction channel
  FastDiv by_ow;
};

template <typename T, int KS, int MT, int NT, int NW, int KW, bool FLIP>
struct ConvTile {
  static constexpr int kPositions = 16 * MT * (NW / KW), kElems = kPositions * 16 * NT;
  float b[2][NT][KS];
  const T* flat;
  int w_off, w_end, n0, units;

  __device__ __forceinline__ void fetch(float (&row)[NT][KS], int u, const TileGeom& g) {
    if (u >= units) return;               // uniform
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)flat, 0, (int)(w_end * sizeof(T)), 0x00020000);
    const int lane = threadIdx.x & 63, quad = u / KS, kh = u - quad * KS, c = 4 * quad + (lane >> 4);
#pragma unroll
    for (int j = 0; j < NT; j++) {
      const int n = n0 + 16 * j + (lane & 15);
      const int off = (c < g.C && n < g.K) ? (w_off + n * g.sn + c * g.sc + (FLIP ? KS - 1 - kh : kh) * KS) * (int)sizeof(T) : (int)kOOB;
      fetch_row<KS>(rw, off, row[j], (const T*)nullptr);
    }
  }
  __device__ __forceinline__ void begin(const T* flat_, int w_off_, int w_elems, const TileGeom& g, int n0_) {
    flat = flat_;
    w_off = w_off_;
    w_end = w_off_ + w_elems;
    n0 = n0_;
    units = ((g.C + 3) >> 2) * KS;
    fetch(b[0], __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % KW, g);
  }
  // after the patch has been written (the barrier is in here)
  __device__ __forceinline__ void run(float* lds, const TileGeom& g, int p0, int r0) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15, q = lane >> 4;
    const int first = wave % KW;
    floatx4 acc[MT][NT];
    int base[MT];
#pragma unroll
    for (int i = 0; i < MT; i++) {
      const int p = min(p0 + (wave / KW * MT + i) * 16 + col, g.OH * g.OW - 1);    // rows beyond the image repeat its last position, never stored
      const int oh = g.by_ow(p), ow = p - oh * g.OW;
      base[i] = ((oh - r0) * g.cols + ow) * g.stride * g.CS + q;
#pragma unroll
      for (int j = 0; j < NT; j++)
#pragma unroll
        for (int r = 0; r < 4; r++) acc[i][j][r] = 0.f;
    }
    auto multiply = [&](const float (&row)[NT][KS], int u) {
      const int quad = u / KS, kh = u - quad * KS;
      const float* a0 = lds + kh * g.cols * g.CS + 4 * quad;
      float a[KS][MT];
#pragma unroll
      for (int kw = 0; kw < KS; kw++)
#pragma unroll
        for (int i = 0; i < MT; i++) a[kw][i] = a0[base[i] + kw * g.CS];
#pragma unroll
      for (int kw = 0; kw < KS; kw++)
#pragma unroll
        for (int i = 0; i < MT; i++)
#pragma unroll
          for (int j = 0; j < NT; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[kw][i], row[j][FLIP ? KS - 1 - kw : kw], acc[i][j], 0, 0, 0);
    };
    __syncthreads();
#pragma unroll 1
    for (int u = first; u < units; u += 2 * KW) {
      fetch(b[1], u + KW, g);
      multiply(b[0], u);
      if (u + KW >= units) break;
      fetch(b[0], u + 2 * KW, g);
      multiply(b[1], u + KW);
    }
    // the wavefronts' partial tiles: element (position m, channel n) of the tile at m * 16 NT + n
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++)
#pragma unroll
        for (int r = 0; r < 4; r++) lds[wave * (256 * MT * NT) + (16 * i + 4 * q + r) * (16 * NT) + 16 * j + col] = acc[i][j][r];
    __syncthreads();
  }
  static __device__ __forceinline__ float sum(const float* lds, int e) {   // element (position, channel), in wavefront order
    const float* part = lds + e / (256 * MT * NT) * ((KW - 1) * 256 * MT * NT) + e;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < KW; w++) v += part[w * (256 * MT * NT)];
    return v;
  }
};

// ---------------------------------------------------------------- forward
template <typename T, int KS, int MT, int NT, int NW, int KW>
__global__ __launch_bounds__(64 * NW, 4) void compact_fwd_kernel(PtrTab ws, CPtrTab wts, CPtrTab imgs, CompactConv v, CompactSrc src, int relu,
                                                                size_t y_off, const float* mean) {
  extern __shared__ __attribute__((aligned(16))) float compact_lds[];
  float* lds = compact_lds;
  const int z = blockIdx.z;
  char* wsb = (char*)ws.p[z];
  const T* W = (const T*)wts.p[z];
  typedef ConvTile<T, KS, MT, NT, NW, KW, false> Tile;
  constexpr int M = Tile::kPositions;
  const int OHW = v.OH * v.OW, tiles = (OHW + M - 1) / M;
  const int n = blockIdx.x / tiles, t = blockIdx.x - n * tiles;
  const int p0 = t * M, p1 = min(p0 + M, OHW) - 1;
  const int r0 = v.by_ow(p0), r1 = v.by_ow(p1);
  TileGeom g;
  g.C = v.C; g.K = v.K; g.OH = v.OH; g.OW = v.OW;
  g.cols = (v.OW - 1) * v.stride + KS;
  g.CS = compact_pixel_stride(v.C);
  g.stride = v.stride;
  g.sn = v.C * KS * KS; g.sc = KS * KS;
  g.by_ow = v.by_ow;
  const int n0 = blockIdx.y * 16 * NT;
  Tile tile;
  tile.begin(W, (int)v.w_off, v.K * g.sn, g, n0);
  // pooled rows this workgroup keeps for the backward pass: from behind the previous tile's last row to its own last row
  const int last = r1 * v.stride - v.pad + KS, prev = t == 0 ? 0 : v.by_ow(p0 - 1) * v.stride - v.pad + KS;
  const bool owner = blockIdx.y == 0;
  load_patch<T, true, 64 * NW>(lds, src, wsb, (const float*)imgs.p[z], mean, n, r0 * v.stride - v.pad, (r1 - r0) * v.stride + KS, -v.pad, g.cols,
                               v.by_cols, g.CS, owner ? prev : 0, owner ? (t == tiles - 1 ? v.H : last) : 0);
  tile.run(lds, g, p0, r0);
  T* y = (T*)wsb + y_off;
  for (int e = threadIdx.x; e < Tile::kElems; e += 64 * NW) {
    const int p = p0 + e / (16 * NT), nn = n0 + e % (16 * NT);
    if (p > p1 || nn >= v.K) continue;
    float f = Tile::sum(lds, e) + ldf(W + v.b_off + nn);
    if (relu) f = fmaxf(f, 0.f);
    stf(y + ((uint32_t)(n * OHW + p) * v.K + nn), f);
  }
}

// ---------------------------------------------------------------- weight and bias gradient
// Workgroup: 32 output channels x up to NW column blocks of 32 filter columns j = tap * C + c, over every splits-th tile of
// bw.tile output positions.  Rows of the product are channels of dy, columns filter elements, the contraction runs over positions.
// A wavefront has one column block and, where there are few of them (first layers), a share of the positions.
template <typename T, int KS, int NW>
__device__ __forceinline__ void wgrad_part(float* lds, char* wsb, const float* img, const float* mean, float* dst, const CompactConv& v,
                                           const CompactSrc& x, const CompactGrad& gr, int nblk, int cblk, int sp, const CompactBwd& bw) {
  constexpr int NTH = 64 * NW;
  const int PT = bw.tile, splits = bw.splits, per = bw.blocks_per_group;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 31, h = lane >> 5;
  const int OHW = v.OH * v.OW, tiles = (OHW + PT - 1) / PT, total = v.N * tiles;
  const int cols = (v.OW - 1) * v.stride + KS, CS = compact_pixel_stride(v.C);
  const int ncol = KS * KS * v.C, cblocks = (ncol + 31) / 32;
  const int mine = min(cblocks - cblk * per, per);              // column blocks of this workgroup
  const int cgw = wgrad_waves_across(mine, NW), PG = NW / cgw;
  const int cgi = wave & (cgw - 1), pg = wave / cgw;
  const bool active = cgi < mine;
  const int n0 = nblk * 32;
  const int j = (cblk * per + cgi) * 32 + col;
  int koff = 0;
  if (j < ncol) {
    const int tap = x.by_c(j), kh = tap / KS;
    koff = (kh * cols + (tap - kh * KS)) * CS + (j - tap * v.C);
  }
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; r++) acc[r] = 0.f;
  float bsum = 0.f;
  float* dyt = lds;                                           // [PT][kDyLd]
  int* ptab = reinterpret_cast<int*>(lds + PT * kDyLd);       // window origin of each position in the patch
  float* patch = lds + PT * kDyLd + PT;
  for (int it = sp; it < total; it += splits) {
    const int n = it / tiles, p0 = (it - n * tiles) * PT, p1 = min(p0 + PT, OHW) - 1;
    const int r0 = v.by_ow(p0), r1 = v.by_ow(p1);
    // the first dy values are requested, then the patch is loaded, then they are turned into gradients
    auto both = [&](auto width) {
      constexpr int V = decltype(width)::value;
      const int TOT = 32 / V * PT;
      GradAt<T, V> ga;
      int idx = threadIdx.x, oh = 0, ow = 0;
      bool ok = false;
      auto request = [&]() {
        const int p = p0 + idx / (32 / V), c = n0 + (idx % (32 / V)) * V;
        ok = idx < TOT && p <= p1 && c < v.K;
        oh = v.by_ow(p);
        ow = p - oh * v.OW;
        if (ok) ga.request(wsb, gr, n, oh, ow, c);
      };
      auto finish = [&]() {
        float val[V];
#pragma unroll
        for (int e = 0; e < V; e++) val[e] = 0.f;
        if (ok) ga.value(gr, oh, ow, val);
        if (idx < TOT) put<V>(dyt + (idx / (32 / V)) * kDyLd + (idx % (32 / V)) * V, val);
      };
      request();
      load_patch<T, false, NTH>(patch, x, wsb, img, mean, n, r0 * v.stride - v.pad, (r1 - r0) * v.stride + KS, -v.pad, cols, v.by_cols, CS, 0, 0);
      finish();
#pragma unroll 1
      for (idx += NTH; idx < TOT; idx += NTH) {
        request();
        finish();
      }
    };
    if (gr.K % 4 == 0) both(std::integral_constant<int, 4>{});
    else both(std::integral_constant<int, 1>{});
    if ((int)threadIdx.x < PT) {
      const int p = min(p0 + (int)threadIdx.x, p1), oh = v.by_ow(p), ow = p - oh * v.OW;
      ptab[threadIdx.x] = ((oh - r0) * cols + ow) * v.stride * CS;
    }
    __syncthreads();
    if (active) {
      for (int k = pg; k < PT / 2; k += PG) {
        const float a = dyt[(2 * k + h) * kDyLd + col], b = patch[ptab[2 * k + h] + koff];
        bsum += a;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
      }
    }
    __syncthreads();
  }
  // shares of the positions: halve until one is left
  for (int s = PG >> 1; s >= 1; s >>= 1) {
    if (pg >= s && pg < 2 * s) {
      float* red = lds + ((pg - s) * cgw + cgi) * kRedFloats;
#pragma unroll
      for (int r = 0; r < 16; r++) red[r * 64 + lane] = acc[r];
      red[1024 + lane] = bsum;
    }
    __syncthreads();
    if (pg < s) {
      const float* from = lds + (pg * cgw + cgi) * kRedFloats;
#pragma unroll
      for (int r = 0; r < 16; r++) acc[r] += from[r * 64 + lane];
      bsum += from[1024 + lane];
    }
    __syncthreads();
  }
  if (pg != 0 || !active) return;
  // partial sums [K][KS KS C + 1], the bias behind a channel's columns; compact_finish_kernel puts them in flat order (stored
  // in flat order from here every lane's element would lie in a cache line of its own)
  if (j < ncol) {
#pragma unroll
    for (int r = 0; r < 16; r++) {
      const int nn = n0 + 8 * (r >> 2) + 4 * h + (r & 3);
      if (nn < v.K) dst[(uint32_t)nn * (ncol + 1) + j] = acc[r];
    }
  }
  if (cblk == 0 && cgi == 0) {                                // bias gradient: the two lane halves hold odd and even positions
    bsum += __shfl_xor(bsum, 32, 64);
    if (h == 0 && n0 + col < v.K) dst[(uint32_t)(n0 + col) * (ncol + 1) + ncol] = bsum;
  }
}

// Input gradient (workgroups 0 .. dgrad_blocks - 1) and weight gradient (the rest) of one layer.
template <typename T, int KS, int MT, int NT, int NW, int KW>
__global__ __launch_bounds__(64 * NW, 4) void compact_bwd_kernel(PtrTab ws, CPtrTab wts, CPtrTab imgs, CompactConv v, CompactSrc x, CompactGrad gr,
                                                                CompactBwd bw, const float* mean) {
  extern __shared__ __attribute__((aligned(16))) float compact_lds[];
  float* lds = compact_lds;
  const int z = blockIdx.z;
  char* wsb = (char*)ws.p[z];
  if ((int)blockIdx.x < bw.dgrad_blocks) {
    typedef ConvTile<T, KS, MT, NT, NW, KW, true> Tile;
    constexpr int M = Tile::kPositions;
    const int HW = v.H * v.W, tiles = (HW + M - 1) / M, cb = (v.C + 16 * NT - 1) / (16 * NT);
    const int i = blockIdx.x / cb, c0 = (blockIdx.x - i * cb) * 16 * NT;
    const int n = i / tiles, p0 = (i - n * tiles) * M, p1 = min(p0 + M, HW) - 1;
    const int r0 = v.by_w(p0), r1 = v.by_w(p1), pad = KS - 1 - v.pad;
    TileGeom g;
    g.C = v.K; g.K = v.C; g.OH = v.H; g.OW = v.W;
    g.cols = v.W - 1 + KS;
    g.CS = compact_pixel_stride(v.K);
    g.stride = 1;
    g.sn = KS * KS; g.sc = v.C * KS * KS;
    g.by_ow = v.by_w;
    Tile tile;
    tile.begin((const T*)wts.p[z], (int)v.w_off, v.K * g.sc, g, c0);
    load_grad_patch<T, 64 * NW>(lds, gr, wsb, n, r0 - pad, r1 - r0 + KS, -pad, g.cols, v.by_dcols, g.CS);
    tile.run(lds, g, p0, r0);
    T* dx = (T*)wsb + bw.dx_off;
    const T* mask = (const T*)wsb + bw.mask_off;
    for (int e = threadIdx.x; e < Tile::kElems; e += 64 * NW) {
      const int p = p0 + e / (16 * NT), c = c0 + e % (16 * NT);
      if (p > p1 || c >= v.C) continue;
      const uint32_t o = (uint32_t)(n * HW + p) * v.C + c;
      float f = Tile::sum(lds, e);
      if (bw.use_mask && !(ldf(mask + o) > 0.f)) f = 0.f;
      stf(dx + o, f);
    }
    return;
  }
  const int id = blockIdx.x - bw.dgrad_blocks, nb = (v.K + 31) / 32;
  const int sp = id / (nb * bw.col_groups), rest = id - sp * nb * bw.col_groups;
  float* dst = reinterpret_cast<float*>(wsb + bw.part_off) + (int64_t)sp * bw.part_elems;
  wgrad_part<T, KS, NW>(lds, wsb, (const float*)imgs.p[z], mean, dst, v, x, gr, rest % nb, rest / nb, sp, bw);
}

// ---------------------------------------------------------------- pooling / flattening in front of a fully connected layer
// x [N][C H W] in (C, H, W) order from a pooled or plain NHWC tensor; one thread per element, channels innermost.
template <typename T>
__global__ __launch_bounds__(256) void compact_flatten_kernel(PtrTab ws, CompactSrc s, size_t flat_off, int N) {
  char* wsb = (char*)ws.p[blockIdx.z];
  const int64_t total = (int64_t)N * s.H * s.W * s.C;
  const int HW = s.H * s.W;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int c = (int)(i % s.C), pix = (int)(i / s.C), n = pix / HW, hw = pix - n * HW;
    float val[1];
    if (s.kind == CSRC_TENSOR) {
      val[0] = ldf((const T*)wsb + s.off + i);
    } else {
      uint32_t best[1];
      pooled_at<T, 1>((const T*)wsb + s.off, s, n, hw / s.W, hw % s.W, c, val, best);
      stf((T*)wsb + s.out_off + i, val[0]);
      if (s.kind == CSRC_MAXPOOL) *((uint8_t*)wsb + s.arg_off + i) = (uint8_t)best[0];
    }
    stf((T*)wsb + flat_off + ((int64_t)n * s.C + c) * HW + hw, val[0]);
  }
}

// ---------------------------------------------------------------- last fully connected layer, softmax, loss, input gradient
// One workgroup per image, whose inputs stay in LDS; a wavefront takes two classes at a time.  rank_out: evaluation.
template <typename T, int V, int TH>
__global__ __launch_bounds__(TH) void compact_head_kernel(PtrTab ws, CPtrTab wts, CPtrTab labels, CompactSrc src, CompactHead hd, int32_t* rank_out) {
  extern __shared__ __attribute__((aligned(16))) float compact_lds[];
  float* xs = compact_lds;                        // [in]
  float* zs = compact_lds + ((hd.in + 3) & ~3);   // [K] scores, then their gradient
  __shared__ float red[TH / 64];
  const int z = blockIdx.z, n = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  char* wsb = (char*)ws.p[z];
  const T* W = (const T*)wts.p[z] + hd.w_off;
  const T* B = (const T*)wts.p[z] + hd.b_off;
  const int in = hd.in, K = hd.K;
  if (src.kind == CSRC_FLAT) {
    const T* x = (const T*)wsb + src.off + (uint32_t)n * in;
    for (int i = tid * V; i < in; i += TH * V) {
      float f[V];
      ldv<T, V>(x + i, f);
      put<V>(xs + i, f);
    }
  } else {
    const int HW = src.H * src.W;
    T* xf = (T*)wsb + hd.flat_off + (uint32_t)n * in;
    for (int i = tid * V; i < in; i += TH * V) {           // i = pixel * C + channel
      const int hw = src.by_c(i), c = i - hw * src.C;
      const uint32_t e = (uint32_t)n * in + i;
      float val[V];
      if (src.kind == CSRC_TENSOR) {
        ldv<T, V>((const T*)wsb + src.off + e, val);
      } else {
        uint32_t best[V];
        pooled_at<T, V>((const T*)wsb + src.off, src, n, hw / src.W, hw % src.W, c, val, best);
        if (src.kind == CSRC_MAXPOOL) store_winners<V>((uint8_t*)wsb + src.arg_off + e, best);
      }
#pragma unroll
      for (int v = 0; v < V; v++) {
        xs[(c + v) * HW + hw] = val[v];
        stf(xf + (c + v) * HW + hw, val[v]);
      }
    }
  }
  const int y = ((const int32_t*)labels.p[z])[n];
  __syncthreads();
  for (int k0 = wave * 2; k0 < K; k0 += 2 * (TH / 64)) {
    const T *w0 = W + (uint32_t)k0 * in, *w1 = W + (uint32_t)min(k0 + 1, K - 1) * in;
    float a0 = 0.f, a1 = 0.f;
#pragma unroll 4
    for (int i = lane * V; i < in; i += 64 * V) {
      float f0[V], f1[V];
      ldv<T, V>(w0 + i, f0);
      ldv<T, V>(w1 + i, f1);
#pragma unroll
      for (int v = 0; v < V; v++) {
        a0 = fmaf(xs[i + v], f0[v], a0);
        a1 = fmaf(xs[i + v], f1[v], a1);
      }
    }
    a0 = wave_sum(a0);
    a1 = wave_sum(a1);
    if (lane == 0) {
      zs[k0] = a0 + ldf(B + k0);
      if (k0 + 1 < K) zs[k0 + 1] = a1 + ldf(B + k0 + 1);
    }
  }
  __syncthreads();
  const bool y_ok = y >= 0 && y < K;
  float m = -INFINITY;
  for (int j = lane; j < K; j += 64) m = fmaxf(m, zs[j]);     // every wavefront on its own: no barrier
  m = wave_max(m);
  float sum = 0.f;
  for (int j = lane; j < K; j += 64) sum += expf(zs[j] - m);
  sum = wave_sum(sum);
  if (tid == 0) reinterpret_cast<float*>(wsb + hd.loss_off)[n] = y_ok ? -(zs[y] - m - logf(sum)) : NAN;   // a bad label poisons the loss
  if (rank_out) {
    int cnt = 0;
    const float zy = y_ok ? zs[y] : 0.f;
    for (int j = tid; j < K; j += TH) cnt += (zs[j] > zy || (zs[j] == zy && j < y)) ? 1 : 0;
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_down(cnt, o, 64);
    if (lane == 0) red[wave] = (float)cnt;
    __syncthreads();
    if (tid == 0) {
      float tot = 0.f;
#pragma unroll
      for (int w = 0; w < TH / 64; w++) tot += red[w];
      rank_out[(int64_t)z * hd.N + n] = y_ok ? (int)tot : K;
    }
    return;
  }
  __syncthreads();
  const float inv = 1.0f / sum, invN = 1.0f / (float)hd.N;
  T* dz = (T*)wsb + hd.dz_off + (uint32_t)n * K;
  for (int j = tid; j < K; j += TH) {
    const float d = stored((expf(zs[j] - m) * inv - (j == y ? 1.f : 0.f)) * invN, (const T*)nullptr);
    stf(dz + j, d);
    zs[j] = d;                                    // each score is read and replaced by its own thread
  }
  __syncthreads();
  T* dx = (T*)wsb + hd.dx_off + (uint32_t)n * in;
  for (int i = tid * V; i < in; i += TH * V) {
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; v++) acc[v] = 0.f;
#pragma unroll 5
    for (int k = 0; k < K; k++) {
      float f[V];
      ldv<T, V>(W + (uint32_t)k * in + i, f);
#pragma unroll
      for (int v = 0; v < V; v++) acc[v] = fmaf(zs[k], f[v], acc[v]);
    }
    // stored channels innermost, as the convolution below reads it
#pragma unroll
    for (int v = 0; v < V; v++) {
      if (hd.use_mask && !(xs[i + v] > 0.f)) acc[v] = 0.f;
      const int c = hd.by_hw(i + v), hw = i + v - c * hd.HW;
      stf(dx + hw * hd.C + c, acc[v]);
    }
  }
}

// ---------------------------------------------------------------- hidden fully connected layers
// Tiles of 16 images x 16 columns; the 16 wavefronts divide the contraction in steps of 16 (lane quarter q holds four
// consecutive elements from 4 q: four matrix instructions a step), operands straight from memory.  Bound by the rate at which
// the few workgroups read the weights (16 of them: 64 GB/s each), hence f.splits workgroups along the contraction where there
// are few tiles; compact_fc_sum_kernel then adds their partial tiles.
//   forward         y[n][u]  = sum_i x[n][i] W[u][i]       columns = units, both operands contiguous along the contraction
//   input gradient  dx[n][i] = sum_k dy[n][k] W[k][i]      columns = inputs, a step reads four weight rows per lane quarter
template <typename T>
__device__ __forceinline__ void fetch4(const T* p, int left, bool ok, bool aligned, float (&f)[4]) {   // zeros beyond `left` elements
  if (aligned) {
#pragma unroll
    for (int e = 0; e < 4; e++) f[e] = 0.f;
    if (ok && left > 0) ldv<T, 4>(p, f);
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++) f[e] = ok && e < left ? ldf(p + e) : 0.f;
  }
}
template <typename T, bool DGRAD>
__device__ __forceinline__ void fc_store(char* wsb, const T* wts, const CompactFc& f, int n, int c, float s) {
  if (DGRAD) {
    if (f.use_mask && !(ldf((const T*)wsb + f.x_off + (uint32_t)n * f.in + c) > 0.f)) s = 0.f;
    // behind a flattening: channels innermost.  A plain division: c goes up to channels x pixels, beyond what FastDiv divides
    const int ch = c / f.HW, hw = c - ch * f.HW;
    stf((T*)wsb + f.dx_off + (uint32_t)n * f.in + hw * (f.in / f.HW) + ch, s);
  } else {
    s += ldf(wts + f.b_off + c);
    if (f.relu) s = fmaxf(s, 0.f);
    stf((T*)wsb + f.y_off + (uint32_t)n * f.out + c, s);
  }
}
template <typename T, bool DGRAD>
__global__ __launch_bounds__(1024) void compact_fc_kernel(PtrTab ws, CPtrTab wts, CompactFc f) {
  __shared__ float red[16 * 256];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15, q = lane >> 4, z = blockIdx.z;
  char* wsb = (char*)ws.p[z];
  const T* W = (const T*)wts.p[z] + f.w_off;
  const int K = DGRAD ? f.out : f.in, C = DGRAD ? f.in : f.out;       // contraction length, columns
  const int rows = (f.N + 15) / 16, sp = blockIdx.y / rows, row = blockIdx.y - sp * rows;
  const int c = blockIdx.x * 16 + col, n = row * 16 + col;            // this lane's column (B) and image (A)
  const T* a = (const T*)wsb + (DGRAD ? f.dy_off : f.x_off) + (uint32_t)n * K;
  const bool a_ok = n < f.N, c_ok = c < C;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 4;                                                // steps whose operands are requested together
  const int step = 256 * f.splits;
#pragma unroll 1
  for (int k = (sp * 16 + wave) * 16; k < K; k += U * step) {
    float av[U][4], bv[U][4];
#pragma unroll
    for (int t = 0; t < U; t++) {
      const int k0 = k + t * step + 4 * q;                            // beyond K: zeros
      fetch4(a + k0, K - k0, a_ok, f.aligned, av[t]);
      if (DGRAD) {
#pragma unroll
        for (int e = 0; e < 4; e++) bv[t][e] = c_ok && k0 + e < K ? ldf(W + (uint32_t)(k0 + e) * f.in + c) : 0.f;
      } else {
        fetch4(W + (uint32_t)c * f.in + k0, K - k0, c_ok, f.aligned, bv[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < U; t++)
#pragma unroll
      for (int e = 0; e < 4; e++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t][e], bv[t][e], acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; r++) red[wave * 256 + (4 * q + r) * 16 + col] = acc[r];
  __syncthreads();
  const int e = threadIdx.x;
  if (e >= 256) return;
  const int nn = row * 16 + e / 16, cc = blockIdx.x * 16 + e % 16;
  if (nn >= f.N || cc >= C) return;
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < 16; w++) s += red[w * 256 + e];
  if (f.splits > 1) reinterpret_cast<float*>(wsb + f.part_off)[((uint32_t)sp * f.N + nn) * C + cc] = s;
  else fc_store<T, DGRAD>(wsb, (const T*)wts.p[z], f, nn, cc, s);
}
template <typename T, bool DGRAD>
__global__ __launch_bounds__(64) void compact_fc_sum_kernel(PtrTab ws, CPtrTab wts, CompactFc f) {
  const int z = blockIdx.z, C = DGRAD ? f.in : f.out, total = f.N * C, i = blockIdx.x * 64 + threadIdx.x;
  if (i >= total) return;
  char* wsb = (char*)ws.p[z];
  const float* part = reinterpret_cast<const float*>(wsb + f.part_off) + i;
  float s = 0.f;
#pragma unroll 8
  for (int sp = 0; sp < f.splits; sp++) s += part[(int64_t)sp * total];
  const int n = i / C;
  fc_store<T, DGRAD>(wsb, (const T*)wts.p[z], f, n, i - n * C, s);
}

// ---------------------------------------------------------------- everything that is left at the end
// Jobs one after the other in the launch index: sums of split weight gradients (a split's partial lies as wgrad_part left it, a
// channel's columns by tap and then its bias: read in that order, each sum written to its place in the flat order), fully
// connected weight gradients (kFinU output units per thread, their dy of up to kFinN images in LDS), mean losses.
constexpr int kFinU = 8, kFinN = 32;
template <typename T>
__global__ __launch_bounds__(256) void compact_finish_kernel(PtrTab ws, PtrTab grads, CompactFinish fin, size_t loss_off, int N, float* loss_out) {
  const int z = blockIdx.z;
  char* wsb = (char*)ws.p[z];
  int j = 0;
  while (j + 1 < fin.count && (int)blockIdx.x >= fin.job[j + 1].first_block) j++;
  const CompactJob& jb = fin.job[j];
  const int b = blockIdx.x - jb.first_block;
  if (jb.kind == CJOB_SUM) {                       // element (channel n, column j = tap C + c, or the bias behind the columns)
    // many splits: dealt out to jb.groups groups of lanes, which take four each a round (two rounds for 64 splits, eight for 256)
    __shared__ float red[256];
    const int per = 256 / jb.groups, g = threadIdx.x / per, e = threadIdx.x - g * per, i = b * per + e;
    const float* part = reinterpret_cast<const float*>(wsb + jb.part_off) + min(i, (int)jb.elems - 1);
    float s = 0.f;
    for (int s0 = g; s0 < jb.splits; s0 += 4 * jb.groups) {
      float f[4];
#pragma unroll
      for (int u = 0; u < 4; u++) f[u] = part[(int64_t)min(s0 + u * jb.groups, jb.splits - 1) * jb.elems];
#pragma unroll
      for (int u = 0; u < 4; u++) s += s0 + u * jb.groups < jb.splits ? f[u] : 0.f;
    }
    if (jb.groups > 1) {
      red[threadIdx.x] = s;
      __syncthreads();
      s = 0.f;
      if (g == 0)
        for (int k = 0; k < jb.groups; k++) s += red[k * per + e];
    }
    if (g != 0 || i >= jb.elems) return;
    const int row = jb.taps * jb.C, n = i / (row + 1), k = i - n * (row + 1), tap = k / jb.C, c = k - tap * jb.C;
    ((float*)grads.p[z])[jb.w_off + (k == row ? (int64_t)jb.K * row + n : (int64_t)n * row + c * jb.taps + tap)] = s;
  } else if (jb.kind == CJOB_FC) {
    __shared__ __attribute__((aligned(16))) float dys[kFinN * kFinU];
    const int cols = (jb.in + 255) / 256;
    const int i = (b % cols) * 256 + threadIdx.x, k0 = (b / cols) * kFinU;
    const T* x = (const T*)wsb + jb.x_off + min(i, jb.in - 1);
    const T* dy = (const T*)wsb + jb.dy_off;
    float* dw = (float*)grads.p[z] + jb.w_off;
    float acc[kFinU], bias = 0.f;
#pragma unroll
    for (int u = 0; u < kFinU; u++) acc[u] = 0.f;
    for (int n0 = 0; n0 < N; n0 += kFinN) {
      const int nn = min(N - n0, kFinN), tn = threadIdx.x / kFinU, tu = threadIdx.x % kFinU;
      __syncthreads();
      if (tn < nn) dys[threadIdx.x] = k0 + tu < jb.out ? ldf(dy + (int64_t)(n0 + tn) * jb.out + k0 + tu) : 0.f;
      __syncthreads();
#pragma unroll 2
      for (int n = 0; n < nn; n++) {
        const float xv = ldf(x + (int64_t)(n0 + n) * jb.in);
#pragma unroll
        for (int u = 0; u < kFinU; u++) acc[u] = fmaf(dys[n * kFinU + u], xv, acc[u]);
      }
      if (i < kFinU)
        for (int n = 0; n < nn; n++) bias += dys[n * kFinU + i];
    }
    if (i < kFinU && k0 + i < jb.out) dw[(int64_t)jb.out * jb.in + k0 + i] = bias;
    if (i >= jb.in) return;
#pragma unroll
    for (int u = 0; u < kFinU; u++)
      if (k0 + u < jb.out) dw[(int64_t)(k0 + u) * jb.in + i] = acc[u];
  } else if (threadIdx.x == 0) {                   // CJOB_LOSS
    const float* img = reinterpret_cast<const float*>(wsb + loss_off);
    float tot = 0.f;
#pragma unroll 8
    for (int n = 0; n < N; n++) tot += img[n];
    loss_out[z] = tot / (float)N;
  }
}

// ---------------------------------------------------------------- host side
// Floats of LDS the patch under `positions` consecutive positions of an OH x OW grid needs.
int64_t patch_floats(int positions, int OH, int OW, int ks, int stride, int C) {
  const int rows = std::min(OH, (positions + OW - 2) / OW + 1);
  return ((int64_t)(rows - 1) * stride + ks) * ((int64_t)(OW - 1) * stride + ks) * compact_pixel_stride(C) + 1;
}
struct Shape {
  int MT, NT, NW, KW;
  int positions() const { return 16 * MT * (NW / KW); }
};
constexpr Shape kSmall = {2, 1, 16, 16}, kLarge = {2, 2, 8, 8}, kWide = {2, 2, 8, 2};    // template arguments of the kernels below
size_t fwd_lds(const CompactConv& v, Shape s) {
  return (size_t)std::max<int64_t>(patch_floats(s.positions(), v.OH, v.OW, v.ks, v.stride, v.C), (int64_t)s.NW * s.MT * s.NT * 256) * 4;
}
size_t dgrad_lds(const CompactConv& v, Shape s) {
  return (size_t)std::max<int64_t>(patch_floats(s.positions(), v.H, v.W, v.ks, 1, v.K), (int64_t)s.NW * s.MT * s.NT * 256) * 4;
}
int col_blocks(const CompactConv& v) { return (v.ks * v.ks * v.C + 31) / 32; }
int col_groups(const CompactConv& v, int NW) { return (col_blocks(v) + NW - 1) / NW; }
size_t wgrad_lds(const CompactConv& v, int NW, int tile) {
  const int64_t floats = tile * kDyLd + tile + patch_floats(tile, v.OH, v.OW, v.ks, v.stride, v.C);
  return (size_t)std::max<int64_t>(floats, (int64_t)(NW / 2) * kRedFloats) * 4;
}
constexpr size_t kLdsMost = 64 * 1024;
// Tiles of 32 x 32 once they alone are a workgroup per compute unit, else 32 x 16 tiles of 16 wavefronts.  CIFAR-shaped net,
// fp32, whole call at 4 / 16 / 32 / 80 images: small tiles 69 / 105 / 178 / 420 us, large ones 77 / 108 / 165 / 370 us (16 x 16
// tiles: 68 / 117 / 200 / 458 us).
// Tiles of 128 positions, whose wavefronts share a filter row more and a partial tile less often, from two workgroups per
// compute unit: 480 images 874 us with them, 960 without; not where a fifth of the last tile would be empty.
int64_t tiles_of(int N, int positions, int channels, Shape s) {
  return (int64_t)N * ((positions + s.positions() - 1) / s.positions()) * ((channels + 16 * s.NT - 1) / (16 * s.NT));
}
template <typename Lds>
Shape choose(int N, int positions, int channels, int count, Lds lds) {
  const int wide = kWide.positions();
  if (tiles_of(N, positions, channels, kWide) * count >= 512 && lds(kWide) <= kLdsMost && (positions + wide - 1) / wide * wide * 4 <= positions * 5)
    return kWide;
  return tiles_of(N, positions, channels, kLarge) * count >= 256 && lds(kLarge) <= kLdsMost ? kLarge : kSmall;
}

}  // namespace

bool compact_conv_ok(const CompactConv& v, bool need_dx) {
  const int k = v.ks;
  if (!(k == 1 || k == 2 || k == 3 || k == 4 || k == 5 || k == 7 || k == 11)) return false;
  if (need_dx && v.stride != 1) return false;
  if ((v.w_off + (int64_t)v.K * v.C * k * k) * 4 >= ((int64_t)1 << 31)) return false;
  // every division of the kernels: positions by row lengths, filter columns and patch elements (of which LDS holds at most
  // kLdsMost / 4) by channels and patch columns
  const int64_t patch = (int64_t)kLdsMost / 4, filter = (int64_t)k * k * v.C;
  if (!FastDiv::exact(v.OW, (int64_t)v.OH * v.OW - 1) || !FastDiv::exact(v.W, (int64_t)v.H * v.W - 1) ||
      !FastDiv::exact(v.C, std::max(patch, filter)) || !FastDiv::exact(v.K, patch) || !FastDiv::exact((v.OW - 1) * v.stride + k, patch) ||
      !FastDiv::exact(v.W - 1 + k, patch))
    return false;
  return fwd_lds(v, kSmall) <= kLdsMost && wgrad_lds(v, kSmall.NW, 32) <= kLdsMost &&
         (!need_dx || dgrad_lds(v, kSmall) <= kLdsMost);
}
size_t compact_head_lds(int in, int K) { return ((((size_t)in + 3) & ~(size_t)3) + K) * 4; }
// (its divisions stay below 2^14 x 2^14: the inputs lie in LDS)
bool compact_head_ok(int in, int K) { return (int64_t)in * K <= (int64_t)1 << 18 && compact_head_lds(in, K) <= 48 * 1024; }
bool compact_fc_ok(int in, int out) { return (int64_t)in * out < ((int64_t)1 << 29); }

static Shape bwd_shape(const CompactConv& v, bool need_dx, int count) {
  return choose(v.N, need_dx ? v.H * v.W : v.OH * v.OW, need_dx ? v.C : v.K, count, [&](Shape s) { return need_dx ? dgrad_lds(v, s) : wgrad_lds(v, s.NW, 32); });
}
static int wgrad_tile(const CompactConv& v, Shape sh) {
  int tile = sh.NW == kSmall.NW ? 32 : 128;
  while (tile > 32 && wgrad_lds(v, sh.NW, tile) > kLdsMost) tile /= 2;
  return tile;
}
// Splits of a weight gradient: about 512 workgroups with the launch's other learners, never fewer than one tile each.
int compact_splits(const CompactConv& v, bool need_dx, int count, int most) {
  const Shape sh = bwd_shape(v, need_dx, count);
  const int tile = wgrad_tile(v, sh);
  const int64_t base = (int64_t)((v.K + 31) / 32) * col_groups(v, sh.NW) * count, tiles = (int64_t)v.N * ((v.OH * v.OW + tile - 1) / tile);
  int64_t sp = (512 + base - 1) / base;
  sp = std::min<int64_t>(std::min<int64_t>(sp, tiles), most);
  return sp < 1 ? 1 : (int)sp;
}

#define COMPACT_KS(ks, X)          \
  switch (ks) {                    \
    case 1: X(1); break;           \
    case 2: X(2); break;           \
    case 3: X(3); break;           \
    case 4: X(4); break;           \
    case 5: X(5); break;           \
    case 7: X(7); break;           \
    case 11: X(11); break;         \
    default: return hipErrorInvalidValue; \
  }

template <typename T>
static hipError_t fwd_t(const PtrTab& ws, const CPtrTab& wts, const CPtrTab& imgs, const CompactConv& v, const CompactSrc& src, bool relu, size_t y_off,
                        const float* mean, int count, hipStream_t s) {
  const Shape sh = choose(v.N, v.OH * v.OW, v.K, count, [&](Shape c) { return fwd_lds(v, c); });
  const int m = sh.positions();
  const dim3 grid((unsigned)(v.N * ((v.OH * v.OW + m - 1) / m)), (unsigned)((v.K + 16 * sh.NT - 1) / (16 * sh.NT)), (unsigned)count);
  const size_t lds = fwd_lds(v, sh);
#define Y(KS, ...) hipLaunchKernelGGL((compact_fwd_kernel<T, KS, __VA_ARGS__>), grid, dim3(64 * sh.NW), lds, s, ws, wts, imgs, v, src, relu ? 1 : 0, y_off, mean)
#define X(KS)                                    \
  if (sh.KW == kWide.KW) Y(KS, 2, 2, 8, 2);      \
  else if (sh.KW == kLarge.KW) Y(KS, 2, 2, 8, 8); \
  else Y(KS, 2, 1, 16, 16)
  COMPACT_KS(v.ks, X)
#undef X
#undef Y
  return hipGetLastError();
}
hipError_t launch_compact_fwd(bool bf, const PtrTab& ws, const CPtrTab& wts, const CPtrTab& imgs, const CompactConv& v, const CompactSrc& src, bool relu,
                              size_t y_off, const float* mean, int count, hipStream_t s) {
  return bf ? fwd_t<bf16_t>(ws, wts, imgs, v, src, relu, y_off, mean, count, s) : fwd_t<float>(ws, wts, imgs, v, src, relu, y_off, mean, count, s);
}

template <typename T>
static hipError_t bwd_t(const PtrTab& ws, const CPtrTab& wts, const CPtrTab& imgs, const CompactConv& v, const CompactSrc& x,
                        const CompactGrad& gr, const CompactBwd& bw_in, const float* mean, bool need_dx, int count, hipStream_t s) {
  CompactBwd bw = bw_in;
  const Shape sh = bwd_shape(v, need_dx, count);
  bw.dgrad_blocks = 0;
  bw.col_groups = col_groups(v, sh.NW);
  bw.blocks_per_group = (col_blocks(v) + bw.col_groups - 1) / bw.col_groups;
  bw.tile = wgrad_tile(v, sh);
  size_t lds = wgrad_lds(v, sh.NW, bw.tile);
  if (need_dx) {
    bw.dgrad_blocks = (int)tiles_of(v.N, v.H * v.W, v.C, sh);
    lds = std::max(lds, dgrad_lds(v, sh));
  }
  const dim3 grid((unsigned)(bw.dgrad_blocks + ((v.K + 31) / 32) * bw.col_groups * bw.splits), 1, (unsigned)count);
#define Y(KS, ...) hipLaunchKernelGGL((compact_bwd_kernel<T, KS, __VA_ARGS__>), grid, dim3(64 * sh.NW), lds, s, ws, wts, imgs, v, x, gr, bw, mean)
#define X(KS)                                    \
  if (sh.KW == kWide.KW) Y(KS, 2, 2, 8, 2);      \
  else if (sh.KW == kLarge.KW) Y(KS, 2, 2, 8, 8); \
  else Y(KS, 2, 1, 16, 16)
  COMPACT_KS(v.ks, X)
#undef X
#undef Y
  return hipGetLastError();
}
hipError_t launch_compact_bwd(bool bf, const PtrTab& ws, const CPtrTab& wts, const CPtrTab& imgs, const CompactConv& v,
                              const CompactSrc& x, const CompactGrad& gr, const CompactBwd& bw, const float* mean, bool need_dx, int count, hipStream_t s) {
  return bf ? bwd_t<bf16_t>(ws, wts, imgs, v, x, gr, bw, mean, need_dx, count, s)
            : bwd_t<float>(ws, wts, imgs, v, x, gr, bw, mean, need_dx, count, s);
}

hipError_t launch_compact_flatten(bool bf, const PtrTab& ws, const CompactSrc& src, size_t flat_off, int N, int count, hipStream_t s) {
  const int64_t total = (int64_t)N * src.C * src.H * src.W;
  const dim3 grid((unsigned)std::min<int64_t>((total + 255) / 256, 4096), 1, (unsigned)count);
  if (bf) hipLaunchKernelGGL(compact_flatten_kernel<bf16_t>, grid, dim3(256), 0, s, ws, src, flat_off, N);
  else hipLaunchKernelGGL(compact_flatten_kernel<float>, grid, dim3(256), 0, s, ws, src, flat_off, N);
  return hipGetLastError();
}

hipError_t launch_compact_head(bool bf, const PtrTab& ws, const CPtrTab& wts, const CPtrTab& labels, const CompactSrc& src, const CompactHead& hd,
                               int32_t* rank_out, int count, hipStream_t s) {
  const dim3 grid((unsigned)hd.N, 1, (unsigned)count);
  const size_t lds = compact_head_lds(hd.in, hd.K);
  // four elements at a time where every row of the weights and of the inputs starts at a multiple of four
  const bool v4 = hd.in % 4 == 0 && hd.w_off % 4 == 0 && (src.kind == CSRC_FLAT || src.C % 4 == 0);
  // few images: as many lanes to each as help; many: half as many lanes leave a compute unit room for twice as many images (64 input channels of
  // 4 x 4, 3 classes, 2 304 images: 28 us with 512 lanes, 19 with 256; 256 images 9.2 and 9.5; 64 x 4 x 4 and 10 classes 30 / 29 and 9.2 / 12.5)
  const bool many = (int64_t)hd.N * count >= 1024;
  auto go = [&](auto kernel, int threads) { hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, s, ws, wts, labels, src, hd, rank_out); };
#define X(T, V) many ? go(compact_head_kernel<T, V, 256>, 256) : go(compact_head_kernel<T, V, 512>, 512)
  if (bf) { if (v4) X(bf16_t, 4); else X(bf16_t, 1); }
  else { if (v4) X(float, 4); else X(float, 1); }
#undef X
  return hipGetLastError();
}

template <typename T, bool DGRAD>
static hipError_t fc_t(const PtrTab& ws, const CPtrTab& wts, const CompactFc& f_in, size_t part_bytes, int count, hipStream_t s) {
  CompactFc f = f_in;
  const int K = DGRAD ? f.out : f.in, C = DGRAD ? f.in : f.out;
  const int64_t tiles = (int64_t)((C + 15) / 16) * ((f.N + 15) / 16);
  // along the contraction: about 256 workgroups with the launch's other learners, at least 1 024 elements each
  int64_t sp = std::min<int64_t>(256 / std::max<int64_t>(tiles * count, 1), K / 1024);
  sp = std::min<int64_t>(sp, (int64_t)(part_bytes / ((size_t)f.N * C * 4)));
  f.splits = sp < 1 ? 1 : (int)sp;
  f.aligned = K % 4 == 0 && f.w_off % 4 == 0;
  hipLaunchKernelGGL((compact_fc_kernel<T, DGRAD>), dim3((unsigned)((C + 15) / 16), (unsigned)((f.N + 15) / 16 * f.splits), (unsigned)count), dim3(1024), 0, s,
                     ws, wts, f);
  if (f.splits > 1)
    hipLaunchKernelGGL((compact_fc_sum_kernel<T, DGRAD>), dim3((unsigned)(((int64_t)f.N * C + 63) / 64), 1, (unsigned)count), dim3(64), 0, s, ws, wts, f);
  return hipGetLastError();
}
hipError_t launch_compact_fc(bool bf, const PtrTab& ws, const CPtrTab& wts, const CompactFc& f, bool dgrad, size_t part_bytes, int count, hipStream_t s) {
  if (bf) return dgrad ? fc_t<bf16_t, true>(ws, wts, f, part_bytes, count, s) : fc_t<bf16_t, false>(ws, wts, f, part_bytes, count, s);
  return dgrad ? fc_t<float, true>(ws, wts, f, part_bytes, count, s) : fc_t<float, false>(ws, wts, f, part_bytes, count, s);
}

hipError_t launch_compact_finish(bool bf, const PtrTab& ws, const PtrTab& grads, const CompactFinish& fin_in, size_t loss_off, int N, float* loss_out,
                                 int count, hipStream_t s) {
  CompactFinish fin = fin_in;
  int64_t blocks = 0;
  for (int j = 0; j < fin.count; j++) {
    CompactJob& jb = fin.job[j];
    jb.first_block = (int)blocks;
    if (jb.kind == CJOB_SUM) {
      jb.groups = 1;
      while (jb.groups < 8 && jb.splits > 8 * jb.groups) jb.groups *= 2;
      blocks += (jb.elems + 256 / jb.groups - 1) / (256 / jb.groups);
    }
    else if (jb.kind == CJOB_FC) blocks += (int64_t)((jb.in + 255) / 256) * ((jb.out + kFinU - 1) / kFinU);
    else blocks += 1;
  }
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks, 1, (unsigned)count);
  if (bf) hipLaunchKernelGGL(compact_finish_kernel<bf16_t>, grid, dim3(256), 0, s, ws, grads, fin, loss_off, N, loss_out);
  else hipLaunchKernelGGL(compact_finish_kernel<float>, grid, dim3(256), 0, s, ws, grads, fin, loss_off, N, loss_out);
  return hipGetLastError();
}

}  // namespace sasgd
