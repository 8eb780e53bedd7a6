// Element-wise and windowed layers of calcGradient (Section 2.1; layer types of Section 4.1): input
// re-layout, max / average pooling with clipped ceil-mode windows, flattening, softmax cross-entropy.
// All are bandwidth-bound; lanes walk the channel-innermost (NHWC) index so loads and stores coalesce,
// reductions over classes use one wavefront per image.  blockIdx.z selects the learner.
#include "dev_common.hpp"
#include "kernels.hpp"

namespace sasgd {

static inline dim3 grid_for(int64_t total, int count, int cap = 4096) {
  int64_t b = (total + 255) / 256;
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return dim3((unsigned)b, 1, (unsigned)count);
}

struct bf8 {
  uint4 v;
  __device__ __forceinline__ float get(int i) const {
    uint32_t w = i < 2 ? v.x : (i < 4 ? v.y : (i < 6 ? v.z : v.w));
    return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
  }
};
__device__ __forceinline__ uint4 pack8(const float* f) {
  uint4 o;
  o.x = pack2bf(f[0], f[1]);
  o.y = pack2bf(f[2], f[3]);
  o.z = pack2bf(f[4], f[5]);
  o.w = pack2bf(f[6], f[7]);
  return o;
}

// ------------------------------------------------------------------ input NCHW fp32 -> NHWC T
template <typename T>
__global__ __launch_bounds__(256) void pack_input_kernel(CPtrTab images, PtrTab ws, size_t out_off, int N, InPack ip,
                                                         const float* __restrict__ mean) {
  const float* in = (const float*)images.p[blockIdx.z];
  T* out = (T*)ws.p[blockIdx.z] + out_off;
  const int64_t total = (int64_t)N * ip.Hp * ip.Wp * ip.Cp;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    int cp = (int)(i % ip.Cp);
    int64_t r = i / ip.Cp;
    int X = (int)(r % ip.Wp);
    r /= ip.Wp;
    int Y = (int)(r % ip.Hp);
    int n = (int)(r / ip.Hp);
    float v = 0.f;
    if (ip.s2d == 1) {
      if (cp < ip.C) {
        const int64_t pix = ((int64_t)cp * ip.H + Y) * ip.W + X;
        v = in[(int64_t)n * ip.C * ip.H * ip.W + pix] - (mean ? mean[pix] : 0.f);
      }
    } else {
      int g = cp / ip.C, c = cp % ip.C;
      int h = ip.s2d * Y + g / ip.s2d, w = ip.s2d * X + g % ip.s2d;
      if (g < ip.s2d * ip.s2d && h < ip.H && w < ip.W) {
        const int64_t pix = ((int64_t)c * ip.H + h) * ip.W + w;
        v = in[(int64_t)n * ip.C * ip.H * ip.W + pix] - (mean ? mean[pix] : 0.f);
      }
    }
    stf(out + i, v);
  }
}

// One lane per destination pixel (bf16, Cp % 8 == 0): the Cp channels are assembled in registers and written as 16-byte chunks;
// neighbouring lanes read neighbouring source columns.  Pixels are counted through all images: with a workgroup per image, images of
// 16 pixels left most lanes idle (2 048 of them, 16 learners: 24 us, 8 here).
__global__ __launch_bounds__(256) void pack_input_pixel_kernel(CPtrTab images, PtrTab ws, size_t out_off, int N, InPack ip,
                                                               const float* __restrict__ mean) {
  const float* in = (const float*)images.p[blockIdx.z];
  bf16_t* out = (bf16_t*)ws.p[blockIdx.z] + out_off;
  const uint32_t total = (uint32_t)N * (uint32_t)ip.Hp * (uint32_t)ip.Wp;     // of at least 32 bytes each, below 2 GiB together
  const int64_t plane = (int64_t)ip.H * ip.W;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const uint32_t row = i / (uint32_t)ip.Wp;
    const int X = (int)(i - row * (uint32_t)ip.Wp), n = (int)(row / (uint32_t)ip.Hp), Y = (int)(row - (uint32_t)n * (uint32_t)ip.Hp);
    const float* src = in + (int64_t)n * ip.C * plane;
    for (int c0 = 0; c0 < ip.Cp; c0 += 8) {
      float f[8];
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const int cp = c0 + e;
        float v = 0.f;
        if (ip.s2d == 1) {
          if (cp < ip.C) {
            const int64_t pix = cp * plane + (int64_t)Y * ip.W + X;
            v = src[pix] - (mean ? mean[pix] : 0.f);
          }
        } else {
          int g = cp / ip.C, c = cp - g * ip.C;
          int h = ip.s2d * Y + g / ip.s2d, w = ip.s2d * X + g % ip.s2d;
          if (g < ip.s2d * ip.s2d && h < ip.H && w < ip.W) {
            const int64_t pix = c * plane + (int64_t)h * ip.W + w;
            v = src[pix] - (mean ? mean[pix] : 0.f);
          }
        }
        f[e] = v;
      }
      *reinterpret_cast<uint4*>(out + (int64_t)i * ip.Cp + c0) = pack8(f);
    }
  }
}

// Space-to-depth by 4 of a 3-channel image (the 11 x 11 / 4 first layer): a workgroup makes `width` pixels of one row of destination
// pixels (input_row_piece).  A thread reads the three channels' aligned float4 (row 4Y + dh, columns 4X .. 4X + 3) and puts
// their twelve values, channels (dh * 4 + dw) * 3 + c, into LDS; the pixels leave as they lie there.  Needs W % 4 == 0 and 16-byte
// aligned images (and mean).  Bound by HBM: 18 learners x 16 images 3 x 224 x 224, 260 MB, in 42 us inside a training step; a lane per pixel, which
// writes its 96 bytes on its own, took 78.  The images are read once, past the caches (54 us with ordinary loads, which drive out of them
// what the step wrote; one learner of 256 images 48 -> 37; level in a validation pass, 33 and 34, which writes little).
typedef float float4v __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void pack_input_s2d4_kernel(CPtrTab images, PtrTab ws, size_t out_off, InPack ip, int width,
                                                              int pieces, const float* __restrict__ mean) {
  extern __shared__ __attribute__((aligned(16))) uint2 s2d_row[];       // [width][96 bytes]
  const int Y = blockIdx.x / pieces, x0 = (blockIdx.x - Y * pieces) * width;
  const int n = blockIdx.y, pixels = min(width, ip.Wp - x0);
  const uint32_t plane = (uint32_t)ip.H * (uint32_t)ip.W;
  const float* src = (const float*)images.p[blockIdx.z] + (int64_t)n * 3 * plane;
  for (int t = threadIdx.x; t < 4 * pixels; t += 256) {
    const int dh = t / pixels, X = t - dh * pixels, h = 4 * Y + dh;
    float f[12];
#pragma unroll
    for (int c = 0; c < 3; c++) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (h < ip.H) {
        const uint32_t pix = c * plane + (uint32_t)h * (uint32_t)ip.W + 4 * (x0 + X);
        const float4v once = __builtin_nontemporal_load(reinterpret_cast<const float4v*>(src + pix));
        v = make_float4(once.x, once.y, once.z, once.w);
        if (mean) {
          const float4 mv = *reinterpret_cast<const float4*>(mean + pix);
          v.x -= mv.x; v.y -= mv.y; v.z -= mv.z; v.w -= mv.w;
        }
      }
      f[c] = v.x; f[3 + c] = v.y; f[6 + c] = v.z; f[9 + c] = v.w;
    }
#pragma unroll
    for (int q = 0; q < 3; q++) s2d_row[X * 12 + dh * 3 + q] = make_uint2(pack2bf(f[4 * q], f[4 * q + 1]), pack2bf(f[4 * q + 2], f[4 * q + 3]));
  }
  __syncthreads();
  uint4* out = reinterpret_cast<uint4*>((bf16_t*)ws.p[blockIdx.z] + out_off) + (((int64_t)n * ip.Hp + Y) * ip.Wp + x0) * 6;
  for (int t = threadIdx.x; t < pixels * 6; t += 256) out[t] = reinterpret_cast<const uint4*>(s2d_row)[t];
}

hipError_t launch_pack_input(bool is_bf16, const CPtrTab& images, const PtrTab& ws, size_t out_off, int count, int N,
                             const InPack& ip, const float* mean, hipStream_t s) {
  bool aligned = ip.W % 4 == 0 && ((uintptr_t)mean & 15) == 0;
  for (int k = 0; k < count; k++) aligned = aligned && ((uintptr_t)images.p[k] & 15) == 0;
  const InputLayout layout = out_off % 8 == 0 ? input_layout(is_bf16, ip.s2d, ip.C, ip.Cp, aligned) : InputLayout::kValues;
  if (layout == InputLayout::kRows) {
    const int width = input_row_piece(ip.Wp), pieces = (ip.Wp + width - 1) / width;
    hipLaunchKernelGGL(pack_input_s2d4_kernel, dim3((unsigned)(ip.Hp * pieces), (unsigned)N, (unsigned)count), dim3(256), (size_t)width * 96, s, images,
                       ws, out_off, ip, width, pieces, mean);
    return hipGetLastError();
  }
  if (layout == InputLayout::kPixels) {
    const dim3 grid((unsigned)input_pixel_groups(N, ip.Hp, ip.Wp), 1, (unsigned)count);
    hipLaunchKernelGGL(pack_input_pixel_kernel, grid, dim3(256), 0, s, images, ws, out_off, N, ip, mean);
    return hipGetLastError();
  }
  dim3 g = grid_for((int64_t)N * ip.Cp * ip.Hp * ip.Wp, count);
  if (is_bf16) hipLaunchKernelGGL(pack_input_kernel<bf16_t>, g, dim3(256), 0, s, images, ws, out_off, N, ip, mean);
  else hipLaunchKernelGGL(pack_input_kernel<float>, g, dim3(256), 0, s, images, ws, out_off, N, ip, mean);
  return hipGetLastError();
}

// ------------------------------------------------------------------ pooling
// Windows start at (oh*stride, ow*stride) and are clipped at the border.  Max: the first maximum in
// row-major window order wins and its position inside the window is kept (one byte) for the backward
// pass.  Where the input is a ReLU's output (`marks`), a window whose maximum is not positive keeps 255 instead, a position it
// does not have: no gradient passes that ReLU, and the backward pass need not read the input again to know it.
// Average: the divisor is the number of in-bounds elements.
template <typename T, bool MAX>
__global__ __launch_bounds__(256) void pool_fwd_kernel(PtrTab ws, size_t x_off, size_t y_off, size_t arg_byte_off, PoolShape sh,
                                                       int relu, int marks) {
  const T* x = (const T*)ws.p[blockIdx.z] + x_off;
  T* y = (T*)ws.p[blockIdx.z] + y_off;
  uint8_t* arg = (uint8_t*)ws.p[blockIdx.z] + arg_byte_off;
  const int64_t total = (int64_t)sh.N * sh.OH * sh.OW * sh.C;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    int c = (int)(i % sh.C);
    int64_t r = i / sh.C;
    int ow = (int)(r % sh.OW);
    r /= sh.OW;
    int oh = (int)(r % sh.OH);
    int n = (int)(r / sh.OH);
    const int h0 = oh * sh.stride, w0 = ow * sh.stride;
    float acc = 0.f;
    int best = 0, cnt = 0;
    for (int kh = 0; kh < sh.ks && h0 + kh < sh.H; kh++)
      for (int kw = 0; kw < sh.ks && w0 + kw < sh.W; kw++) {
        float v = ldf(x + (((int64_t)n * sh.H + h0 + kh) * sh.W + w0 + kw) * sh.C + c);
        if (MAX) {
          if (cnt == 0 || v > acc) { acc = v; best = kh * sh.ks + kw; }
        } else {
          acc += v;
        }
        cnt++;
      }
    if (!MAX) acc /= (float)cnt;
    if (MAX && marks && !(acc > 0.f)) best = 255;
    if (relu) acc = fmaxf(acc, 0.f);
    stf(y + i, acc);
    if (MAX) arg[i] = (uint8_t)best;
  }
}

template <typename T, bool MAX>
__global__ __launch_bounds__(256) void pool_bwd_kernel(PtrTab ws, size_t dy_off, size_t dx_off, size_t arg_byte_off, PoolShape sh,
                                                       int use_mask, size_t mask_off) {
  const T* dy = (const T*)ws.p[blockIdx.z] + dy_off;
  T* dx = (T*)ws.p[blockIdx.z] + dx_off;
  const T* mask = (const T*)ws.p[blockIdx.z] + mask_off;
  const uint8_t* arg = (const uint8_t*)ws.p[blockIdx.z] + arg_byte_off;
  const int64_t total = (int64_t)sh.N * sh.H * sh.W * sh.C;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    int c = (int)(i % sh.C);
    int64_t r = i / sh.C;
    int iw = (int)(r % sh.W);
    r /= sh.W;
    int ih = (int)(r % sh.H);
    int n = (int)(r / sh.H);
    float acc = 0.f;
    if (MAX || !use_mask || ldf(mask + i) > 0.f) {          // (max: the winners know)
      // windows that contain (ih, iw): oh*stride <= ih < oh*stride + ks
      int oh_lo = ih - sh.ks + 1 > 0 ? (ih - sh.ks + sh.stride) / sh.stride : 0;
      int oh_hi = min(sh.OH - 1, ih / sh.stride);
      int ow_lo = iw - sh.ks + 1 > 0 ? (iw - sh.ks + sh.stride) / sh.stride : 0;
      int ow_hi = min(sh.OW - 1, iw / sh.stride);
      for (int oh = oh_lo; oh <= oh_hi; oh++)
        for (int ow = ow_lo; ow <= ow_hi; ow++) {
          const int64_t o = (((int64_t)n * sh.OH + oh) * sh.OW + ow) * sh.C + c;
          if (MAX) {
            if (arg[o] == (uint8_t)((ih - oh * sh.stride) * sh.ks + (iw - ow * sh.stride))) acc += ldf(dy + o);
          } else {
            int ch = min(oh * sh.stride + sh.ks, sh.H) - oh * sh.stride;
            int cw = min(ow * sh.stride + sh.ks, sh.W) - ow * sh.stride;
            acc += ldf(dy + o) / (float)(ch * cw);
          }
        }
    }
    stf(dx + i, acc);
  }
}

// ------------------------------------------------------------------ pooling, 8 channels per lane (bf16, C % 8 == 0)
// Same arithmetic as the scalar kernels; each lane moves 16-byte channel chunks, so a wavefront reads and
// writes 1 KiB contiguous runs.
template <bool MAX>
__global__ __launch_bounds__(256) void pool_fwd_vec8_kernel(PtrTab ws, size_t x_off, size_t y_off, size_t arg_byte_off, PoolShape sh,
                                                            int relu, int marks) {
  const bf16_t* x = (const bf16_t*)ws.p[blockIdx.z] + x_off;
  bf16_t* y = (bf16_t*)ws.p[blockIdx.z] + y_off;
  uint8_t* arg = (uint8_t*)ws.p[blockIdx.z] + arg_byte_off;
  const int C8 = sh.C / 8;
  const int64_t total = (int64_t)sh.N * sh.OH * sh.OW * C8;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    // 32-bit index arithmetic: a tensor of one learner has fewer than 2^31 elements
    uint32_t r = (uint32_t)i;
    const int c8 = (int)(r % (uint32_t)C8);
    r /= (uint32_t)C8;
    const int ow = (int)(r % (uint32_t)sh.OW);
    r /= (uint32_t)sh.OW;
    const int oh = (int)(r % (uint32_t)sh.OH);
    const int n = (int)(r / (uint32_t)sh.OH);
    const int h0 = oh * sh.stride, w0 = ow * sh.stride;
    float acc[8];
    int best[8];
#pragma unroll
    for (int e = 0; e < 8; e++) { acc[e] = 0.f; best[e] = 0; }
    int cnt = 0;
    for (int kh = 0; kh < sh.ks && h0 + kh < sh.H; kh++)
      for (int kw = 0; kw < sh.ks && w0 + kw < sh.W; kw++) {
        bf8 v;
        v.v = *reinterpret_cast<const uint4*>(x + (((int64_t)n * sh.H + h0 + kh) * sh.W + w0 + kw) * sh.C + c8 * 8);
#pragma unroll
        for (int e = 0; e < 8; e++) {
          float f = v.get(e);
          if (MAX) {
            if (cnt == 0 || f > acc[e]) { acc[e] = f; best[e] = kh * sh.ks + kw; }
          } else {
            acc[e] += f;
          }
        }
        cnt++;
      }
#pragma unroll
    for (int e = 0; e < 8; e++) {
      if (!MAX) acc[e] /= (float)cnt;
      if (MAX && marks && !(acc[e] > 0.f)) best[e] = 255;
      if (relu) acc[e] = fmaxf(acc[e], 0.f);
    }
    *reinterpret_cast<uint4*>(y + i * 8) = pack8(acc);
    if (MAX) {
      uint2 a;
      a.x = (uint32_t)best[0] | ((uint32_t)best[1] << 8) | ((uint32_t)best[2] << 16) | ((uint32_t)best[3] << 24);
      a.y = (uint32_t)best[4] | ((uint32_t)best[5] << 8) | ((uint32_t)best[6] << 16) | ((uint32_t)best[7] << 24);
      *reinterpret_cast<uint2*>(arg + i * 8) = a;
    }
  }
}

// Divisions of a flat index by the 8-channel chunks of a pixel, then by the columns and the rows it runs over.
struct PoolDiv {
  FastDiv c8, w, h;
};
static bool pool_divides(PoolDiv* d, int64_t total, int C8, int W, int H) {
  d->c8.set(C8);
  d->w.set(W);
  d->h.set(H);
  return FastDiv::exact(C8, total) && FastDiv::exact(W, total / C8) && FastDiv::exact(H, total / C8 / W);
}

// 3 x 3 windows (every pooling layer of the two reference networks): the nine 16-byte reads of a window are all
// requested before the first is used (the general kernel above walks the window in a loop whose trip count the
// compiler does not know, one dependent read after the other).  Same arithmetic and the same winner on ties.
template <bool MAX>
__global__ __launch_bounds__(256) void pool_fwd_3x3_kernel(PtrTab ws, size_t x_off, size_t y_off, size_t arg_byte_off, PoolShape sh, PoolDiv dv, int relu, int marks) {
  const bf16_t* x = (const bf16_t*)ws.p[blockIdx.z] + x_off;
  bf16_t* y = (bf16_t*)ws.p[blockIdx.z] + y_off;
  uint8_t* arg = (uint8_t*)ws.p[blockIdx.z] + arg_byte_off;
  const int C8 = sh.C / 8;
  const uint32_t total = (uint32_t)sh.N * sh.OH * sh.OW * C8;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const int r1 = dv.c8((int)i), c8 = (int)i - r1 * C8, r2 = dv.w(r1), ow = r1 - r2 * sh.OW, n = dv.h(r2), oh = r2 - n * sh.OH;
    const int h0 = oh * sh.stride, w0 = ow * sh.stride;
    const int nh = min(3, sh.H - h0), nw = min(3, sh.W - w0);          // rows and columns of the window inside the image
    const bf16_t* base = x + (((int64_t)n * sh.H + h0) * sh.W + w0) * sh.C + c8 * 8;
    bf8 v[9];
#pragma unroll
    for (int kh = 0; kh < 3; kh++)
#pragma unroll
      for (int kw = 0; kw < 3; kw++) {
        const bool in = kh < nh && kw < nw;
        v[kh * 3 + kw].v = *reinterpret_cast<const uint4*>(base + (in ? ((int64_t)kh * sh.W + kw) * sh.C : 0));   // outside: the first element again
      }
    float acc[8];
    int best[8];
#pragma unroll
    for (int e = 0; e < 8; e++) { acc[e] = v[0].get(e); best[e] = 0; }
#pragma unroll
    for (int t = 1; t < 9; t++) {
      const bool in = t / 3 < nh && t % 3 < nw;
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const float f = v[t].get(e);
        if (MAX) {
          if (in && f > acc[e]) { acc[e] = f; best[e] = t; }
        } else {
          if (in) acc[e] += f;
        }
      }
    }
    const float cnt = (float)(nh * nw);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      if (!MAX) acc[e] /= cnt;
      if (MAX && marks && !(acc[e] > 0.f)) best[e] = 255;
      if (relu) acc[e] = fmaxf(acc[e], 0.f);
    }
    *reinterpret_cast<uint4*>(y + (size_t)i * 8) = pack8(acc);
    if (MAX) {
      uint2 a;
      a.x = (uint32_t)best[0] | ((uint32_t)best[1] << 8) | ((uint32_t)best[2] << 16) | ((uint32_t)best[3] << 24);
      a.y = (uint32_t)best[4] | ((uint32_t)best[5] << 8) | ((uint32_t)best[6] << 16) | ((uint32_t)best[7] << 24);
      *reinterpret_cast<uint2*>(arg + (size_t)i * 8) = a;
    }
  }
}

template <bool MAX>
__global__ __launch_bounds__(256) void pool_bwd_vec8_kernel(PtrTab ws, size_t dy_off, size_t dx_off, size_t arg_byte_off, PoolShape sh,
                                                            int use_mask, size_t mask_off) {
  const bf16_t* dy = (const bf16_t*)ws.p[blockIdx.z] + dy_off;
  bf16_t* dx = (bf16_t*)ws.p[blockIdx.z] + dx_off;
  const bf16_t* mask = (const bf16_t*)ws.p[blockIdx.z] + mask_off;
  const uint8_t* arg = (const uint8_t*)ws.p[blockIdx.z] + arg_byte_off;
  const int C8 = sh.C / 8;
  const int64_t total = (int64_t)sh.N * sh.H * sh.W * C8;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    uint32_t r = (uint32_t)i;
    const int c8 = (int)(r % (uint32_t)C8);
    r /= (uint32_t)C8;
    const int iw = (int)(r % (uint32_t)sh.W);
    r /= (uint32_t)sh.W;
    const int ih = (int)(r % (uint32_t)sh.H);
    const int n = (int)(r / (uint32_t)sh.H);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; e++) acc[e] = 0.f;
    int oh_lo = ih - sh.ks + 1 > 0 ? (ih - sh.ks + sh.stride) / sh.stride : 0;
    int oh_hi = min(sh.OH - 1, ih / sh.stride);
    int ow_lo = iw - sh.ks + 1 > 0 ? (iw - sh.ks + sh.stride) / sh.stride : 0;
    int ow_hi = min(sh.OW - 1, iw / sh.stride);
    for (int oh = oh_lo; oh <= oh_hi; oh++)
      for (int ow = ow_lo; ow <= ow_hi; ow++) {
        const int64_t o = ((((int64_t)n * sh.OH + oh) * sh.OW + ow) * C8 + c8) * 8;
        bf8 d;
        d.v = *reinterpret_cast<const uint4*>(dy + o);
        if (MAX) {
          const uint2 a = *reinterpret_cast<const uint2*>(arg + o);
          const uint32_t pos = (uint32_t)((ih - oh * sh.stride) * sh.ks + (iw - ow * sh.stride));
#pragma unroll
          for (int e = 0; e < 8; e++) {
            uint32_t ae = ((e < 4 ? a.x : a.y) >> (8 * (e & 3))) & 0xffu;
            if (ae == pos) acc[e] += d.get(e);
          }
        } else {
          int ch = min(oh * sh.stride + sh.ks, sh.H) - oh * sh.stride;
          int cw = min(ow * sh.stride + sh.ks, sh.W) - ow * sh.stride;
          const float inv = (float)(ch * cw);
#pragma unroll
          for (int e = 0; e < 8; e++) acc[e] += d.get(e) / inv;
        }
      }
    if (!MAX && use_mask) {
      bf8 mk;
      mk.v = *reinterpret_cast<const uint4*>(mask + i * 8);
#pragma unroll
      for (int e = 0; e < 8; e++)
        if (!(mk.get(e) > 0.f)) acc[e] = 0.f;
    }
    *reinterpret_cast<uint4*>(dx + i * 8) = pack8(acc);
  }
}

// 3 x 3 windows at stride 2 (every pooling layer of the two reference networks): one lane owns 8 channels of a 2 x 2
// block of the input, rows 2a, 2a+1 and columns 2b, 2b+1.  Only the four windows (a-1 | a, b-1 | b) reach into the
// block, so they are read once for the four results instead of once per covered element (nine reads per block).
// Max: neither the mask nor the input is read (the winners know both); AlexNet-shaped net, 256 images, its three layers from the input on
// 61 / 43 / 16 -> 45 / 31 / 11 us.
template <bool MAX>
__global__ __launch_bounds__(256) void pool_bwd_3x3s2_kernel(PtrTab ws, size_t dy_off, size_t dx_off, size_t arg_byte_off, PoolShape sh, PoolDiv dv,
                                                             int use_mask, size_t mask_off) {
  const bf16_t* dy = (const bf16_t*)ws.p[blockIdx.z] + dy_off;
  bf16_t* dx = (bf16_t*)ws.p[blockIdx.z] + dx_off;
  const bf16_t* mask = (const bf16_t*)ws.p[blockIdx.z] + mask_off;
  const uint8_t* arg = (const uint8_t*)ws.p[blockIdx.z] + arg_byte_off;
  const int C8 = sh.C / 8, HB = (sh.H + 1) / 2, WB = (sh.W + 1) / 2;
  const uint32_t total = (uint32_t)sh.N * HB * WB * C8;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const int r1 = dv.c8((int)i), c8 = (int)i - r1 * C8, r2 = dv.w(r1), b = r1 - r2 * WB, n = dv.h(r2), a = r2 - n * HB;
    // All reads are requested before the first is used: windows outside the output and block elements outside the
    // input read a clamped (valid) address and are discarded by a predicate instead of a branch around the load.
    bool w_ok[4];
    uint4 dw[4];
    uint2 av[4];
    float inv[4];
#pragma unroll
    for (int wh = 0; wh < 2; wh++)
#pragma unroll
      for (int ww = 0; ww < 2; ww++) {
        const int oh = a - 1 + wh, ow = b - 1 + ww;
        const int q = 2 * wh + ww;
        w_ok[q] = oh >= 0 && oh < sh.OH && ow >= 0 && ow < sh.OW;
        const int ohc = min(max(oh, 0), sh.OH - 1), owc = min(max(ow, 0), sh.OW - 1);
        const int64_t o = ((((int64_t)n * sh.OH + ohc) * sh.OW + owc) * C8 + c8) * 8;
        dw[q] = *reinterpret_cast<const uint4*>(dy + o);
        av[q] = make_uint2(0u, 0u);
        if (MAX) av[q] = *reinterpret_cast<const uint2*>(arg + o);
        inv[q] = 1.f;
        if (!MAX) {
          const int ch = min(ohc * 2 + 3, sh.H) - ohc * 2, cw = min(owc * 2 + 3, sh.W) - owc * 2;
          inv[q] = 1.f / (float)(ch * cw);
        }
      }
    bool x_ok[4];
    int64_t xo[4];
    uint4 mv[4];
#pragma unroll
    for (int dh = 0; dh < 2; dh++)
#pragma unroll
      for (int dw = 0; dw < 2; dw++) {
        const int ih = 2 * a + dh, iw = 2 * b + dw;
        const int q = 2 * dh + dw;
        x_ok[q] = ih < sh.H && iw < sh.W;
        xo[q] = ((((int64_t)n * sh.H + min(ih, sh.H - 1)) * sh.W + min(iw, sh.W - 1)) * C8 + c8) * 8;
        mv[q] = make_uint4(0u, 0u, 0u, 0u);
        if (!MAX && use_mask) mv[q] = *reinterpret_cast<const uint4*>(mask + xo[q]);
      }
    float acc[4][8];                                    // [2 * dh + dw][channel]
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int e = 0; e < 8; e++) acc[q][e] = 0.f;
#pragma unroll
    for (int wh = 0; wh < 2; wh++)
#pragma unroll
      for (int ww = 0; ww < 2; ww++) {
        const int wq = 2 * wh + ww;
        bf8 d;
        d.v = w_ok[wq] ? dw[wq] : make_uint4(0u, 0u, 0u, 0u);
        const uint2 ar = av[wq];
        // window (oh, ow) = (a - 1 + wh, b - 1 + ww) starts at row 2 oh, column 2 ow: block row dh sits at window row
        // 2 (a - oh) + dh, i.e. 2, 3 for the window above (only 2 is inside), 0, 1 for the own one
#pragma unroll
        for (int dh = 0; dh < 2; dh++) {
          const int wr = 2 * (1 - wh) + dh;
          if (wr > 2) continue;
#pragma unroll
          for (int dw = 0; dw < 2; dw++) {
            const int wc = 2 * (1 - ww) + dw;
            if (wc > 2) continue;
            const uint32_t pos = (uint32_t)(wr * 3 + wc);
#pragma unroll
            for (int e = 0; e < 8; e++) {
              if (MAX) {
                const uint32_t ae = ((e < 4 ? ar.x : ar.y) >> (8 * (e & 3))) & 0xffu;
                if (ae == pos) acc[2 * dh + dw][e] += d.get(e);
              } else {
                acc[2 * dh + dw][e] += d.get(e) * inv[wq];
              }
            }
          }
        }
      }
#pragma unroll
    for (int q = 0; q < 4; q++) {
      if (!x_ok[q]) continue;
      if (!MAX && use_mask) {
        bf8 mk;
        mk.v = mv[q];
#pragma unroll
        for (int e = 0; e < 8; e++)
          if (!(mk.get(e) > 0.f)) acc[q][e] = 0.f;
      }
      *reinterpret_cast<uint4*>(dx + xo[q]) = pack8(acc[q]);
    }
  }
}

hipError_t launch_pool_fwd(bool is_bf16, bool is_max, const PtrTab& ws, size_t x_off, size_t y_off, size_t arg_byte_off,
                           const PoolShape& sh, bool relu, bool input_relu, int count, hipStream_t s) {
  dim3 g = grid_for((int64_t)sh.N * sh.OH * sh.OW * sh.C, count);
  const int r = relu ? 1 : 0, m = is_max && input_relu ? 1 : 0;
  if (is_bf16 && sh.C % 8 == 0 && x_off % 8 == 0 && y_off % 8 == 0 && arg_byte_off % 8 == 0) {
    dim3 gv = grid_for((int64_t)sh.N * sh.OH * sh.OW * (sh.C / 8), count, 16384);
    PoolDiv dv;
    if (sh.ks == 3 && (int64_t)sh.N * sh.H * sh.W * sh.C < ((int64_t)1 << 31) &&
        pool_divides(&dv, (int64_t)sh.N * sh.OH * sh.OW * (sh.C / 8), sh.C / 8, sh.OW, sh.OH)) {
      if (is_max) hipLaunchKernelGGL((pool_fwd_3x3_kernel<true>), gv, dim3(256), 0, s, ws, x_off, y_off, arg_byte_off, sh, dv, r, m);
      else hipLaunchKernelGGL((pool_fwd_3x3_kernel<false>), gv, dim3(256), 0, s, ws, x_off, y_off, arg_byte_off, sh, dv, r, m);
      return hipGetLastError();
    }
    if (is_max) hipLaunchKernelGGL((pool_fwd_vec8_kernel<true>), gv, dim3(256), 0, s, ws, x_off, y_off, arg_byte_off, sh, r, m);
    else hipLaunchKernelGGL((pool_fwd_vec8_kernel<false>), gv, dim3(256), 0, s, ws, x_off, y_off, arg_byte_off, sh, r, m);
    return hipGetLastError();
  }
  if (is_bf16) {
    if (is_max) hipLaunchKernelGGL((pool_fwd_kernel<bf16_t, true>), g, dim3(256), 0, s, ws, x_off, y_off, arg_byte_off, sh, r, m);
    else hipLaunchKernelGGL((pool_fwd_kernel<bf16_t, false>), g, dim3(256), 0, s, ws, x_off, y_off, arg_byte_off, sh, r, m);
  } else {
    if (is_max) hipLaunchKernelGGL((pool_fwd_kernel<float, true>), g, dim3(256), 0, s, ws, x_off, y_off, arg_byte_off, sh, r, m);
    else hipLaunchKernelGGL((pool_fwd_kernel<float, false>), g, dim3(256), 0, s, ws, x_off, y_off, arg_byte_off, sh, r, m);
  }
  return hipGetLastError();
}

hipError_t launch_pool_bwd(bool is_bf16, bool is_max, const PtrTab& ws, size_t dy_off, size_t dx_off, size_t arg_byte_off,
                           const PoolShape& sh, bool use_mask, size_t mask_off, int count, hipStream_t s) {
  dim3 g = grid_for((int64_t)sh.N * sh.H * sh.W * sh.C, count);
  const int um = use_mask && !is_max ? 1 : 0;      // max: the winners know (launch_pool_fwd's input_relu)
  if (is_bf16 && sh.C % 8 == 0 && dy_off % 8 == 0 && dx_off % 8 == 0 && arg_byte_off % 8 == 0 && mask_off % 8 == 0) {
    PoolDiv dv;
    if (sh.ks == 3 && sh.stride == 2 &&
        pool_divides(&dv, (int64_t)sh.N * ((sh.H + 1) / 2) * ((sh.W + 1) / 2) * (sh.C / 8), sh.C / 8, (sh.W + 1) / 2, (sh.H + 1) / 2)) {
      dim3 gb = grid_for((int64_t)sh.N * ((sh.H + 1) / 2) * ((sh.W + 1) / 2) * (sh.C / 8), count, 16384);
      if (is_max) hipLaunchKernelGGL((pool_bwd_3x3s2_kernel<true>), gb, dim3(256), 0, s, ws, dy_off, dx_off, arg_byte_off, sh, dv, um, mask_off);
      else hipLaunchKernelGGL((pool_bwd_3x3s2_kernel<false>), gb, dim3(256), 0, s, ws, dy_off, dx_off, arg_byte_off, sh, dv, um, mask_off);
      return hipGetLastError();
    }
    dim3 gv = grid_for((int64_t)sh.N * sh.H * sh.W * (sh.C / 8), count, 16384);
    if (is_max) hipLaunchKernelGGL((pool_bwd_vec8_kernel<true>), gv, dim3(256), 0, s, ws, dy_off, dx_off, arg_byte_off, sh, um, mask_off);
    else hipLaunchKernelGGL((pool_bwd_vec8_kernel<false>), gv, dim3(256), 0, s, ws, dy_off, dx_off, arg_byte_off, sh, um, mask_off);
    return hipGetLastError();
  }
  if (is_bf16) {
    if (is_max) hipLaunchKernelGGL((pool_bwd_kernel<bf16_t, true>), g, dim3(256), 0, s, ws, dy_off, dx_off, arg_byte_off, sh, um, mask_off);
    else hipLaunchKernelGGL((pool_bwd_kernel<bf16_t, false>), g, dim3(256), 0, s, ws, dy_off, dx_off, arg_byte_off, sh, um, mask_off);
  } else {
    if (is_max) hipLaunchKernelGGL((pool_bwd_kernel<float, true>), g, dim3(256), 0, s, ws, dy_off, dx_off, arg_byte_off, sh, um, mask_off);
    else hipLaunchKernelGGL((pool_bwd_kernel<float, false>), g, dim3(256), 0, s, ws, dy_off, dx_off, arg_byte_off, sh, um, mask_off);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ flatten (NHWC -> C,H,W order) and back
// A workgroup turns up to 64 channels of up to 64 positions of one image around through LDS, so that a call of any shape has a workgroup for every
// 4 096 values (or 8 192, below), and both sides' accesses are of neighbouring addresses: channels on one side in whole 16-byte pieces where they come in such, positions
// on the other where an image's do, or where the tile holds the whole image (its 64 channels lie one after the other then).
// Bound by the launch and two round trips to memory in small calls, by HBM in large ones.  bf16, forward and backward in us, with a value a lane and
// three 64-bit divisions / here: 64 channels of 32 x 32, 16 images 7 / 4 and 5 / 5, 576 images 148 / 25 and 115 / 30; 72 of 45 x 45, 576 images
// 371 / 110 and 323 / 123; 256 of 6 x 6, 256 images 9.6 / 5.2 and 10.5 / 5.4.  (With a workgroup for all positions of 64 channels, the 16 images took 54 and 47.)
template <typename T>
struct FlatTile {
  static constexpr int V = 16 / sizeof(T), kPitch = kFlat + 16 / sizeof(T);     // elements
};
__device__ __forceinline__ uint32_t flat_bits(bf16_t v) { return v; }
__device__ __forceinline__ uint32_t flat_bits(float v) { return __float_as_uint(v); }
__device__ __forceinline__ void flat_store(bf16_t* to, uint32_t v) { *to = (bf16_t)v; }
__device__ __forceinline__ void flat_store(float* to, uint32_t v) { *to = __uint_as_float(v); }
struct FlatArgs {
  int C, HW, cblocks;            // blocks of channels
  FastDiv by_c, by_p;            // channels and positions of a full tile
};

// A step of the workgroup's way over a tile: position and channel of this lane's value or piece, false behind the last one.  Neighbouring lanes
// take neighbouring channels, or positions.
template <int V>
__device__ __forceinline__ bool flat_channels(const FlatArgs& a, int cn, int pn, int i, int& p, int& c) {
  if (V > 1) { p = i / (kFlat / V); c = i % (kFlat / V) * V; }
  else { p = a.by_c(i); c = i - p * min(a.C, kFlat); }
  return p < pn && c < cn;
}
template <int V>
__device__ __forceinline__ bool flat_positions(const FlatArgs& a, int cn, int pn, int i, int& p, int& c) {
  if (V > 1) { c = i / (kFlat / V); p = i % (kFlat / V) * V; }
  else { c = a.by_p(i); p = i - c * min(a.HW, kFlat); }
  return p < pn && c < cn;
}
// All of a lane's reads (get) are on their way before the first is used (put): one after the other they take a memory latency each.  Of `all` steps
// of all lanes.  (Values of 16 bits in registers of their own: a load into half a register waits for the other half's.)
template <int STEPS, typename R, typename At, typename Get>
__device__ __forceinline__ void flat_get(R (&v)[STEPS], int all, At at, Get get) {
#pragma unroll
  for (int k = 0; k < STEPS; k++) {
    int p, c;
    if (256 * k < all && at((int)threadIdx.x + 256 * k, p, c)) v[k] = get(p, c);
  }
}
template <int STEPS, typename R, typename At, typename Put>
__device__ __forceinline__ void flat_put(const R (&v)[STEPS], int all, At at, Put put) {
#pragma unroll
  for (int k = 0; k < STEPS; k++) {
    int p, c;
    if (256 * k < all && at((int)threadIdx.x + 256 * k, p, c)) put(p, c, v[k]);
  }
}

template <typename T, bool PIECES, int ROWS>
__global__ __launch_bounds__(256) void flatten_fwd_kernel(PtrTab ws, size_t x_off, size_t y_off, FlatArgs a) {
  constexpr int V = FlatTile<T>::V, PITCH = FlatTile<T>::kPitch, POS = flat_positions_of(ROWS), ALL = kFlat * POS / 256;
  constexpr bool BLOCK = ROWS == FLAT_BLOCK || ROWS == FLAT_BLOCK_128;
  __shared__ __attribute__((aligned(16))) T tile[POS * PITCH];
  const int n = blockIdx.y, c0 = (int)blockIdx.x % a.cblocks * kFlat, p0 = (int)blockIdx.x / a.cblocks * POS;
  const int cn = min(kFlat, a.C - c0), pn = min(POS, a.HW - p0), wc = min(kFlat, a.C), wp = min(kFlat, a.HW);
  const T* x = (const T*)ws.p[blockIdx.z] + x_off + ((int64_t)n * a.HW + p0) * a.C + c0;
  T* y = (T*)ws.p[blockIdx.z] + y_off + ((int64_t)n * a.C + c0) * a.HW + p0;
  if constexpr (PIECES) {
    uint4 v[ALL / V];
    auto at = [&](int i, int& p, int& c) { return flat_channels<V>(a, cn, pn, i, p, c); };
    flat_get(v, pn * (kFlat / V), at, [&](int p, int c) { return *reinterpret_cast<const uint4*>(x + p * a.C + c); });
    flat_put(v, pn * (kFlat / V), at, [&](int p, int c, const uint4& q) { *reinterpret_cast<uint4*>(tile + p * PITCH + c) = q; });
  } else {
    uint32_t v[ALL];
    auto at = [&](int i, int& p, int& c) { return flat_channels<1>(a, cn, pn, i, p, c); };
    flat_get(v, pn * wc, at, [&](int p, int c) { return flat_bits(x[p * a.C + c]); });
    flat_put(v, pn * wc, at, [&](int p, int c, uint32_t q) { flat_store(tile + p * PITCH + c, q); });
  }
  __syncthreads();
  if constexpr (ROWS == FLAT_ELEMENTS) {
    uint32_t v[ALL];
    auto at = [&](int i, int& p, int& c) { return flat_positions<1>(a, cn, pn, i, p, c); };
    flat_get(v, cn * wp, at, [&](int p, int c) { return flat_bits(tile[p * PITCH + c]); });
    flat_put(v, cn * wp, at, [&](int p, int c, uint32_t q) { flat_store(y + c * a.HW + p, q); });
  } else {
#pragma unroll
    for (int k = 0; k < ALL / V; k++) {
      const int i = (int)threadIdx.x + 256 * k;
      union { uint4 q; T e[V]; } o;
      int p, c;
      if (BLOCK) {
        c = a.by_p(i * V);
        p = i * V - c * a.HW;
        if (i * V >= cn * a.HW) continue;
      } else if (!flat_positions<V>(a, cn, pn, i, p, c)) {
        continue;
      }
      T* to = y + c * a.HW + p;
#pragma unroll
      for (int e = 0; e < V; e++) {
        o.e[e] = tile[p * PITCH + c];
        if (++p == a.HW && BLOCK) { p = 0; c++; }
      }
      *reinterpret_cast<uint4*>(to) = o.q;
    }
  }
}

template <typename T, bool PIECES, int ROWS>
__global__ __launch_bounds__(256) void flatten_bwd_kernel(PtrTab ws, size_t dy_off, size_t dx_off, FlatArgs a, int use_mask, size_t mask_off) {
  constexpr int V = FlatTile<T>::V, PITCH = FlatTile<T>::kPitch, POS = flat_positions_of(ROWS), ALL = kFlat * POS / 256;
  constexpr bool BLOCK = ROWS == FLAT_BLOCK || ROWS == FLAT_BLOCK_128;
  __shared__ __attribute__((aligned(16))) T tile[POS * PITCH];
  const int n = blockIdx.y, c0 = (int)blockIdx.x % a.cblocks * kFlat, p0 = (int)blockIdx.x / a.cblocks * POS;
  const int cn = min(kFlat, a.C - c0), pn = min(POS, a.HW - p0), wc = min(kFlat, a.C), wp = min(kFlat, a.HW);
  const int64_t first = ((int64_t)n * a.HW + p0) * a.C + c0;
  const T* dy = (const T*)ws.p[blockIdx.z] + dy_off + ((int64_t)n * a.C + c0) * a.HW + p0;
  T* dx = (T*)ws.p[blockIdx.z] + dx_off + first;
  const T* mask = (const T*)ws.p[blockIdx.z] + mask_off + first;
  constexpr int OUT = PIECES ? ALL / V : ALL;
  union Piece { uint4 q; T e[V]; };
  uint4 mq[PIECES ? ALL / V : 1];
  uint32_t me[PIECES ? 1 : ALL];
  auto out = [&](int i, int& p, int& c) { return flat_channels<PIECES ? V : 1>(a, cn, pn, i, p, c); };
  const int out_steps = pn * (PIECES ? kFlat / V : wc);
  if (use_mask) {
    if constexpr (PIECES) flat_get(mq, out_steps, out, [&](int p, int c) { return *reinterpret_cast<const uint4*>(mask + p * a.C + c); });
    else flat_get(me, out_steps, out, [&](int p, int c) { return flat_bits(mask[p * a.C + c]); });
  }
  if constexpr (ROWS == FLAT_ELEMENTS) {
    uint32_t v[ALL];
    auto at = [&](int i, int& p, int& c) { return flat_positions<1>(a, cn, pn, i, p, c); };
    flat_get(v, cn * wp, at, [&](int p, int c) { return flat_bits(dy[c * a.HW + p]); });
    flat_put(v, cn * wp, at, [&](int p, int c, uint32_t q) { flat_store(tile + p * PITCH + c, q); });
  } else {
    Piece v[ALL / V];
    auto at = [&](int i, int& p, int& c) {
      if (!BLOCK) return flat_positions<V>(a, cn, pn, i, p, c);
      c = a.by_p(i * V);
      p = i * V - c * a.HW;
      return i * V < cn * a.HW;
    };
    flat_get(v, cn * (POS / V), at, [&](int p, int c) { Piece o; o.q = *reinterpret_cast<const uint4*>(dy + c * a.HW + p); return o; });
    flat_put(v, cn * (POS / V), at, [&](int p, int c, const Piece& o) {
#pragma unroll
      for (int e = 0; e < V; e++) {
        tile[p * PITCH + c] = o.e[e];
        if (++p == a.HW && BLOCK) { p = 0; c++; }
      }
    });
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < OUT; k++) {
    int p, c;
    if (256 * k >= out_steps || !out((int)threadIdx.x + 256 * k, p, c)) continue;
    if constexpr (PIECES) {
      Piece o, m;
      o.q = *reinterpret_cast<const uint4*>(tile + p * PITCH + c);
      m.q = mq[k];
#pragma unroll
      for (int e = 0; e < V; e++)
        if (use_mask && !(ldf(&m.e[e]) > 0.f)) o.e[e] = (T)0;
      *reinterpret_cast<uint4*>(dx + p * a.C + c) = o.q;
    } else {
      T v = tile[p * PITCH + c], m;
      flat_store(&m, me[k]);
      if (use_mask && !(ldf(&m) > 0.f)) v = (T)0;
      dx[p * a.C + c] = v;
    }
  }
}

// A value a lane straight from memory to memory: few values, whose time is one round trip (flatten_direct).
template <typename T>
__global__ __launch_bounds__(256) void flatten_fwd_direct_kernel(PtrTab ws, size_t x_off, size_t y_off, int C, int HW) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= C * HW) return;
  const int c = (int)((unsigned)i / (unsigned)HW), p = i - c * HW;
  const int64_t image = (int64_t)blockIdx.y * C * HW;
  ((T*)ws.p[blockIdx.z] + y_off + image)[i] = ((const T*)ws.p[blockIdx.z] + x_off + image)[p * C + c];
}
template <typename T>
__global__ __launch_bounds__(256) void flatten_bwd_direct_kernel(PtrTab ws, size_t dy_off, size_t dx_off, int C, int HW, int use_mask, size_t mask_off) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= C * HW) return;
  const int p = (int)((unsigned)i / (unsigned)C), c = i - p * C;
  const int64_t image = (int64_t)blockIdx.y * C * HW;
  T v = ((const T*)ws.p[blockIdx.z] + dy_off + image)[c * HW + p];
  if (use_mask && !(ldf((const T*)ws.p[blockIdx.z] + mask_off + image + i) > 0.f)) v = (T)0;
  ((T*)ws.p[blockIdx.z] + dx_off + image)[i] = v;
}

// f(kernel of the form): the template arguments as types
template <typename F>
static void flat_form(bool pieces, int rows, F f) {
  if (pieces) {
    if (rows == FLAT_BLOCK) f(std::true_type{}, std::integral_constant<int, FLAT_BLOCK>{});
    else if (rows == FLAT_BLOCK_128) f(std::true_type{}, std::integral_constant<int, FLAT_BLOCK_128>{});
    else if (rows == FLAT_PIECES) f(std::true_type{}, std::integral_constant<int, FLAT_PIECES>{});
    else f(std::true_type{}, std::integral_constant<int, FLAT_ELEMENTS>{});
  } else {
    if (rows == FLAT_PIECES) f(std::false_type{}, std::integral_constant<int, FLAT_PIECES>{});
    else f(std::false_type{}, std::integral_constant<int, FLAT_ELEMENTS>{});
  }
}

// (Tensors begin at multiples of 64 elements, so that whole rows of pieces are all that pieces take.)
static FlatArgs flat_args(int C, int HW, const FlattenPlan& pl) {
  FlatArgs a;
  a.C = C;
  a.HW = HW;
  a.cblocks = (C + kFlat - 1) / kFlat;
  a.by_c.set(std::min(C, kFlat));
  a.by_p.set(std::min(HW, flat_positions_of(pl.rows)));
  return a;
}

hipError_t launch_flatten_fwd(bool is_bf16, const PtrTab& ws, size_t x_off, size_t y_off, int N, int C, int H, int W, int count,
                              hipStream_t s) {
  if (x_off % 8 || y_off % 8) return hipErrorInvalidValue;
  const FlattenPlan pl = flatten_plan((int64_t)N * count, C, H * W, is_bf16);
  const dim3 g((unsigned)pl.groups, (unsigned)N, (unsigned)count);
  if (pl.direct) {
    if (is_bf16) hipLaunchKernelGGL(flatten_fwd_direct_kernel<bf16_t>, g, dim3(256), 0, s, ws, x_off, y_off, C, H * W);
    else hipLaunchKernelGGL(flatten_fwd_direct_kernel<float>, g, dim3(256), 0, s, ws, x_off, y_off, C, H * W);
    return hipGetLastError();
  }
  const FlatArgs a = flat_args(C, H * W, pl);
  flat_form(pl.pieces, pl.rows, [&](auto P, auto R) {
    if (is_bf16) hipLaunchKernelGGL((flatten_fwd_kernel<bf16_t, decltype(P)::value, decltype(R)::value>), g, dim3(256), 0, s, ws, x_off, y_off, a);
    else hipLaunchKernelGGL((flatten_fwd_kernel<float, decltype(P)::value, decltype(R)::value>), g, dim3(256), 0, s, ws, x_off, y_off, a);
  });
  return hipGetLastError();
}

hipError_t launch_flatten_bwd(bool is_bf16, const PtrTab& ws, size_t dy_off, size_t dx_off, int N, int C, int H, int W, bool use_mask,
                              size_t mask_off, int count, hipStream_t s) {
  if (dy_off % 8 || dx_off % 8 || mask_off % 8) return hipErrorInvalidValue;
  const FlattenPlan pl = flatten_plan((int64_t)N * count, C, H * W, is_bf16);
  const dim3 g((unsigned)pl.groups, (unsigned)N, (unsigned)count);
  const int um = use_mask ? 1 : 0;
  if (pl.direct) {
    if (is_bf16) hipLaunchKernelGGL(flatten_bwd_direct_kernel<bf16_t>, g, dim3(256), 0, s, ws, dy_off, dx_off, C, H * W, um, mask_off);
    else hipLaunchKernelGGL(flatten_bwd_direct_kernel<float>, g, dim3(256), 0, s, ws, dy_off, dx_off, C, H * W, um, mask_off);
    return hipGetLastError();
  }
  const FlatArgs a = flat_args(C, H * W, pl);
  flat_form(pl.pieces, pl.rows, [&](auto P, auto R) {
    if (is_bf16) hipLaunchKernelGGL((flatten_bwd_kernel<bf16_t, decltype(P)::value, decltype(R)::value>), g, dim3(256), 0, s, ws, dy_off, dx_off, a, um, mask_off);
    else hipLaunchKernelGGL((flatten_bwd_kernel<float, decltype(P)::value, decltype(R)::value>), g, dim3(256), 0, s, ws, dy_off, dx_off, a, um, mask_off);
  });
  return hipGetLastError();
}

// ------------------------------------------------------------------ softmax cross-entropy
// One workgroup per image: dz = (softmax(z) - onehot(label)) / N, i.e. the gradient of the MEAN loss: this is
// where the division by the mini-batch size enters (Section 2.1).  The per-image losses go to a small array and
// are summed in image order by a second tiny kernel, so the result does not depend on scheduling.
template <typename T, typename Z>
__global__ __launch_bounds__(256) void softmax_ce_kernel(PtrTab ws, CPtrTab labels, size_t z_off, size_t dz_off, size_t loss_byte_off,
                                                         int N, int K) {
  __shared__ float red[4];
  const int l = blockIdx.z, n = blockIdx.x;
  const Z* zn = reinterpret_cast<const Z*>((const T*)ws.p[l] + z_off) + (int64_t)n * K;
  T* dz = (T*)ws.p[l] + dz_off + (int64_t)n * K;
  float* img_loss = reinterpret_cast<float*>((char*)ws.p[l] + loss_byte_off);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float m = -INFINITY;
  for (int j = threadIdx.x; j < K; j += 256) m = fmaxf(m, ldf(zn + j));
  m = wave_max(m);
  if (lane == 0) red[wave] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float sum = 0.f;
  for (int j = threadIdx.x; j < K; j += 256) sum += expf(ldf(zn + j) - m);
  sum = wave_sum(sum);
  if (lane == 0) red[wave] = sum;
  __syncthreads();
  sum = (red[0] + red[1]) + (red[2] + red[3]);
  const int y = ((const int32_t*)labels.p[l])[n];
  const float inv = 1.0f / sum, invN = 1.0f / (float)N;
  for (int j = threadIdx.x; j < K; j += 256) stf(dz + j, (expf(ldf(zn + j) - m) * inv - (j == y ? 1.f : 0.f)) * invN);
  if (threadIdx.x == 0) img_loss[n] = (y >= 0 && y < K) ? -(ldf(zn + y) - m - logf(sum)) : NAN;   // a bad label poisons the loss
}

// Sums stay in image order: the losses come to LDS together (one dependent read after the other, 256 images took 11 us).
constexpr int kLossChunk = 1024;
__global__ __launch_bounds__(256) void loss_mean_kernel(PtrTab ws, size_t loss_byte_off, int N, float* loss_out) {
  __shared__ __attribute__((aligned(16))) float part[kLossChunk];
  const float* img_loss = reinterpret_cast<const float*>((const char*)ws.p[blockIdx.x] + loss_byte_off);
  float tot = 0.f;
  for (int n0 = 0; n0 < N; n0 += kLossChunk) {
    const int len = min(kLossChunk, N - n0);
    if (n0) __syncthreads();
    for (int i = threadIdx.x; i < (len + 15) / 16 * 16; i += 256) part[i] = i < len ? img_loss[n0 + i] : -0.f;    // -0 changes no sum
    __syncthreads();
    if (threadIdx.x == 0)
      for (int i = 0; i < len; i += 16) {
        float4 v[4];
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = *reinterpret_cast<const float4*>(part + i + 4 * k);
#pragma unroll
        for (int k = 0; k < 4; k++) { tot += v[k].x; tot += v[k].y; tot += v[k].z; tot += v[k].w; }
      }
  }
  if (threadIdx.x == 0) loss_out[blockIdx.x] = tot / (float)N;
}

hipError_t launch_loss_mean(const PtrTab& ws, size_t loss_byte_off, int N, float* loss_out, int count, hipStream_t s) {
  hipLaunchKernelGGL(loss_mean_kernel, dim3(count), dim3(256), 0, s, ws, loss_byte_off, N, loss_out);
  return hipGetLastError();
}

hipError_t launch_softmax_ce(bool is_bf16, bool z_f32, const PtrTab& ws, const CPtrTab& labels, size_t z_off, size_t dz_off,
                             size_t loss_byte_off, int N, int K, float* loss_out, int count, hipStream_t s) {
  dim3 g((unsigned)N, 1, (unsigned)count);
  if (is_bf16 && z_f32) hipLaunchKernelGGL((softmax_ce_kernel<bf16_t, float>), g, dim3(256), 0, s, ws, labels, z_off, dz_off, loss_byte_off, N, K);
  else if (is_bf16) hipLaunchKernelGGL((softmax_ce_kernel<bf16_t, bf16_t>), g, dim3(256), 0, s, ws, labels, z_off, dz_off, loss_byte_off, N, K);
  else hipLaunchKernelGGL((softmax_ce_kernel<float, float>), g, dim3(256), 0, s, ws, labels, z_off, dz_off, loss_byte_off, N, K);
  return loss_out ? launch_loss_mean(ws, loss_byte_off, N, loss_out, count, s) : hipGetLastError();
}

// ------------------------------------------------------------------ evaluation: rank of the true class
// rank[n] = number of classes ordered before the label's class when scores are sorted in descending order (equal
// scores: lower class index first).  rank < k  <=>  the label is among the k best: top-1 / top-5 errors (Section 4.3)
// are counts of rank >= 1 / rank >= 5.  A label outside [0, K) gets rank K.  One workgroup per image.
template <typename T, typename Z>
__global__ __launch_bounds__(256) void label_rank_kernel(PtrTab ws, CPtrTab labels, size_t z_off, int N, int K, int32_t* rank_out) {
  __shared__ int red[4];
  const int l = blockIdx.z, n = blockIdx.x;
  const Z* zn = reinterpret_cast<const Z*>((const T*)ws.p[l] + z_off) + (int64_t)n * K;
  const int y = ((const int32_t*)labels.p[l])[n];
  const bool ok = y >= 0 && y < K;
  const float zy = ok ? ldf(zn + y) : 0.f;
  int cnt = 0;
  for (int j = threadIdx.x; j < K; j += 256) {
    const float zj = ldf(zn + j);
    cnt += (zj > zy || (zj == zy && j < y)) ? 1 : 0;
  }
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_down(cnt, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) rank_out[(int64_t)l * N + n] = ok ? (red[0] + red[1]) + (red[2] + red[3]) : K;
}

hipError_t launch_label_rank(bool is_bf16, bool z_f32, const PtrTab& ws, const CPtrTab& labels, size_t z_off, int N, int K,
                             int32_t* rank_out, int count, hipStream_t s) {
  dim3 g((unsigned)N, 1, (unsigned)count);
  if (is_bf16 && z_f32) hipLaunchKernelGGL((label_rank_kernel<bf16_t, float>), g, dim3(256), 0, s, ws, labels, z_off, N, K, rank_out);
  else if (is_bf16) hipLaunchKernelGGL((label_rank_kernel<bf16_t, bf16_t>), g, dim3(256), 0, s, ws, labels, z_off, N, K, rank_out);
  else hipLaunchKernelGGL((label_rank_kernel<float, float>), g, dim3(256), 0, s, ws, labels, z_off, N, K, rank_out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ fully connected weight gradient as factors
// The weight gradient of a fully connected layer over a mini-batch of N images is the rank-N product
// dW[o][i] = sum_n dy[n][o] x[n][i].  Instead of writing out * in values, keep the factors, both with the images
// innermost: x transposed to [in][NP] and dy transposed to [out][NP] (NP = N rounded up to 8, zero-filled), so that the
// update kernel reads the N values of one unit as contiguous 16-byte pieces (the k-contiguous operands of an MFMA).
// The bias gradient db[o] = sum_n dy[n][o] is written out.
// A thread turns 8 units x 8 images around; neighbouring threads take neighbouring images, up to 64 of them, then neighbouring units, so that both
// the reads of the mini-batch's rows and the writes are of whole lines.  Three layers, 9 216 -> 4 096 -> 4 096 -> 1 000, one learner
// of 256 images: 18 us; 18 learners of 16: 30 us with a thread per unit (all images in turn), 21 here.
constexpr int kSaveSegments = 8;              // of a bias gradient's images: their sums are added in order
__global__ __launch_bounds__(256) void fc_save_factors_kernel(PtrTab ws, PtrTab grads, size_t x_off, size_t dy_off, size_t fx_off,
                                                              size_t fdy_off, int64_t b_off, int N, int in, int out, int NP, int x_blocks,
                                                              int dy_blocks) {
  __shared__ float part[256];
  const bf16_t* dy = (const bf16_t*)ws.p[blockIdx.z] + dy_off;
  if ((int)blockIdx.x >= x_blocks + dy_blocks) {      // bias: 32 units of a workgroup, the images in segments
    if (blockIdx.y > 0) return;
    const int o = ((int)blockIdx.x - x_blocks - dy_blocks) * (256 / kSaveSegments) + threadIdx.x % (256 / kSaveSegments);
    const int per = (N + kSaveSegments - 1) / kSaveSegments, n0 = threadIdx.x / (256 / kSaveSegments) * per, n1 = min(N, n0 + per);
    float sum = 0.f;
    if (o < out)
#pragma unroll 8
      for (int n = n0; n < n1; n++) sum += bf2f(dy[(int64_t)n * out + o]);
    part[threadIdx.x] = sum;
    __syncthreads();
    if ((int)threadIdx.x < 256 / kSaveSegments && o < out) {
      float v = 0.f;
#pragma unroll
      for (int k = 0; k < kSaveSegments; k++) v += part[threadIdx.x + k * (256 / kSaveSegments)];
      ((float*)grads.p[blockIdx.z] + b_off)[o] = v;
    }
    return;
  }
  const bool is_x = (int)blockIdx.x < x_blocks;
  const bf16_t* src_t = is_x ? (const bf16_t*)ws.p[blockIdx.z] + x_off : dy;
  bf16_t* dst_t = (bf16_t*)ws.p[blockIdx.z] + (is_x ? fx_off : fdy_off);
  const int units = is_x ? in : out;
  const uint32_t pieces = min(8u, (uint32_t)NP / 8u);                 // of 8 images, side by side
  const uint32_t t = (blockIdx.x - (is_x ? 0u : (uint32_t)x_blocks)) * 256u + threadIdx.x;
  const int n0 = (int)(blockIdx.y * 64u + (t % pieces) * 8u), u0 = (int)(t / pieces) * 8;
  if (u0 >= units || n0 >= NP) return;
  union { uint4 q; bf16_t h[8]; } src[8], dst[8];
#pragma unroll
  for (int k = 0; k < 8; k++) {
    src[k].q = make_uint4(0u, 0u, 0u, 0u);
    if (n0 + k >= N) continue;
    src[k].q = *reinterpret_cast<const uint4*>(src_t + (int64_t)(n0 + k) * units + u0);
  }
#pragma unroll
  for (int e = 0; e < 8; e++)
#pragma unroll
    for (int k = 0; k < 8; k++) dst[e].h[k] = src[k].h[e];
#pragma unroll
  for (int e = 0; e < 8; e++) *reinterpret_cast<uint4*>(dst_t + (int64_t)(u0 + e) * NP + n0) = dst[e].q;
}

hipError_t launch_fc_save_factors(const PtrTab& ws, const PtrTab& grads, size_t x_off, size_t dy_off, size_t fx_off, size_t fdy_off,
                                  int64_t b_off, int N, int in, int out, int NP, int count, hipStream_t s) {
  if (in % 8 || out % 8) return hipErrorInvalidValue;          // (the matrix kernels take no other layers)
  const int pieces = std::min(8, NP / 8);
  auto blocks = [&](int units) { return (units / 8 * pieces + 255) / 256; };
  const int per_bias = 256 / kSaveSegments;
  hipLaunchKernelGGL(fc_save_factors_kernel, dim3((unsigned)(blocks(in) + blocks(out) + (out + per_bias - 1) / per_bias), (unsigned)((NP + 63) / 64), (unsigned)count),
                     dim3(256), 0, s, ws, grads, x_off, dy_off, fx_off, fdy_off, b_off, N, in, out, NP, blocks(in), blocks(out));
  return hipGetLastError();
}

}  // namespace sasgd
