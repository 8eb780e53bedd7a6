// The first convolution of a network and the 3 x 3 / 2 max pooling behind it in one kernel (bf16 compute; Section 2.1 learner step, layer shapes
// of Section 4.1).  Nothing but the pooling reads that convolution's output -- the first layer has no input gradient, and the winners
// carry what the backward pass needs -- so it never leaves LDS: a first layer has few input channels and large images, and its output is the
// largest tensor of the network.
//
// A workgroup walks down one image (or a segment of its pooled rows), `CR` convolution rows at a time: the input patch under them goes to LDS (as in
// conv_halo_seq_kernel: whole pixels, the contraction walks the packed filters' 16-k blocks in order), four wavefronts multiply 64 positions
// each by all output channels, bias and ReLU are applied and the rows are put, as the bf16 values that would have been stored, where the patch
// was; then every pooled row whose windows are complete is written, and the last two convolution rows are kept beside for the next ones.
// Products come out channel by position (filters as the first operand), so that a lane holds four neighbouring channels of a position.
//
// Rows are kept as 16-bit integers in the order of their values, so that a window's maximum and the place of the first one are one integer
// maximum each (compared and selected as floats: 153 us of the first figure below).  What bounds it: a round's patch load, products, pooling and
// stores follow each other, and only the other workgroups of the compute unit fill the gaps.
// Convolution and pooling, us, separate kernels / this one: AlexNet-shaped net (11 x 11 / 4, 96 channels), 256 images 149 / 113, 18 learners of 16
// 180 / 136, one of 16 21 / 17; CIFAR-shaped net, 18 learners of 128 104 / 70, 4 of 64 19 / 16; 3 x 3, 64 channels of 64 x 64 images, 18 of 32 187 / 124.
#include <algorithm>
#include "dev_common.hpp"
#include "kernels.hpp"

namespace sasgd {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef int v4i_t __attribute__((ext_vector_type(4)));

namespace {
constexpr uint32_t kOutOfRange = 0x80000000u;   // buffer offset beyond any tensor: the load returns zeros
constexpr int kTM = 2;                          // blocks of 32 positions per wavefront

// Two bf16 values as 16-bit integers of their order (RELU: no value has a sign); NaNs, which come with every bit set, below all others.
template <bool RELU>
__device__ __forceinline__ uint32_t ordered(uint32_t two) {
  if (RELU) return two;
  const uint32_t sign = (two >> 15) & 0x00010001u;
  return two ^ ((sign << 15) - sign);
}
}  // namespace

struct ConvPoolArgs {
  int PW, spp, pixb, C16;      // patch width in pixels; 16-byte slots and bytes per pixel (data + padding); 16-channel blocks per tap
  int CR;                      // convolution rows per round
  int segs, per;               // segments of an image, pooled rows of one
  int PH, PWo;                 // pooled size
  int pitch;                   // bytes of a staged position
  int carry_off, bias_off, tab_off;   // LDS: the two kept rows, biases, slot table (the patch and the round's rows lie at 0)
  int pool_relu;               // ReLU behind the pooling (RELU: in front of it, and winners mark the windows that no gradient passes)
  size_t y_off, arg_off;       // pooled tensor (elements), winners (bytes)
  FastDiv by_pw, by_spp, by_ow, by_segs, by_pwo, by_c8;
};

template <int TN, bool C8, bool RELU>
__global__ __launch_bounds__(256, 2) void conv_pool_kernel(PtrTab ws, CPtrTab wts, IGemm g, Epilogue ep, ConvPoolArgs h) {
  extern __shared__ __attribute__((aligned(16))) char conv_pool_lds[];
  char* lds = conv_pool_lds;
  char* const base = (char*)ws.p[blockIdx.z];
  const bf16_t* wv = (const bf16_t*)wts.p[blockIdx.z];
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void*)((const bf16_t*)base + g.a_off), 0, (int)g.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc((void*)(wv + g.b_off), 0, (int)g.b_bytes, 0x00020000);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), hl = lane >> 5;
  const int n = h.by_segs((int)blockIdx.x), seg = (int)blockIdx.x - n * h.segs;
  const int p_begin = seg * h.per, p_end = min(h.PH, p_begin + h.per);
  const int row_end = min(2 * p_end + 1, g.OH);
  const int ks = g.ks, KB16 = g.ldb / 16, NB = (g.Ncols + 31) / 32;
  bf16_t* const y = (bf16_t*)base + h.y_off;
  uint8_t* const arg = (uint8_t*)base + h.arg_off;

  int boff[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) boff[j] = j < NB ? (j * KB16 * 512 + lane * 8) * 2 : (int)kOutOfRange;
  // filters of k-block kb; behind the last one: out of range, zeros for nobody
  auto load_b = [&](bf16x8 (&bt)[TN], int kb) {
#pragma unroll
    for (int j = 0; j < TN; j++) bt[j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc_b, boff[j], kb * 1024, 0));
  };
  const int taps = ks * ks, blocks = C8 ? (taps + 1) / 2 : taps * h.C16;
  const int row_step = (h.PW - ks) * h.pixb;           // patch bytes from behind a window's row to its next one
  float* const bias = reinterpret_cast<float*>(lds + h.bias_off);
  if (tid < 32 * TN) bias[tid] = ep.has_bias && tid < g.Ncols ? bf2f(wv[ep.bias_off + tid]) : 0.f;
  const int c8s = g.Ncols / 8;
  // where the patch's slots come from, but for the round's first row: bytes, or out of range (padding of a pixel, columns outside)
  int* const tab = reinterpret_cast<int*>(lds + h.tab_off);
  for (int sl = tid; sl < (h.CR + ks - 1) * h.PW * h.spp; sl += 256) {
    const int px = h.by_spp(sl), sub = sl - px * h.spp, pr = h.by_pw(px), iw = px - pr * h.PW - g.pad;
    tab[sl] = sub * 8 < g.C && (unsigned)iw < (unsigned)g.W ? (pr * g.W + iw) * g.C * 2 + sub * 16 : (int)kOutOfRange;
  }
  __syncthreads();
  int next_p = p_begin;
#pragma unroll 1
  for (int r0 = 2 * p_begin; r0 < row_end; r0 += h.CR) {
    const int rows = min(h.CR, row_end - r0), M = rows * g.OW;
    // ---- the input patch: LDS-direct loads, 64 consecutive 16-byte slots per wavefront and instruction
    const int row_slots = h.PW * h.spp, slots = (rows + ks - 1) * row_slots, wave_slot = wave * 64;
    const int sl_lo = max(0, g.pad - r0) * row_slots, sl_hi = min(rows + ks - 1, g.H + g.pad - r0) * row_slots;   // rows inside the image
    const int first = (n * g.H + r0 - g.pad) * g.W * g.C * 2;
#pragma unroll 2
    for (int s0 = 0; s0 < slots; s0 += 256) {
      const int sl = s0 + tid, t = tab[min(sl, slots - 1)];
      const int off = t >= 0 && sl >= sl_lo && sl < sl_hi ? t + first : (int)kOutOfRange;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (__attribute__((address_space(3))) void*)(lds + (s0 + wave_slot) * 16), 16, off, 0, 0, 0);
    }
    bf16x8 b0[TN], b1[TN], b2[TN];
    load_b(b0, 0);
    load_b(b1, 1);
    load_b(b2, 2);
    int abase[kTM];
#pragma unroll
    for (int i = 0; i < kTM; i++) {
      const int m = min((wave * kTM + i) * 32 + (lane & 31), M - 1);     // positions behind the round's last one repeat it, never stored
      const int row = h.by_ow(m);
      abase[i] = (row * h.PW + m - row * g.OW) * h.pixb + (C8 ? 0 : 16 * hl);
    }
    floatx16 acc[kTM][TN];
#pragma unroll
    for (int i = 0; i < kTM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    auto lds_a = [&](bf16x8 (&a)[kTM], int off) {
#pragma unroll
      for (int i = 0; i < kTM; i++) a[i] = *reinterpret_cast<const bf16x8*>(lds + abase[i] + off);
    };
    auto multiply = [&](const bf16x8 (&b)[TN], const bf16x8 (&a)[kTM]) {
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < kTM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_s_setprio(0);
    };
    if (wave * kTM * 32 < M) {                           // the whole wavefront
      // patch byte offset that the lanes of the running k-block add to their window origin: the block's tap and 16 channels, or, of 8
      // channels, two taps, one for each half of the lanes (behind the last tap: zero filters, the last tap again)
      int off = 0, kw = 0, c16 = 0, tap = 0;
      auto next_tap = [&]() {
        const bool last = tap + 1 >= taps, wrap = kw + 1 == ks;
        off += last ? 0 : h.pixb + (wrap ? row_step : 0);
        kw = wrap ? 0 : kw + 1;
        tap++;
      };
      int lane_off = 0;
      auto advance = [&]() {                             // lane_off for the next k-block
        if (C8) {
          const int o0 = off;
          next_tap();
          lane_off = hl ? off : o0;
          next_tap();
        } else {
          lane_off = off + c16 * 32;
          c16++;
          if (c16 == h.C16) { c16 = 0; next_tap(); }
        }
      };
      bf16x8 fa[kTM], fb[kTM];
      advance();
      lds_a(fa, lane_off);
      int kb = 0;
      // a k-block: the next one's positions are read, this one's products run, its filters' place takes those of three blocks on
      auto block = [&](bf16x8 (&bc)[TN], bf16x8 (&cur)[kTM], bf16x8 (&nxt)[kTM]) {
        advance();
        lds_a(nxt, lane_off);
        multiply(bc, cur);
        load_b(bc, kb + 3);
        kb++;
      };
      const int sixes = blocks / 6, rest = blocks - 6 * sixes;
#pragma unroll 1
      for (int t = 0; t < sixes; t++) {
        block(b0, fa, fb); block(b1, fb, fa); block(b2, fa, fb);
        block(b0, fb, fa); block(b1, fa, fb); block(b2, fb, fa);
      }
      if (rest > 0) block(b0, fa, fb);
      if (rest > 1) block(b1, fb, fa);
      if (rest > 2) block(b2, fa, fb);
      if (rest > 3) block(b0, fb, fa);
      if (rest > 4) block(b1, fa, fb);
    }
    __syncthreads();                                     // the patch has been read: the convolution's rows take its place
    if (wave * kTM * 32 < M) {
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const int c = 32 * j + 8 * q + 4 * hl;
          if (c >= g.Ncols) continue;
          const float4 bq = *reinterpret_cast<const float4*>(bias + c);
          const float bs[4] = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
          for (int i = 0; i < kTM; i++) {
            const int m = (wave * kTM + i) * 32 + (lane & 31);
            float f[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
              f[e] = acc[i][j][4 * q + e] + bs[e];
              if (RELU) {
                f[e] = f[e] > 0.f ? f[e] : 0.f;
              } else {
                if (fabsf(f[e]) < 0x1p-134f) f[e] = 0.f;              // what rounds to -0
                if (f[e] != f[e]) f[e] = __uint_as_float(0xffffffffu);
              }
            }
            const uint32_t lo = ordered<RELU>(pack2bf(f[0], f[1])), hi = ordered<RELU>(pack2bf(f[2], f[3]));
            if (m < M) *reinterpret_cast<uint2*>(lds + m * h.pitch + c * 2) = make_uint2(lo, hi);
          }
        }
    }
    __syncthreads();
    // ---- pooled rows that are complete: window rows 2 p .. min(2 p + 2, OH - 1)
    const int done = r0 + rows - 1;
    const int p_hi = min(p_end, done == g.OH - 1 ? h.PH : done / 2);       // the first that is not
    const int items = (p_hi - next_p) * h.PWo * c8s;
    for (int it = tid; it < items; it += 256) {
      const int px = h.by_c8(it), c = (it - px * c8s) * 8;
      const int pr = h.by_pwo(px), pw = px - pr * h.PWo, ph = next_p + pr;
      const int h0 = 2 * ph, w0 = 2 * pw, nh = min(3, g.OH - h0), nw = min(3, g.OW - w0);
      // the largest of (value, 8 - place in the window): of equal values the first
      int key[8];
      uint4 v0;
#pragma unroll
      for (int t = 0; t < 9; t++) {                      // outside the image: the first element again, behind itself
        const bool in = t / 3 < nh && t % 3 < nw;
        const int row = h0 + (in ? t / 3 : 0), col = w0 + (in ? t % 3 : 0);
        const char* src = row < r0 ? lds + h.carry_off + ((row - r0 + 2) * g.OW + col) * h.pitch : lds + ((row - r0) * g.OW + col) * h.pitch;
        const uint4 v = *reinterpret_cast<const uint4*>(src + c * 2);
        if (t == 0) v0 = v;
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 8; e++) {
          const int k = (int)((e & 1 ? w[e / 2] & 0xffff0000u : w[e / 2] << 16) | (uint32_t)(8 - t));
          key[e] = t == 0 ? k : max(key[e], k);
        }
      }
      const uint32_t w0s[4] = {v0.x, v0.y, v0.z, v0.w};
      uint32_t best[8], won[8];
#pragma unroll
      for (int e = 0; e < 8; e++) {
        const int val = key[e] >> 16;
        won[e] = 8u - ((uint32_t)key[e] & 15u);
        if (RELU) {
          best[e] = (uint32_t)val;
          if (val == 0) won[e] = 255;
        } else {
          // a window that begins with a NaN is one; others do not see theirs, which order below every number
          const bool nan = (e & 1 ? w0s[e / 2] >> 16 : w0s[e / 2] & 0xffffu) == 0x8000u;
          best[e] = nan ? 0x7fc0u : (uint32_t)(val ^ ((val >> 31) & 0x7fff)) & 0xffffu;
          if (nan) won[e] = 0;
          if (h.pool_relu && !(val > 0 && !nan)) best[e] = 0;
        }
      }
      const uint32_t o = ((uint32_t)(n * h.PH + ph) * h.PWo + pw) * g.Ncols + c;
      *reinterpret_cast<uint4*>(y + o) = make_uint4(best[0] | best[1] << 16, best[2] | best[3] << 16, best[4] | best[5] << 16, best[6] | best[7] << 16);
      *reinterpret_cast<uint2*>(arg + o) = make_uint2(won[0] | won[1] << 8 | won[2] << 16 | won[3] << 24, won[4] | won[5] << 8 | won[6] << 16 | won[7] << 24);
    }
    next_p = max(next_p, p_hi);
    if (r0 + h.CR >= row_end) break;
    __syncthreads();
    // ---- the last two rows (rows == CR >= 2 here) are kept for the next windows
    const int bytes = 2 * g.OW * h.pitch;
    for (int b = tid * 16; b < bytes; b += 256 * 16)
      *reinterpret_cast<uint4*>(lds + h.carry_off + b) = *reinterpret_cast<const uint4*>(lds + (rows - 2) * g.OW * h.pitch + b);
    __syncthreads();
  }
}

// Fills in everything that does not depend on the number of learners; false: the pair is not for this kernel.
static bool plan(const IGemm& g, const PoolShape& ps, ConvPoolArgs* h, size_t* lds_bytes) {
  const bool c8 = g.C == 8;
  if (ps.ks != 3 || ps.stride != 2 || ps.C != g.Ncols || ps.H != g.OH || ps.W != g.OW) return false;
  if (!(c8 || (g.C % 16 == 0 && g.C <= 112)) || g.Ncols % 8 || g.Ncols > 128 || g.OW + g.ks - 1 != g.W + 2 * g.pad) return false;
  h->PW = g.OW + g.ks - 1;
  h->spp = c8 ? 1 : g.C / 8 + 1;
  h->pixb = 16 * h->spp;
  h->C16 = c8 ? 1 : g.C / 16;
  h->CR = 128 * kTM / g.OW;
  if (h->CR < 2) return false;
  h->PH = ps.OH;
  h->PWo = ps.OW;
  h->pitch = g.Ncols * 2 + 16;
  const int slots = (h->CR + g.ks - 1) * h->PW * h->spp;
  h->carry_off = std::max((slots + 255) / 256 * 4096, h->CR * g.OW * h->pitch);
  h->bias_off = h->carry_off + 2 * g.OW * h->pitch;
  h->tab_off = h->bias_off + 128 * 4;
  *lds_bytes = (size_t)h->tab_off + (size_t)slots * 4;
  if (*lds_bytes > 80 * 1024) return false;              // two workgroups on a compute unit cover each other's patch loads
  const int images = g.M / (g.OH * g.OW);
  if (!FastDiv::exact(h->spp, slots + 255) || !FastDiv::exact(h->PW, slots + 255) || !FastDiv::exact(g.OW, 128 * kTM) ||
      (int64_t)images * h->PH >= ((int64_t)1 << 31) || (int64_t)h->PH * h->PWo * (g.Ncols / 8) >= ((int64_t)1 << 24))
    return false;
  h->by_pw.set(h->PW); h->by_spp.set(h->spp); h->by_ow.set(g.OW); h->by_pwo.set(h->PWo); h->by_c8.set(g.Ncols / 8);
  return FastDiv::exact(h->PWo, (int64_t)h->PH * h->PWo) && FastDiv::exact(g.Ncols / 8, (int64_t)h->PH * h->PWo * (g.Ncols / 8));
}

bool conv_pool_ok(const IGemm& g, const PoolShape& ps) {
  ConvPoolArgs h;
  size_t bytes;
  return plan(g, ps, &h, &bytes);
}

template <int TN>
static void launch_t(const PtrTab& ws, const CPtrTab& wts, const IGemm& g, const Epilogue& ep, const ConvPoolArgs& h, size_t bytes, int images, int count,
                     hipStream_t s) {
  const dim3 grid((unsigned)(images * h.segs), 1, (unsigned)count);
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), bytes, s, ws, wts, g, ep, h); };
  if (g.C == 8) ep.relu ? go(conv_pool_kernel<TN, true, true>) : go(conv_pool_kernel<TN, true, false>);
  else ep.relu ? go(conv_pool_kernel<TN, false, true>) : go(conv_pool_kernel<TN, false, false>);
}

hipError_t launch_conv_pool(const PtrTab& ws, const CPtrTab& wts, const IGemm& g, const Epilogue& ep, const PoolShape& ps, size_t y_off, size_t arg_off,
                            bool pool_relu, int count, hipStream_t s) {
  ConvPoolArgs h;
  size_t bytes;
  if (!plan(g, ps, &h, &bytes) || ep.use_mask || ep.out_f32 || g.ldb % 32) return hipErrorInvalidValue;
  const int images = g.M / (g.OH * g.OW);
  const int tn = (g.Ncols + 31) / 32, by_registers = tn == 1 ? 5 : tn == 2 ? 3 : 2;
  h.per = conv_pool_rows(h.PH, h.CR, (int64_t)images * count, std::min(by_registers, (int)(160 * 1024 / bytes)));
  h.segs = (h.PH + h.per - 1) / h.per;
  h.by_segs.set(h.segs);
  if (!FastDiv::exact(h.segs, (int64_t)images * h.segs)) return hipErrorInvalidValue;
  h.y_off = y_off;
  h.arg_off = arg_off;
  h.pool_relu = pool_relu ? 1 : 0;
  switch (tn) {
    case 1: launch_t<1>(ws, wts, g, ep, h, bytes, images, count, s); break;
    case 2: launch_t<2>(ws, wts, g, ep, h, bytes, images, count, s); break;
    case 3: launch_t<3>(ws, wts, g, ep, h, bytes, images, count, s); break;
    default: launch_t<4>(ws, wts, g, ep, h, bytes, images, count, s); break;
  }
  return hipGetLastError();
}

}  // namespace sasgd
