// bf16 MFMA implicit-GEMM kernels for calcGradient's convolutions, and the weight gradients of fully connected layers
// (Section 2.1 learner step; layer shapes of Section 4.1), written for gfx950 (CDNA4):
// v_mfma_f32_32x32x16_bf16 tiles, fp32 accumulation, LDS-staged im2col tiles, 64-wide wavefronts.
//
// GEMM views (activations NHWC bf16, "chunk" = 8 consecutive channels = 16 bytes):
//   forward  y[m][n]  = sum_k im2col(x)[m][k] * Wp[n][k]      m = (image, oh, ow), k = (kh, kw, c)
//   dgrad    dx[m][c] = sum_k im2col(dy)[m][k] * Wt[c][k]     the same kernel on dy with flipped, transposed
//                                                             filters (stride 1)
//   wgrad    dW[n][k] = sum_m dy[m][n] * im2col(x)[m][k]      both operands are contraction-major in memory;
//                                                             they are staged as they lie and read with the
//                                                             LDS transpose load (ds_read_b64_tr_b16)
// The im2col matrix is never materialised: a tile loader gathers 16-byte chunks straight from the NHWC
// tensor (zero outside the image).  Only stride-1 windows are handled here; a strided first layer is
// turned into a stride-1 layer by a space-to-depth re-layout of the input (see pack_input).
#include <algorithm>
#include <type_traits>
#include "dev_common.hpp"
#include "kernels.hpp"

namespace sasgd {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short shortx4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int BK = 32;           // contraction elements per step (4 chunks)

// ------------------------------------------------------------------ filter packing (once per weight version)
// Filters are stored in MFMA operand ("fragment") order so that a wavefront fetches the B operand of one
// 32x32x16 MFMA as one contiguous 1 KiB read, straight into registers:
//   frag[(nb * KB16 + kb) * 512 + lane * 8 + t] = B[row 32 nb + lane%32][k = 16 kb + 8 (lane/32) + t]
// fwd: B = Wp[n][tap][cp] (k = tap * C + cp, Kp = padded ks*ks*C);   rows beyond K and k beyond the filter are zero
// bwd: B = Wt[c][tap'][n] (k = tap' * K + n, tap' = flipped tap, Kpt = padded ks*ks*K), stride-1 layers only
// One thread produces one lane's 16-byte chunk (8 consecutive k of one row); index arithmetic is 32-bit.
__global__ __launch_bounds__(256) void pack_filters_kernel(PackVersions pv, PackTable t) {
  const bf16_t* __restrict__ flat = (const bf16_t*)pv.flat[blockIdx.y];      // blockIdx.y = weight version
  bf16_t* __restrict__ packed = (bf16_t*)pv.packed[blockIdx.y];
  const int64_t chunks = t.total >> 3;
  for (int64_t gc = (int64_t)blockIdx.x * 256 + threadIdx.x; gc < chunks; gc += (int64_t)gridDim.x * 256) {
    int li = 0;                                   // layer this chunk belongs to
    while (li + 1 < t.count && gc * 8 >= t.job[li + 1].start) li++;
    const PackJob& jb = t.job[li];
    const VConv& v = jb.v;
    const uint32_t i = (uint32_t)(gc * 8 - jb.start);
    const uint32_t nf = (uint32_t)((v.K + 31) & ~31) * (uint32_t)jb.Kp;
    const bool fwd = i < nf;
    const uint32_t e = fwd ? i : i - nf;
    const uint32_t KB16 = (uint32_t)(fwd ? jb.Kp : jb.Kpt) / 16u;
    const uint32_t lane = (e >> 3) & 63u, blk = e >> 9;
    const uint32_t rb = blk / KB16, kb = blk - rb * KB16;
    const int row = (int)(32u * rb + (lane & 31u));
    const uint32_t k0 = 16u * kb + 8u * (lane >> 5);
    const int taps = v.ks * v.ks;
    union { bf16_t h[8]; uint4 q; } out;
    out.q = make_uint4(0u, 0u, 0u, 0u);
    if (fwd) {
      // k = tap * C + cp; C is a multiple of 8, so the 8 elements share the tap
      const int tap = (int)(k0 / (uint32_t)v.C), cp0 = (int)(k0 - (uint32_t)tap * (uint32_t)v.C);
      if (row < v.K && tap < taps) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const int64_t src = filter_src(v, row, tap, cp0 + j);
          if (src >= 0) out.h[j] = flat[jb.w_off + src];
        }
      }
      *reinterpret_cast<uint4*>(packed + jb.fwd_off + e) = out.q;
    } else {
      // k = tap' * K + n; K is a multiple of 8
      const int tap = (int)(k0 / (uint32_t)v.K), n0 = (int)(k0 - (uint32_t)tap * (uint32_t)v.K);
      if (row < v.C && tap < taps) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const int64_t src = filter_src(v, n0 + j, taps - 1 - tap, row);   // flipped tap (ks-1-kh, ks-1-kw)
          if (src >= 0) out.h[j] = flat[jb.w_off + src];
        }
      }
      *reinterpret_cast<uint4*>(packed + jb.bwd_off + e) = out.q;
    }
  }
}

// Layers with a multiple of 32 input and 16 output channels and no re-layout of the first layer: the repack is a
// transposition ([n][c][tap] -> [n][tap][c] and [c][tap'][n]), done through LDS so that both the reads of the flat
// filter and the writes of the fragments are contiguous.
//   forward block  (32 output channels, 16 input channels): reads 32 runs of 16 T elements, writes T fragment blocks
//   backward block (32 input channels, 16 output channels): reads 16 runs of 32 T elements, writes T fragment blocks
// Fragment blocks of the zero padding (k beyond the filter) are never written: they keep the zeros the ring was
// created with.
struct PackFastJob {
  int64_t w_off, fwd_off, bwd_off;
  int C, K, T, KB16, KB16t;          // T = taps; fragment k-blocks per row of the two copies
  int first_block, fwd_blocks;       // workgroups [first_block, next job's first_block): forward ones first
};
struct PackFastTable {
  PackFastJob job[kMaxPackJobs];
  int count;
};
constexpr int kPackMaxTaps = 25;

__global__ __launch_bounds__(256) void pack_filters_lds_kernel(PackVersions pv, PackFastTable t) {
  const bf16_t* __restrict__ flat = (const bf16_t*)pv.flat[blockIdx.y];      // blockIdx.y = weight version
  bf16_t* __restrict__ packed = (bf16_t*)pv.packed[blockIdx.y];
  __shared__ __attribute__((aligned(16))) bf16_t tile[32 * 16 * kPackMaxTaps];
  int li = 0;
  while (li + 1 < t.count && (int)blockIdx.x >= t.job[li + 1].first_block) li++;
  const PackFastJob& jb = t.job[li];
  const int b = blockIdx.x - jb.first_block;
  const int T = jb.T, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = lane & 31, h = lane >> 5;
  const bf16_t* W = flat + jb.w_off;
  if (b < jb.fwd_blocks) {
    const int groups = jb.C / 16, rb = b / groups, cg = b - rb * groups;
    const int run = 16 * T;                                  // contiguous elements of one output channel
    for (int ch = tid; ch < 64 * T; ch += 256) {             // 16-byte pieces: 2 T per run
      const int r = ch / (2 * T), rem = (ch - r * 2 * T) * 8, n = 32 * rb + r;
      uint4 q = make_uint4(0u, 0u, 0u, 0u);
      if (n < jb.K) q = *reinterpret_cast<const uint4*>(W + ((int64_t)n * jb.C + 16 * cg) * T + rem);
      *reinterpret_cast<uint4*>(tile + r * run + rem) = q;
    }
    __syncthreads();
    for (int tap = wave; tap < T; tap += 4) {
      union { bf16_t e[8]; uint4 q; } o;
#pragma unroll
      for (int j = 0; j < 8; j++) o.e[j] = tile[row * run + (8 * h + j) * T + tap];
      const int kb = tap * groups + cg;
      *reinterpret_cast<uint4*>(packed + jb.fwd_off + ((int64_t)rb * jb.KB16 + kb) * 512 + lane * 8) = o.q;
    }
  } else {
    const int bb = b - jb.fwd_blocks;
    const int groups = jb.K / 16, cb = bb / groups, ng = bb - cb * groups;
    const int run = 32 * T;                                  // contiguous elements of 32 input channels of one filter
    for (int ch = tid; ch < 64 * T; ch += 256) {             // 16-byte pieces: 4 T per run (the 32 channels all exist)
      const int nn = ch / (4 * T), rem = (ch - nn * 4 * T) * 8;
      *reinterpret_cast<uint4*>(tile + nn * run + rem) =
          *reinterpret_cast<const uint4*>(W + ((int64_t)(16 * ng + nn) * jb.C + 32 * cb) * T + rem);
    }
    __syncthreads();
    for (int tap = wave; tap < T; tap += 4) {                // tap' of the flipped filter
      union { bf16_t e[8]; uint4 q; } o;
#pragma unroll
      for (int j = 0; j < 8; j++) o.e[j] = tile[(8 * h + j) * run + row * T + (T - 1 - tap)];
      const int kb = tap * groups + ng;
      *reinterpret_cast<uint4*>(packed + jb.bwd_off + ((int64_t)cb * jb.KB16t + kb) * 512 + lane * 8) = o.q;
    }
  }
}

hipError_t launch_pack_filters(const PackVersions& pv, int versions, const PackTable& t, hipStream_t s) {
  if (t.count == 0 || t.total == 0 || versions < 1) return hipSuccess;
  if (versions > kMaxPackVersions) return hipErrorInvalidValue;
  PackTable slow;
  PackFastTable fast;
  slow.count = 0; slow.total = 0;
  fast.count = 0;
  int blocks_fast = 0;
  for (int k = 0; k < t.count; k++) {
    const PackJob& jb = t.job[k];
    const VConv& v = jb.v;
    const int T = v.ks * v.ks;
    if (v.s2d == 1 && v.C == v.Creal && v.ks == v.ksr && v.C % 32 == 0 && v.K % 16 == 0 && T <= kPackMaxTaps && jb.Kpt > 0 && jb.w_off % 8 == 0) {
      PackFastJob& f = fast.job[fast.count++];
      f.w_off = jb.w_off; f.fwd_off = jb.fwd_off; f.bwd_off = jb.bwd_off;
      f.C = v.C; f.K = v.K; f.T = T; f.KB16 = jb.Kp / 16; f.KB16t = jb.Kpt / 16;
      f.first_block = blocks_fast;
      f.fwd_blocks = ((v.K + 31) / 32) * (v.C / 16);
      blocks_fast += f.fwd_blocks + ((v.C + 31) / 32) * (v.K / 16);
    } else {
      PackJob& o = slow.job[slow.count++];
      o = jb;
      o.start = slow.total;
      slow.total += (int64_t)((v.K + 31) & ~31) * jb.Kp + (jb.Kpt > 0 ? (int64_t)((v.C + 31) & ~31) * jb.Kpt : 0);
    }
  }
  if (slow.count > 0) {
    const int64_t chunks = slow.total / 8;
    int blocks = (int)((chunks + 255) / 256 < 8192 ? (chunks + 255) / 256 : 8192);
    hipLaunchKernelGGL(pack_filters_kernel, dim3(blocks, (unsigned)versions), dim3(256), 0, s, pv, slow);
  }
  if (fast.count > 0)
    hipLaunchKernelGGL(pack_filters_lds_kernel, dim3((unsigned)blocks_fast, (unsigned)versions), dim3(256), 0, s, pv, fast);
  return hipGetLastError();
}

// ------------------------------------------------------------------ im2col rows
__device__ __forceinline__ uint32_t fastdiv(uint32_t n, int d, uint32_t magic) { return d == 1 ? n : __umulhi(n, magic); }

struct RowPos {
  const bf16_t* base;   // &t[n][oh - pad][ow - pad][0]  (may point outside; only dereferenced when in range)
  int oh, ow;           // already offset by -pad
  bool valid;
};

__device__ __forceinline__ RowPos row_pos(const bf16_t* t, const IGemm& g, int m) {
  RowPos r;
  r.valid = m < g.M;
  const uint32_t mm = r.valid ? (uint32_t)m : 0u;
  const uint32_t rest = fastdiv(mm, g.OW, g.mg_ow);
  const int ow = (int)(mm - rest * (uint32_t)g.OW);
  const uint32_t n = fastdiv(rest, g.OH, g.mg_oh);
  const int oh = (int)(rest - n * (uint32_t)g.OH);
  r.oh = oh - g.pad;
  r.ow = ow - g.pad;
  r.base = t + (((int64_t)n * g.H + r.oh) * g.W + r.ow) * g.C;
  return r;
}

typedef int v2i_t __attribute__((ext_vector_type(2)));
typedef int v4i_t __attribute__((ext_vector_type(4)));
// Bias, ReLU, ReLU mask of the input gradient, conversion and store of one wavefront's WM x WN accumulator tile whose
// origin is (mw, nw).  `lds` is the workgroup's tile memory, free once every wavefront has passed the barrier inside.
template <int WM, int WN>
__device__ __forceinline__ void frag_epilogue(floatx16 (&acc)[WM / 32][WN / 32], bf16_t* lds, void* ws_base, const void* wt_base,
                                              const IGemm& g, const Epilogue& ep, int mw, int nw, int lane, int wave) {
  constexpr int TM = WM / 32, TN = WN / 32;
  bf16_t* out = (bf16_t*)ws_base + ep.out_off;
  const bf16_t* mask = (const bf16_t*)ws_base + ep.mask_off;
  const bf16_t* bias = (const bf16_t*)wt_base + ep.bias_off;
  if (!ep.out_f32) {
    // bf16 output: a lane holds single elements of 16 different rows, which written straight out are 2-byte stores.
    // Each wavefront turns its 32-row blocks around in its own piece of LDS (the tiles there are no longer needed) and
    // writes 16 bytes per lane, 8 lanes per row; the ReLU mask of the input gradient is read the same way.
    constexpr int LDE = WN + 8;                          // row stride of the staging piece (elements)
    __syncthreads();                                     // every wavefront has finished reading the last tile
    bf16_t* stage = lds + wave * (32 * LDE);
    constexpr int CPRW = WN / 8;                         // 16-byte chunks per row of the wavefront's tile
    static_assert(32 * CPRW % 64 == 0, "a block leaves in whole passes of 64 chunks");
#pragma unroll
    for (int i = 0; i < TM; i++) {
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const int n = nw + 32 * j + (lane & 31);
        const float bv = (ep.has_bias && n < g.Ncols) ? bf2f(bias[n]) : 0.f;
#pragma unroll
        for (int r = 0; r < 16; r++) {
          float v = acc[i][j][r] + bv;
          if (ep.relu) v = fmaxf(v, 0.f);
          stage[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * LDE + 32 * j + (lane & 31)] = f2bf(v);
        }
      }
      // LDS operations of one wavefront complete in order, so its reads below see its writes above; the compiler is
      // told not to move LDS accesses across the two phases
      __builtin_amdgcn_wave_barrier();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int it = 0; it < 32 * CPRW / 64; it++) {
        const int row = (lane + 64 * it) / CPRW, rchunk = (lane + 64 * it) % CPRW;
        const int m = mw + 32 * i + row, n = nw + rchunk * 8;
        uint4 q = *reinterpret_cast<const uint4*>(stage + row * LDE + rchunk * 8);
        if (m < g.M && n < g.Ncols) {
          const int64_t o = (int64_t)m * g.Ncols + n;
          if (ep.use_mask) {
            const uint4 mk = *reinterpret_cast<const uint4*>(mask + o);
            const uint32_t mw[4] = {mk.x, mk.y, mk.z, mk.w};
            uint32_t qw[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int w = 0; w < 4; w++) {                // keep a 16-bit half where the forward value is positive
              const uint32_t lo = mw[w] & 0xffffu, hi = mw[w] >> 16;
              const uint32_t keep = (((lo & 0x8000u) == 0 && (lo & 0x7fffu) != 0) ? 0x0000ffffu : 0u) |
                                    (((hi & 0x8000u) == 0 && (hi & 0x7fffu) != 0) ? 0xffff0000u : 0u);
              qw[w] &= keep;
            }
            q = make_uint4(qw[0], qw[1], qw[2], qw[3]);
          }
          *reinterpret_cast<uint4*>(out + o) = q;
        }
      }
      __builtin_amdgcn_wave_barrier();
      asm volatile("" ::: "memory");
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const int n = nw + 32 * j + (lane & 31);
    if (n >= g.Ncols) continue;
    const float bv = ep.has_bias ? bf2f(bias[n]) : 0.f;
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int m = mw + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (m >= g.M) continue;
        float v = acc[i][j][r] + bv;
        if (ep.relu) v = fmaxf(v, 0.f);
        const int64_t o = (int64_t)m * g.Ncols + n;
        if (ep.use_mask && !(bf2f(mask[o]) > 0.f)) v = 0.f;
        reinterpret_cast<float*>(out)[o] = v;
      }
  }
}

// ------------------------------------------------------------------ convolution forward / dgrad, B from fragments
// Only the gathered im2col tile goes through LDS; the filter operand comes from the fragment-packed copy, one coalesced 1 KiB read
// per MFMA operand, prefetched one step ahead.  This halves the LDS traffic per MFMA, which bounds a kernel with both operands there.
constexpr uint32_t kOutOfRange = 0x80000000u;   // buffer offset beyond any tensor: the load returns zeros

// NT = threads per workgroup = 64 x number of wave tiles.
// UNI: every contraction step stays inside one filter tap (channels per tap are a multiple of the step) and the
// window has at most 32 taps.  Then the tap is wavefront-uniform and advances in scalar registers, the per-row
// bounds test is one bit of a mask computed once, and a step costs a handful of vector instructions besides the
// loads and MFMAs.  Otherwise (first layer, large windows) the tap is decoded per lane and step.
template <int BM, int BN, int WM, int WN, int BKT, int NT, bool UNI>
__global__ __launch_bounds__(NT, (WM * WN > 64 * 64 ? 2 : 1)) void igemm_frag_kernel(PtrTab ws, CPtrTab wts, IGemm g, Epilogue ep) {
  constexpr int WAVES_N = BN / WN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int LDF = BKT + 8;                 // 80 or 144 byte rows: conflict-free 16-byte reads
  constexpr int CPS = BKT / 8;                 // chunks per contraction step
  constexpr int KK = BKT / 16;                 // MFMA k-blocks per step
  constexpr int A_ELEMS = BM * LDF;
  __shared__ __attribute__((aligned(16))) bf16_t lds[2 * A_ELEMS];

  const int z = blockIdx.z / g.splits, sp = blockIdx.z % g.splits;
  const bf16_t* act = (const bf16_t*)ws.p[z] + g.a_off;
  const bf16_t* Bf = (const bf16_t*)wts.p[z] + g.b_off;
  // Buffer resources: an offset at or beyond the size reads as zero in hardware, so padding taps, ragged rows
  // and ragged columns need no branch, no select on the data and no 64-bit address arithmetic.
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void*)act, 0, (int)g.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc((void*)Bf, 0, (int)g.b_bytes, 0x00020000);
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  const int KB16 = g.ldb / 16;
  const int NB = (g.Ncols + 31) / 32;

  constexpr int A_LOADS = (BM * CPS + NT - 1) / NT;
  constexpr int RPP = NT / CPS;                // tile rows covered per loader pass
  constexpr bool FULL = (BM % RPP) == 0;       // every loader pass lies inside the tile
  const int cc = tid % CPS, lrow = tid / CPS;
  // per tile row handled by this thread: byte offset of its window origin (plus this thread's chunk in UNI mode),
  // and either the origin's coordinates or (UNI) a mask with one bit per tap that falls outside the tensor
  int row_off[A_LOADS], row_oh[A_LOADS], row_ow[A_LOADS];
  uint32_t row_bad[A_LOADS];
#pragma unroll
  for (int i = 0; i < A_LOADS; i++) {
    const RowPos r = row_pos(act, g, m0 + lrow + RPP * i);
    row_off[i] = (int)((r.base - act) * 2) + (UNI ? cc * 16 : 0);
    row_oh[i] = r.valid ? r.oh : -0x40000000;  // an invalid row fails every bounds test below
    row_ow[i] = r.ow;
    if (UNI) {
      uint32_t good = 0;
      if (r.valid) {
        const int kw_lo = max(0, -r.ow), kw_hi = min(g.ks, g.W - r.ow);              // valid kw: [kw_lo, kw_hi)
        const uint32_t kwmask = kw_hi > kw_lo ? (((1u << kw_hi) - 1u) & ~((1u << kw_lo) - 1u)) : 0u;
        for (int kh = 0; kh < g.ks; kh++)
          if ((unsigned)(r.oh + kh) < (unsigned)g.H) good |= kwmask << (kh * g.ks);
      }
      row_bad[i] = ~good;
    }
  }

  const int all_steps = (g.Kchunks + CPS - 1) / CPS;
  const int per = (all_steps + g.splits - 1) / g.splits;
  const int ks_begin = __builtin_amdgcn_readfirstlane(sp * per);
  const int ksteps = __builtin_amdgcn_readfirstlane(min(all_steps, ks_begin + per));

  // UNI: tap state of the step that load_a fetches next, kept in scalar registers
  int u_tap = 0, u_c8 = 0, u_kw = 0, u_koff = 0;
  if (UNI) {
    const uint32_t q0 = (uint32_t)(ks_begin * CPS);
    u_tap = (int)fastdiv(q0, g.CPT, g.mg_cpt);
    u_c8 = (int)q0 - u_tap * g.CPT;
    const int kh = (int)fastdiv((uint32_t)u_tap, g.ks, g.mg_ks);
    u_kw = u_tap - kh * g.ks;
    u_koff = ((kh * g.W + u_kw) * g.C + u_c8 * 8) * 2;
    u_tap = __builtin_amdgcn_readfirstlane(u_tap);
    u_c8 = __builtin_amdgcn_readfirstlane(u_c8);
    u_kw = __builtin_amdgcn_readfirstlane(u_kw);
    u_koff = __builtin_amdgcn_readfirstlane(u_koff);
  }
  const int u_row_step = __builtin_amdgcn_readfirstlane((g.W - g.ks) * g.C * 2);   // extra bytes when kw wraps to the next kh

  v4i_t ra[A_LOADS];
  auto load_a = [&](int ks) {
    if (UNI) {
#pragma unroll
      for (int i = 0; i < A_LOADS; i++) {
        const int bad = __builtin_amdgcn_sbfe((int)row_bad[i], u_tap, 1);            // 0 or -1
        const int off = (row_off[i] + u_koff) | (bad & (int)kOutOfRange);
        ra[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, off, 0, 0);
      }
      // advance to the next step: CPS more chunks of the same tap, or the first chunks of the next tap
      u_c8 += CPS;
      u_koff += CPS * 16;
      const bool next_tap = u_c8 >= g.CPT;
      u_c8 = next_tap ? 0 : u_c8;
      u_tap += next_tap ? 1 : 0;
      u_kw += next_tap ? 1 : 0;
      const bool next_row = u_kw == g.ks;
      u_kw = next_row ? 0 : u_kw;
      u_koff += next_row ? u_row_step : 0;
    } else {
      const int q = ks * CPS + cc;
      const uint32_t tap = fastdiv((uint32_t)q, g.CPT, g.mg_cpt);
      const int c8 = q - (int)tap * g.CPT;
      const int kh = (int)fastdiv(tap, g.ks, g.mg_ks), kw = (int)tap - kh * g.ks;
      const int koff = ((kh * g.W + kw) * g.C + c8 * 8) * 2;
      const bool qok = q < g.Kchunks;
#pragma unroll
      for (int i = 0; i < A_LOADS; i++) {
        const bool ok = qok && (unsigned)(row_oh[i] + kh) < (unsigned)g.H && (unsigned)(row_ow[i] + kw) < (unsigned)g.W;
        ra[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, ok ? (row_off[i] + koff) : (int)kOutOfRange, 0, 0);
      }
    }
  };
  auto store_a = [&](int buf) {
    bf16_t* A = lds + buf * A_ELEMS;
#pragma unroll
    for (int i = 0; i < A_LOADS; i++)
      if (FULL || lrow + RPP * i < BM) *reinterpret_cast<v4i_t*>(A + (lrow + RPP * i) * LDF + cc * 8) = ra[i];
  };
  // B fragments: one fixed byte offset per column block of this wavefront; the step advances a scalar offset
  uint32_t boff[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const int nb = (n0 + wn0) / 32 + j;
    boff[j] = nb < NB ? (uint32_t)(((int64_t)nb * KB16 * 512 + lane * 8) * 2) : kOutOfRange;
  }
  int b_step = ks_begin * KK * 1024;           // scalar byte offset of the step that load_b fetches next
  auto load_b = [&](bf16x8 (&bt)[KK][TN]) {
#pragma unroll
    for (int kk = 0; kk < KK; kk++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        union { v4i_t u; bf16x8 v; } f;
        f.u = __builtin_amdgcn_raw_buffer_load_b128(rsrc_b, (int)(boff[j] + kk * 1024), b_step, 0);
        bt[kk][j] = f.v;
      }
    b_step += KK * 1024;
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  // One contraction step ks on LDS buffer `buf`.  At entry the A fragments of its first k-block (`a0`) are already in
  // registers.  The im2col chunks of step ks+1 (fetched during step ks-1, now in staging registers) go to the other
  // LDS buffer, the chunks of step ks+2 and the filter fragments of step ks+1 (into `bnext`) are requested, the A
  // fragments of the second k-block are read, and the first k-block's MFMAs run.  The single barrier of the step
  // sits in the middle: after it every wavefront has finished reading `buf` and writing the other buffer, so the
  // first A fragments of step ks+1 (`a0n`) are read while the second k-block's MFMAs run, and nothing waits on LDS
  // right after a barrier.  Fragment sets swap roles from step to step: two steps per loop iteration, no copies.
  auto lds_frag = [&](int buf, int i, int kk) {
    return *reinterpret_cast<const bf16x8*>(lds + buf * A_ELEMS + (wm0 + 32 * i + (lane & 31)) * LDF + 16 * kk + 8 * (lane >> 5));
  };
  auto step = [&](bf16x8 (&bcur)[KK][TN], bf16x8 (&bnext)[KK][TN], bf16x8 (&a0)[TM], bf16x8 (&a0n)[TM], int ks, int buf, bool has1,
                  bool has2) {
    static_assert(KK == 2, "two k-blocks per step");
    if (has1) store_a(buf ^ 1);
    if (has2) load_a(ks + 2);
    if (has1) load_b(bnext);
    bf16x8 a1[TM];
#pragma unroll
    for (int i = 0; i < TM; i++) a1[i] = lds_frag(buf, i, 1);
    __builtin_amdgcn_sched_barrier(0);         // requests and LDS traffic first: they need the step to complete
    __builtin_amdgcn_s_setprio(1);             // a wavefront in its MFMA phase keeps the matrix pipe; others issue memory work
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[i], bcur[0][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    if (has1) {
#pragma unroll
      for (int i = 0; i < TM; i++) a0n[i] = lds_frag(buf ^ 1, i, 0);
    }
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[i], bcur[1][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };

  bf16x8 b0[KK][TN], b1[KK][TN], fa[TM], fb[TM];
  int ks = ks_begin;
  if (ks < ksteps) {
    load_a(ks);
    load_b(b0);
    store_a(0);
    if (ks + 1 < ksteps) load_a(ks + 1);
  }
  __syncthreads();
  if (ks < ksteps) {
#pragma unroll
    for (int i = 0; i < TM; i++) fa[i] = lds_frag(0, i, 0);
  }
  // Inside the loop both steps prefetch unconditionally: a branch around the loads would make the compiler wait
  // for the most pessimistic count of outstanding loads where the paths join.
  for (; ks + 3 < ksteps; ks += 2) {
    step(b0, b1, fa, fb, ks, 0, true, true);
    step(b1, b0, fb, fa, ks + 1, 1, true, true);
  }
  for (; ks + 1 < ksteps; ks += 2) {          // at most once: two or three steps remain
    step(b0, b1, fa, fb, ks, 0, true, ks + 2 < ksteps);
    step(b1, b0, fb, fa, ks + 1, 1, ks + 2 < ksteps, false);
  }
  if (ks < ksteps) step(b0, b1, fa, fb, ks, 0, false, false);

  if (g.splits > 1) {
    float* part = reinterpret_cast<float*>((char*)ws.p[z] + g.scratch_off) + (int64_t)sp * g.M * g.Ncols;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int n = n0 + wn0 + 32 * j + (lane & 31);
      if (n >= g.Ncols) continue;
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int m = m0 + wm0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (m < g.M) part[(int64_t)m * g.Ncols + n] = acc[i][j][r];
        }
    }
    return;
  }
  static_assert(4 * 32 * (WN + 8) <= 2 * A_ELEMS || NT != 256, "the epilogue's staging piece fits the tile buffers");
  frag_epilogue<WM, WN>(acc, lds, ws.p[z], wts.p[z], g, ep, m0 + wm0, n0 + wn0, lane, wave);
}

// ------------------------------------------------------------------ convolution forward / dgrad, input patch in LDS
// For windows larger than 1 x 1 the im2col tile of one tap is the tile of the neighbouring tap shifted by one
// pixel, so gathering it tap by tap moves every input pixel ks*ks times from the L1 into LDS.  This kernel puts
// the input patch under a tile of BM output positions into LDS once per 32 input channels (zero padding and the
// halo rows included, 80 bytes per pixel) and reads the MFMA A operand of tap (kh, kw) from it at the address of the
// output position's window origin plus a wavefront-uniform offset.  The ks*ks contraction steps of one channel
// chunk run without a barrier; the filter operand comes from the fragment-packed copy as in igemm_frag_kernel
// (k = tap * C + c, so the 32 channels of a chunk are two 16-k blocks at tap * C/16 + 2 * chunk).
//   patch rows: the output rows gr = m / OW of the tile, gr_lo .. gr_hi, may belong to several images; image n owns
//   a band of (its output rows in the tile) + ks - 1 input rows, so the row of (gr, kh) is
//   (gr - gr_lo) + kh + (ks - 1)(n - n_lo);  patch columns: OW + ks - 1 = W + 2 pad.
// The contraction may be split over channel chunks (g.splits <= C / 32).
// Workgroups are handed to the eight XCDs round-robin in launch order, and each XCD has its own L2.  This turns the
// launch-order index around so that every XCD works through one contiguous eighth of the (x, y, z) tile space: tiles
// that share filter fragments and halo rows then share an L2 instead of being spread over all eight.
struct TileIdx { int x, y, z; };
__device__ __forceinline__ TileIdx xcd_tile(int on) {
  uint32_t lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  const uint32_t per = (gridDim.x * gridDim.y * gridDim.z) >> 3;
  if (on && lin < per * 8u) lin = (lin & 7u) * per + (lin >> 3);   // the last (count mod 8) workgroups keep their place
  TileIdx t;
  const uint32_t q = lin / gridDim.x;
  t.x = (int)(lin - q * gridDim.x);
  t.z = (int)(q / gridDim.y);
  t.y = (int)(q - (uint32_t)t.z * gridDim.y);
  return t;
}

struct HaloArgs {
  int PW;              // patch width in pixels
  uint32_t mg_pw;      // multiplier for division by PW
  int n_px_max;        // pixels the LDS patch has room for
  int xcd;             // 1: XCD-contiguous tile order (see xcd_tile)
  int tab_off;         // bytes from the start of LDS to the pixel table (behind the patch, rounded up to whole refill rounds)
};

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN), (WM * WN > 64 * 64 ? 2 : 3)) void conv_halo_kernel(PtrTab ws, CPtrTab wts, IGemm g, Epilogue ep, HaloArgs h) {
  constexpr int NT = 64 * (BM / WM) * (BN / WN);
  constexpr int WAVES_N = BN / WN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int PST = 40;                      // elements per patch pixel: 32 channels + 8 of padding (conflict-free 16-byte reads)
  extern __shared__ __attribute__((aligned(16))) bf16_t halo_lds[];
  bf16_t* lds = halo_lds;
  int* tab = reinterpret_cast<int*>(reinterpret_cast<char*>(lds) + h.tab_off);   // byte offset of every patch pixel in the tensor

  const TileIdx tile = xcd_tile(h.xcd);
  const int z = tile.z / g.splits, sp = tile.z % g.splits;
  const bf16_t* act = (const bf16_t*)ws.p[z] + g.a_off;
  const bf16_t* Bf = (const bf16_t*)wts.p[z] + g.b_off;
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void*)act, 0, (int)g.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc((void*)Bf, 0, (int)g.b_bytes, 0x00020000);
  const int m0 = tile.x * BM, n0 = tile.y * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  const int KB16 = g.ldb / 16;
  const int NB = (g.Ncols + 31) / 32;

  const int ks = g.ks, PW = h.PW;
  const int m_last = min(m0 + BM, g.M) - 1;
  const int gr_lo = (int)fastdiv((uint32_t)m0, g.OW, g.mg_ow), gr_hi = (int)fastdiv((uint32_t)m_last, g.OW, g.mg_ow);
  const int n_lo = (int)fastdiv((uint32_t)gr_lo, g.OH, g.mg_oh), n_hi = (int)fastdiv((uint32_t)gr_hi, g.OH, g.mg_oh);
  const int oh_lo = gr_lo - n_lo * g.OH;
  const int NR = gr_hi - gr_lo + 1;
  const int n_px = (NR + (ks - 1) * (n_hi - n_lo + 1)) * PW;   // <= h.n_px_max (checked by the launcher's bound)

  for (int p = tid; p < n_px; p += NT) {
    const int pr = (int)fastdiv((uint32_t)p, PW, h.mg_pw), pc = p - pr * PW;
    int start = 0, rem = NR, n = n_lo, first = oh_lo, ih = -1, nn = -1;
    while (rem > 0) {
      const int rows = min(g.OH - first, rem), len = rows + ks - 1;
      if (pr < start + len) { nn = n; ih = first - g.pad + (pr - start); break; }
      start += len; rem -= rows; n++; first = 0;
    }
    const int iw = pc - g.pad;
    const bool ok = nn >= 0 && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
    tab[p] = ok ? ((nn * g.H + ih) * g.W + iw) * g.C * 2 : (int)kOutOfRange;
  }

  // window origin of this lane's rows in the patch (bytes); rows beyond M repeat the last one and are never stored
  int abase[TM];
#pragma unroll
  for (int i = 0; i < TM; i++) {
    const uint32_t m = (uint32_t)min(m0 + wm0 + 32 * i + (lane & 31), g.M - 1);
    const uint32_t gr = fastdiv(m, g.OW, g.mg_ow), ow = m - gr * (uint32_t)g.OW;
    const uint32_t n = fastdiv(gr, g.OH, g.mg_oh);
    const int pr0 = ((int)gr - gr_lo) + (ks - 1) * ((int)n - n_lo);
    abase[i] = ((pr0 * PW + (int)ow) * PST + 8 * (lane >> 5)) * 2;
  }
  __syncthreads();

  // Patch refill: LDS-direct loads, 64 consecutive 16-byte slots per wavefront and instruction.  Slot s holds piece
  // s % 5 of pixel s / 5; the fifth piece of a pixel is its padding and, like the slots beyond the patch, is
  // requested out of range (the hardware writes zeros).
  const int n_slots = n_px * 5;
  const int dma_rounds = (n_slots + NT - 1) / NT;
  const int wave_slot = __builtin_amdgcn_readfirstlane(wave * 64);
  auto refill = [&](int cc) {
#pragma unroll 1
    for (int r = 0; r < dma_rounds; r++) {
      const int sl = r * NT + tid;
      const int px = (int)(__umulhi((uint32_t)sl, 0xCCCCCCCDu) >> 2);   // sl / 5
      const int sub = sl - 5 * px;
      const int voff = (sub < 4 && sl < n_slots) ? tab[min(px, n_px - 1)] + sub * 16 : (int)kOutOfRange;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (__attribute__((address_space(3))) void*)(reinterpret_cast<char*>(lds) + (r * NT + wave_slot) * 16),
                                               16, voff, cc * 64, 0, 0);
    }
  };

  uint32_t boff[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const int nb = (n0 + wn0) / 32 + j;
    boff[j] = nb < NB ? (uint32_t)(((int64_t)nb * KB16 * 512 + lane * 8) * 2) : kOutOfRange;
  }
  const int b_tap = __builtin_amdgcn_readfirstlane((g.C / 16) * 1024);   // bytes from one tap's k-blocks to the next tap's
  auto load_b = [&](bf16x8 (&bt)[2][TN], int s_off) {
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        union { v4i_t u; bf16x8 v; } f;
        f.u = __builtin_amdgcn_raw_buffer_load_b128(rsrc_b, (int)(boff[j] + kk * 1024), s_off, 0);
        bt[kk][j] = f.v;
      }
  };
  auto lds_a = [&](int i, int toff, int kk) {
    return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(lds) + abase[i] + toff + kk * 32);
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  const int chunks = g.C >> 5;
  const int per = (chunks + g.splits - 1) / g.splits;
  const int cc_begin = __builtin_amdgcn_readfirstlane(sp * per);
  const int cc_end = __builtin_amdgcn_readfirstlane(min(chunks, cc_begin + per));
  const int T = ks * ks;
  const int a_wrap = (PW - ks) * PST * 2;

  // patch byte offset of the running tap (c_aoff); patch offset, kw and filter byte offset of the tap after it (n_*)
  int c_aoff = 0, n_aoff = 0, n_kw = 0, n_boff = 0;
  auto advance = [&]() {
    c_aoff = n_aoff;
    n_kw++; n_aoff += PST * 2; n_boff += b_tap;
    const bool wrap = n_kw == ks;
    n_kw = wrap ? 0 : n_kw;
    n_aoff += wrap ? a_wrap : 0;
  };
  // One tap.  The filter fragments travel two taps ahead through a ring of three register sets (the L2 round trip is
  // longer than one tap's MFMAs): `bld` receives tap t + 2 while `bcur` (tap t) is consumed.  The second k-block's A
  // fragments are read, the first k-block's MFMAs run, the next tap's first A fragments are read, the second
  // k-block's MFMAs run.
  bf16x8 a0[TM];
  auto step = [&](bf16x8 (&bcur)[2][TN], bf16x8 (&bld)[2][TN], bool ld, bool has_next) {
    if (ld) load_b(bld, n_boff + b_tap);
    bf16x8 a1[TM];
#pragma unroll
    for (int i = 0; i < TM; i++) a1[i] = lds_a(i, c_aoff, 1);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[i], bcur[0][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if (has_next) {                              // straight into a0: its last readers have been issued
#pragma unroll
      for (int i = 0; i < TM; i++) a0[i] = lds_a(i, n_aoff, 0);
    }
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[i], bcur[1][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    advance();
  };

  bf16x8 bq0[2][TN], bq1[2][TN], bq2[2][TN];
  if (cc_begin < cc_end) {
    refill(cc_begin);
    load_b(bq0, cc_begin * 2048);
    load_b(bq1, cc_begin * 2048 + b_tap);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // ks * ks leaves the remainder 0 or 1 when divided by three, so after the full groups of three taps either three
  // or four taps remain.  They are written out straight-line in two copies of the chunk loop: with a joined tail the
  // compiler kept a second set of accumulators.
  auto run = [&](auto four) {
    const int groups = (T - 2) / 3;
#pragma unroll 1
    for (int cc = cc_begin; cc < cc_end; cc++) {
      n_aoff = 0; n_kw = 0; n_boff = cc * 2048;
      advance();                                 // c_aoff = tap 0, n_* = tap 1
#pragma unroll
      for (int i = 0; i < TM; i++) a0[i] = lds_a(i, 0, 0);
#pragma unroll 1
      for (int t = 0; t < groups; t++) {
        step(bq0, bq2, true, true);
        step(bq1, bq0, true, true);
        step(bq2, bq1, true, true);
      }
      if constexpr (decltype(four)::value) {
        step(bq0, bq2, true, true);
        step(bq1, bq0, true, true);
        step(bq2, bq1, false, true);
        step(bq0, bq2, false, false);
      } else {
        step(bq0, bq2, true, true);
        step(bq1, bq0, false, true);
        step(bq2, bq1, false, false);
      }
      const bool more = cc + 1 < cc_end;
      if (more) {
        load_b(bq0, (cc + 1) * 2048);
        load_b(bq1, (cc + 1) * 2048 + b_tap);
      }
      __syncthreads();                           // every wavefront has finished reading the patch
      if (more) refill(cc + 1);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
    }
  };
  if (T % 3 == 1) run(std::true_type{});
  else run(std::false_type{});

  if (g.splits > 1) {
    float* part = reinterpret_cast<float*>((char*)ws.p[z] + g.scratch_off) + (int64_t)sp * g.M * g.Ncols;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int n = n0 + wn0 + 32 * j + (lane & 31);
      if (n >= g.Ncols) continue;
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int m = m0 + wm0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (m < g.M) part[(int64_t)m * g.Ncols + n] = acc[i][j][r];
        }
    }
    return;
  }
  frag_epilogue<WM, WN>(acc, lds, ws.p[z], wts.p[z], g, ep, m0 + wm0, n0 + wn0, lane, wave);
}

// ------------------------------------------------------------------ patch-in-LDS convolution for few input channels
// First layers: 8 channels (3 padded) or a multiple of 16 that is not one of 32 (48 after the space-to-depth
// re-layout).  The whole pixel goes into the patch, loaded once per tile, and the contraction walks the 16-k blocks
// of the packed filters in their own order, k = tap * C + c:
//   C % 16 == 0: block b is channels 16 (b % (C/16)) ... + 15 of tap b / (C/16); the lane halves take its two 8-channel
//                halves, as in conv_halo_kernel, but each of a step's two blocks has a patch offset of its own;
//   C == 8:      block b is taps 2 b (lane half 0) and 2 b + 1 (lane half 1), all 8 channels each.
// Pixels are C * 2 bytes plus 16 bytes of padding (none for C == 8, where consecutive pixels are consecutive
// 16-byte reads).  Blocks behind the last tap exist only as zero padding of the filters; they read the last tap.
// The contraction may be split over steps (two blocks each).
struct HaloSeqArgs {
  int PW;              // patch width in pixels
  uint32_t mg_pw;      // multiplier for division by PW
  int n_px_max;        // pixels the LDS patch has room for
  int tab_off;         // bytes from the start of LDS to the pixel table
  int spp;             // 16-byte slots per pixel in LDS (data + padding)
  uint32_t mg_spp;     // multiplier for division by spp
  int pixb;            // bytes per pixel in LDS = 16 spp
  int C16;             // 16-channel blocks per tap (C % 16 == 0)
  uint32_t mg_c16;     // multiplier for division by C16
};

template <int BM, int BN, int WM, int WN, bool C8>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN), (WM * WN > 64 * 64 ? 2 : 3)) void conv_halo_seq_kernel(PtrTab ws, CPtrTab wts, IGemm g, Epilogue ep, HaloSeqArgs h) {
  constexpr int NT = 64 * (BM / WM) * (BN / WN);
  constexpr int WAVES_N = BN / WN;
  constexpr int TM = WM / 32, TN = WN / 32;
  extern __shared__ __attribute__((aligned(16))) bf16_t halo_seq_lds[];
  bf16_t* lds = halo_seq_lds;
  int* tab = reinterpret_cast<int*>(reinterpret_cast<char*>(lds) + h.tab_off);

  const int z = blockIdx.z / g.splits, sp = blockIdx.z % g.splits;
  const bf16_t* act = (const bf16_t*)ws.p[z] + g.a_off;
  const bf16_t* Bf = (const bf16_t*)wts.p[z] + g.b_off;
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void*)act, 0, (int)g.a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc((void*)Bf, 0, (int)g.b_bytes, 0x00020000);
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WAVES_N) * WM, wn0 = (wave % WAVES_N) * WN;
  const int KB16 = g.ldb / 16;
  const int NB = (g.Ncols + 31) / 32;

  // patch geometry and pixel table: as in conv_halo_kernel
  const int ks = g.ks, PW = h.PW, pixb = h.pixb;
  const int m_last = min(m0 + BM, g.M) - 1;
  const int gr_lo = (int)fastdiv((uint32_t)m0, g.OW, g.mg_ow), gr_hi = (int)fastdiv((uint32_t)m_last, g.OW, g.mg_ow);
  const int n_lo = (int)fastdiv((uint32_t)gr_lo, g.OH, g.mg_oh), n_hi = (int)fastdiv((uint32_t)gr_hi, g.OH, g.mg_oh);
  const int oh_lo = gr_lo - n_lo * g.OH;
  const int NR = gr_hi - gr_lo + 1;
  const int n_px = (NR + (ks - 1) * (n_hi - n_lo + 1)) * PW;
  for (int p = tid; p < n_px; p += NT) {
    const int pr = (int)fastdiv((uint32_t)p, PW, h.mg_pw), pc = p - pr * PW;
    int start = 0, rem = NR, n = n_lo, first = oh_lo, ih = -1, nn = -1;
    while (rem > 0) {
      const int rows = min(g.OH - first, rem), len = rows + ks - 1;
      if (pr < start + len) { nn = n; ih = first - g.pad + (pr - start); break; }
      start += len; rem -= rows; n++; first = 0;
    }
    const int iw = pc - g.pad;
    const bool ok = nn >= 0 && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
    tab[p] = ok ? ((nn * g.H + ih) * g.W + iw) * g.C * 2 : (int)kOutOfRange;
  }
  int abase[TM];
#pragma unroll
  for (int i = 0; i < TM; i++) {
    const uint32_t m = (uint32_t)min(m0 + wm0 + 32 * i + (lane & 31), g.M - 1);
    const uint32_t gr = fastdiv(m, g.OW, g.mg_ow), ow = m - gr * (uint32_t)g.OW;
    const uint32_t n = fastdiv(gr, g.OH, g.mg_oh);
    const int pr0 = ((int)gr - gr_lo) + (ks - 1) * ((int)n - n_lo);
    abase[i] = (pr0 * PW + (int)ow) * pixb + (C8 ? 0 : 16 * (lane >> 5));
  }
  __syncthreads();
  {
    const int dpp = g.C / 8;                               // data slots per pixel
    const int n_slots = n_px * h.spp;
    const int dma_rounds = (n_slots + NT - 1) / NT;
    const int wave_slot = __builtin_amdgcn_readfirstlane(wave * 64);
#pragma unroll 1
    for (int r = 0; r < dma_rounds; r++) {
      const int sl = r * NT + tid;
      const int px = (int)fastdiv((uint32_t)sl, h.spp, h.mg_spp), sub = sl - px * h.spp;
      const int voff = (sub < dpp && sl < n_slots) ? tab[min(px, n_px - 1)] + sub * 16 : (int)kOutOfRange;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, (__attribute__((address_space(3))) void*)(reinterpret_cast<char*>(lds) + (r * NT + wave_slot) * 16),
                                               16, voff, 0, 0, 0);
    }
  }

  uint32_t boff[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const int nb = (n0 + wn0) / 32 + j;
    boff[j] = nb < NB ? (uint32_t)(((int64_t)nb * KB16 * 512 + lane * 8) * 2) : kOutOfRange;
  }
  auto load_b = [&](bf16x8 (&bt)[2][TN], int step) {
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        union { v4i_t u; bf16x8 v; } f;
        f.u = __builtin_amdgcn_raw_buffer_load_b128(rsrc_b, (int)(boff[j] + kk * 1024), step * 2048, 0);
        bt[kk][j] = f.v;
      }
  };
  // patch byte offset of tap t (clamped to the last tap)
  const int T = ks * ks;
  auto tap_off = [&](int t) {
    t = min(t, T - 1);
    const int kh = (int)fastdiv((uint32_t)t, ks, g.mg_ks), kw = t - kh * ks;
    return (kh * PW + kw) * pixb;
  };
  // patch byte offset the lanes of k-block b add to their window origin
  const bool upper = lane >= 32;
  auto blk_off = [&](int b) {
    if (C8) {
      const int o0 = tap_off(2 * b), o1 = tap_off(2 * b + 1);
      return upper ? o1 : o0;
    }
    const int t = (int)fastdiv((uint32_t)b, h.C16, h.mg_c16), c16 = b - t * h.C16;
    return tap_off(t) + c16 * 32;
  };
  auto lds_a = [&](int i, int off) { return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(lds) + abase[i] + off); };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  const int all_steps = (KB16 + 1) / 2;
  const int per = (all_steps + g.splits - 1) / g.splits;
  const int s_begin = __builtin_amdgcn_readfirstlane(sp * per);
  const int s_end = __builtin_amdgcn_readfirstlane(min(all_steps, s_begin + per));

  // One step = two k-blocks.  The filter fragments of the next step are requested, the second block's A fragments
  // are read, the first block's MFMAs run, the next step's first A fragments are read, the second block's MFMAs run.
  auto step = [&](bf16x8 (&bcur)[2][TN], bf16x8 (&bnext)[2][TN], bf16x8 (&a0)[TM], bf16x8 (&a0n)[TM], int s, bool has_next) {
    if (has_next) load_b(bnext, s + 1);
    const int o1 = blk_off(2 * s + 1);
    bf16x8 a1[TM];
#pragma unroll
    for (int i = 0; i < TM; i++) a1[i] = lds_a(i, o1);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[i], bcur[0][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    if (has_next) {
      const int o0 = blk_off(2 * s + 2);
#pragma unroll
      for (int i = 0; i < TM; i++) a0n[i] = lds_a(i, o0);
    }
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[i], bcur[1][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };

  bf16x8 b0[2][TN], b1[2][TN], fa[TM], fb[TM];
  if (s_begin < s_end) load_b(b0, s_begin);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (s_begin < s_end) {
    const int o0 = blk_off(2 * s_begin);
#pragma unroll
    for (int i = 0; i < TM; i++) fa[i] = lds_a(i, o0);
  }
  // two copies for an odd and an even number of steps: the last steps written out straight-line (see conv_halo_kernel)
  auto run = [&](auto odd) {
    int s = s_begin;
    const int pairs = (s_end - s_begin - 1) >> 1;
#pragma unroll 1
    for (int t = 0; t < pairs; t++, s += 2) {
      step(b0, b1, fa, fb, s, true);
      step(b1, b0, fb, fa, s + 1, true);
    }
    if constexpr (decltype(odd)::value) {
      step(b0, b1, fa, fb, s, false);
    } else {
      step(b0, b1, fa, fb, s, true);
      step(b1, b0, fb, fa, s + 1, false);
    }
  };
  if (s_begin < s_end) {
    if ((s_end - s_begin) & 1) run(std::true_type{});
    else run(std::false_type{});
  }

  if (g.splits > 1) {
    float* part = reinterpret_cast<float*>((char*)ws.p[z] + g.scratch_off) + (int64_t)sp * g.M * g.Ncols;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int n = n0 + wn0 + 32 * j + (lane & 31);
      if (n >= g.Ncols) continue;
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int m = m0 + wm0 + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (m < g.M) part[(int64_t)m * g.Ncols + n] = acc[i][j][r];
        }
    }
    return;
  }
  frag_epilogue<WM, WN>(acc, lds, ws.p[z], wts.p[z], g, ep, m0 + wm0, n0 + wn0, lane, wave);
}

// Sum of the split partials in split order, then bias / ReLU / mask / conversion.
__global__ __launch_bounds__(256) void igemm_finish_kernel(PtrTab ws, CPtrTab wts, IGemm g, Epilogue ep) {
  const int z = blockIdx.z;
  const float4* part = reinterpret_cast<const float4*>((const char*)ws.p[z] + g.scratch_off);
  bf16_t* out = (bf16_t*)ws.p[z] + ep.out_off;
  const bf16_t* mask = (const bf16_t*)ws.p[z] + ep.mask_off;
  const bf16_t* bias = (const bf16_t*)wts.p[z] + ep.bias_off;
  // four consecutive columns per thread (the column count is a multiple of 8)
  const uint32_t total4 = (uint32_t)(((int64_t)g.M * g.Ncols) >> 2);
  for (uint32_t o4 = blockIdx.x * 256 + threadIdx.x; o4 < total4; o4 += gridDim.x * 256) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int sp = 0; sp < g.splits; sp++) {   // loads of several splits in flight; the additions keep split order
      const float4 p = part[(size_t)sp * total4 + o4];
      v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    const int64_t o = (int64_t)o4 * 4;
    float f[4] = {v.x, v.y, v.z, v.w};
    if (ep.has_bias) {
      const int n = (int)((o4 * 4u) % (uint32_t)g.Ncols);
#pragma unroll
      for (int e = 0; e < 4; e++) f[e] += bf2f(bias[n + e]);
    }
    if (ep.relu) {
#pragma unroll
      for (int e = 0; e < 4; e++) f[e] = fmaxf(f[e], 0.f);
    }
    if (ep.use_mask) {
      const uint2 mk = *reinterpret_cast<const uint2*>(mask + o);
      const bf16_t m4[4] = {(bf16_t)(mk.x & 0xffffu), (bf16_t)(mk.x >> 16), (bf16_t)(mk.y & 0xffffu), (bf16_t)(mk.y >> 16)};
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (!(bf2f(m4[e]) > 0.f)) f[e] = 0.f;
    }
    if (ep.out_f32) {
      reinterpret_cast<float4*>(out)[o4] = make_float4(f[0], f[1], f[2], f[3]);
    } else {
      uint2 w;
      w.x = pack2bf(f[0], f[1]);
      w.y = pack2bf(f[2], f[3]);
      *reinterpret_cast<uint2*>(out + o) = w;
    }
  }
}

template <int BM, int BN, int WM, int WN>
static void launch_frag_t(const PtrTab& ws, const CPtrTab& wts, const IGemm& g_in, const Epilogue& ep, int count, hipStream_t s) {
  IGemm g = g_in;
  g.splits = worthwhile_splits(g.splits, (int64_t)((g.M + BM - 1) / BM) * ((g.Ncols + BN - 1) / BN) * count, 256 * (WM * WN > 64 * 64 ? 2 : 3));
  dim3 grid((unsigned)((g.M + BM - 1) / BM), (unsigned)((g.Ncols + BN - 1) / BN), (unsigned)(count * g.splits));
  constexpr int NT = 64 * (BM / WM) * (BN / WN);
  const bool uni = g.CPT % 4 == 0 && g.ks * g.ks <= 32 && g.Kchunks % 4 == 0;
  if (uni) hipLaunchKernelGGL((igemm_frag_kernel<BM, BN, WM, WN, 32, NT, true>), grid, dim3(NT), 0, s, ws, wts, g, ep);
  else hipLaunchKernelGGL((igemm_frag_kernel<BM, BN, WM, WN, 32, NT, false>), grid, dim3(NT), 0, s, ws, wts, g, ep);
  if (g.splits > 1) {
    int64_t total = ((int64_t)g.M * g.Ncols) >> 2;
    unsigned blocks = (unsigned)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048);
    hipLaunchKernelGGL(igemm_finish_kernel, dim3(blocks, 1, (unsigned)count), dim3(256), 0, s, ws, wts, g, ep);
  }
}

// Convolution forward / input gradient with fragment-packed filters (g.b_off points at the fragment copy).
// The patch-in-LDS kernel applies to windows larger than 1 x 1 over a multiple of 32 channels whose patch (plus the
// pixel table, 84 bytes per pixel) fits 64 KiB of LDS; the contraction is split at most once per channel chunk.
// decided: g.splits is the split to take, not the most.
template <int BM, int BN, int WM, int WN>
static bool launch_halo_t(const PtrTab& ws, const CPtrTab& wts, const IGemm& g_in, const Epilogue& ep, int count, bool xcd_order, hipStream_t s,
                          bool decided = false) {
  if (g_in.ks < 2 || g_in.C % 32 || g_in.OW + g_in.ks - 1 != g_in.W + 2 * g_in.pad) return false;
  IGemm g = g_in;
  g.splits = std::min(g.splits, g.C / 32);
  if (!decided) g.splits = worthwhile_splits(g.splits, (int64_t)((g.M + BM - 1) / BM) * ((g.Ncols + BN - 1) / BN) * count, 256 * (WM * WN > 64 * 64 ? 2 : 3));
  HaloArgs h;
  h.PW = g.OW + g.ks - 1;
  h.xcd = xcd_order ? 1 : 0;
  h.mg_pw = magic_u32(h.PW);
  const int rows = (BM + g.OW - 2) / g.OW + 1;               // output rows a tile of BM positions can touch
  const int images = (rows + g.OH - 2) / g.OH + 1;           // and images those rows can belong to
  h.n_px_max = (rows + (g.ks - 1) * images) * h.PW;
  constexpr int NT = 64 * (BM / WM) * (BN / WN);
  const size_t stage = (size_t)(NT / 64) * 32 * (WN + 8) * 2;   // the epilogue's staging pieces
  const size_t slot_round = (size_t)NT * 16;                 // bytes one refill instruction per thread covers
  h.tab_off = (int)(((size_t)h.n_px_max * 80 + slot_round - 1) / slot_round * slot_round);
  const size_t bytes = std::max((size_t)h.tab_off + (size_t)h.n_px_max * 4, stage);
  if (bytes > 64 * 1024) return false;
  dim3 grid((unsigned)((g.M + BM - 1) / BM), (unsigned)((g.Ncols + BN - 1) / BN), (unsigned)(count * g.splits));
  hipLaunchKernelGGL((conv_halo_kernel<BM, BN, WM, WN>), grid, dim3(NT), bytes, s, ws, wts, g, ep, h);
  if (g.splits > 1) {
    int64_t total = ((int64_t)g.M * g.Ncols) >> 2;
    unsigned blocks = (unsigned)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048);
    hipLaunchKernelGGL(igemm_finish_kernel, dim3(blocks, 1, (unsigned)count), dim3(256), 0, s, ws, wts, g, ep);
  }
  return true;
}

// Layers over 8 channels, or over a multiple of 16 (not of 32, at most 112) with windows of 4 x 4 and more:
// conv_halo_seq_kernel, if one tile's patch fits 64 KiB of LDS.  CIFAR-shaped conv1 (5 x 5 over 3 -> 8 channels, 18
// learners x 128 images): 63 us against 95 us for the tap-by-tap gather.
template <int BM, int BN, int WM, int WN>
static bool launch_halo_seq_t(const PtrTab& ws, const CPtrTab& wts, const IGemm& g_in, const Epilogue& ep, int count, hipStream_t s) {
  const bool c8 = g_in.C == 8;
  // (with 3 x 3 windows over 48 channels, the first layer of the AlexNet shape after space-to-depth, one fill of the
  // 50 KiB patch per tile costs more than nine-fold reuse saves: 155 us against 140 us for the tap-by-tap gather)
  if (g_in.ks < 2 || !(c8 || (g_in.C % 16 == 0 && g_in.C % 32 != 0 && g_in.C <= 112 && g_in.ks >= 4)) ||
      g_in.OW + g_in.ks - 1 != g_in.W + 2 * g_in.pad)
    return false;
  IGemm g = g_in;
  const int all_steps = (g.ldb / 16 + 1) / 2;
  g.splits = std::min(g.splits, std::max(1, all_steps / 2));
  g.splits = worthwhile_splits(g.splits, (int64_t)((g.M + BM - 1) / BM) * ((g.Ncols + BN - 1) / BN) * count, 256 * (WM * WN > 64 * 64 ? 2 : 3));
  HaloSeqArgs h;
  h.PW = g.OW + g.ks - 1;
  h.mg_pw = magic_u32(h.PW);
  h.spp = c8 ? 1 : g.C / 8 + 1;
  h.mg_spp = magic_u32(h.spp);
  h.pixb = 16 * h.spp;
  h.C16 = c8 ? 1 : g.C / 16;
  h.mg_c16 = magic_u32(h.C16);
  const int rows = (BM + g.OW - 2) / g.OW + 1;
  const int images = (rows + g.OH - 2) / g.OH + 1;
  h.n_px_max = (rows + (g.ks - 1) * images) * h.PW;
  constexpr int NT = 64 * (BM / WM) * (BN / WN);
  const size_t stage = (size_t)(NT / 64) * 32 * (WN + 8) * 2;
  const size_t slot_round = (size_t)NT * 16;
  h.tab_off = (int)(((size_t)h.n_px_max * h.pixb + slot_round - 1) / slot_round * slot_round);
  const size_t bytes = std::max((size_t)h.tab_off + (size_t)h.n_px_max * 4, stage);
  if (bytes > 64 * 1024) return false;
  dim3 grid((unsigned)((g.M + BM - 1) / BM), (unsigned)((g.Ncols + BN - 1) / BN), (unsigned)(count * g.splits));
  if (c8) hipLaunchKernelGGL((conv_halo_seq_kernel<BM, BN, WM, WN, true>), grid, dim3(NT), bytes, s, ws, wts, g, ep, h);
  else hipLaunchKernelGGL((conv_halo_seq_kernel<BM, BN, WM, WN, false>), grid, dim3(NT), bytes, s, ws, wts, g, ep, h);
  if (g.splits > 1) {
    int64_t total = ((int64_t)g.M * g.Ncols) >> 2;
    unsigned blocks = (unsigned)((total + 255) / 256 < 2048 ? (total + 255) / 256 : 2048);
    hipLaunchKernelGGL(igemm_finish_kernel, dim3(blocks, 1, (unsigned)count), dim3(256), 0, s, ws, wts, g, ep);
  }
  return true;
}

hipError_t launch_igemm_frag(const PtrTab& ws, const CPtrTab& wts, const IGemm& g, const Epilogue& ep, int count, hipStream_t s) {
  if (g.C % 8 || g.ldb % 32 || g.splits < 1) return hipErrorInvalidValue;
  if (g.C % 32 != 0) {
    bool done;
    if (g.Ncols <= 32) {
      const bool many = (int64_t)((g.M + 255) / 256) * count >= 1024;
      done = many ? launch_halo_seq_t<256, 32, 64, 32>(ws, wts, g, ep, count, s) : launch_halo_seq_t<128, 32, 32, 32>(ws, wts, g, ep, count, s);
    } else if (g.Ncols <= 64) {
      done = launch_halo_seq_t<128, 64, 64, 32>(ws, wts, g, ep, count, s);
    } else {
      done = launch_halo_seq_t<128, 128, 64, 64>(ws, wts, g, ep, count, s);
    }
    if (done) return hipGetLastError();
  }
  // own: most learners of this call read a weight version of their own (lambda-softsync) rather than a shared one
  int same = 0;
  for (int k = 1; k < count; k++) same += wts.p[k] == wts.p[0] ? 1 : 0;
  const bool own = count > 1 && 2 * same < count;
  const ConvProduct product{g.M, g.Ncols, g.C, g.ks, count, own, g.splits};
  // Narrow layers: 256-row tiles (64 x 32 per wavefront) once there are enough of them to fill the chip, else 128 rows.
  // Measured on the CIFAR-shaped layers (18 learners x 128 images): 5x5 over 32 channels, 16x16 images, 39 us against
  // 46 us with 128-row tiles and 68 us for the tap-by-tap gather; 8x8 images 27 us against 33 us and 43 us.
  if (g.Ncols <= 32) {
    const bool many = (int64_t)((g.M + 255) / 256) * count >= 1024;
    const bool done = many ? launch_halo_t<256, 32, 64, 32>(ws, wts, g, ep, count, own, s) : launch_halo_t<128, 32, 32, 32>(ws, wts, g, ep, count, own, s);
    if (done) return hipGetLastError();
  } else if (g.Ncols <= 64) {
    if (launch_halo_t<128, 64, 64, 32>(ws, wts, g, ep, count, own, s)) return hipGetLastError();
  }
  if (g.Ncols > 64 && g.Ncols % 256 == 0) {     // whole 256-column tiles: every filter fragment serves four products
    if (launch_halo_t<128, 256, 128, 64>(ws, wts, g, ep, count, own, s)) return hipGetLastError();
  } else if (g.Ncols > 64) {
    // (also measured slower: 128 x 64 wave tiles in two-wavefront blocks, eight-wavefront 256 x 128 blocks, 256 x 256)
    ConvChoice choice[3];
    const int n = conv_choices(product, choice);
    for (int k = 0; k < n; k++) {                // the next one where a patch does not fit
      IGemm gs = g;
      gs.splits = choice[k].splits;
      const bool done = choice[k].tile == ConvTile::k256x96   ? launch_halo_t<256, 96, 64, 96>(ws, wts, gs, ep, count, own, s, true)
                        : choice[k].tile == ConvTile::k256x128 ? launch_halo_t<256, 128, 128, 64>(ws, wts, gs, ep, count, own, s, true)
                                                               : launch_halo_t<128, 128, 64, 64>(ws, wts, gs, ep, count, own, s, true);
      if (done) return hipGetLastError();
    }
  }
  // Wave tile 128 x 64 (two wavefronts per SIMD, accumulators in ordinary registers) wins where the columns fill
  // whole 256-wide tiles: each B fragment then serves four MFMAs instead of two.  Measured slower: 256 x 128 blocks,
  // 192-wide tiles of three wavefronts for 384 columns, and taking the filters
  // through LDS as well (tiles 128 x 128 to 256 x 256, staging registers two steps deep): with both operands in
  // LDS its bandwidth becomes the limit instead of the vector L1's.
  if (g.Ncols <= 32) launch_frag_t<128, 32, 32, 32>(ws, wts, g, ep, count, s);
  else if (g.Ncols <= 64) launch_frag_t<128, 64, 64, 32>(ws, wts, g, ep, count, s);
  else if (frag_takes_96(product, (g.Kchunks + 3) / 4)) {
    IGemm gs = g;
    gs.splits = 1;
    launch_frag_t<256, 96, 64, 96>(ws, wts, gs, ep, count, s);
  } else if (g.Ncols % 256 == 0) launch_frag_t<128, 256, 128, 64>(ws, wts, g, ep, count, s);
  else launch_frag_t<128, 128, 64, 64>(ws, wts, g, ep, count, s);
  return hipGetLastError();
}

// ------------------------------------------------------------------ weight gradient
// A wavefront's piece of the weight-gradient tile: 32 TM output channels from n_base, 32 TN im2col columns from k_base.
template <int TM, int TN>
__device__ __forceinline__ void wgrad_write(const floatx16 (&acc)[TM][TN], const PtrTab& ws, const PtrTab& grads, const IGemm& g, const VConv& v,
                                            int64_t w_off, int64_t b_off, int partial, int z, int sp, int n_base, int k_base, int lane) {
  const int kcols = g.Kchunks * 8;
  if (partial) {   // fp32 partial [split][n][kcols + 8]; wgrad_finish_kernel adds and writes the flat gradient in its order
    const int ldk = kcols + 8;
    float* part = reinterpret_cast<float*>((char*)ws.p[z] + g.scratch_off) + (int64_t)sp * g.Ncols * ldk;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int k = k_base + 32 * j + (lane & 31);
      if (k > kcols) continue;
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int n = n_base + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
          if (n < g.Ncols) part[(int64_t)n * ldk + k] = acc[i][j][r];
        }
    }
    return;
  }
  float* dw = (float*)grads.p[z] + w_off;
  float* db = (float*)grads.p[z] + b_off;
  if (v.ks == 1 && v.s2d == 1 && v.C == v.Creal) {
    // fully connected layer: dW[n][k] is the tile itself, row length C; 32 lanes write 128 contiguous bytes
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int k = k_base + 32 * j + (lane & 31);
      if (k > kcols) continue;
#pragma unroll
      for (int i = 0; i < TM; i++) {
        const int nb = n_base + 32 * i + 4 * (lane >> 5);
        float* row = dw + (int64_t)nb * v.C + k;
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int dn = 8 * (r >> 2) + (r & 3);
          if (nb + dn >= g.Ncols) continue;
          if (k == kcols) db[nb + dn] = acc[i][j][r];
          else row[(int64_t)dn * v.C] = acc[i][j][r];
        }
      }
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const int k = k_base + 32 * j + (lane & 31);       // im2col column = tap * C + cp; column kcols = bias
    if (k > kcols) continue;
    const int tap = k / g.C, cp = k - tap * g.C;
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int n = n_base + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (n >= g.Ncols) continue;
        if (k == kcols) { db[n] = acc[i][j][r]; continue; }
        const int64_t dst = filter_src(v, n, tap, cp);
        if (dst >= 0) dw[dst] = acc[i][j][r];
      }
  }
}

// dW tile [BMG output channels][BNG im2col columns], contraction over output positions m in steps of 32.
// dy tile  [32 m][BMG n]  and  im2col tile [32 m][BNG k]  are staged as they lie in memory (rows = m) and
// read with the transpose load.  The result is scattered into the flat fp32 gradient through filter_src().
// INCR: the output position (image, oh, ow) of a thread's tile row advances from step to step by additions and
// two conditional wraps (possible when 32 / OW + 1 <= OH); otherwise it is decoded from the row index every step.
template <int BMG, int BNG, int WMG, int WNG, bool INCR>
__global__ __launch_bounds__(256) void igemm_wgrad_kernel(PtrTab ws, PtrTab grads, IGemm g, VConv v, size_t dy_off, int64_t w_off,
                                                          int64_t b_off, int partial) {
  constexpr int WAVES_NG = BNG / WNG;                  // four wavefronts: (BMG / WMG) x (BNG / WNG)
  constexpr int TM = WMG / 32, TN = WNG / 32;
  constexpr int LDT_A = BMG + 32 - (BMG == 32 ? 32 : 0);
  constexpr int LDT_B = BNG + 32 - (BNG == 32 ? 32 : 0);
  constexpr int A_ELEMS = BK * LDT_A, B_ELEMS = BK * LDT_B;
  __shared__ __attribute__((aligned(16))) bf16_t lds[2 * (A_ELEMS + B_ELEMS)];

  const TileIdx tile = xcd_tile(1);   // a learner's tiles share dy and x: keep them on one XCD's L2 (AlexNet layers 3-9 % faster)
  const int z = tile.z / g.splits, sp = tile.z % g.splits;
  const bf16_t* x = (const bf16_t*)ws.p[z] + g.a_off;
  const bf16_t* dy = (const bf16_t*)ws.p[z] + dy_off;
  const int n0 = tile.x * BMG, k0 = tile.y * BNG;           // output-channel and im2col-column origins
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WAVES_NG) * WMG, wn0 = (wave % WAVES_NG) * WNG;

  constexpr int CPR_A = BMG / 8, CPR_B = BNG / 8;
  constexpr int TPR = 256 / BK;                        // threads per tile row of the im2col tile
  constexpr int A_LOADS = (BK * CPR_A + 255) / 256, B_LOADS = CPR_B / TPR;
  static_assert(CPR_B % TPR == 0, "im2col tile: whole chunks per thread");
  const int all_steps = (g.M + BK - 1) / BK;
  const int per = (all_steps + g.splits - 1) / g.splits;
  const int ms_begin = __builtin_amdgcn_readfirstlane(sp * per);
  const int msteps = __builtin_amdgcn_readfirstlane(min(all_steps, ms_begin + per));

  // Hardware-bounds-checked buffer loads (an offset at or beyond the tensor reads as zero): rows beyond M, columns
  // beyond the layer and taps in the zero padding need no branch and no patching of loaded data.
  const __amdgpu_buffer_rsrc_t rsrc_dy = __builtin_amdgcn_make_buffer_rsrc((void*)dy, 0, (int)((int64_t)g.M * g.Ncols * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, (int)g.a_bytes, 0x00020000);
  // dy tile: chunk (row r, 8 channels from n) per thread; its offset advances by a constant every step
  uint32_t a_off[A_LOADS];
  const uint32_t a_step = (uint32_t)(BK * g.Ncols * 2);
#pragma unroll
  for (int i = 0; i < A_LOADS; i++) {
    const int idx = tid + 256 * i;
    const int r = idx / CPR_A, n = n0 + (idx % CPR_A) * 8;
    a_off[i] = (r < BK && n < g.Ncols) ? (uint32_t)((((int64_t)ms_begin * BK + r) * g.Ncols + n) * 2) : kOutOfRange;
  }
  // im2col tile: a thread owns B_LOADS chunks of ONE tile row; their filter taps are fixed, only the row's output
  // position changes from step to step
  const int b_row = tid / TPR;
  int b_dkh[B_LOADS], b_dkw[B_LOADS], b_koff[B_LOADS];
  bool b_ok[B_LOADS], b_ones[B_LOADS];
#pragma unroll
  for (int i = 0; i < B_LOADS; i++) {
    const int q = k0 / 8 + tid % TPR + TPR * i;
    const uint32_t tap = fastdiv((uint32_t)q, g.CPT, g.mg_cpt);
    const int c8 = q - (int)tap * g.CPT;
    const int kh = (int)fastdiv(tap, g.ks, g.mg_ks), kw = (int)tap - kh * g.ks;
    b_dkh[i] = kh - g.pad;
    b_dkw[i] = kw - g.pad;
    b_koff[i] = ((b_dkh[i] * g.W + b_dkw[i]) * g.C + c8 * 8) * 2;
    b_ok[i] = q < g.Kchunks;
    b_ones[i] = q == g.Kchunks;                  // the bias column: im2col value 1 for every real output position
  }
  // position of the row that load_regs fetches next: m, its (oh, ow) and the byte offset of x[image][oh][ow][0]
  int r_m = ms_begin * BK + b_row, r_oh, r_ow, r_off;
  auto decode_row = [&]() {
    const uint32_t mm = r_m < g.M ? (uint32_t)r_m : 0u;
    const uint32_t rest = fastdiv(mm, g.OW, g.mg_ow);
    const uint32_t n = fastdiv(rest, g.OH, g.mg_oh);
    r_ow = (int)(mm - rest * (uint32_t)g.OW);
    r_oh = (int)(rest - n * (uint32_t)g.OH);
    r_off = (int)(((n * (uint32_t)g.H + (uint32_t)r_oh) * (uint32_t)g.W + (uint32_t)r_ow) * (uint32_t)g.C * 2u);
  };
  decode_row();
  const int d_ow = BK / g.OW, m_ow = BK - d_ow * g.OW;          // 32 rows further: d_ow lines down, m_ow positions right
  const int inc0 = (d_ow * g.W + m_ow) * g.C * 2;               // the same in bytes of x
  const int inc_w = (g.W - g.OW) * g.C * 2;                      // extra when ow wraps into the next line
  const int inc_h = (g.H - g.OH) * g.W * g.C * 2;                // extra when oh wraps into the next image

  v4i_t ra[A_LOADS], rb[B_LOADS];
  uint32_t bias_one[B_LOADS];
  auto load_regs = [&]() {
#pragma unroll
    for (int i = 0; i < A_LOADS; i++) {
      ra[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_dy, (int)a_off[i], 0, 0);
      a_off[i] += a_step;
    }
    const bool valid = r_m < g.M;
#pragma unroll
    for (int i = 0; i < B_LOADS; i++) {
      const bool ok = b_ok[i] && valid && (unsigned)(r_oh + b_dkh[i]) < (unsigned)g.H && (unsigned)(r_ow + b_dkw[i]) < (unsigned)g.W;
      rb[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, ok ? r_off + b_koff[i] : (int)kOutOfRange, 0, 0);
      bias_one[i] = (b_ones[i] && valid) ? 0x3F80u : 0u;
    }
    // advance the row by BK output positions
    r_m += BK;
    if (INCR) {
      r_ow += m_ow;
      const bool c1 = r_ow >= g.OW;
      r_ow -= c1 ? g.OW : 0;
      r_oh += d_ow + (c1 ? 1 : 0);
      const bool c2 = r_oh >= g.OH;
      r_oh -= c2 ? g.OH : 0;
      r_off += inc0 + (c1 ? inc_w : 0) + (c2 ? inc_h : 0);
    } else {
      decode_row();
    }
  };
  auto store_lds = [&](int buf) {
    bf16_t* A = lds + buf * (A_ELEMS + B_ELEMS);
    bf16_t* B = A + A_ELEMS;
#pragma unroll
    for (int i = 0; i < A_LOADS; i++) {
      int idx = tid + 256 * i;
      int r = idx / CPR_A, ch = idx % CPR_A;
      if (BK * CPR_A % 256 == 0 || r < BK) *reinterpret_cast<v4i_t*>(A + r * LDT_A + ch * 8) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < B_LOADS; i++) {
      v4i_t val = rb[i];
      val.x |= (int)bias_one[i];                 // the chunk of the bias column loads as zeros; its first element becomes 1.0
      *reinterpret_cast<v4i_t*>(B + b_row * LDT_B + (tid % TPR + TPR * i) * 8) = val;
    }
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  const int j16 = lane & 15, half = (lane >> 4) & 1;
  // One step: the tiles of step ms+1 (fetched during step ms-1) go to the other LDS buffer, the tiles of step ms+2 are
  // requested, then the MFMAs run on buffer `buf`: a global load has a whole step to arrive.  Two steps per loop
  // iteration make `buf` a constant.
  auto step = [&](int buf, bool has1, bool has2) {
    const bf16_t* A = lds + buf * (A_ELEMS + B_ELEMS);
    const bf16_t* B = A + A_ELEMS;
#pragma unroll
    for (int kk = 0; kk < 2; kk++) {
      const int kb = 16 * kk + 8 * (lane >> 5);
      bf16x8 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; i++) {
        const bf16_t* p = A + (kb + (j16 >> 2)) * LDT_A + wm0 + 32 * i + 16 * half + 4 * (j16 & 3);
        union { bf16x8 v; shortx4 h[2]; } u;
        u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p));
        u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p + 4 * LDT_A));
        a[i] = u.v;
      }
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const bf16_t* p = B + (kb + (j16 >> 2)) * LDT_B + wn0 + 32 * j + 16 * half + 4 * (j16 & 3);
        union { bf16x8 v; shortx4 h[2]; } u;
        u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p));
        u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p + 4 * LDT_B));
        b[j] = u.v;
      }
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    // the wait for the next tiles' global loads falls behind this step's MFMAs instead of in front of its LDS reads
    __builtin_amdgcn_sched_barrier(0);
    if (has1) store_lds(buf ^ 1);
    if (has2) load_regs();
    __syncthreads();
  };

  int ms = ms_begin;
  if (ms < msteps) {
    load_regs();
    store_lds(0);
    if (ms + 1 < msteps) load_regs();
  }
  __syncthreads();
  for (; ms + 3 < msteps; ms += 2) {            // no branch around the loads inside the loop
    step(0, true, true);
    step(1, true, true);
  }
  for (; ms + 1 < msteps; ms += 2) {            // at most once: two or three steps remain
    step(0, true, ms + 2 < msteps);
    step(1, ms + 2 < msteps, false);
  }
  if (ms < msteps) step(0, false, false);

  wgrad_write<TM, TN>(acc, ws, grads, g, v, w_off, b_off, partial, z, sp, n0 + wm0, k0 + wn0, lane);
}

// The same product for more than 64 output channels, with the tiles going from memory to LDS without passing through
// registers.  Tiles are stored as panels of 32 columns, [panel][32 m][32 columns]: the 64 lanes of an LDS-direct load fill half
// a panel (16 rows of 64 bytes, a piece the vector L1 serves at its full rate), a panel is the operand of one 32-wide MFMA
// block, and four neighbouring rows lie 16 banks apart, so that the transpose load meets no conflict and needs no padding.
// Three buffers: the tiles of step s + 2 are requested before the MFMAs of step s and waited for by count at the end of step
// s + 1; one barrier a step.  Every step issues the same number of loads; rows behind the split's last one are out of range
// and arrive as zeros.  The buffers are arrays of their own and the step is written out once per buffer: only then does the
// compiler know that an LDS read of one does not wait for the loads into another.
// What bounds it: the transposing LDS reads (32 KiB a step at 82 B/clk per compute unit) and the arriving tiles.  AlexNet-shaped
// net, 288 images, average of its five layers: 147 us against 173 us with staging registers and two buffers.  128 x 256 tiles
// (64 x 128 per wavefront) read a quarter less but leave two wavefronts a SIMD and too few tiles: 152 us.  Where there is enough
// work for a round of its larger tiles, wgrad_wide_kernel below is the faster one (wgrad_tiles).
template <bool INCR>
__global__ __launch_bounds__(256, 3) void wgrad_panel_kernel(PtrTab ws, PtrTab grads, IGemm g, VConv v, size_t dy_off, int64_t w_off,
                                                             int64_t b_off, int partial) {
  constexpr int BMG = 128, BNG = 128, TM = 2, TN = BNG / 64;
  constexpr int PA = BMG / 32, PB = BNG / 32, PANEL = BK * 32;
  __shared__ __attribute__((aligned(16))) bf16_t buf0[(PA + PB) * PANEL], buf1[(PA + PB) * PANEL], buf2[(PA + PB) * PANEL];

  const TileIdx tile = xcd_tile(1);
  const int z = tile.z / g.splits, sp = tile.z % g.splits;
  const bf16_t* x = (const bf16_t*)ws.p[z] + g.a_off;
  const bf16_t* dy = (const bf16_t*)ws.p[z] + dy_off;
  const int n0 = tile.x * BMG, k0 = tile.y * BNG;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * 64, wn0 = (wave & 1) * (BNG / 2);

  const int all_steps = (g.M + BK - 1) / BK;
  const int per = (all_steps + g.splits - 1) / g.splits;
  const int ms_begin = __builtin_amdgcn_readfirstlane(sp * per);
  const int ms_end = __builtin_amdgcn_readfirstlane(min(all_steps, ms_begin + per));
  const int m_end = min(g.M, ms_end * BK);

  // the bias column is an im2col column of ones: its chunk {1, 0, ...} comes from the constant block of the workspace, which
  // only the workgroups that hold this column can reach
  const int one_off = (int)((g.zero_off + 128 - g.a_off) * 2);
  const bool has_bias = g.Kchunks * 8 >= k0 && g.Kchunks * 8 < k0 + BNG;
  const __amdgpu_buffer_rsrc_t rsrc_dy = __builtin_amdgcn_make_buffer_rsrc((void*)dy, 0, (int)((int64_t)m_end * g.Ncols * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, has_bias ? one_off + 16 : (int)g.a_bytes, 0x00020000);
  const int row = lane >> 2, ch = lane & 3;
  uint32_t a_off[2];
  const uint32_t a_step = (uint32_t)(BK * g.Ncols * 2);
#pragma unroll
  for (int h = 0; h < 2; h++) {
    const int n = n0 + wave * 32 + ch * 8;
    a_off[h] = n < g.Ncols ? (uint32_t)((((int64_t)ms_begin * BK + 16 * h + row) * g.Ncols + n) * 2) : kOutOfRange;
  }
  const int q = k0 / 8 + wave * 4 + ch;                  // this lane's im2col chunk: one tap, 8 channels
  const uint32_t tap = fastdiv((uint32_t)q, g.CPT, g.mg_cpt);
  const int c8 = q - (int)tap * g.CPT;
  const int kh = (int)fastdiv(tap, g.ks, g.mg_ks), kw = (int)tap - kh * g.ks;
  const int b_dkh = q < g.Kchunks ? kh - g.pad : (int)kOutOfRange;      // a row that no input has
  const int b_dkw = kw - g.pad;
  const int b_koff = ((kh - g.pad) * g.W * g.C + (kw - g.pad) * g.C + c8 * 8) * 2;
  const int b_else = q == g.Kchunks ? one_off : (int)kOutOfRange;
  // position of the rows that `issue` fetches next
  int r_m[2], r_oh[2], r_ow[2], r_off[2];
  auto decode_row = [&](int h) {
    const uint32_t mm = r_m[h] < g.M ? (uint32_t)r_m[h] : 0u;
    const uint32_t rest = fastdiv(mm, g.OW, g.mg_ow);
    const uint32_t n = fastdiv(rest, g.OH, g.mg_oh);
    r_ow[h] = (int)(mm - rest * (uint32_t)g.OW);
    r_oh[h] = (int)(rest - n * (uint32_t)g.OH);
    r_off[h] = (int)(((n * (uint32_t)g.H + (uint32_t)r_oh[h]) * (uint32_t)g.W + (uint32_t)r_ow[h]) * (uint32_t)g.C * 2u);
  };
#pragma unroll
  for (int h = 0; h < 2; h++) {
    r_m[h] = ms_begin * BK + 16 * h + row;
    decode_row(h);
  }
  const int d_ow = BK / g.OW, m_ow = BK - d_ow * g.OW;
  const int inc0 = (d_ow * g.W + m_ow) * g.C * 2;
  const int inc_w = (g.W - g.OW) * g.C * 2;
  const int inc_h = (g.H - g.OH) * g.W * g.C * 2;

  auto issue = [&](bf16_t* S) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_dy, (__attribute__((address_space(3))) void*)(S + wave * PANEL + h * (PANEL / 2)), 16, (int)a_off[h], 0, 0, 0);
      a_off[h] += a_step;
      const bool ok = r_m[h] < m_end && (unsigned)(r_oh[h] + b_dkh) < (unsigned)g.H && (unsigned)(r_ow[h] + b_dkw) < (unsigned)g.W;
      const int off = ok ? r_off[h] + b_koff : b_else;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (__attribute__((address_space(3))) void*)(S + (PA + wave) * PANEL + h * (PANEL / 2)), 16,
                                               off, 0, 0, 0);
      r_m[h] += BK;
      if (INCR) {
        r_ow[h] += m_ow;
        const bool c1 = r_ow[h] >= g.OW;
        r_ow[h] -= c1 ? g.OW : 0;
        r_oh[h] += d_ow + (c1 ? 1 : 0);
        const bool c2 = r_oh[h] >= g.OH;
        r_oh[h] -= c2 ? g.OH : 0;
        r_off[h] += inc0 + (c1 ? inc_w : 0) + (c2 ? inc_h : 0);
      } else {
        decode_row(h);
      }
    }
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  const int j16 = lane & 15;
  const int lane_off = (8 * (lane >> 5) + (j16 >> 2)) * 32 + 16 * ((lane >> 4) & 1) + 4 * (j16 & 3);
  const int pa_off = (wm0 / 32) * PANEL + lane_off, pb_off = (PA + wn0 / 32) * PANEL + lane_off;
  auto read_frag = [&](const bf16_t* p) {
    union { bf16x8 v; shortx4 h[2]; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p + 4 * 32));
    return u.v;
  };
  auto multiply = [&](const bf16_t* S) {
#pragma unroll
    for (int kk = 0; kk < 2; kk++) {
      bf16x8 a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; i++) a[i] = read_frag(S + pa_off + i * PANEL + kk * 16 * 32);
#pragma unroll
      for (int j = 0; j < TN; j++) b[j] = read_frag(S + pb_off + j * PANEL + kk * 16 * 32);
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };
  // The older of two steps' loads has landed (each wavefront waits for its own, the barrier for everyone's), and this
  // wavefront's LDS reads are done, so that the buffer it leaves may be overwritten.
  auto turn = [&]() {
    asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // four loads a step and wavefront
  };

  const int steps = ms_end - ms_begin;
  issue(buf0);
  issue(buf1);
  turn();
  int s = 0;
  for (; s + 3 <= steps; s += 3) {
    issue(buf2); multiply(buf0); turn();
    issue(buf0); multiply(buf1); turn();
    issue(buf1); multiply(buf2); turn();
  }
  if (s < steps) {
    issue(buf2); multiply(buf0); turn();
    if (s + 1 < steps) multiply(buf1);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no load is left on its way to this workgroup's LDS
  wgrad_write<TM, TN>(acc, ws, grads, g, v, w_off, b_off, partial, z, sp, n0 + wm0, k0 + wn0, lane);
}
// All but the youngest N loads of this wavefront have landed, its LDS reads are done, and so for every wavefront.
template <int N>
__device__ __forceinline__ void landed_and_read() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// Large products: tiles of 32 TM WM output channels x 128 (4 / WM) im2col columns, one wavefront a SIMD with 32 TM x 128 of them
// in its accumulators.  What bounds wgrad_panel_kernel is the rate at which a compute unit issues transposing LDS reads (6.2 cycles
// each, four a product of 64 x 64 wavefront tiles' 32 cycles): a 128 x 128 wavefront tile needs half as many for the same
// products.  With one wavefront a SIMD nothing else covers a latency, so every read is issued a k-block ahead, between the
// products of the one before, and four stages are in LDS, two of them on their way.  Panels, addresses and the bias column are
// wgrad_panel_kernel's.  AlexNet-shaped net, 256 images of one learner, its five layers from the input on: 159 / 229 / 99 / 122 / 100 us
// there, 90 / 182 / 76 / 105 / 72 us here (1.26 PFLOP/s in the second).
template <int TM, int WM>
__global__ __launch_bounds__(256, 1) void wgrad_wide_kernel(PtrTab ws, PtrTab grads, IGemm g, VConv v, size_t dy_off, int64_t w_off, int64_t b_off) {
  constexpr int TN = 4, BMG = 32 * TM * WM, BNG = 128 * (4 / WM);
  constexpr int PA = BMG / 32, PB = BNG / 32, PANEL = BK * 32;
  constexpr int LA = (PA * 2 + 3) / 4, LB = PB * 2 / 4;    // half panels a wavefront loads per stage (dy: the last one perhaps none)
  static_assert(LB % 2 == 0 && (PA * 2 % 4 == 0 || PA * 2 == LA * 3), "shares");
  __shared__ __attribute__((aligned(16))) bf16_t buf0[(PA + PB) * PANEL], buf1[(PA + PB) * PANEL], buf2[(PA + PB) * PANEL], buf3[(PA + PB) * PANEL];

  const TileIdx tile = xcd_tile(1);
  const int z = tile.z / g.splits, sp = tile.z % g.splits;
  const bf16_t* x = (const bf16_t*)ws.p[z] + g.a_off;
  const bf16_t* dy = (const bf16_t*)ws.p[z] + dy_off;
  const int n0 = tile.x * BMG, k0 = tile.y * BNG;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave % WM) * (32 * TM), wn0 = (wave / WM) * 128;

  const int all_steps = (g.M + BK - 1) / BK;
  const int per = (all_steps + g.splits - 1) / g.splits;
  const int ms_begin = __builtin_amdgcn_readfirstlane(sp * per);
  const int ms_end = __builtin_amdgcn_readfirstlane(min(all_steps, ms_begin + per));
  const int m_end = min(g.M, ms_end * BK);

  const int one_off = (int)((g.zero_off + 128 - g.a_off) * 2);
  const bool has_bias = g.Kchunks * 8 >= k0 && g.Kchunks * 8 < k0 + BNG;
  const __amdgpu_buffer_rsrc_t rsrc_dy = __builtin_amdgcn_make_buffer_rsrc((void*)dy, 0, (int)((int64_t)m_end * g.Ncols * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, has_bias ? one_off + 16 : (int)g.a_bytes, 0x00020000);
  const int row = lane >> 2, ch = lane & 3;
  // dy: half panel a = LA * wave + l is panel a / 2, rows 16 (a % 2) .. + 15
  int a_off[LA];
  const int a_step = BK * g.Ncols * 2;
#pragma unroll
  for (int l = 0; l < LA; l++) {
    const int a = LA * wave + l, n = n0 + (a >> 1) * 32 + ch * 8;
    a_off[l] = n < g.Ncols ? (int)((((int64_t)ms_begin * BK + 16 * (a & 1) + row) * g.Ncols + n) * 2) : (int)kOutOfRange;
  }
  // x: panels (LB / 2) * wave + p, both halves; a lane's chunk of a panel is one tap, 8 channels
  int b_dkh[LB / 2], b_dkw[LB / 2], b_koff[LB / 2], b_else[LB / 2];
#pragma unroll
  for (int p = 0; p < LB / 2; p++) {
    const int q = k0 / 8 + (LB / 2 * wave + p) * 4 + ch;
    const uint32_t tap = fastdiv((uint32_t)q, g.CPT, g.mg_cpt);
    const int c8 = q - (int)tap * g.CPT;
    const int kh = (int)fastdiv(tap, g.ks, g.mg_ks), kw = (int)tap - kh * g.ks;
    b_dkh[p] = q < g.Kchunks ? kh - g.pad : (int)kOutOfRange;      // a row that no input has
    b_dkw[p] = kw - g.pad;
    b_koff[p] = ((kh - g.pad) * g.W * g.C + (kw - g.pad) * g.C + c8 * 8) * 2;
    b_else[p] = q == g.Kchunks ? one_off : (int)kOutOfRange;
  }
  int r_m[2], r_oh[2], r_ow[2], r_off[2];
#pragma unroll
  for (int h = 0; h < 2; h++) {
    r_m[h] = ms_begin * BK + 16 * h + row;
    const uint32_t mm = r_m[h] < g.M ? (uint32_t)r_m[h] : 0u;
    const uint32_t rest = fastdiv(mm, g.OW, g.mg_ow);
    const uint32_t n = fastdiv(rest, g.OH, g.mg_oh);
    r_ow[h] = (int)(mm - rest * (uint32_t)g.OW);
    r_oh[h] = (int)(rest - n * (uint32_t)g.OH);
    r_off[h] = (int)(((n * (uint32_t)g.H + (uint32_t)r_oh[h]) * (uint32_t)g.W + (uint32_t)r_ow[h]) * (uint32_t)g.C * 2u);
  }
  const int d_ow = BK / g.OW, m_ow = BK - d_ow * g.OW;
  const int inc0 = (d_ow * g.W + m_ow) * g.C * 2;
  const int inc_w = (g.W - g.OW) * g.C * 2;
  const int inc_h = (g.H - g.OH) * g.W * g.C * 2;

  auto issue = [&](bf16_t* S) {
    if (PA * 2 % 4 == 0 || wave < 3)
#pragma unroll
    for (int l = 0; l < LA; l++) {
      const int off = a_off[l];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_dy, (__attribute__((address_space(3))) void*)(S + (LA * wave + l) * (PANEL / 2)), 16, off, 0, 0, 0);
      a_off[l] += a_step;
    }
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const bool in = r_m[h] < m_end;
#pragma unroll
      for (int p = 0; p < LB / 2; p++) {
        const bool ok = in & ((unsigned)(r_oh[h] + b_dkh[p]) < (unsigned)g.H) & ((unsigned)(r_ow[h] + b_dkw[p]) < (unsigned)g.W);
        const int off = ok ? r_off[h] + b_koff[p] : b_else[p];
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (__attribute__((address_space(3))) void*)(S + (PA + LB / 2 * wave + p) * PANEL + h * (PANEL / 2)), 16,
                                                 off, 0, 0, 0);
      }
      r_m[h] += BK;
      r_ow[h] += m_ow;
      const bool c1 = r_ow[h] >= g.OW;
      r_ow[h] -= c1 ? g.OW : 0;
      r_oh[h] += d_ow + (c1 ? 1 : 0);
      const bool c2 = r_oh[h] >= g.OH;
      r_oh[h] -= c2 ? g.OH : 0;
      r_off[h] += inc0 + (c1 ? inc_w : 0) + (c2 ? inc_h : 0);
    }
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  const int j16 = lane & 15;
  const int lane_off = (8 * (lane >> 5) + (j16 >> 2)) * 32 + 16 * ((lane >> 4) & 1) + 4 * (j16 & 3);
  const int pa_off = (wm0 / 32) * PANEL + lane_off, pb_off = (PA + wn0 / 32) * PANEL + lane_off;
  auto read_frag = [&](const bf16_t* p) {
    union { bf16x8 v; shortx4 h[2]; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p + 4 * 32));
    return u.v;
  };
  auto read = [&](bf16x8 (&a)[TM], bf16x8 (&b)[TN], const bf16_t* S, int kk) {
#pragma unroll
    for (int i = 0; i < TM; i++) a[i] = read_frag(S + pa_off + i * PANEL + kk * 16 * 32);
#pragma unroll
    for (int j = 0; j < TN; j++) b[j] = read_frag(S + pb_off + j * PANEL + kk * 16 * 32);
  };
  auto multiply = [&](const bf16x8 (&a)[TM], const bf16x8 (&b)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  };
  // Step s on stage buffer `cur`: the second k-block is read while the first one's products run.  Then the next stage has landed
  // (one more is on its way), every wavefront's reads of `cur` are done, and the stage after those is requested into the buffer
  // that was left a step ago; the next stage's first k-block is read while the second one's products run.
  bf16x8 a0[TM], b0[TN], a1[TM], b1[TN];
  auto step = [&](bf16_t* cur, bf16_t* next, bf16_t* free_) {
    read(a1, b1, cur, 1);
    multiply(a0, b0);
#pragma unroll
    for (int k = 0; k < TM * TN; k++) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // a product ...
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);       // ... and a read behind it
    }
    __builtin_amdgcn_sched_barrier(0);
    if (PA * 2 % 4 == 0 || wave < 3) landed_and_read<LA + LB>();
    else landed_and_read<LB>();
    read(a0, b0, next, 0);
    multiply(a1, b1);
    issue(free_);
#pragma unroll
    for (int k = 0; k < TM * TN; k++) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);       // addresses of the loads
      if (k & 1) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  const int steps = ms_end - ms_begin;
  issue(buf0);
  issue(buf1);
  issue(buf2);
  if (PA * 2 % 4 == 0 || wave < 3) landed_and_read<2 * (LA + LB)>();
  else landed_and_read<2 * LB>();
  read(a0, b0, buf0, 0);
  // stages 0, 1, 2 are requested; step s requests stage s + 3
#pragma unroll 1
  for (int s = 0; s < steps; s += 4) {           // stages behind the last one are zeros
    step(buf0, buf1, buf3);
    step(buf1, buf2, buf0);
    step(buf2, buf3, buf1);
    step(buf3, buf0, buf2);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // no load is left on its way to this workgroup's LDS
  wgrad_write<TM, TN>(acc, ws, grads, g, v, w_off, b_off, 1, z, sp, n0 + wm0, k0 + wn0, lane);
}
// Up to 64 output channels.  Gathered tap by tap, a narrow tile's im2col columns pass the vector L1 once per tap and 128 columns,
// which took longer than anything else (32 channels of 16 x 16 images, 5 x 5 over 32: 1.3 GB for 37 MB of input).  Here
// the input patch under a tile of MT output positions is in LDS, all channels of a pixel, and the transposing reads pick every
// tap's columns out of it: a lane's address is its position's place in the patch plus an offset that depends on its column only.
// A workgroup of eight wavefronts holds 32 WN TN columns (the last place of the last group is the bias: a fragment of ones),
// its 8 / WN position groups take a tile's 16-position steps in turn and are added through LDS at the end.  Patch, dy and the
// positions' places are double-buffered: the next tile's are requested before this one is multiplied, one barrier a tile.
// Bound by the transposing LDS reads.  CIFAR-shaped net, 18 learners x 128 images: its three layers 96 / 79 / 36 us gathered,
// 51 / 45 / 31 here.
//
// POOL: a first layer with a 3 x 3 / 2 max pooling behind it reads the pooled tensor's gradient and the winners, a third of the bytes, instead of
// its own output's, the largest tensor of the network, which then is neither written nor read and of which this was the only reader.  A
// thread owns 8 channels of a 2 x 2 block of the tile, reads the four windows that reach it (a tile ahead, in registers) and puts the four
// results where the dy of the tile would have landed.  Four of the wavefronts do that in front of their products and four behind, so that
// vector and matrix instructions of the two of a SIMD meet.  First layer above: pooling backward and this 54 + 54 us, 63 in one kernel (68 with
// all wavefronts behind; 71 with a compare and a select for each channel and window instead of four channels' compares in one subtraction).
struct StripArgs {
  int PW;                    // patch width in pixels
  int tiles, per;            // tiles of MT positions, and how many a workgroup takes
  int patch, buf;            // bytes of a patch and of a whole buffer (dy, patch, places) in LDS
  FastDiv by_pw, by_cpt, by_band;   // divisions by PW, by 8-channel chunks of a pixel and by OH + ks - 1 (rows of a whole image in the patch)
  int PH, PWo;               // POOL: pooled size
  size_t arg_off;            // and its winners (bytes)
};

template <int TM, int WN, int TN, int MT, bool POOL>
__global__ __launch_bounds__(512, 2) void wgrad_strip_kernel(PtrTab ws, IGemm g, size_t dy_off, StripArgs h) {
  constexpr int WK = 8 / WN, NT = 512, DY = TM * MT * 64;
  static_assert(TM * MT <= NT, "POOL: 8 channels of a 2 x 2 block a thread");
  extern __shared__ __attribute__((aligned(16))) char strip_lds[];
  char* lds = strip_lds;
  const int z = blockIdx.z / g.splits, sp = blockIdx.z % g.splits, cg = blockIdx.y;
  const bf16_t* x = (const bf16_t*)ws.p[z] + g.a_off;
  const bf16_t* dy = (const bf16_t*)ws.p[z] + dy_off;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % WN, wk = wave / WN;
  const int ks = g.ks, PW = h.PW;
  const int kcols = g.Kchunks * 8;
  const int j16 = lane & 15;
  // this lane's columns of each block: the offset of their tap and channels in the patch
  int off[TN];
#pragma unroll
  for (int p = 0; p < TN; p++) {
    const int panel = (cg * WN + wn) * TN + p, col = panel * 32 + 16 * ((lane >> 4) & 1) + 4 * (j16 & 3);
    const uint32_t tap = fastdiv((uint32_t)col >> 3, g.CPT, g.mg_cpt);
    const int kh = (int)fastdiv(tap, ks, g.mg_ks), kw = (int)tap - kh * ks;
    off[p] = col < kcols ? ((kh * PW + kw) * g.C + col - (int)tap * g.C) * 2 : 0;
  }
  const bool last_group = cg == (int)gridDim.y - 1, bias = last_group && wn == WN - 1;   // (its block TN - 1)
  bf16x8 ones;
  {
    union { bf16x8 v; bf16_t e[8]; } u;
#pragma unroll
    for (int e = 0; e < 8; e++) u.e[e] = lane % 32 == 0 ? (bf16_t)0x3F80 : (bf16_t)0;
    ones = u.v;
  }

  v4i_t rsrc_dy, rsrc_x;
  rsrc_dy.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)dy);
  rsrc_dy.y = __builtin_amdgcn_readfirstlane((int)((uintptr_t)dy >> 32) & 0xffff);
  rsrc_dy.z = (int)((int64_t)g.M * g.Ncols * 2);
  rsrc_dy.w = 0x00020000;
  // POOL: dy is the pooled tensor's
  const uint32_t out_rows = POOL ? fastdiv((uint32_t)g.M, g.OW, g.mg_ow) : 0;
  const int pooled = POOL ? (int)fastdiv(out_rows, g.OH, g.mg_oh) * h.PH * h.PWo * g.Ncols : 0;
  const __amdgpu_buffer_rsrc_t rsrc_pooled = __builtin_amdgcn_make_buffer_rsrc((void*)dy, 0, pooled * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_arg = __builtin_amdgcn_make_buffer_rsrc((char*)ws.p[z] + (POOL ? h.arg_off : 0), 0, pooled, 0x00020000);
  rsrc_x.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)x);
  rsrc_x.y = __builtin_amdgcn_readfirstlane((int)((uintptr_t)x >> 32) & 0xffff);
  rsrc_x.z = (int)g.a_bytes;
  rsrc_x.w = 0x00020000;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  // Written out because the compiler, which cannot tell the buffers apart, would wait for all of them in front of every LDS read.
  // m0 is a register that it never allocates (hence its warning) but whose values it shares between neighbouring uses of its own.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  auto dma = [&](const v4i_t& rsrc, uint32_t dst, int voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(lds0 + dst), "v"(voff), "s"(rsrc) : "memory", "m0");
  };
#pragma clang diagnostic pop
  // POOL: this thread's 8 channels of a 2 x 2 block of the tile's positions
  const PoolBlock block = pool_block(tid, TM, g.OW, [&](uint32_t n) { return fastdiv(n, g.OW, g.mg_ow); });
  v4i_t wd[4];                 // the windows above left, above, left and its own: their gradients
  v2i_t wa[4];                 // and winners
  auto request_windows = [&](int t) {
    const uint32_t gr = fastdiv((uint32_t)t * MT, g.OW, g.mg_ow) + 2 * block.row;      // (a tile begins with an even row)
    const int n = (int)fastdiv(gr, g.OH, g.mg_oh), a = (int)(gr - (uint32_t)n * g.OH) >> 1;
    const bool mine = tid < TM * MT && block.chunk * 8 < g.Ncols && gr < out_rows;
#pragma unroll
    for (int w = 0; w < 4; w++) {
      const int oh = a - 1 + (w >> 1), ow = block.col - 1 + (w & 1);
      const bool ok = mine && (unsigned)oh < (unsigned)h.PH && (unsigned)ow < (unsigned)h.PWo;
      const int o = ((n * h.PH + oh) * h.PWo + ow) * g.Ncols + block.chunk * 8;
      wd[w] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_pooled, ok ? o * 2 : (int)kOutOfRange, 0, 0);
      wa[w] = __builtin_amdgcn_raw_buffer_load_b64(rsrc_arg, ok ? o : (int)kOutOfRange, 0, 0);
    }
  };
  const bool early = wave >= 4;
  // the same sums in the same order as pool_bwd_3x3s2_kernel
  auto spread_windows = [&](int buf) {
    if (tid >= TM * MT) return;
    char* to = lds + buf + ((block.chunk >> 2) * MT + block.first) * 64 + (block.chunk & 3) * 16;
    // (255, a window that passes nothing on, becomes 15: no place either, and no borrow below)
#pragma unroll
    for (int w = 0; w < 4; w++) wa[w] &= 0x0f0f0f0f;
    // channels 2 c and 2 c + 1 of window w where their winner is `place`, else zeros: the top bit of each byte that is equal to it,
    // spread over 16 bits
    auto passed = [&](int w, int place, uint32_t (&two)[4]) {
#pragma unroll
      for (int i = 0; i < 2; i++) {
        const uint32_t eq = 0x80808080u - ((uint32_t)wa[w][i] ^ (0x01010101u * place));
        two[2 * i] = __builtin_amdgcn_perm(eq << 8, eq, 0x08080a0au) & (uint32_t)wd[w][2 * i];
        two[2 * i + 1] = __builtin_amdgcn_perm(eq << 8, eq, 0x09090b0bu) & (uint32_t)wd[w][2 * i + 1];
      }
    };
    uint32_t own[4], left[4], above[4], corner[4];
    auto put = [&](int q, const uint32_t (&v)[4]) {
      *reinterpret_cast<uint4*>(to + ((q >> 1) * g.OW + (q & 1)) * 64) = make_uint4(v[0], v[1], v[2], v[3]);
    };
    auto lo = [](uint32_t p) { return __uint_as_float(p << 16); };
    auto hi = [](uint32_t p) { return __uint_as_float(p & 0xffff0000u); };
    passed(3, 4, own);
    put(3, own);
    passed(2, 5, left);
    passed(3, 3, own);
#pragma unroll
    for (int c = 0; c < 4; c++) own[c] = pack2bf(lo(left[c]) + lo(own[c]), hi(left[c]) + hi(own[c]));
    put(2, own);
    passed(1, 7, above);
    passed(3, 1, own);
#pragma unroll
    for (int c = 0; c < 4; c++) own[c] = pack2bf(lo(above[c]) + lo(own[c]), hi(above[c]) + hi(own[c]));
    put(1, own);
    passed(0, 8, corner);
    passed(1, 6, above);
    passed(2, 2, left);
    passed(3, 0, own);
#pragma unroll
    for (int c = 0; c < 4; c++)
      own[c] = pack2bf(lo(corner[c]) + lo(above[c]) + lo(left[c]) + lo(own[c]), hi(corner[c]) + hi(above[c]) + hi(left[c]) + hi(own[c]));
    put(0, own);
  };
  auto request = [&](int t, int buf) {
    const int m0 = t * MT, m_last = min(m0 + MT, g.M) - 1;
#pragma unroll
    for (int i = 0; i < (POOL ? 0 : TM * MT / 128); i++) {      // dy: [32-channel panel][position][64 bytes]
      const int s = i * NT + tid, panel = s / (MT * 4), row = (s / 4) % MT, n = panel * 32 + (s & 3) * 8;
      dma(rsrc_dy, (uint32_t)(buf + (i * NT + wave * 64) * 16), n < g.Ncols ? ((m0 + row) * g.Ncols + n) * 2 : (int)kOutOfRange);
    }
    // patch rows: the first image's output rows of the tile and their halo, then whole images
    const int gr_lo = (int)fastdiv((uint32_t)m0, g.OW, g.mg_ow), gr_hi = (int)fastdiv((uint32_t)m_last, g.OW, g.mg_ow);
    const int n_lo = (int)fastdiv((uint32_t)gr_lo, g.OH, g.mg_oh), n_hi = (int)fastdiv((uint32_t)gr_hi, g.OH, g.mg_oh);
    const int oh_lo = gr_lo - n_lo * g.OH, first = min(g.OH - oh_lo, gr_hi - gr_lo + 1) + ks - 1;
    const int n_slots = (gr_hi - gr_lo + 1 + (ks - 1) * (n_hi - n_lo + 1)) * PW * g.CPT;
#pragma unroll 1
    for (int s0 = wave * 64; s0 < n_slots; s0 += NT) {
      const int s = s0 + lane, px = h.by_cpt(s), sub = s - px * g.CPT, pr = h.by_pw(px), pc = px - pr * PW;
      const int q = pr - first, nb = q < 0 ? 0 : h.by_band(q);
      const int n = q < 0 ? n_lo : n_lo + 1 + nb, ih = (q < 0 ? oh_lo + pr : q - nb * (g.OH + ks - 1)) - g.pad, iw = pc - g.pad;
      const bool ok = s < n_slots && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
      dma(rsrc_x, (uint32_t)(buf + DY + s0 * 16), ok ? (((n * g.H + ih) * g.W + iw) * g.C + sub * 8) * 2 : (int)kOutOfRange);
    }
    // each position's place in the patch; positions behind M repeat the last one, their dy is zero
    static_assert(MT <= NT, "a position a thread");
    if (tid < MT) {
      const uint32_t m = (uint32_t)min(m0 + tid, m_last);
      const uint32_t gr = fastdiv(m, g.OW, g.mg_ow), ow = m - gr * (uint32_t)g.OW, n = fastdiv(gr, g.OH, g.mg_oh);
      const int pr = ((int)gr - gr_lo) + (ks - 1) * ((int)n - n_lo);
      reinterpret_cast<int*>(lds + buf + DY + h.patch)[tid] = (pr * PW + (int)ow) * g.C * 2;
    }
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  auto read_tr = [&](const char* p0, const char* p1) {
    union { bf16x8 v; shortx4 q[2]; } u;
    u.q[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p0));
    u.q[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p1));
    return u.v;
  };
  const int row = 8 * (lane >> 5) + (j16 >> 2), dy_lane = row * 64 + 32 * ((lane >> 4) & 1) + 8 * (j16 & 3);
  const int t_begin = sp * h.per, t_end = min(h.tiles, t_begin + h.per);
  int buf = 0;
  if (t_begin < t_end) {
    request(t_begin, 0);
    if constexpr (POOL) {
      request_windows(t_begin);
      spread_windows(0);
      request_windows(t_begin + 1);
    }
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll 1
  for (int t = t_begin; t < t_end; t++) {
    if (t + 1 < t_end) {
      if constexpr (POOL)
        if (early) spread_windows(h.buf - buf);    // (before the next loads: the compiler would wait for those too)
      request(t + 1, h.buf - buf);
      if constexpr (POOL)
        if (early) request_windows(t + 2);
    }
    const char* D = lds + buf;
    const char* X = D + DY;
    const int* place = reinterpret_cast<const int*>(X + h.patch);
    // a step's operands are read between the products of the step before, its positions' places a step earlier still
    bf16x8 a0[TM], b0[TN], a1[TM], b1[TN];
    int at0[2], at1[2];
    auto places = [&](int (&at)[2], int st) {
      const int k = min(wk + WK * st, MT / 16 - 1);        // behind the last step: read, not used
      at[0] = place[16 * k + row];
      at[1] = place[16 * k + row + 4];
    };
    auto operands = [&](bf16x8 (&a)[TM], bf16x8 (&b)[TN], const int (&at)[2], int st) {
      const int k = min(wk + WK * st, MT / 16 - 1);
#pragma unroll
      for (int i = 0; i < TM; i++) a[i] = read_tr(D + (i * MT + 16 * k) * 64 + dy_lane, D + (i * MT + 16 * k + 4) * 64 + dy_lane);
#pragma unroll
      for (int j = 0; j < TN; j++) b[j] = read_tr(X + at[0] + off[j], X + at[1] + off[j]);
    };
    auto multiply = [&](const bf16x8 (&a)[TM], const bf16x8 (&b)[TN]) {
#pragma unroll
      for (int j = 0; j < TN; j++) {
        bf16x8 bj = b[j];
        if (j == TN - 1 && bias) bj = ones;
#pragma unroll
        for (int i = 0; i < TM; i++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], bj, acc[i][j], 0, 0, 0);
      }
    };
    auto interleave = [&]() {
#pragma unroll
      for (int q = 0; q < TM * TN; q++) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, TM == 1 ? 3 : 2, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int kSteps = MT / 16 / WK;
    static_assert(kSteps % 2 == 0, "two steps a turn");
    places(at0, 0);
    places(at1, 1);
    operands(a0, b0, at0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
    for (int st = 0; st < kSteps; st += 2) {
      operands(a1, b1, at1, st + 1);
      places(at0, st + 2);
      multiply(a0, b0);
      interleave();
      operands(a0, b0, at0, st + 2);
      places(at1, st + 3);
      multiply(a1, b1);
      interleave();
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (POOL)
      if (!early && t + 1 < t_end) {
        spread_windows(h.buf - buf);
        request_windows(t + 2);                    // on their way across the barrier
      }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the next tile is there, this one read
    buf = h.buf - buf;
  }

  // the position groups' sums, block by block, in group order
  const int ldk = kcols + 8;
  float* part = reinterpret_cast<float*>((char*)ws.p[z] + g.scratch_off) + (int64_t)sp * g.Ncols * ldk;
  float* red = reinterpret_cast<float*>(lds);                // [wavefront][1024]
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) {
#pragma unroll
      for (int r = 0; r < 16; r++) red[wave * 1024 + r * 64 + lane] = acc[i][j][r];
      __syncthreads();
#pragma unroll
      for (int e = tid; e < WN * 1024; e += NT) {
        float v = red[e];
#pragma unroll
        for (int w = 1; w < WK; w++) v += red[w * WN * 1024 + e];
        const int c = e / 1024, r = (e / 64) % 16, l = e % 64;
        const int n = 32 * i + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
        int kc = ((cg * WN + c) * TN + j) * 32 + (l & 31);
        const bool last = last_group && c == WN - 1 && j == TN - 1;
        if (last) kc = (l & 31) == 0 ? kcols : kcols + 1;
        if (n < g.Ncols && (last ? kc == kcols : kc < kcols)) part[(int64_t)n * ldk + kc] = v;
      }
      __syncthreads();
    }
}

// Row length of a second pass's sums in LDS, per tap: whole float4s and an odd number of them, so that the taps of a channel,
// which the write to the flat gradient takes one after the other, lie in different banks.
__host__ __device__ inline int wgrad_finish_ld(int cw) { return 4 * (((cw + 3) >> 2) | 1); }

// Second pass of the weight gradient.  One workgroup per output channel n and group of input channels: the partial sums are
// added in split order into LDS (four columns a lane, up to eight reads in flight), then written to the flat gradient in ITS
// order (coalesced).
// What bounds it: HBM, the sums read once and the gradient written once.  AlexNet-shaped net, 288 images of 18 learners, average
// of its five layers: 22 us against 31 us with one column a lane, one read after the other below eight splits, and the taps of
// a channel in one LDS bank.
__global__ __launch_bounds__(256) void wgrad_finish_kernel(PtrTab ws, PtrTab grads, IGemm g, VConv v, int64_t w_off, int64_t b_off,
                                                           int cgroup) {
  extern __shared__ __attribute__((aligned(16))) float row[];   // sums of this workgroup's columns
  const int z = blockIdx.z, n = blockIdx.x;
  const int kcols = g.Kchunks * 8, ldk = kcols + 8;
  const float* part = reinterpret_cast<const float*>((const char*)ws.p[z] + g.scratch_off) + (int64_t)n * ldk;
  const int64_t split_stride = (int64_t)g.Ncols * ldk;
  float* dw = (float*)grads.p[z] + w_off + (int64_t)n * v.Creal * v.ksr * v.ksr;
  // channels [c_lo, c_hi) of this filter, all taps: columns tap * C + c are read tap by tap (contiguous runs), the
  // run [c_lo * T, c_hi * T) of the flat gradient is written in its own order.  The bias gradient, the extra im2col
  // column, is one more read of the first group.
  const int T = v.ks * v.ks;
  const int c_lo = blockIdx.y * cgroup, c_hi = min(v.Creal, c_lo + cgroup), cw = c_hi - c_lo;
  if (cw <= 0) return;
  const int cw4 = (cw + 3) >> 2, ld = wgrad_finish_ld(cw);
  const int units = T * cw4, all = units + (blockIdx.y == 0 ? 1 : 0);
  for (int u0 = threadIdx.x; u0 < all; u0 += 2 * 256) {
    const float* src[2];
    int dst[2];
    float4 acc[2];
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int u = min(u0 + 256 * q, all - 1);
      const int tap = u / cw4, cc = 4 * (u - tap * cw4);
      dst[q] = u0 + 256 * q >= all ? -2 : u == units ? -1 : tap * ld + cc;
      src[q] = part + (u == units ? kcols : tap * g.C + c_lo + cc);
      acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int sp = 0; sp < g.splits; sp += 4) {
      float4 p[4][2];
#pragma unroll
      for (int t = 0; t < 4; t++)
#pragma unroll
        for (int q = 0; q < 2; q++)
          if (sp + t < g.splits) p[t][q] = *reinterpret_cast<const float4*>(src[q] + (sp + t) * split_stride);
#pragma unroll
      for (int t = 0; t < 4; t++)
        if (sp + t < g.splits)
#pragma unroll
          for (int q = 0; q < 2; q++) {
            acc[q].x += p[t][q].x;
            acc[q].y += p[t][q].y;
            acc[q].z += p[t][q].z;
            acc[q].w += p[t][q].w;
          }
    }
#pragma unroll
    for (int q = 0; q < 2; q++) {
      if (dst[q] >= 0) *reinterpret_cast<float4*>(row + dst[q]) = acc[q];
      else if (dst[q] == -1) ((float*)grads.p[z] + b_off)[n] = acc[q].x;
    }
  }
  __syncthreads();
  int cc = threadIdx.x / T, tap = threadIdx.x - cc * T;
  const int dc = 256 / T, dt = 256 - dc * T;
  for (int j = threadIdx.x; j < T * cw; j += 256) {
    dw[(int64_t)c_lo * T + j] = row[tap * ld + cc];
    cc += dc;
    tap += dt;
    if (tap >= T) { tap -= T; cc++; }
  }
}

// The same where there are many splits and few columns, for a first layer seen through a space-to-depth input, and for a window
// too large for the sums in LDS: a lane adds four im2col columns of every W-th split, the W wavefronts' sums are added through
// LDS, and each column's place in the flat filter is looked up and written on its own.  blockIdx.y selects a run of 256
// columns.  Of 818 layers of random networks and the AlexNet-shaped one with 1 to 256 splits, sixteen wavefronts were the faster ones
// nowhere, at 64 and more splits level (5 us), and below 16 splits up to three times as slow, most of them with nothing to add
// (344 filters of 576 columns, 29 learners, 3 splits: 92 us, 33 with four); at 503 splits 7 us, 11 with four.
template <int W>
__global__ __launch_bounds__(64 * W) void wgrad_columns_kernel(PtrTab ws, PtrTab grads, IGemm g, VConv v, int64_t w_off, int64_t b_off) {
  static_assert(W >= 4, "a thread a column");
  __shared__ float4 sums[W][64];
  const int z = blockIdx.z, n = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kcols = g.Kchunks * 8, ldk = kcols + 8, k = blockIdx.y * 256 + 4 * lane;
  const float* part = reinterpret_cast<const float*>((const char*)ws.p[z] + g.scratch_off) + (int64_t)n * ldk;
  const int64_t split_stride = (int64_t)g.Ncols * ldk;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (k < ldk) {                                          // column kcols is the bias gradient, the row's rest padding
#pragma unroll 8
    for (int sp = wave; sp < g.splits; sp += W) {
      const float4 p = *reinterpret_cast<const float4*>(part + sp * split_stride + k);
      acc.x += p.x; acc.y += p.y; acc.z += p.z; acc.w += p.w;
    }
  }
  sums[wave][lane] = acc;
  __syncthreads();
  const int col = blockIdx.y * 256 + threadIdx.x;
  if (threadIdx.x >= 256 || col > kcols) return;
  const float* f = reinterpret_cast<const float*>(sums) + threadIdx.x;
  float total = f[0];
#pragma unroll
  for (int w = 1; w < W; w++) total += f[w * 256];
  if (col == kcols) {
    ((float*)grads.p[z] + b_off)[n] = total;
    return;
  }
  const int tap = col / g.C, cp = col - tap * g.C;
  const int64_t dst = filter_src(v, 0, tap, cp);          // position inside one filter, or -1 for padding
  if (dst >= 0) ((float*)grads.p[z] + w_off + (int64_t)n * v.Creal * v.ksr * v.ksr)[dst] = total;
}

template <int F>
static void launch_strip_t(const PtrTab& ws, const IGemm& g, size_t dy_off, const StripPlan& p, const PooledDy* pooled, int count, hipStream_t s) {
  constexpr StripForm f = kStripForms[F];
  StripArgs h;
  h.PW = p.PW;
  h.tiles = p.tiles;
  h.per = p.per;
  h.patch = p.patch;
  h.buf = p.buf;
  h.by_pw.set(p.PW);
  h.by_cpt.set(g.CPT);
  h.by_band.set(g.OH + g.ks - 1);
  h.PH = pooled ? pooled->OH : 0;
  h.PWo = pooled ? pooled->OW : 0;
  h.arg_off = pooled ? pooled->arg_off : 0;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(1, (unsigned)p.groups, (unsigned)(count * p.splits)), dim3(512), p.lds, s, ws, g, dy_off, h);
  };
  pooled ? go(wgrad_strip_kernel<f.TM, f.WN, f.TN, f.MT, true>) : go(wgrad_strip_kernel<f.TM, f.WN, f.TN, f.MT, false>);
}

bool wgrad_takes_pooled(const IGemm& g, const VConv& v, const PoolShape& ps, size_t scratch_bytes, int count) {
  StripPlan p;
  return (v.ks > 1 || v.s2d > 1) && ps.ks == 3 && ps.stride == 2 && ps.H == g.OH && ps.W == g.OW &&
         strip_plan(StripLayer{g.M, g.Ncols, g.C, g.ks, g.OH, g.OW, g.W, g.pad, count, scratch_bytes}, &p) && strip_pools(p, g.OH, g.OW);
}

hipError_t launch_igemm_wgrad(const PtrTab& ws, const PtrTab& grads, const IGemm& g_in, const VConv& v, size_t dy_off, int64_t w_off,
                              int64_t b_off, size_t scratch_bytes, const PooledDy* pooled, int count, hipStream_t s) {
  IGemm g = g_in;
  if (g.C % 8 || g.Ncols % 8) return hipErrorInvalidValue;
  const int cols = g.Kchunks * 8 + 1;          // im2col columns plus the bias column
  const bool incr = BK / g.OW + 1 <= g.OH;      // one wrap of oh per step at most
  // A convolution's tile holds one tap of many channels, the flat gradient wants all taps of one channel together:
  // written straight from the tile every 4-byte element lands alone and every cache line is completed by as many
  // workgroups as the window has taps (measured: 65-125 us per AlexNet layer at 18 learners).  So convolutions
  // always go through the partial buffer and the second pass, which reads and writes whole lines (28-51 us).
  const bool conv = v.ks > 1 || v.s2d > 1;
  // the constant block has to lie within a 31-bit byte offset from the layer's input
  const bool near = g.zero_off >= g.a_off && (g.zero_off - g.a_off + 256) * 2 < ((size_t)1 << 31);
  WgradTile shape = WgradTile::k128x128;
  if (conv && g.Ncols > 64 && near) {
    const WgradTiles t = wgrad_tiles(WgradProduct{g.M, g.Ncols, cols, count, scratch_bytes}, incr);
    shape = t.tile;
    g.splits = t.splits;
  } else {
    // narrow layers run small tiles (24-32 KiB of LDS, few registers): six and more workgroups fit a compute
    // unit and each one alone is latency-bound, so they want more of them
    // (CIFAR-shaped layers, 18 learners x 128 images: 1200 workgroups against 600 take conv1 from 148 to 97 us and
    // conv2 from 112 to 80 us; 900 and 1500 are slower again)
    const int64_t tiles = (int64_t)((g.Ncols + 127) / 128) * ((cols + 127) / 128);
    g.splits = choose_splits(tiles, count, (g.M + 31) / 32, (size_t)g.Ncols * (g.Kchunks * 8 + 8) * 4, scratch_bytes, g.Ncols <= 64 ? 1200 : 600);
  }
  const int partial = (g.splits > 1 || conv) ? 1 : 0;
  StripPlan strip;
  const bool done = conv && strip_plan(StripLayer{g.M, g.Ncols, g.C, g.ks, g.OH, g.OW, g.W, g.pad, count, scratch_bytes}, &strip);
  if (pooled && !done) return hipErrorInvalidValue;
  if (done) {
    g.splits = strip.splits;
    switch (strip.form) {
      case 0: launch_strip_t<0>(ws, g, dy_off, strip, pooled, count, s); break;
      case 1: launch_strip_t<1>(ws, g, dy_off, strip, pooled, count, s); break;
      case 2: launch_strip_t<2>(ws, g, dy_off, strip, pooled, count, s); break;
      case 3: launch_strip_t<3>(ws, g, dy_off, strip, pooled, count, s); break;
      default: launch_strip_t<4>(ws, g, dy_off, strip, pooled, count, s); break;
    }
  }
#define SASGD_WGRAD(BMG, BNG, WMG, WNG)                                                                                          \
  do {                                                                                                                           \
    if (incr) hipLaunchKernelGGL((igemm_wgrad_kernel<BMG, BNG, WMG, WNG, true>), grid, dim3(256), 0, s, ws, grads, g, v, dy_off, w_off, b_off, partial); \
    else hipLaunchKernelGGL((igemm_wgrad_kernel<BMG, BNG, WMG, WNG, false>), grid, dim3(256), 0, s, ws, grads, g, v, dy_off, w_off, b_off, partial);    \
  } while (0)
  auto grid_of = [&](int rows, int columns) {
    return dim3((unsigned)((g.Ncols + rows - 1) / rows), (unsigned)((cols + columns - 1) / columns), (unsigned)(count * g.splits));
  };
  if (done) {
  } else if (g.Ncols <= 32) {
    const dim3 grid = grid_of(32, 128);
    SASGD_WGRAD(32, 128, 32, 32);
  } else if (g.Ncols <= 64) {
    const dim3 grid = grid_of(64, 128);
    SASGD_WGRAD(64, 128, 32, 64);
  } else if (shape == WgradTile::k96x512) {
    hipLaunchKernelGGL((wgrad_wide_kernel<3, 1>), grid_of(96, 512), dim3(256), 0, s, ws, grads, g, v, dy_off, w_off, b_off);
  } else if (shape == WgradTile::k256x256) {
    hipLaunchKernelGGL((wgrad_wide_kernel<4, 2>), grid_of(256, 256), dim3(256), 0, s, ws, grads, g, v, dy_off, w_off, b_off);
  } else if (shape == WgradTile::k384x128) {
    hipLaunchKernelGGL((wgrad_wide_kernel<3, 4>), grid_of(384, 128), dim3(256), 0, s, ws, grads, g, v, dy_off, w_off, b_off);
  } else {
    const dim3 grid = grid_of(128, 128);
    if (near) {
      if (incr) hipLaunchKernelGGL((wgrad_panel_kernel<true>), grid, dim3(256), 0, s, ws, grads, g, v, dy_off, w_off, b_off, partial);
      else hipLaunchKernelGGL((wgrad_panel_kernel<false>), grid, dim3(256), 0, s, ws, grads, g, v, dy_off, w_off, b_off, partial);
    } else {
      SASGD_WGRAD(128, 128, 64, 64);
    }
  }
#undef SASGD_WGRAD
  if (partial) {
    const int cap = (15360 / (v.ks * v.ks) - 4) & ~3;    // input channels whose sums fit 60 KiB of LDS
    // (few columns, at most 256 K values over all learners: the kernel below 7 / 10 / 14 us at 16 / 32 / 64 and more splits, this one 5 / 5 / 5)
    if (v.s2d > 1 || cap < 4 || (g.splits >= 16 && (int64_t)g.Ncols * count * cols <= 256 * 1024)) {
      const dim3 grid((unsigned)g.Ncols, (unsigned)((cols + 255) / 256), (unsigned)count);
      if (g.splits > 256) hipLaunchKernelGGL(wgrad_columns_kernel<16>, grid, dim3(1024), 0, s, ws, grads, g, v, w_off, b_off);
      else hipLaunchKernelGGL(wgrad_columns_kernel<4>, grid, dim3(256), 0, s, ws, grads, g, v, w_off, b_off);
      return hipGetLastError();
    }
    // enough workgroups to keep the chip busy: the channels of a filter are divided among several of them
    int groups = (int)((1536 + (int64_t)g.Ncols * count - 1) / ((int64_t)g.Ncols * count));
    if (groups > v.Creal / 8) groups = v.Creal / 8;
    if (groups < 1) groups = 1;
    int cgroup = ((v.Creal + groups - 1) / groups + 3) & ~3;            // channels are read four at a time
    if (cgroup > cap) cgroup = cap;
    groups = (v.Creal + cgroup - 1) / cgroup;
    const size_t lds = (size_t)wgrad_finish_ld(cgroup) * v.ks * v.ks * sizeof(float);
    hipLaunchKernelGGL(wgrad_finish_kernel, dim3((unsigned)g.Ncols, (unsigned)groups, (unsigned)count), dim3(256), lds, s, ws, grads, g, v,
                       w_off, b_off, cgroup);
  }
  return hipGetLastError();
}

}  // namespace sasgd
