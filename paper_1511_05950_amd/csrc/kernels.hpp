// Launch wrappers of the calcGradient kernels (Section 2.1 learner step; layer types of Section 4.1).
// Every launch covers `count` learners at once: blockIdx.z (or .y) selects the learner, and per-learner
// base addresses come from small by-value tables.  Activations are NHWC ([image][h][w][channel]) of type
// T = float (fp32 compute) or bf16 bits (bf16 compute); parameters and parameter gradients use the flat
// order of the C ABI.
#pragma once
#include "ctx.hpp"
#include "fastdiv.hpp"
#include "tile_rules.hpp"

namespace sasgd {

struct PtrTab {
  void* p[kMaxLearners];
};
struct CPtrTab {
  const void* p[kMaxLearners];
};

struct ConvShape {
  int N;                 // images per learner (mu)
  int C, H, W;           // input
  int K, OH, OW;         // output channels and size
  int ks, stride, pad;   // square window
};

struct PoolShape {
  int N, C, H, W, OH, OW, ks, stride;
};

// Re-layout of the caller's images.  s2d == 1: NCHW fp32 -> NHWC with channels zero-padded to Cp.
// s2d == s > 1 (space to depth): out[n][Y][X][(dy*s+dx)*C + c] = in[n][c][s*Y+dy][s*X+dx], zero outside the
// image and in the padding channels; a stride-s convolution on the image is a stride-1 one on this tensor.
struct InPack {
  int C, H, W;      // source
  int Cp, Hp, Wp;   // destination
  int s2d;
};

// A convolution as the MFMA kernels see it (stride 1): C = effective (padded or space-to-depth) input
// channels, ks = effective window, K = output channels; Creal / ksr describe the flat filter [K][Creal][ksr][ksr].
struct VConv {
  int C, ks, K, s2d, Creal, ksr;
};

// Source index, in the flat [K][Creal][ksr][ksr] filter, of packed element (n, tap, cp) of a virtual
// stride-1 layer, or -1 for padding.  s2d > 1: the layer is a strided one seen through a
// space-to-depth input: channel cp = (dy*s2d + dx)*Creal + c, tap = (KY, KX), kh = s2d*KY + dy.
__host__ __device__ inline int64_t filter_src(const VConv& v, int n, int tap, int cp) {
  int kh, kw, c;
  if (v.s2d == 1) {
    if (cp >= v.Creal) return -1;
    c = cp; kh = tap / v.ks; kw = tap % v.ks;
  } else {
    int g = cp / v.Creal;
    c = cp % v.Creal;
    if (g >= v.s2d * v.s2d) return -1;
    kh = v.s2d * (tap / v.ks) + g / v.s2d;
    kw = v.s2d * (tap % v.ks) + g % v.s2d;
    if (kh >= v.ksr || kw >= v.ksr) return -1;
  }
  return (((int64_t)n * v.Creal + c) * v.ksr + kh) * v.ksr + kw;
}

// One implicit GEMM: D[m][n] = sum_k im2col(t)[m][k] * B(n, k).  t = NHWC tensor [*][H][W][C] at a_off (elements
// of bf16 from the workspace base), output positions OH x OW, window ks, zero padding pad, stride 1.
struct IGemm {
  size_t a_off;
  int64_t b_off;            // elements of bf16 from the learner's weight-version base
  int M, Ncols;             // M = images * OH * OW
  int H, W, C, OH, OW, ks, pad;
  int Kchunks, CPT;         // ks*ks*C/8 and C/8
  int ldb;                  // row length of B in elements
  // Split of the contraction over `splits` workgroups per tile (fills the chip when there are few tiles):
  // each writes an fp32 partial tile to scratch (byte offset from the workspace base), a second kernel adds
  // them in split order and applies the epilogue, so the result does not depend on scheduling.
  int splits;
  size_t scratch_off;
  // multipliers for division by CPT, ks, OW, OH without a divide (set by igemm_set_magics)
  uint32_t mg_cpt, mg_ks, mg_ow, mg_oh;
  // 256 bytes of zeros inside the workspace (elements of bf16 from its base): the address out-of-range chunk
  // loads are redirected to, so that no load is conditional and no loaded value needs patching
  size_t zero_off;
  // byte sizes of the gathered tensor (one learner) and of the fragment-packed B, for hardware-bounds-checked
  // buffer loads (both below 2 GiB)
  uint32_t a_bytes, b_bytes;
};

// The multipliers are FastDiv's, with its limits; d == 1 is handled apart.
inline uint32_t magic_u32(int d) {
  FastDiv f;
  f.set(d);
  return f.m;
}
// Are all of an implicit GEMM's divisions exact?  Rows go up to M, contraction chunks up to Kchunks.  Not so e.g. for 33 images of
// 512 x 512, or a fully connected layer of 307 200 inputs in fp32: such layers stay on the direct kernels.
inline bool igemm_divides(const IGemm& g) {
  return FastDiv::exact(g.OW, g.M - 1) && FastDiv::exact(g.OH, g.M / g.OW - 1) && FastDiv::exact(g.CPT, g.Kchunks - 1) &&
         FastDiv::exact(g.ks, g.ks * g.ks - 1);
}
inline void igemm_set_magics(IGemm& g, int elem_bytes) {
  if (g.OH > 0 && g.OW > 0) g.a_bytes = (uint32_t)((int64_t)(g.M / (g.OH * g.OW)) * g.H * g.W * g.C * elem_bytes);
  g.b_bytes = (uint32_t)((int64_t)((g.Ncols + 31) & ~31) * g.ldb * 2);
  g.mg_cpt = magic_u32(g.CPT);
  g.mg_ks = magic_u32(g.ks);
  g.mg_ow = magic_u32(g.OW);
  g.mg_oh = magic_u32(g.OH);
}

struct Epilogue {
  size_t out_off, mask_off; // elements of bf16 from the workspace base
  int64_t bias_off;         // elements of bf16 from the weight-version base
  int has_bias, relu, use_mask, out_f32;
};

// is_bf16 selects T.  All offsets are in elements of T from the learner's workspace base, except where noted.
hipError_t launch_pack_input(bool is_bf16, const CPtrTab& images, const PtrTab& ws, size_t out_off, int count, int N,
                             const InPack& ip, const float* mean, hipStream_t s);

// ---- bf16 MFMA path (conv_mfma.hip)
// One launch repacks the filters of every MFMA convolution of a weight version.
struct PackJob {
  VConv v;
  int64_t w_off, fwd_off, bwd_off;   // flat source, fragment destinations (elements)
  int64_t start;                     // first global element index of this layer in the launch
  int Kp, Kpt;                       // padded row lengths; Kpt == 0: no transposed copy
};
constexpr int kMaxPackJobs = 24;
struct PackTable {
  PackJob job[kMaxPackJobs];
  int count;
  int64_t total;
};
// Several weight versions in one launch (blockIdx.y): flat bf16 vector and packed-filter region of each.
constexpr int kMaxPackVersions = 32;
struct PackVersions {
  const void* flat[kMaxPackVersions];
  void* packed[kMaxPackVersions];
};
hipError_t launch_pack_filters(const PackVersions& pv, int versions, const PackTable& t, hipStream_t s);
// ---- fp32 MFMA path (conv_mfma_f32.hip); dgrad: g gathers over dy, the filter is read transposed and flipped
hipError_t launch_igemm_f32(const PtrTab& ws, const CPtrTab& wts, const IGemm& g, const VConv& v, const Epilogue& ep, int64_t w_off,
                            bool dgrad, int count, hipStream_t s);
hipError_t launch_igemm_wgrad_f32(const PtrTab& ws, const PtrTab& grads, const IGemm& g, const VConv& v, size_t dy_off, int64_t w_off,
                                  int64_t b_off, int count, hipStream_t s);
// The first convolution and the 3 x 3 / 2 max pooling behind it in one launch (conv_pool.hip): the convolution's output is not stored.
// y_off / arg_off: the pooled tensor (elements) and its winners (bytes), which mark dead windows where ep.relu is set.
bool conv_pool_ok(const IGemm& g, const PoolShape& ps);
hipError_t launch_conv_pool(const PtrTab& ws, const CPtrTab& wts, const IGemm& g, const Epilogue& ep, const PoolShape& ps, size_t y_off, size_t arg_off,
                            bool pool_relu, int count, hipStream_t s);
hipError_t launch_igemm_frag(const PtrTab& ws, const CPtrTab& wts, const IGemm& g, const Epilogue& ep, int count, hipStream_t s);
// dW and db of one layer (the bias gradient rides along as one extra im2col column of ones).  pooled: dy_off is the gradient of the 3 x 3 / 2 max
// pooling's output behind the layer, whose winners are here; only where wgrad_takes_pooled() says so.
struct PooledDy {
  int OH, OW;
  size_t arg_off;    // bytes
};
bool wgrad_takes_pooled(const IGemm& g, const VConv& v, const PoolShape& ps, size_t scratch_bytes, int count);
hipError_t launch_igemm_wgrad(const PtrTab& ws, const PtrTab& grads, const IGemm& g, const VConv& v, size_t dy_off, int64_t w_off,
                              int64_t b_off, size_t scratch_bytes, const PooledDy* pooled, int count, hipStream_t s);

// y = conv(x, w) + b, optional ReLU.  w_off / b_off: element offsets into the learner's flat weight vector.
// out_f32: y is stored as fp32 whatever T is (class scores).
hipError_t launch_conv_fwd_simple(bool is_bf16, const PtrTab& ws, const CPtrTab& wts, size_t x_off, size_t y_off, int64_t w_off,
                                  int64_t b_off, const ConvShape& sh, bool relu, bool out_f32, int count, hipStream_t s);
// dx = conv^T(dy, w), optionally zeroed where mask (the forward tensor at mask_off) <= 0.
hipError_t launch_conv_dgrad_simple(bool is_bf16, const PtrTab& ws, const CPtrTab& wts, size_t dy_off, size_t dx_off, int64_t w_off,
                                    const ConvShape& sh, bool use_mask, size_t mask_off, int count, hipStream_t s);
// dW, db into the learner's fp32 gradient vector at w_off / b_off.
hipError_t launch_conv_wgrad_simple(bool is_bf16, const PtrTab& ws, const PtrTab& grads, size_t x_off, size_t dy_off, int64_t w_off,
                                    int64_t b_off, const ConvShape& sh, int count, hipStream_t s);

// input_relu: the input holds ReLU outputs (max: the winners then keep which windows no gradient passes, and the backward
// pass of a max pooling ignores use_mask).
hipError_t launch_pool_fwd(bool is_bf16, bool is_max, const PtrTab& ws, size_t x_off, size_t y_off, size_t arg_byte_off,
                           const PoolShape& sh, bool relu, bool input_relu, int count, hipStream_t s);
hipError_t launch_pool_bwd(bool is_bf16, bool is_max, const PtrTab& ws, size_t dy_off, size_t dx_off, size_t arg_byte_off,
                           const PoolShape& sh, bool use_mask, size_t mask_off, int count, hipStream_t s);

// NHWC [N][H][W][C] <-> [N][C*H*W] (C,H,W order), the flattening the fully connected weights expect.
hipError_t launch_flatten_fwd(bool is_bf16, const PtrTab& ws, size_t x_off, size_t y_off, int N, int C, int H, int W, int count,
                              hipStream_t s);
hipError_t launch_flatten_bwd(bool is_bf16, const PtrTab& ws, size_t dy_off, size_t dx_off, int N, int C, int H, int W, bool use_mask,
                              size_t mask_off, int count, hipStream_t s);

// loss[l] = mean_n -log softmax(z_n)[label_n];  dz = (softmax(z) - onehot) / N.  loss_out may be null.
// z_f32: the scores at z_off (an offset in elements of T) are fp32; dz is always of type T.
// loss_byte_off: N floats of per-image losses in the workspace (bytes from its base).
hipError_t launch_softmax_ce(bool is_bf16, bool z_f32, const PtrTab& ws, const CPtrTab& labels, size_t z_off, size_t dz_off,
                             size_t loss_byte_off, int N, int K, float* loss_out, int count, hipStream_t s);
// loss_out[l] = mean of learner l's per-image losses
hipError_t launch_loss_mean(const PtrTab& ws, size_t loss_byte_off, int N, float* loss_out, int count, hipStream_t s);
hipError_t launch_label_rank(bool is_bf16, bool z_f32, const PtrTab& ws, const CPtrTab& labels, size_t z_off, int N, int K,
                             int32_t* rank_out, int count, hipStream_t s);
// ---- fully connected layers over all rows of a weight version (fc_rows.hip)
// Version k = members first[k] .. first[k] + members[k] - 1 of the pointer tables handed to the launch.
struct alignas(4) GroupTab {
  uint8_t first[kMaxLearners];
  uint8_t members[kMaxLearners];
};
// A layer of `in` inputs is within reach of the kernels' 32-bit offsets.
inline bool fc_rows_layer_ok(int in) { return in < 1 << 23; }
// y = x W^T + b (optional ReLU, optional fp32 output), or dx = dy W (optionally zeroed where the forward tensor at ep.mask_off is
// <= 0), for every version of the table; g = the layer's product for ONE learner (M = mu).  scratch_off / scratch_bytes: the
// split-partial area of a workspace (a version's first member's is used).
hipError_t launch_fc_rows(const PtrTab& ws, const CPtrTab& wts, const GroupTab& gt, int groups, const IGemm& g, const Epilogue& ep, bool dgrad,
                          size_t scratch_off, size_t scratch_bytes, hipStream_t s);

hipError_t launch_fc_save_factors(const PtrTab& ws, const PtrTab& grads, size_t x_off, size_t dy_off, size_t fx_off, size_t fdy_off,
                                  int64_t b_off, int N, int in, int out, int NP, int count, hipStream_t s);

// ---- small networks and mini-batches in few launches (compact.hip)
// Where a layer's input comes from.
enum { CSRC_TENSOR = 0, CSRC_IMAGES = 1, CSRC_MAXPOOL = 2, CSRC_AVGPOOL = 3, CSRC_FLAT = 4 };
struct CompactSrc {
  int kind;
  int C, H, W;                 // the input as the layer sees it (behind the pooling)
  size_t off;                  // tensor that is read (elements)
  int YH, YW, pks, pst, relu;  // pooled sources: size of that tensor, window, stride, ReLU behind the pooling
  size_t out_off, arg_off;     // pooled sources: where the pooled tensor (elements) and its winners (bytes) are kept
  FastDiv by_c, by_c4;         // C and C / 4
};
// Gradient of a convolution's output: stored (masked), or behind the pooling layer that follows the convolution.
enum { CGRAD_PLAIN = 0, CGRAD_MAXPOOL = 1, CGRAD_AVGPOOL = 2 };
struct CompactGrad {
  int kind;
  int use_mask;                // pooled kinds: zero where the convolution's output (at mask_off) is not positive
  int OH, OW, K, PH, PW, pks, pst;
  size_t off, mask_off, arg_off;
  FastDiv by_k, by_k4, by_pst;
};
struct CompactConv {
  int N, C, H, W, K, OH, OW, ks, stride, pad;
  int64_t w_off, b_off;
  FastDiv by_ow, by_w, by_cols, by_dcols;   // OW, W, patch columns of the forward pass and of the input gradient
};
struct CompactBwd {
  int dgrad_blocks, col_groups, blocks_per_group, tile;   // set by the launcher
  int splits;
  size_t dx_off, mask_off;        // elements
  int use_mask;
  size_t part_off;                // bytes from the workspace base: `splits` partial gradients of part_elems floats, [K][ks ks C + 1]
  int64_t part_elems;
};
struct CompactHead {
  int N, in, K;
  int64_t w_off, b_off;
  size_t flat_off, dz_off, dx_off, loss_off;   // elements; loss_off bytes
  int use_mask;
  int C, HW;                   // the input in front of a flattening: channels, pixels (HW = 1, C = in: none)
  FastDiv by_hw;
};
struct CompactFc {
  int N, in, out, relu, use_mask;
  int HW;                      // pixels of the input in front of a flattening (1: none)
  int64_t w_off, b_off;
  size_t x_off, y_off, dy_off, dx_off;
  int splits, aligned;         // set by the launcher
  size_t part_off;             // bytes: partial tiles [splits][N][columns]
};
enum { CJOB_SUM = 0, CJOB_FC = 1, CJOB_LOSS = 2 };
struct CompactJob {
  int kind, first_block, splits, groups;
  int64_t elems, w_off;
  size_t part_off;
  int K, C, taps;
  int in, out;
  size_t x_off, dy_off;
};
constexpr int kMaxCompactJobs = 16;
struct CompactFinish {
  CompactJob job[kMaxCompactJobs];
  int count;
};
// Floats per pixel of an LDS patch: room for C rounded up to a multiple of four, and 4 (mod 8).
__host__ __device__ inline int compact_pixel_stride(int C) { return ((C + 3) & ~7) + 4; }
// Wavefronts of a weight-gradient workgroup side by side across its column blocks (a power of two).
__host__ __device__ inline int wgrad_waves_across(int blocks, int waves) {
  int w = 1;
  while (w < blocks && w < waves) w *= 2;
  return w;
}
bool compact_conv_ok(const CompactConv& v, bool need_dx);
bool compact_head_ok(int in, int K);
bool compact_fc_ok(int in, int out);
int compact_splits(const CompactConv& v, bool need_dx, int count, int most);
hipError_t launch_compact_fwd(bool is_bf16, const PtrTab& ws, const CPtrTab& wts, const CPtrTab& imgs, const CompactConv& v, const CompactSrc& src,
                              bool relu, size_t y_off, const float* mean, int count, hipStream_t s);
hipError_t launch_compact_bwd(bool is_bf16, const PtrTab& ws, const CPtrTab& wts, const CPtrTab& imgs, const CompactConv& v,
                              const CompactSrc& x, const CompactGrad& gr, const CompactBwd& bw, const float* mean, bool need_dx, int count, hipStream_t s);
hipError_t launch_compact_flatten(bool is_bf16, const PtrTab& ws, const CompactSrc& src, size_t flat_off, int N, int count, hipStream_t s);
hipError_t launch_compact_head(bool is_bf16, const PtrTab& ws, const CPtrTab& wts, const CPtrTab& labels, const CompactSrc& src, const CompactHead& hd,
                               int32_t* rank_out, int count, hipStream_t s);
hipError_t launch_compact_fc(bool is_bf16, const PtrTab& ws, const CPtrTab& wts, const CompactFc& f, bool dgrad, size_t part_bytes, int count, hipStream_t s);
hipError_t launch_compact_finish(bool is_bf16, const PtrTab& ws, const PtrTab& grads, const CompactFinish& fin, size_t loss_off, int N, float* loss_out,
                                 int count, hipStream_t s);

}  // namespace sasgd
