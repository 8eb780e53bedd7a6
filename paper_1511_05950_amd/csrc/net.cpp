// Network plan and executor of calcGradient (Section 2.1): the layer list is turned into a list of
// device operations with fixed offsets into one per-learner workspace; a calcGradient call walks the list
// forward and backward, every launch covering all listed learners at once.  ReLU layers are fused into the
// operation that produces their input (its output is stored after the ReLU; the backward mask is applied
// by whichever kernel produces the gradient of that tensor).
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "kernels.hpp"

namespace sasgd {

enum OpKind { OP_CONV, OP_POOL_MAX, OP_POOL_AVG, OP_FLATTEN };

struct Op {
  OpKind kind;
  bool relu = false;           // output stored after ReLU
  bool is_fc = false;
  bool out_f32 = false;        // output kept in fp32 (class scores)
  ConvShape cs{};              // OP_CONV
  PoolShape ps{};              // pools; OP_FLATTEN uses N,C,H,W
  int64_t w_off = 0, b_off = 0;
  int in_t = 0, out_t = 0;     // tensor indices
  size_t arg_off = 0;          // byte offset of the max-pool argmax, from the workspace base
  // bf16 MFMA path (conv / fc ops that qualify)
  bool mfma = false;
  VConv vc{};
  IGemm gf{};                  // forward implicit GEMM
  IGemm gd{};                  // input-gradient implicit GEMM
  bool dgrad_bt = false;       // fc: B operand is the flat weight matrix read transposed
  int64_t pack_fwd = -1, pack_bwd = -1;   // element offsets in the packed-filter region of a version slot
  int Kp = 0, Kpt = 0;
  // first convolution that the max pooling behind it can share a kernel with (conv_pool_wins decides per call): its output is not stored then
  bool with_pool = false;
  // fully connected layer whose weight gradient is kept as the factors x^T [in][NP] and dy^T [out][NP]
  bool factored = false;
  size_t fx_off = 0, fdy_off = 0;         // element offsets of the two factor copies in the workspace
  int NP = 0;
};

struct Tensor {
  size_t off = 0;              // element offset in the workspace
  size_t elems = 0;
  bool relu = false;           // values are post-ReLU (a gradient flowing into it must be masked)
};

// The network as the compact kernels run it (compact.hip): convolutions with the pooling layer behind each, then fully
// connected layers.  Indices into ops.
struct CompactStage {
  int conv = -1, pool = -1;
  CompactConv v{};
  size_t part_off = 0;         // bytes: partial weight gradients
  int most_splits = 1;
};
struct CompactPlan {
  bool ok = false;             // the network fits
  bool always = false;         // every call of this context goes there: nothing is laid out for the layer-by-layer kernels
  // what a call's cost is made of (compact_wins), in units of 2^20: multiply-adds of an image's forward pass in convolutions that
  // have a matrix-instruction kernel of their own (and in the last layer) and in those that do not ("odd"), weights of hidden
  // fully connected layers with and without one, values of an image's layer outputs; output units of the odd hidden layers
  double macs = 0, odd_macs = 0, fc = 0, odd_fc = 0, values = 0;
  int odd_units = 0;
  bool any_odd() const { return odd_macs + odd_fc > 0; }
  std::vector<CompactStage> stages;
  std::vector<int> fcs;
  std::vector<size_t> fc_dy;   // element offset of every fully connected layer's output gradient
};

struct Net {
  int mu = 0;
  // layer by layer: the last fully connected layer, loss and its input gradient in one kernel, from operation `head` on (an average
  // pooling, the flattening or the layer itself); -1: separate kernels
  int head = -1;
  CompactPlan compact;
  bool bf16 = false;
  int classes = 0;
  bool scores_f32 = false;
  int64_t P = 0;
  std::vector<Op> ops;
  std::vector<Tensor> tensors; // tensor 0 = re-laid-out input
  int inC = 0, inH = 0, inW = 0;
  InPack inpack{};
  size_t Ppad = 0;             // start of the packed-filter region inside a version slot (elements)
  PackTable pack{};            // filter repacking jobs of one weight version
  size_t pack_elems = 0;
  size_t grad_a = 0, grad_b = 0, grad_elems = 0;   // two gradient-activation buffers (element offsets)
  size_t ws_bytes = 0;
  size_t loss_off = 0;         // per-image losses, mu floats (byte offset)
  size_t zero_off = 0;         // 256 zero bytes (element offset), target of out-of-range loads
  size_t scratch_off = 0, scratch_bytes = 0;   // split-contraction partials (bytes from the workspace base)
  void* ws[kMaxLearners] = {nullptr};
  const float* pixel_mean = nullptr;   // optional [C][H][W] fp32, subtracted while the input is re-laid out
};

// Recognises networks the compact kernels take: conv (pool)? repeated, (flatten)?, fc repeated.
static CompactPlan compact_plan(const Net* net) {
  CompactPlan cp;
  const std::vector<Op>& ops = net->ops;
  const int n = (int)ops.size();
  int i = 0;
  while (i < n && ops[(size_t)i].kind == OP_CONV && !ops[(size_t)i].is_fc) {
    CompactStage st;
    st.conv = i;
    const ConvShape& cs = ops[(size_t)i].cs;
    st.v = CompactConv{cs.N, cs.C, cs.H, cs.W, cs.K, cs.OH, cs.OW, cs.ks, cs.stride, cs.pad, ops[(size_t)i].w_off, ops[(size_t)i].b_off, {}, {}, {}, {}};
    st.v.by_ow.set(cs.OW);
    st.v.by_w.set(cs.W);
    st.v.by_cols.set((cs.OW - 1) * cs.stride + cs.ks);
    st.v.by_dcols.set(cs.W - 1 + cs.ks);
    if (!compact_conv_ok(st.v, !cp.stages.empty())) return cp;
    i++;
    if (i < n && (ops[(size_t)i].kind == OP_POOL_MAX || ops[(size_t)i].kind == OP_POOL_AVG)) {
      const PoolShape& ps = ops[(size_t)i].ps;
      if (ps.ks > 2 * ps.stride) return cp;                          // more than two windows per direction reach a position
      if (!FastDiv::exact(ps.stride, std::max(ps.H, ps.W))) return cp;
      st.pool = i++;
    }
    cp.stages.push_back(st);
  }
  if (cp.stages.empty()) return cp;
  if (i < n && ops[(size_t)i].kind == OP_FLATTEN) i++;
  for (; i < n; i++) {
    if (!ops[(size_t)i].is_fc) return cp;
    cp.fcs.push_back(i);
  }
  if (cp.fcs.empty() || cp.stages.size() + cp.fcs.size() + 1 > (size_t)kMaxCompactJobs) return cp;
  for (size_t k = 0; k < cp.fcs.size(); k++) {
    const ConvShape& cs = ops[(size_t)cp.fcs[k]].cs;
    if (k + 1 == cp.fcs.size() ? !compact_head_ok(cs.C, cs.K) : !compact_fc_ok(cs.C, cs.K)) return cp;
  }
  for (int k = 0; k < n; k++) {
    const Op& op = ops[(size_t)k];
    cp.values += (op.kind == OP_CONV ? (double)op.cs.K * op.cs.OH * op.cs.OW : (double)op.ps.C * op.ps.OH * op.ps.OW) / (1 << 20);
    const double m = (double)op.cs.K * op.cs.C * op.cs.ks * op.cs.ks * op.cs.OH * op.cs.OW / (1 << 20);
    if (k == cp.fcs.back()) cp.macs += m;
    else if (op.is_fc) (op.mfma ? cp.fc : cp.odd_fc) += m;
    else (op.mfma ? cp.macs : cp.odd_macs) += m;
    if (op.is_fc && !op.mfma && k != cp.fcs.back()) cp.odd_units += op.cs.K;
  }
  cp.ok = true;
  return cp;
}

// Are the compact kernels the faster ones for a call of `count` learners?  They save launches, and layers without a
// matrix-instruction kernel of their own (channel counts that are no multiple of 8 in bf16, 4 in fp32; strided first layers with
// padding; such hidden layers) are scalar kernels on the other path.  They lose where work is large: fp32 matrix instructions
// whatever the type, the weights of a hidden layer read again for every learner and every 16 images and its gradient written out.
// The differences in us, per unit of CompactPlan's terms, from both paths' times of 24 networks at 1 to 2 304 images a call:
// what this takes is the faster path or within 10 % of it in all but a few cases, and behind the layer-by-layer path by 13 % at
// most (20 us of a call on 1 x 1 convolutions).  E.g. 64- and 96-channel convolutions in front of a
// hidden layer of 137 units, bf16, 18 x 128 images 2 189 us layer by layer, 8 422 us compact; 1 x 8 images 165 against 102; two
// hidden layers of 4 096 units behind a convolution of 30 channels, 18 x 4 images 649 against 3 437; the CIFAR-shaped net in
// fp32 at 4 / 64 / 128 images 62 / 162 / 274 us compact, 139 / 256 / 358 layer by layer, in bf16 at 8 / 32 / 64 images
// 86 / 125 / 217 against 123 / 149 / 169.
struct CompactCost {
  double launches, hidden;     // saved, us a call and us per hidden layer
  double odd_units;            // saved: the scalar input gradient walks a layer's units one after the other
  double macs, odd_macs;       // per image (odd: saved)
  double fc, odd_fc;           // per image and weight
  double learner;              // per learner
  double fc_once, odd_fc_once; // per learner and weight
  double fc_again;             // per learner, weight and 16 images behind the first
  double values;               // per image
};
static const CompactCost kCompactCost[2][2] = {   // [bf16][evaluation]
    {{72, 0, 0.08, 0.045, 4.5, 0.08, 0.45, 0, -6.5, 0, 0, 0}, {50, 0, 0, 0, 0.9, 0, 0.13, 0, -2.5, 0, 1, 0.4}},
    {{84, 12, 0.08, 0.145, 3.8, 0.1, 0.9, 2, 3, 3.5, 1.2, 12}, {40, 8, 0, 0.05, 1, 0.012, 0.18, 0, 0.7, 0.8, 0.4, 5}}};
static bool compact_wins(const CompactPlan& p, bool bf16, int mu, int count, bool evaluation) {
  const CompactCost& k = kCompactCost[bf16][evaluation];
  const double image = k.macs * p.macs - k.odd_macs * p.odd_macs + k.fc * p.fc - k.odd_fc * p.odd_fc + k.values * p.values;
  const double learner = k.learner + k.fc_once * p.fc + k.odd_fc_once * p.odd_fc + k.fc_again * (p.fc + p.odd_fc) * ((mu + 15) / 16 - 1);
  return count * (mu * image + learner) <= k.launches + k.hidden * ((double)p.fcs.size() - 1) + k.odd_units * p.odd_units;
}

static int pool_out_size(int n, int k, int s) {
  int o = (n - k + s - 1) / s + 1;
  if ((o - 1) * s >= n) o--;
  return o < 1 ? 1 : o;
}

static const sasgd_layer kCifar3[] = {
    {SASGD_CONV, 32, 5, 1, 2}, {SASGD_MAXPOOL, 0, 3, 2, 0}, {SASGD_RELU, 0, 0, 0, 0},
    {SASGD_CONV, 32, 5, 1, 2}, {SASGD_RELU, 0, 0, 0, 0},    {SASGD_AVGPOOL, 0, 3, 2, 0},
    {SASGD_CONV, 64, 5, 1, 2}, {SASGD_RELU, 0, 0, 0, 0},    {SASGD_AVGPOOL, 0, 3, 2, 0},
    {SASGD_FC, 10, 0, 0, 0}};

static const sasgd_layer kAlex8[] = {
    {SASGD_CONV, 96, 11, 4, 0}, {SASGD_RELU, 0, 0, 0, 0}, {SASGD_MAXPOOL, 0, 3, 2, 0},
    {SASGD_CONV, 256, 5, 1, 2}, {SASGD_RELU, 0, 0, 0, 0}, {SASGD_MAXPOOL, 0, 3, 2, 0},
    {SASGD_CONV, 384, 3, 1, 1}, {SASGD_RELU, 0, 0, 0, 0},
    {SASGD_CONV, 384, 3, 1, 1}, {SASGD_RELU, 0, 0, 0, 0},
    {SASGD_CONV, 256, 3, 1, 1}, {SASGD_RELU, 0, 0, 0, 0}, {SASGD_MAXPOOL, 0, 3, 2, 0},
    {SASGD_FC, 4096, 0, 0, 0},  {SASGD_RELU, 0, 0, 0, 0},
    {SASGD_FC, 4096, 0, 0, 0},  {SASGD_RELU, 0, 0, 0, 0},
    {SASGD_FC, 1000, 0, 0, 0}};

int net_create(const sasgd_config& cfg, Net** out, int64_t* out_P, size_t* out_pack_elems, std::string& err) {
  const sasgd_layer* layers = nullptr;
  int nl = 0, C = 0, H = 0, W = 0;
  if (cfg.net == SASGD_NET_CIFAR3) {
    layers = kCifar3; nl = (int)(sizeof(kCifar3) / sizeof(kCifar3[0])); C = 3; H = 32; W = 32;
  } else if (cfg.net == SASGD_NET_ALEX8) {
    layers = kAlex8; nl = (int)(sizeof(kAlex8) / sizeof(kAlex8[0])); C = 3; H = 224; W = 224;
  } else if (cfg.net == SASGD_NET_CUSTOM) {
    layers = cfg.layers; nl = cfg.num_layers; C = cfg.in_channels; H = cfg.in_height; W = cfg.in_width;
    if (!layers || nl < 1 || nl > 256 || C < 1 || H < 1 || W < 1) { err = "custom network: bad layer table or input shape"; return SASGD_EINVAL; }
  } else {
    err = "unknown network"; return SASGD_EINVAL;
  }
  if (cfg.mu < 1 || cfg.mu > 4096) { err = "mu out of range (1..4096)"; return SASGD_EINVAL; }

  Net* net = new Net();
  net->mu = cfg.mu;
  net->bf16 = cfg.compute == SASGD_BF16;
  net->inC = C; net->inH = H; net->inW = W;
  const int N = cfg.mu;
  size_t cursor = 0;       // elements of T
  auto new_tensor = [&](size_t elems) {
    Tensor t;
    t.off = cursor;
    t.elems = elems;
    cursor += (elems + 63) & ~(size_t)63;
    net->tensors.push_back(t);
    return (int)net->tensors.size() - 1;
  };
  // The MFMA kernels gather 16-byte chunks of `chunk` channels (8 bf16 or 4 fp32).  The first convolution runs on
  // the MFMA path when it can: its input is channel-padded to a multiple of the chunk (stride 1) or
  // space-to-depth transformed (stride s, no padding).
  const int chunk = net->bf16 ? 8 : 4;
  int n_factored = 0;
  auto round_chunk = [&](int x) { return (x + chunk - 1) / chunk * chunk; };
  net->inpack = InPack{C, H, W, C, H, W, 1};
  bool first_mfma = false;
  if (layers[0].kind == SASGD_CONV && layers[0].units % chunk == 0 && layers[0].window >= 1 && layers[0].stride >= 1) {
    const sasgd_layer& L0 = layers[0];
    const int oh = (H + 2 * L0.pad - L0.window) / L0.stride + 1, ow = (W + 2 * L0.pad - L0.window) / L0.stride + 1;
    if (oh < 1 || ow < 1 || !FastDiv::exact(ow, (int64_t)N * oh * ow - 1) || !FastDiv::exact(oh, (int64_t)N * oh - 1)) {
      // refused below, or more positions than the matrix kernels can divide (igemm_divides)
    } else if (L0.stride == 1) {
      net->inpack.Cp = round_chunk(C);
      first_mfma = true;
    } else if (L0.pad == 0 && L0.window <= H && L0.window <= W) {
      const int sd = L0.stride;
      net->inpack = InPack{C, H, W, round_chunk(sd * sd * C), (H + sd - 1) / sd, (W + sd - 1) / sd, sd};
      first_mfma = true;
    }
  }
  int cur = new_tensor((size_t)N * net->inpack.Cp * net->inpack.Hp * net->inpack.Wp);
  bool flat = false;       // current tensor already in (C,H,W)-flattened order (after a flatten or an fc)
  size_t pack_cursor = 0;
  auto round32 = [](int x) { return (x + 31) & ~31; };
  int64_t P = 0;
  size_t arg_bytes = 0;
  for (int li = 0; li < nl; li++) {
    const sasgd_layer& L = layers[li];
    if (L.kind == SASGD_RELU) {
      if (net->ops.empty() || net->tensors[(size_t)cur].relu) { delete net; err = "relu must directly follow a conv, fc or pooling layer"; return SASGD_EINVAL; }
      net->ops.back().relu = true;
      net->tensors[(size_t)cur].relu = true;
      continue;
    }
    Op op;
    if (L.kind == SASGD_CONV) {
      if (flat || L.units < 1 || L.window < 1 || L.stride < 1 || L.pad < 0 || L.pad >= L.window || H + 2 * L.pad < L.window || W + 2 * L.pad < L.window) {
        delete net; err = "conv layer: bad shape"; return SASGD_EINVAL;
      }
      op.kind = OP_CONV;
      op.cs = ConvShape{N, C, H, W, L.units, (H + 2 * L.pad - L.window) / L.stride + 1, (W + 2 * L.pad - L.window) / L.stride + 1, L.window, L.stride, L.pad};
      op.w_off = P;
      P += (int64_t)L.units * C * L.window * L.window;
      op.b_off = P;
      P += L.units;
      op.in_t = cur;
      if (cur == 0 && first_mfma) {
        const InPack& ip = net->inpack;
        const int kse = (L.window + ip.s2d - 1) / ip.s2d;
        op.mfma = true;
        op.vc = VConv{ip.Cp, kse, L.units, ip.s2d, C, L.window};
        op.gf = IGemm{0, 0, N * op.cs.OH * op.cs.OW, L.units, ip.Hp, ip.Wp, ip.Cp, op.cs.OH, op.cs.OW, kse, ip.s2d == 1 ? L.pad : 0,
                      kse * kse * ip.Cp / chunk, ip.Cp / chunk, 0};
        if (net->bf16) {
          op.Kp = round32(kse * kse * ip.Cp);
          op.pack_fwd = (int64_t)pack_cursor;
          pack_cursor += (size_t)round32(L.units) * op.Kp;
        }
      } else if (cur != 0 && L.stride == 1 && C % chunk == 0 && L.units % chunk == 0) {
        op.vc = VConv{C, L.window, L.units, 1, C, L.window};
        op.gf = IGemm{0, 0, N * op.cs.OH * op.cs.OW, L.units, H, W, C, op.cs.OH, op.cs.OW, L.window, L.pad,
                      L.window * L.window * C / chunk, C / chunk, 0};
        op.gd = IGemm{0, 0, N * H * W, C, op.cs.OH, op.cs.OW, L.units, H, W, L.window, L.window - 1 - L.pad,
                      L.window * L.window * L.units / chunk, L.units / chunk, 0};
        op.mfma = igemm_divides(op.gf) && igemm_divides(op.gd);
        if (net->bf16 && op.mfma) {
          op.Kp = round32(L.window * L.window * C);
          op.Kpt = round32(L.window * L.window * L.units);
          op.pack_fwd = (int64_t)pack_cursor;
          pack_cursor += (size_t)round32(L.units) * op.Kp;
          op.pack_bwd = (int64_t)pack_cursor;
          pack_cursor += (size_t)round32(C) * op.Kpt;
        }
      }
      C = L.units; H = op.cs.OH; W = op.cs.OW;
      cur = op.out_t = new_tensor((size_t)N * C * H * W);
    } else if (L.kind == SASGD_MAXPOOL || L.kind == SASGD_AVGPOOL) {
      if (flat || L.window < 1 || L.window > 15 || L.stride < 1 || L.window > H || L.window > W) { delete net; err = "pooling layer: bad shape"; return SASGD_EINVAL; }
      op.kind = L.kind == SASGD_MAXPOOL ? OP_POOL_MAX : OP_POOL_AVG;
      op.ps = PoolShape{N, C, H, W, pool_out_size(H, L.window, L.stride), pool_out_size(W, L.window, L.stride), L.window, L.stride};
      op.in_t = cur;
      H = op.ps.OH; W = op.ps.OW;
      cur = op.out_t = new_tensor((size_t)N * C * H * W);
      if (op.kind == OP_POOL_MAX) { op.arg_off = arg_bytes; arg_bytes += ((size_t)N * C * H * W + 255) & ~(size_t)255; }
    } else if (L.kind == SASGD_FC) {
      if (L.units < 1) { delete net; err = "fc layer: bad shape"; return SASGD_EINVAL; }
      if (!flat && H * W > 1) {           // bring the tensor into the (C,H,W) order of the fc weights
        Op fl;
        fl.kind = OP_FLATTEN;
        fl.ps = PoolShape{N, C, H, W, 0, 0, 0, 0};
        fl.in_t = cur;
        cur = fl.out_t = new_tensor((size_t)N * C * H * W);
        net->ops.push_back(fl);
      }
      const int in = C * H * W;
      op.kind = OP_CONV;
      op.is_fc = true;
      op.cs = ConvShape{N, in, 1, 1, L.units, 1, 1, 1, 1, 0};
      op.w_off = P;
      P += (int64_t)L.units * in;
      op.b_off = P;
      P += L.units;
      op.in_t = cur;
      if (cur != 0 && in % chunk == 0 && L.units % chunk == 0 && (!net->bf16 || op.w_off % 8 == 0)) {
        // fully connected: the flat weight matrix [out][in] is the B operand as it lies (forward), and is read
        // transposed for the input gradient; no packed copy
        op.dgrad_bt = true;
        op.vc = VConv{in, 1, L.units, 1, in, 1};
        op.gf = IGemm{0, op.w_off, N, L.units, 1, 1, in, 1, 1, 1, 0, in / chunk, in / chunk, in};
        op.gd = IGemm{0, op.w_off, N, in, 1, 1, L.units, 1, 1, 1, 0, L.units / chunk, L.units / chunk, in};
        op.mfma = igemm_divides(op.gf) && igemm_divides(op.gd);
        if (net->bf16) op.mfma = op.mfma && fc_rows_layer_ok(in);
        // rank-N weight gradient kept as factors: worth it while the products per weight and pending gradient stay far
        // below what the update's streaming rate leaves room for; with more than 32 images where every update is a pass of its own
        // (and where the factors' rounded-up rows stay within a tensor's limit, below, as the layer's own tensors may)
        const int c_upd = cfg.lambda / cfg.n, NP = (N + 7) & ~7;
        if (op.mfma && net->bf16 && !(cfg.flags & SASGD_FLAG_FLAT_FC_GRADIENT) && N <= (cfg.n == 1 ? kMaxFactorRows : kFactorRowsAlways) && (int64_t)c_upd * N <= 1024 &&
            op.w_off % 4 == 0 && L.units % 4 == 0 && in % 8 == 0 && n_factored < kMaxFactoredLayers &&
            (int64_t)std::max(in, L.units) * NP * 4 < ((int64_t)1 << 31)) {
          op.factored = true;
          op.NP = NP;
          n_factored++;
        }
      }
      C = L.units; H = 1; W = 1;
      flat = true;
      cur = op.out_t = new_tensor((size_t)N * C);
    } else {
      delete net; err = "unknown layer kind"; return SASGD_EINVAL;
    }
    net->ops.push_back(op);
  }
  if (P < 1) { delete net; err = "network has no parameters"; return SASGD_EINVAL; }
  if (net->tensors[(size_t)cur].relu) { delete net; err = "the class scores must not pass through a relu"; return SASGD_EINVAL; }
  net->classes = C * H * W;
  if (net->classes < 2) { delete net; err = "network output must have at least two classes"; return SASGD_EINVAL; }
  if (!flat && H * W > 1) {               // scores must be one vector per image in class order
    Op fl;
    fl.kind = OP_FLATTEN;
    fl.ps = PoolShape{N, C, H, W, 0, 0, 0, 0};
    fl.in_t = cur;
    cur = fl.out_t = new_tensor((size_t)N * C * H * W);
    net->ops.push_back(fl);
  }
  if (net->ops.back().kind == OP_CONV) {   // class scores produced by a conv / fc: keep them in fp32
    net->ops.back().out_f32 = true;
    net->scores_f32 = true;
    if (net->bf16) { new_tensor(net->tensors[(size_t)cur].elems); }   // room for the wider elements (tensor is last in the arena)
  }
  // small networks and mini-batches: the compact kernels
  net->compact = compact_plan(net);
  if (net->compact.ok) {
    CompactPlan& cp = net->compact;
    bool any_factored = false;
    for (const Op& op : net->ops) any_factored = any_factored || op.factored;
    // they write every gradient out: not where the factors of few images are kept and all layers have kernels of their own
    if (any_factored && N <= kFactorRowsAlways && !cp.any_odd()) cp.ok = false;
    // the cost is linear in the learners of a call, so that the largest call decides for all of them
    cp.always = cp.ok && compact_wins(cp, net->bf16, N, cfg.lambda, false) && compact_wins(cp, net->bf16, N, cfg.lambda, true);
    if (cp.always)
      for (Op& op : net->ops) op.factored = false;
    if (cp.ok)
      for (int f : cp.fcs) cp.fc_dy.push_back(net->tensors[(size_t)new_tensor((size_t)N * net->ops[(size_t)f].cs.K)].off);
  }
  for (Op& op : net->ops) {
    if (!op.factored) continue;
    op.fx_off = net->tensors[(size_t)new_tensor((size_t)op.cs.C * op.NP)].off;
    op.fdy_off = net->tensors[(size_t)new_tensor((size_t)op.cs.K * op.NP)].off;
  }
  net->P = P;
  net->Ppad = ((size_t)P + 63) & ~(size_t)63;
  net->pack_elems = pack_cursor;
  for (Op& op : net->ops) {
    if (!op.mfma) continue;
    op.gf.zero_off = op.gd.zero_off = 0;   // filled below, once the arena is laid out
    const Tensor& ti = net->tensors[(size_t)op.in_t];
    op.gf.a_off = ti.off;
    if (!op.dgrad_bt && net->bf16) {
      op.gf.b_off = (int64_t)(net->Ppad + (size_t)op.pack_fwd);
      op.gf.ldb = op.Kp;
      if (op.pack_bwd >= 0) { op.gd.b_off = (int64_t)(net->Ppad + (size_t)op.pack_bwd); op.gd.ldb = op.Kpt; }
    }
    igemm_set_magics(op.gf, net->bf16 ? 2 : 4);
    igemm_set_magics(op.gd, net->bf16 ? 2 : 4);
    if (!net->bf16)   // the fp32 kernels read the flat filter itself: its byte size bounds their loads
      op.gf.b_bytes = op.gd.b_bytes = (uint32_t)((int64_t)op.vc.K * op.vc.Creal * op.vc.ksr * op.vc.ksr * 4);
  }
  if (net->bf16 && net->ops.size() > 1) {
    Op &conv = net->ops[0], &pool = net->ops[1];
    conv.with_pool = conv.kind == OP_CONV && conv.mfma && !conv.is_fc && pool.kind == OP_POOL_MAX && conv_pool_ok(conv.gf, pool.ps);
  }
  {
    // a last layer of few classes, which has no matrix-instruction kernel: one workgroup per image reads its weights twice
    const int last = (int)net->ops.size() - 1;
    const Op& fc = net->ops[(size_t)last];
    if (fc.is_fc && !fc.mfma && last > 0 && compact_head_ok(fc.cs.C, fc.cs.K) && head_kernel_wins(fc.cs.C, fc.cs.K)) {
      net->head = last;
      if (net->ops[(size_t)last - 1].kind == OP_FLATTEN && net->ops[(size_t)last - 1].in_t != 0) {
        net->head = last - 1;
        const Op* pool = last > 1 ? &net->ops[(size_t)last - 2] : nullptr;
        if (pool && pool->kind == OP_POOL_AVG && pool->in_t != 0) net->head = last - 2;
      } else if (!net->ops[(size_t)last - 1].is_fc) {
        net->head = -1;                                  // flattened images, or a layer of 1 x 1 pixels
      }
    }
  }
  size_t maxe = 0;
  for (const Tensor& t : net->tensors) maxe = t.elems > maxe ? t.elems : maxe;
  // the kernels address an activation tensor through 32-bit byte offsets with the top bit reserved for "out of range"
  if (maxe * 4 >= ((size_t)1 << 31)) { delete net; err = "an activation tensor of mu images exceeds 2 GiB: lower mu"; return SASGD_ERANGE; }
  net->grad_elems = (maxe + 63) & ~(size_t)63;
  net->grad_a = cursor;
  net->grad_b = cursor + net->grad_elems;
  cursor += 2 * net->grad_elems;
  net->zero_off = cursor;
  cursor += 256;
  for (Op& op : net->ops) op.gf.zero_off = op.gd.zero_off = net->zero_off;
  for (const Op& op : net->ops) {
    if (!op.mfma || op.pack_fwd < 0 || net->compact.always) continue;
    if (net->pack.count == kMaxPackJobs) { delete net; err = "too many convolution layers for the MFMA path"; return SASGD_EINVAL; }
    PackJob& jb = net->pack.job[net->pack.count++];
    jb.v = op.vc;
    jb.w_off = op.w_off;
    jb.fwd_off = op.pack_fwd;
    jb.bwd_off = op.pack_bwd < 0 ? 0 : op.pack_bwd;
    jb.Kp = op.Kp;
    jb.Kpt = op.pack_bwd < 0 ? 0 : op.Kpt;
    jb.start = net->pack.total;
    net->pack.total += (int64_t)((op.vc.K + 31) & ~31) * op.Kp + (op.pack_bwd < 0 ? 0 : (int64_t)((op.vc.C + 31) & ~31) * op.Kpt);
  }
  const size_t esz = net->bf16 ? 2 : 4;
  size_t bytes = (cursor * esz + 255) & ~(size_t)255;
  for (Op& op : net->ops) op.arg_off += bytes;
  bytes += arg_bytes;
  net->loss_off = bytes;
  bytes += ((size_t)N * 4 + 255) & ~(size_t)255;
  // scratch for split contractions: room for 8 partial copies of the largest output, within 16..128 MiB
  size_t need = 0;
  const int cw = net->bf16 ? 8 : 4;                // channels per im2col chunk
  for (const Op& op : net->ops) {
    if (!op.mfma) continue;
    size_t fwd = (size_t)op.gf.M * op.gf.Ncols * 4, wg = (size_t)op.gf.Ncols * (op.gf.Kchunks * cw + cw) * 4;
    size_t dg = (size_t)op.gd.M * op.gd.Ncols * 4;
    need = fwd > need ? fwd : need;
    need = wg > need ? wg : need;
    need = dg > need ? dg : need;
  }
  size_t sb = net->compact.always ? 0 : std::min(need * 8, std::max(need, (size_t)128 << 20));
  if (net->compact.ok) {
    // partial weight gradients of all convolutions side by side: one tile of 32 positions per workgroup where that costs
    // little memory, and fewer partial copies of the largest where all together would take more than 128 MiB a learner
    // (eight 512 x 512 x 3 x 3 convolutions at 32 images: 2.4 GiB uncapped)
    std::vector<CompactStage>& stages = net->compact.stages;
    auto elems = [](const CompactStage& st) { return (int64_t)st.v.K * st.v.C * st.v.ks * st.v.ks + st.v.K; };
    for (CompactStage& st : stages)
      st.most_splits = (int)std::min<int64_t>(std::min<int64_t>(256, std::max<int64_t>(32, ((int64_t)1 << 20) / elems(st))),
                                              (int64_t)st.v.N * ((st.v.OH * st.v.OW + 31) / 32));
    const size_t most = std::max(sb, (size_t)128 << 20);
    size_t parts;
    for (;;) {
      parts = 0;
      CompactStage* largest = nullptr;
      for (CompactStage& st : stages) {
        st.part_off = parts;
        parts += ((size_t)st.most_splits * elems(st) * 4 + 255) & ~(size_t)255;
        if (st.most_splits > 1 && (!largest || st.most_splits * elems(st) > largest->most_splits * elems(*largest))) largest = &st;
      }
      if (parts <= most || !largest) break;
      largest->most_splits = (largest->most_splits + 1) / 2;
    }
    sb = std::max(sb, parts);
  }
  if (sb > 0) {
    net->scratch_off = (bytes + 255) & ~(size_t)255;
    net->scratch_bytes = sb;
    bytes = net->scratch_off + sb;
  }
  net->ws_bytes = bytes + 256;
  *out = net;
  *out_P = P;
  *out_pack_elems = net->pack_elems;
  return SASGD_OK;
}

void net_destroy(Net* net) { delete net; }
size_t net_workspace_bytes(const Net* net) { return net->ws_bytes; }
hipError_t net_set_workspace(Net* net, int learner, void* ws, hipStream_t stream) {
  net->ws[learner] = ws;
  hipError_t e = hipMemsetAsync(ws, 0, net->ws_bytes, stream);
  if (e != hipSuccess) return e;
  // second half of the constant block: one 16-byte chunk holding 1.0 followed by zeros (the im2col "bias column")
  static const uint16_t one_bf16 = 0x3F80;
  static const float one_f32 = 1.0f;
  if (net->bf16) return hipMemcpyAsync((char*)ws + (net->zero_off + 128) * 2, &one_bf16, 2, hipMemcpyHostToDevice, stream);
  return hipMemcpyAsync((char*)ws + (net->zero_off + 128) * 4, &one_f32, 4, hipMemcpyHostToDevice, stream);
}

#define TRY(x) do { hipError_t e__ = (x); if (e__ != hipSuccess) return e__; } while (0)

// Derive the packed bf16 filters of every MFMA convolution from the flat bf16 copy of one weight version.
hipError_t net_prepare_versions(Net* net, const void* const* flat, void* const* packed, int versions, hipStream_t stream) {
  if (net->pack.count == 0) return hipSuccess;
  for (int v0 = 0; v0 < versions; v0 += kMaxPackVersions) {
    PackVersions pv;
    memset(&pv, 0, sizeof(pv));
    const int nv = std::min(kMaxPackVersions, versions - v0);
    for (int k = 0; k < nv; k++) { pv.flat[k] = flat[v0 + k]; pv.packed[k] = packed[v0 + k]; }
    TRY(launch_pack_filters(pv, nv, net->pack, stream));
  }
  return hipSuccess;
}
hipError_t net_prepare_version(Net* net, const void* flat, void* packed, hipStream_t stream) {
  return net_prepare_versions(net, &flat, &packed, 1, stream);
}

// fp32 MFMA path: 128 x 32 tiles, contraction steps of 16 (four 4-channel chunks)
static void set_splits_f32(const Net* net, IGemm& g, int count) {
  const int64_t tiles = (int64_t)((g.M + 127) / 128) * ((g.Ncols + 31) / 32);
  g.scratch_off = net->scratch_off;
  g.splits = choose_splits(tiles, count, (g.Kchunks + 3) / 4, (size_t)g.M * g.Ncols * 4, net->scratch_bytes);
}

// (by 128-row tiles: where a convolution's product takes larger ones, conv_choices takes this as the most it may be split into.  Of up to 32 positions
// columns are counted in 128s also where a tile takes 256: half the splits of many learners' 512-column layers, which is faster or slower by how they
// fill the chip; one image of 3 x 3 to 5 x 5, 512 -> 512, 18 learners 120 us for four products and 130 by tiles of 256, 30 learners 161 and 138)
static void set_splits(const Net* net, IGemm& g, int steps, int count) {
  const int bm = g.M <= 32 ? 32 : 128, bn = g.M <= 32 ? 128 : (g.Ncols <= 32 ? 32 : (g.Ncols <= 64 ? 64 : (g.Ncols % 256 == 0 ? 256 : 128)));
  const int64_t tiles = (int64_t)((g.M + bm - 1) / bm) * ((g.Ncols + bn - 1) / bn);
  g.scratch_off = net->scratch_off;
  g.splits = choose_splits(tiles, count, steps, (size_t)g.M * g.Ncols * 4, net->scratch_bytes);
}

int net_factored_layers(const Net* net, FactoredLayer* out, int max) {
  int k = 0;
  for (const Op& op : net->ops) {
    if (!op.factored) continue;
    if (k < max) out[k] = FactoredLayer{op.w_off, op.cs.C, op.cs.K, op.cs.N, op.NP, op.fx_off, op.fdy_off};
    k++;
  }
  return k;
}

void net_set_pixel_mean(Net* net, const float* mean_dev) { net->pixel_mean = mean_dev; }
void net_input_shape(const Net* net, int* C, int* H, int* W) { *C = net->inC; *H = net->inH; *W = net->inW; }

static CompactSrc compact_src(const Net* net, const CompactStage* st) {
  CompactSrc s;
  memset(&s, 0, sizeof(s));
  if (!st) {
    s.kind = CSRC_IMAGES;
    s.C = net->inC; s.H = net->inH; s.W = net->inW;
    s.by_c.set(s.C);
    return s;
  }
  const Op& conv = net->ops[(size_t)st->conv];
  s.off = net->tensors[(size_t)conv.out_t].off;
  s.C = conv.cs.K; s.H = conv.cs.OH; s.W = conv.cs.OW;
  s.by_c.set(s.C);
  s.by_c4.set(s.C / 4);
  if (st->pool < 0) return s;                        // CSRC_TENSOR
  const Op& pool = net->ops[(size_t)st->pool];
  s.kind = pool.kind == OP_POOL_MAX ? CSRC_MAXPOOL : CSRC_AVGPOOL;
  s.YH = s.H; s.YW = s.W;
  s.H = pool.ps.OH; s.W = pool.ps.OW;
  s.pks = pool.ps.ks; s.pst = pool.ps.stride; s.relu = pool.relu ? 1 : 0;
  s.out_off = net->tensors[(size_t)pool.out_t].off;
  s.arg_off = pool.arg_off;
  return s;
}

static hipError_t compact_gradient(Net* net, const PtrTab& ws, const CPtrTab& wts, const CPtrTab& imgs, const CPtrTab& labs, const PtrTab& grads,
                                   int count, float* out_loss_dev, int32_t* out_rank_dev, hipStream_t stream) {
  const bool bf = net->bf16;
  const CompactPlan& cp = net->compact;
  const std::vector<Tensor>& T = net->tensors;
  const std::vector<Op>& ops = net->ops;
  const int ns = (int)cp.stages.size(), nf = (int)cp.fcs.size();
  // ---- forward
  for (int k = 0; k < ns; k++) {
    const CompactStage& st = cp.stages[(size_t)k];
    const Op& op = ops[(size_t)st.conv];
    TRY(launch_compact_fwd(bf, ws, wts, imgs, st.v, compact_src(net, k ? &cp.stages[(size_t)k - 1] : nullptr), op.relu, T[(size_t)op.out_t].off,
                           net->pixel_mean, count, stream));
  }
  const CompactStage& last = cp.stages.back();
  const size_t flat_off = T[(size_t)ops[(size_t)cp.fcs[0]].in_t].off;        // input of the first fully connected layer, (C, H, W) order
  const bool pooled_relu = last.pool >= 0 && ops[(size_t)last.pool].relu;
  const CompactSrc flat_src = compact_src(net, &last);
  const int flat_hw = flat_src.H * flat_src.W;
  auto fc_of = [&](int k) {
    const Op& op = ops[(size_t)cp.fcs[(size_t)k]];
    CompactFc f;
    memset(&f, 0, sizeof(f));
    f.N = net->mu; f.in = op.cs.C; f.out = op.cs.K;
    f.relu = op.relu ? 1 : 0;
    f.w_off = op.w_off; f.b_off = op.b_off;
    f.x_off = T[(size_t)op.in_t].off;
    f.y_off = T[(size_t)op.out_t].off;
    f.dy_off = cp.fc_dy[(size_t)k];
    f.dx_off = k ? cp.fc_dy[(size_t)k - 1] : net->grad_a;
    f.use_mask = (k ? T[(size_t)op.in_t].relu : pooled_relu) ? 1 : 0;
    f.HW = k ? 1 : flat_hw;
    f.part_off = net->scratch_off;
    return f;
  };
  if (nf > 1) {
    TRY(launch_compact_flatten(bf, ws, compact_src(net, &last), flat_off, net->mu, count, stream));
    for (int k = 0; k + 1 < nf; k++) TRY(launch_compact_fc(bf, ws, wts, fc_of(k), false, net->scratch_bytes, count, stream));
  }
  // ---- last fully connected layer, loss, its input gradient
  {
    const CompactFc f = fc_of(nf - 1);
    CompactSrc s = compact_src(net, &last);
    if (nf > 1) {
      memset(&s, 0, sizeof(s));
      s.kind = CSRC_FLAT;
      s.off = f.x_off;
    }
    CompactHead hd;
    memset(&hd, 0, sizeof(hd));
    hd.N = net->mu; hd.in = f.in; hd.K = f.out;
    hd.w_off = f.w_off; hd.b_off = f.b_off;
    hd.flat_off = flat_off; hd.dz_off = f.dy_off; hd.dx_off = f.dx_off; hd.loss_off = net->loss_off;
    hd.use_mask = f.use_mask;
    hd.HW = f.HW; hd.C = f.in / f.HW;
    hd.by_hw.set(f.HW);
    TRY(launch_compact_head(bf, ws, wts, labs, s, hd, out_rank_dev, count, stream));
  }
  CompactFinish fin;
  memset(&fin, 0, sizeof(fin));
  if (out_loss_dev) fin.job[fin.count++].kind = CJOB_LOSS;
  if (!out_rank_dev) {
    // ---- backward
    for (int k = nf - 2; k >= 0; k--) TRY(launch_compact_fc(bf, ws, wts, fc_of(k), true, net->scratch_bytes, count, stream));
    size_t dy = net->grad_a, dx = net->grad_b;
    for (int k = ns - 1; k >= 0; k--) {
      const CompactStage& st = cp.stages[(size_t)k];
      const Op& op = ops[(size_t)st.conv];
      CompactGrad g;
      memset(&g, 0, sizeof(g));
      g.off = dy;
      g.OH = op.cs.OH; g.OW = op.cs.OW; g.K = op.cs.K;
      g.by_k.set(g.K);
      g.by_k4.set(g.K / 4);
      if (st.pool >= 0) {
        const Op& pool = ops[(size_t)st.pool];
        g.kind = pool.kind == OP_POOL_MAX ? CGRAD_MAXPOOL : CGRAD_AVGPOOL;
        g.PH = pool.ps.OH; g.PW = pool.ps.OW; g.pks = pool.ps.ks; g.pst = pool.ps.stride;
        g.arg_off = pool.arg_off;
      } else if (k == ns - 1) {                       // flattened as it is: a window of one element
        g.kind = CGRAD_AVGPOOL;
        g.PH = g.OH; g.PW = g.OW; g.pks = g.pst = 1;
      }
      g.by_pst.set(g.pst);
      g.use_mask = op.relu ? 1 : 0;                   // plain gradients were masked by their producer
      g.mask_off = T[(size_t)op.out_t].off;
      // the layer's input as kept by the forward pass
      CompactSrc x = compact_src(net, k ? &cp.stages[(size_t)k - 1] : nullptr);
      if (k && x.kind != CSRC_TENSOR) {
        x.kind = CSRC_TENSOR;
        x.off = x.out_off;
      }
      CompactBwd bw;
      memset(&bw, 0, sizeof(bw));
      bw.splits = compact_splits(st.v, k > 0, count, st.most_splits);
      bw.dx_off = dx;
      bw.mask_off = x.off;
      bw.use_mask = k && T[(size_t)op.in_t].relu ? 1 : 0;
      bw.part_off = net->scratch_off + st.part_off;
      bw.part_elems = (int64_t)st.v.K * st.v.C * st.v.ks * st.v.ks + st.v.K;
      TRY(launch_compact_bwd(bf, ws, wts, imgs, st.v, x, g, bw, net->pixel_mean, k > 0, count, stream));
      CompactJob& jb = fin.job[fin.count++];
      jb.kind = CJOB_SUM;
      jb.splits = bw.splits; jb.elems = bw.part_elems; jb.w_off = st.v.w_off; jb.part_off = bw.part_off;
      jb.K = st.v.K; jb.C = st.v.C; jb.taps = st.v.ks * st.v.ks;
      std::swap(dy, dx);
    }
    for (int k = 0; k < nf; k++) {
      const CompactFc f = fc_of(k);
      CompactJob& jb = fin.job[fin.count++];
      jb.kind = CJOB_FC;
      jb.in = f.in; jb.out = f.out; jb.w_off = f.w_off; jb.x_off = f.x_off; jb.dy_off = f.dy_off;
    }
  }
  return launch_compact_finish(bf, ws, grads, fin, net->loss_off, net->mu, out_loss_dev, count, stream);
}

// Forward pass, loss and (unless out_rank_dev is given, which makes this an evaluation pass) backward pass.
hipError_t net_calc_gradient(Net* net, const int* learners, const LearnerBind* binds, int count, float* out_loss_dev,
                             int32_t* out_rank_dev, bool write_out, bool* wrote_factors, hipStream_t stream) {
  PtrTab ws, grads;
  CPtrTab wts, imgs, labs;
  memset(&ws, 0, sizeof(ws)); memset(&grads, 0, sizeof(grads));
  memset(&wts, 0, sizeof(wts)); memset(&imgs, 0, sizeof(imgs)); memset(&labs, 0, sizeof(labs));
  for (int k = 0; k < count; k++) {
    ws.p[k] = net->ws[learners[k]];
    grads.p[k] = binds[k].grad;
    wts.p[k] = binds[k].weights;
    imgs.p[k] = binds[k].images;
    labs.p[k] = binds[k].labels;
  }
  const bool bf = net->bf16;
  const std::vector<Tensor>& T = net->tensors;
  const bool compact = net->compact.ok && (net->compact.always || compact_wins(net->compact, bf, net->mu, count, out_rank_dev != nullptr));
  if (wrote_factors) {
    *wrote_factors = false;
    for (const Op& op : net->ops) *wrote_factors = *wrote_factors || (op.factored && !compact && !write_out);
  }
  if (compact)
    return compact_gradient(net, ws, wts, imgs, labs, grads, count, out_loss_dev, out_rank_dev, stream);
  // The fully connected kernels multiply the rows of all learners of one weight version at once: `wsV` / `wtsV` list the learners
  // version by version, `vtab` says where each version's begin.
  PtrTab wsV;
  CPtrTab wtsV;
  GroupTab vtab;
  int versions = 0;
  bool any_rows = false;
  for (const Op& op : net->ops) any_rows = any_rows || (bf && op.is_fc && op.mfma);
  memset(&wsV, 0, sizeof(wsV)); memset(&wtsV, 0, sizeof(wtsV)); memset(&vtab, 0, sizeof(vtab));
  for (int a = 0, pos = 0; any_rows && a < count; a++) {
    bool seen = false;
    for (int b2 = 0; b2 < a; b2++) seen = seen || wts.p[b2] == wts.p[a];
    if (seen) continue;
    vtab.first[versions] = (uint8_t)pos;
    for (int b2 = a; b2 < count; b2++)
      if (wts.p[b2] == wts.p[a]) { wsV.p[pos] = ws.p[b2]; wtsV.p[pos++] = wts.p[b2]; }
    vtab.members[versions] = (uint8_t)(pos - vtab.first[versions]);
    versions++;
  }
  // ---- forward
  TRY(launch_pack_input(bf, imgs, ws, T[0].off, count, net->mu, net->inpack, net->pixel_mean, stream));
  size_t first = 0;
  if (net->ops[0].with_pool && conv_pool_wins((int64_t)count * net->mu, net->ops[0].gf.OH * net->ops[0].gf.OW, net->ops[0].gf.C, net->ops[0].gf.Ncols, net->ops[0].gf.ks)) {
    const Op &conv = net->ops[0], &pool = net->ops[1];
    const Epilogue ep{0, 0, conv.b_off, 1, conv.relu ? 1 : 0, 0, 0};
    TRY(launch_conv_pool(ws, wts, conv.gf, ep, pool.ps, T[(size_t)pool.out_t].off, pool.arg_off, pool.relu, count, stream));
    first = 2;
  }
  const size_t layers = net->head >= 0 ? (size_t)net->head : net->ops.size();
  for (size_t k = first; k < layers; k++) {
    const Op& op = net->ops[k];
    const size_t xi = T[(size_t)op.in_t].off, yo = T[(size_t)op.out_t].off;
    switch (op.kind) {
      case OP_CONV:
        if (op.mfma && !bf) {
          Epilogue ep{yo, 0, op.b_off, 1, op.relu ? 1 : 0, 0, 1};
          IGemm gf = op.gf;
          set_splits_f32(net, gf, count);
          TRY(launch_igemm_f32(ws, wts, gf, op.vc, ep, op.w_off, false, count, stream));
        } else if (op.mfma && op.is_fc) {
          Epilogue ep{yo, 0, op.b_off, 1, op.relu ? 1 : 0, 0, op.out_f32 ? 1 : 0};
          TRY(launch_fc_rows(wsV, wtsV, vtab, versions, op.gf, ep, false, net->scratch_off, net->scratch_bytes, stream));
        } else if (op.mfma) {
          Epilogue ep{yo, 0, op.b_off, 1, op.relu ? 1 : 0, 0, op.out_f32 ? 1 : 0};
          IGemm gf = op.gf;
          set_splits(net, gf, (gf.Kchunks + 3) / 4, count);
          TRY(launch_igemm_frag(ws, wts, gf, ep, count, stream));
        } else {
          TRY(launch_conv_fwd_simple(bf, ws, wts, xi, yo, op.w_off, op.b_off, op.cs, op.relu, op.out_f32, count, stream));
        }
        break;
      case OP_POOL_MAX:
      case OP_POOL_AVG:
        TRY(launch_pool_fwd(bf, op.kind == OP_POOL_MAX, ws, xi, yo, op.arg_off, op.ps, op.relu, T[(size_t)op.in_t].relu, count, stream));
        break;
      case OP_FLATTEN:
        TRY(launch_flatten_fwd(bf, ws, xi, yo, op.ps.N, op.ps.C, op.ps.H, op.ps.W, count, stream));
        break;
    }
  }
  // ---- loss and its gradient with respect to the class scores
  size_t dy = net->grad_a, dx = net->grad_b;
  if (net->head >= 0) {
    const Op &from = net->ops[(size_t)net->head], &fc = net->ops.back();
    const Tensor& tin = T[(size_t)from.in_t];
    CompactSrc src;
    memset(&src, 0, sizeof(src));
    src.off = tin.off;
    bool relu = tin.relu;                                // of the values the input gradient is masked by
    CompactHead hd;
    memset(&hd, 0, sizeof(hd));
    hd.HW = 1;
    if (from.is_fc) {
      src.kind = CSRC_FLAT;
    } else {
      src.kind = CSRC_TENSOR;
      src.C = from.ps.C; src.H = from.ps.H; src.W = from.ps.W;
      if (from.kind == OP_POOL_AVG) {
        src.kind = CSRC_AVGPOOL;
        src.YH = src.H; src.YW = src.W;
        src.H = from.ps.OH; src.W = from.ps.OW;
        src.pks = from.ps.ks; src.pst = from.ps.stride; src.relu = from.relu ? 1 : 0;
        relu = from.relu;
      }
      src.by_c.set(src.C);
      src.by_c4.set(src.C / 4);
      hd.HW = src.H * src.W;
    }
    hd.N = net->mu; hd.in = fc.cs.C; hd.K = fc.cs.K;
    hd.C = hd.in / hd.HW;
    hd.w_off = fc.w_off; hd.b_off = fc.b_off;
    hd.flat_off = T[(size_t)fc.in_t].off; hd.dz_off = dy; hd.dx_off = dx; hd.loss_off = net->loss_off;
    hd.use_mask = relu ? 1 : 0;
    hd.by_hw.set(hd.HW);
    TRY(launch_compact_head(bf, ws, wts, labs, src, hd, out_rank_dev, count, stream));
    if (out_loss_dev) TRY(launch_loss_mean(ws, net->loss_off, net->mu, out_loss_dev, count, stream));
    if (out_rank_dev) return hipSuccess;
  } else {
    TRY(launch_softmax_ce(bf, net->scores_f32, ws, labs, T[(size_t)net->ops.back().out_t].off, dy, net->loss_off, net->mu, net->classes,
                          out_loss_dev, count, stream));
    if (out_rank_dev)
      return launch_label_rank(bf, net->scores_f32, ws, labs, T[(size_t)net->ops.back().out_t].off, net->mu, net->classes, out_rank_dev,
                               count, stream);
  }
  // ---- backward
  auto fc_dgrad = [&](const Op& op, const Tensor& tin) -> hipError_t {
    IGemm gd = op.gd;
    gd.a_off = dy;
    const Epilogue ep{dx, tin.off, 0, 0, 0, tin.relu ? 1 : 0, 0};
    return launch_fc_rows(wsV, wtsV, vtab, versions, gd, ep, true, net->scratch_off, net->scratch_bytes, stream);
  };
  // the first convolution's gradient has one reader, which may take it through the max pooling behind
  PooledDy pooled{0, 0, 0};
  bool through_pool = false;
  if (bf && net->ops.size() > 1 && net->ops[0].kind == OP_CONV && net->ops[0].mfma && !net->ops[0].is_fc && net->ops[1].kind == OP_POOL_MAX) {
    const Op &conv = net->ops[0], &pool = net->ops[1];
    pooled = PooledDy{pool.ps.OH, pool.ps.OW, pool.arg_off};
    through_pool = wgrad_takes_pooled(conv.gf, conv.vc, pool.ps, net->scratch_bytes, count);
  }
  for (int k = (int)net->ops.size() - 1; k >= 0; k--) {
    const Op& op = net->ops[(size_t)k];
    const Tensor& tin = T[(size_t)op.in_t];
    if (k == 1 && through_pool) continue;       // (dy stays the pooled tensor's gradient)
    const bool need_dx = op.in_t != 0;          // the network input needs no gradient
    switch (op.kind) {
      case OP_CONV:
        if (op.mfma && !bf) {
          {
            IGemm gw = op.gf;
            const int64_t tiles = (int64_t)((gw.Ncols + 31) / 32) * ((gw.Kchunks * 4 + 1 + 127) / 128);
            gw.scratch_off = net->scratch_off;
            gw.splits = choose_splits(tiles, count, (gw.M + 15) / 16, (size_t)gw.Ncols * (gw.Kchunks * 4 + 4) * 4, net->scratch_bytes);
            TRY(launch_igemm_wgrad_f32(ws, grads, gw, op.vc, dy, op.w_off, op.b_off, count, stream));
          }
          if (need_dx) {
            IGemm gd = op.gd;
            gd.a_off = dy;
            set_splits_f32(net, gd, count);
            Epilogue ep{dx, tin.off, 0, 0, 0, tin.relu ? 1 : 0, 1};
            TRY(launch_igemm_f32(ws, wts, gd, op.vc, ep, op.w_off, true, count, stream));
          }
        } else if (op.mfma && op.factored && !write_out) {
          TRY(launch_fc_save_factors(ws, grads, tin.off, dy, op.fx_off, op.fdy_off, op.b_off, op.cs.N, op.cs.C, op.cs.K, op.NP, count, stream));
          if (need_dx) TRY(fc_dgrad(op, tin));
        } else if (op.mfma) {
          IGemm gw = op.gf;
          gw.scratch_off = net->scratch_off;
          TRY(launch_igemm_wgrad(ws, grads, gw, op.vc, dy, op.w_off, op.b_off, net->scratch_bytes,
                                 k == 0 && through_pool ? &pooled : nullptr, count, stream));
          if (need_dx && op.is_fc) {
            TRY(fc_dgrad(op, tin));
          } else if (need_dx) {
            IGemm gd = op.gd;
            gd.a_off = dy;
            set_splits(net, gd, (gd.Kchunks + 3) / 4, count);
            Epilogue ep{dx, tin.off, 0, 0, 0, tin.relu ? 1 : 0, 0};
            TRY(launch_igemm_frag(ws, wts, gd, ep, count, stream));
          }
        } else {
          TRY(launch_conv_wgrad_simple(bf, ws, grads, tin.off, dy, op.w_off, op.b_off, op.cs, count, stream));
          if (need_dx && k == (int)net->ops.size() - 1 && net->head >= 0) {
            // the input gradient has been written: of the pooled tensor where a flattening comes next
            if (k > 0 && net->ops[(size_t)k - 1].kind == OP_FLATTEN) k--;
          } else if (need_dx) TRY(launch_conv_dgrad_simple(bf, ws, wts, dy, dx, op.w_off, op.cs, tin.relu, tin.off, count, stream));
        }
        break;
      case OP_POOL_MAX:
      case OP_POOL_AVG:
        if (need_dx) TRY(launch_pool_bwd(bf, op.kind == OP_POOL_MAX, ws, dy, dx, op.arg_off, op.ps, tin.relu, tin.off, count, stream));
        break;
      case OP_FLATTEN:
        if (need_dx) TRY(launch_flatten_bwd(bf, ws, dy, dx, op.ps.N, op.ps.C, op.ps.H, op.ps.W, tin.relu, tin.off, count, stream));
        break;
    }
    if (need_dx) { size_t t = dy; dy = dx; dx = t; }
  }
  return hipSuccess;
}

}  // namespace sasgd
