// Which kernel and which tiles serve a layer, from its sizes.  No HIP types: host code and host tests include it alone.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace sasgd {

// Re-layout of a mini-batch's images (bf16): whole rows for the space-to-depth layout by 4 of three-channel images, in pieces where
// a row is long; a lane per pixel wherever pixels are whole 16-byte chunks; a lane per value otherwise.
enum class InputLayout { kRows, kPixels, kValues };
inline InputLayout input_layout(bool is_bf16, int s2d, int C, int Cp, bool aligned) {
  if (is_bf16 && aligned && s2d == 4 && C == 3 && Cp == 48) return InputLayout::kRows;
  return is_bf16 && Cp % 8 == 0 ? InputLayout::kPixels : InputLayout::kValues;
}
// Pixels of a row that one workgroup of the kRows kernel makes: the row in even pieces of up to 640, 60 KiB of LDS
// (3072 x 256 pixels, 4 learners x 2 images: 17 us; a lane per pixel takes 50).
inline int input_row_piece(int Wp) {
  const int pieces = (Wp + 639) / 640;
  return (Wp + pieces - 1) / pieces;
}
// Workgroups of the kPixels kernel a learner: 256 pixels each, counted through all images.
inline int64_t input_pixel_groups(int N, int Hp, int Wp) {
  const int64_t groups = ((int64_t)N * Hp * Wp + 255) / 256;
  return groups < 16384 ? groups : 16384;
}

// ---- matrix products
// Splits of a contraction: enough workgroups for the chip, bounded by the contraction's length and the scratch size.
// target = workgroups wanted per launch; 600 by default (256..1024 measured, flat between 400 and 768 at 6 and 18 learners).
inline int choose_splits(int64_t tiles, int count, int steps, size_t bytes_per_split, size_t scratch_bytes, int64_t target = 600) {
  int64_t sp = (target + tiles * count - 1) / (tiles * count);
  if (sp > steps / 4) sp = steps / 4;                // keep at least four contraction steps per workgroup
  if (bytes_per_split > 0 && (int64_t)(scratch_bytes / bytes_per_split) < sp) sp = (int64_t)(scratch_bytes / bytes_per_split);
  if (sp > 64) sp = 64;
  return sp < 2 ? 1 : (int)sp;
}

// ---- forward pass and input gradient of a convolution, bf16

// A split of up to six ways is not worth its partials and second pass once the tiles alone take a fifth of the resident
// places (conv5 forward of the AlexNet shape at 18 learners, 396 tiles on 512 places: 92 us unsplit against
// 104 + 25 us; conv3 forward at 8 learners, 264 tiles: two-way split 60 + 18 us for the second pass; over a run of
// the 18-softsync benchmark the calcGradient phase takes 0.230 ms per update with this rule against 0.237 ms when only two-way
// splits of tiles filling 60 % of the places were dropped, and 0.233 ms when nothing is split).
inline int worthwhile_splits(int splits, int64_t tiles, int places) { return splits <= 6 && tiles * 5 >= places ? 1 : splits; }

// A product: M positions, Ncols columns, ks x ks windows over C channels, `count` learners.  own: most of
// them read a weight version of their own.  splits: what the contraction may be split into (never more than that: it is what
// the scratch memory holds).
struct ConvProduct {
  int64_t M;
  int Ncols, C, ks, count;
  bool own;
  int splits;
};
enum class ConvTile { k128x128, k256x128, k256x96 };
struct ConvChoice {
  ConvTile tile;
  int splits;
  double us;
};
// Times in us: start of a launch, filling a patch with 32 channels (tap by tap: start of a workgroup), a step of 32 values of the
// contraction with one, two, three workgroups on a compute unit (the last the places it has); a chip whose places are partly empty
// is faster by `spare` of the empty part.  Fitted to 1 243 products of 200 random networks and the AlexNet-shaped one (72 to 512
// columns, windows of 2 to 7, 30 to 500 000 positions, 1 to 30 learners), each in every form, split and not: off by 7 to 10 %.
struct ConvTileTimes {
  int rows, cols, places;
  double start, fill, step[3], spare;
  int64_t tiles(const ConvProduct& p) const { return (p.M + rows - 1) / rows * ((p.Ncols + cols - 1) / cols) * p.count; }
};
inline double conv_time(const ConvTileTimes& t, const ConvProduct& p, int splits, int fills, int steps) {
  const int64_t groups = t.tiles(p) * splits, each = (groups + 255) / 256;
  const int left = (int)(each % t.places);
  const double full = t.step[t.places - 1], rounds = (double)(each / t.places) + (left ? t.step[left - 1] / full : 0.);
  const double empty = 1. - (double)groups / (256. * each);
  const double second_pass = splits > 1 ? 3.5 + 4e-6 / 4.5 * splits * (double)p.M * p.Ncols * p.count : 0.;
  return t.start + rounds * (full * (1. - t.spare * empty) * steps + t.fill * fills) + second_pass;
}
// The form in question has to be better than the plain one by more than the times are off.
constexpr double kConvMargin = 1.02;
// Columns that whole 96s cover with fewer to spare than whole 128s: 72 .. 96, 136 .. 192, 264 .. 288, 392 .. 480, ...
inline bool spares_columns_96(int Ncols) { return (Ncols + 95) / 96 * 96 < (Ncols + 127) / 128 * 128; }

// Tiles of a product of the patch-in-LDS kernel with more than 64 columns, no multiple of 256, the cheapest first; returns how many.
//   128 x 128: three workgroups on a compute unit.
//   256 x 128, more than 128 columns: two, which read the filter fragments half as often.
//   256 x 96, where that spares columns: two, and up to a quarter fewer products, in larger steps.  272 columns, 3 x 3 over 128, 15 learners of 2 704
//     positions: 51 us with 128 x 128, 35 here; 448 columns, 5 x 5 over 448, 29 learners of 1 300: 375 and 416; 96 columns, 3 x 3
//     over 96, 4 learners of 5 832: 16, and 25 split three ways.  Taken wherever it spares columns, it was the slower one by
//     more than 3 % in 145 of 544 products, by up to 60 %; by these times in 4, by up to 11 %.
// With a weight version per learner the fragments are the larger part of the traffic, and 128 x 128 has to be better by more than
// that (3 x 3 over 384, 384 columns, 18 learners: 120 us against 101 with 256 x 128).
inline int conv_choices(const ConvProduct& p, ConvChoice (&out)[3]) {
  static const ConvTileTimes k128 = {128, 128, 3, 7.6, 2.7, {0.21, 0.32, 0.47}, 0.36}, k256 = {256, 128, 2, 9.5, 2.0, {0.40, 0.645, 0}, 0.34},
                             k96 = {256, 96, 2, 8.7, 2.0, {0.31, 0.52, 0}, 0.39};
  const int chunks = (p.C + 31) / 32, most = p.splits < chunks ? p.splits : chunks;
  auto time = [&](const ConvTileTimes& t, int splits) {
    const int fills = (chunks + splits - 1) / splits;
    return conv_time(t, p, splits, fills, fills * p.ks * p.ks);
  };
  int n = 0;
  auto add = [&](ConvTile tile, int splits, double us) {
    int at = n++;
    for (; at > 0 && out[at - 1].us > us; at--) out[at] = out[at - 1];
    out[at] = ConvChoice{tile, splits, us};
  };
  const bool wide = p.Ncols > 128;
  const int s128 = worthwhile_splits(most, k128.tiles(p), 256 * 3);
  add(ConvTile::k128x128, s128, time(k128, s128) * (p.own && wide ? 1.18 : 1.));
  if (wide) {
    const int s256 = worthwhile_splits(most, k256.tiles(p), 256 * 2);
    add(ConvTile::k256x128, s256, time(k256, s256) * (p.own ? 1. : kConvMargin));
  }
  if (spares_columns_96(p.Ncols)) {
    const double whole = time(k96, 1) * kConvMargin, split = time(k96, most) * kConvMargin * kConvMargin;
    const bool splits = most > 1 && split < whole;
    add(ConvTile::k256x96, splits ? most : 1, splits ? split : whole);
  }
  return n;
}
// The kernel that gathers tap by tap, `steps` of 32 values: 256 x 96 tiles, never split, instead of 128 x 128?  72 columns, 7 x 7 over 328
// channels, 17 learners of 7 320 positions: 659 us with 128 x 128, 547 with 256 x 96; 448 columns, 3 x 3 over 232, 5 learners of
// 2 772: 132 and 213.
inline bool frag_takes_96(const ConvProduct& p, int steps) {
  static const ConvTileTimes k128 = {128, 128, 3, 4.8, 2.3, {0.43, 0.57, 0.92}, 0.13}, k96 = {256, 96, 2, 5.4, 3.5, {0.68, 1.13, 0}, 0.19};
  if (p.Ncols <= 64 || !spares_columns_96(p.Ncols)) return false;
  const int s128 = worthwhile_splits(p.splits, k128.tiles(p), 256 * 3);
  return conv_time(k96, p, 1, 1, steps) * kConvMargin < conv_time(k128, p, s128, 1, (steps + s128 - 1) / s128);
}

// ---- weight gradient of a convolution with more than 64 output channels, bf16
// M positions, Ncols output channels, cols im2col columns with the bias's, `count` learners.
struct WgradProduct {
  int64_t M;
  int Ncols, cols, count;
  size_t scratch_bytes;
};
// The 128 x 128 tiles of wgrad_panel_kernel, three workgroups on a compute unit, and the three shapes of wgrad_wide_kernel, one.
enum class WgradTile { k128x128, k96x512, k256x256, k384x128 };
struct WgradTiles {
  WgradTile tile;
  int splits;
};
// Times in us: start of a launch, start and end of a workgroup (128 x 128: of three), a step of 32 positions with one (two, three)
// workgroups on a compute unit; steps are faster by `spare` of the part of their loads that brings nothing (output channels and columns
// behind the last, an empty part of the chip).  Fitted to 686 layers of 200 random networks and the AlexNet-shaped one (72 to 512 output
// channels, windows of 2 to 7, 30 to 500 000 positions, 1 to 30 learners), each with every shape at several splits: off by 8
// (the wide shapes) to 13 %.
struct WgradTimes {
  int rows, cols;
  double start, group, step[3], spare;
};
constexpr WgradTimes kWgradTimes[4] = {{128, 128, 2.6, 4.9, {0.37, 0.52, 0.745}, 0.18},
                                       {96, 512, 3.2, 10.0, {0.80, 0, 0}, 0.21},
                                       {256, 256, 2.8, 11.4, {0.78, 0, 0}, 0.31},
                                       {384, 128, 2.9, 9.3, {0.67, 0, 0}, 0.33}};
inline double wgrad_time(WgradTile tile, const WgradProduct& p, int splits) {
  const WgradTimes& t = kWgradTimes[(int)tile];
  const int64_t down = (p.Ncols + t.rows - 1) / t.rows, across = (p.cols + t.cols - 1) / t.cols;
  const int64_t groups = down * across * p.count * splits, each = (groups + 255) / 256, steps = ((p.M + 31) / 32 + splits - 1) / splits;
  const double load = ((double)p.Ncols / down + (double)p.cols / across) / (t.rows + t.cols);
  const double faster = 1. - t.spare * (1. - load * groups / (256. * each));
  double us = t.start + 4.5 + 4e-6 / 6. * splits * p.count * p.Ncols * (p.cols + 7);        // and the second pass
  if (tile == WgradTile::k128x128) {
    const int left = (int)(each % 3);
    us += (each / 3 * t.step[2] + (left ? t.step[left - 1] : 0.)) * steps * faster + (double)((each + 2) / 3) * t.group;
  } else {
    us += each * (t.group + t.step[0] * steps * faster);
  }
  return us;
}
// The cheapest of 128 x 128 tiles at 600 workgroups (choose_splits) and every shape at splits that fill one to six rounds of the chip.
// wide_ok: wgrad_wide_kernel takes the layer.
// Against the first alone: of those layers 16 more than 3 % behind (7 more than 6 %, 10 at most), all together 86 % of its time.  With times
// that were fitted to the AlexNet-shaped layers alone: 99 (46), by up to 29 % (3 x 3 over 160 channels, 144 output channels, 8 learners of
// 2 048 positions: 28 and 36 us), 88 %.
inline WgradTiles wgrad_tiles(const WgradProduct& p, bool wide_ok) {
  const int64_t steps = (p.M + 31) / 32;
  const size_t part = (size_t)p.Ncols * (p.cols + 7) * 4;
  const int64_t held = (int64_t)(p.scratch_bytes / part), most = held < 1 || steps < 8 ? 1 : held < steps / 4 ? held : steps / 4;
  const int64_t plain = (int64_t)((p.Ncols + 127) / 128) * ((p.cols + 127) / 128);
  WgradTiles best{WgradTile::k128x128, choose_splits(plain, p.count, (int)steps, part, p.scratch_bytes)};
  double least = wgrad_time(best.tile, p, best.splits);
  for (int k = 0; k < (wide_ok ? 4 : 1); k++) {
    const WgradTimes& t = kWgradTimes[k];
    const int64_t tiles = (int64_t)((p.Ncols + t.rows - 1) / t.rows) * ((p.cols + t.cols - 1) / t.cols) * p.count;
    for (int round = 0; round <= 6; round++) {
      int64_t sp = round ? round * 256 / tiles : 1;
      if (sp > most) sp = most;
      if (sp < 1) continue;
      const int64_t each = (steps + sp - 1) / sp;
      sp = (steps + each - 1) / each;                  // no workgroup without a step
      const double us = wgrad_time((WgradTile)k, p, (int)sp) * (k ? 1. : 1.01);
      if (us < least) {
        least = us;
        best = WgradTiles{(WgradTile)k, (int)sp};
      }
    }
  }
  return best;
}

// ---- weight gradient of a stride-1 convolution with up to 64 output channels, bf16
// Forms of wgrad_strip_kernel: 32 TM output channels, WN TN blocks of 32 im2col columns a workgroup, MT positions a tile.
struct StripForm {
  int TM, WN, TN, MT;
};
constexpr StripForm kStripForms[5] = {{2, 2, 4, 256}, {2, 4, 4, 256}, {1, 1, 8, 512}, {1, 2, 8, 256}, {1, 4, 7, 256}};
struct StripLayer {
  int M, Ncols, C, ks, OH, OW, W, pad, count;
  size_t scratch_bytes;
};
struct StripPlan {
  int form, PW;              // kStripForms, patch width in pixels
  int groups, tiles, per, splits;   // column groups; tiles of positions, how many a workgroup takes, workgroups along them
  int patch, buf;            // bytes of a patch and of a whole buffer (dy, patch, places) in LDS
  size_t lds;
};
// Does the kernel take the layer, and how?
inline bool strip_plan(const StripLayer& g, StripPlan* p) {
  if (g.Ncols > 64 || g.OW + g.ks - 1 != g.W + 2 * g.pad) return false;
  const int kcols = g.ks * g.ks * g.C, panels = (kcols + 31) / 32;
  p->form = g.Ncols > 32 ? (panels < 8 ? 0 : 1) : panels < 8 ? 2 : panels < 16 ? 3 : 4;
  const StripForm& f = kStripForms[p->form];
  p->PW = g.OW + g.ks - 1;
  const int rows = (f.MT + g.OW - 2) / g.OW + 1;             // output rows a tile can touch
  const int images = (rows + g.OH - 2) / g.OH + 1;           // and images those rows can belong to
  const int64_t patch = ((int64_t)(rows + (g.ks - 1) * images) * p->PW * g.C * 2 + 1023) / 1024 * 1024;
  if (patch > 64 * 1024) return false;
  p->patch = (int)patch;
  p->buf = f.TM * f.MT * 64 + p->patch + f.MT * 4;
  p->lds = 2 * (size_t)p->buf > 8 * 4096 ? 2 * (size_t)p->buf : 8 * 4096;
  if (p->lds > 160 * 1024) return false;
  p->groups = (panels + f.WN * f.TN) / (f.WN * f.TN);        // with the bias's place
  // Below this the tiles a workgroup has to itself are too few to pay for its start and its sum over the position groups
  // (CIFAR-shaped conv2, 64 images of one learner: 11 us with the gathering kernel, 14 here; 8 x 64 images: 25 and 19).
  if ((int64_t)g.M * p->groups * g.count < 65536) return false;
  p->tiles = (g.M + f.MT - 1) / f.MT;
  // one workgroup a compute unit: whole rounds of 256 of them
  const int64_t held = (int64_t)(g.scratch_bytes / ((size_t)g.Ncols * (kcols + 8) * 4));
  const int most = held < 1 ? 1 : held < p->tiles ? (int)held : p->tiles, fill = 256 / (p->groups * g.count);
  const int want = fill < 1 ? 1 : fill < most ? fill : most;
  p->per = (p->tiles + want - 1) / want;
  p->splits = (p->tiles + p->per - 1) / p->per;
  return true;
}

// Can the kernel read the gradient of the 3 x 3 / 2 pooling's output behind the layer instead of the layer's own?  A tile has to be whole
// 2 x 2 blocks of one image each: rows in pairs, and a whole number of pairs a tile.  Wherever it can, it is no slower than the pooling
// layer's kernel in front of it: of 16 calls of one learner x 64 images to 18 x 128, the whole calls took 0.4 to 12 % less.
inline bool strip_pools(const StripPlan& p, int OH, int OW) { return OH % 2 == 0 && OW % 2 == 0 && kStripForms[p.form].MT % (2 * OW) == 0; }
// A thread's part of such a tile there: 8 channels (of 32 * panels) of a 2 x 2 block, which are the output positions `first`, first + 1, first + OW
// and first + OW + 1 of the tile and lie in the window of that block and those above, left and above left of it.  by_ow(n) is n / OW.
struct PoolBlock { int chunk, row, col, first; };
template <class ByOW>
constexpr PoolBlock pool_block(int tid, int panels, int OW, ByOW by_ow) {
  const int block = tid / (panels * 4), row = (int)by_ow((uint32_t)block * 2), col = block - row * (OW >> 1);
  return {tid & (panels * 4 - 1), row, col, row * 2 * OW + 2 * col};
}

// ---- fully connected layers over all rows of a weight version, bf16
// Tiles of 64 tm rows x 128 columns and splits of the contraction (K values, in stages of 64).  The least of: rounds of one
// workgroup per compute unit (two of the smallest fit, but what they wait for is the LDS, which they share), each its start and its
// stages, or the weights at the rate at which they stream in; and, split, the partial sums' way through memory and a second launch.
// In us, fitted to 240 products (K = 104 to 9 216, N = 104 to 9 216, 8 to 576 rows, 1 to 18 versions), each with 4 heights and
// 10 splits: what this takes is within 2 % of the best on average and a third behind it at most (of 12 to 20 us).
struct FcRowsChoice {
  int tm, splits;
};
inline FcRowsChoice fc_rows_choice(int K, int N, int rows, int groups, size_t scratch_bytes) {
  static const double kStage[4] = {0.306, 0.478, 0.611, 0.766};
  const int steps = (K + 63) / 64;
  const int64_t part = (int64_t)rows * N * 4;                     // partial sums of a split, a version
  const double stream = 0.187e-6 * 2. * (double)K * N * groups;
  FcRowsChoice best = {1, 1};
  double least = 0.;
  for (int tm = 1; tm <= 4; tm++) {
    if (tm > 1 && 64 * (tm - 1) >= rows) break;                   // a smaller tile holds them all
    const int64_t tiles = (int64_t)((rows + 64 * tm - 1) / (64 * tm)) * ((N + 127) / 128) * groups;
    // A second pass is a launch more than it costs itself: a contraction of less than 18 stages is not worth it (512 -> 64, 14 rows of 7 versions 10.3 us
    // with that launch, 7.7 without; 1 024 -> 1 024, 64 rows 11.6 and 11).  Beyond 16 splits each keeps nine stages: 184 320 -> 8, 78 rows 58 us with 16
    // splits of two tiles, 25 with 126; 357 216 -> 88, 57 rows 176 and 47 (from 9 729 inputs on).
    const int most = steps < 18 ? 1 : steps / 9 <= 16 ? 16 : steps / 9 < 128 ? steps / 9 : 128;
    for (int sp = 1; sp <= most; sp++) {
      const int per = (steps + sp - 1) / sp;
      if (sp > 1 && (per < 2 || (steps + per - 1) / per != sp || part >= (int64_t)1 << 31 || (uint64_t)part * sp > scratch_bytes)) continue;
      const double work = (double)((tiles * sp + 255) / 256) * (per * kStage[tm - 1] + 0.48 + 0.64 * tm);
      const double w2 = work * work, s2 = stream * stream;
      double us = 0.;
      // (work^4 + stream^4)^(1/4): the larger, and a little more where they are alike
      us = __builtin_sqrt(__builtin_sqrt(w2 * w2 + s2 * s2));
      if (sp > 1) us += 0.344e-6 * (double)part * sp * groups + 1.4;
      if ((tm == 1 && sp == 1) || us < least) { least = us; best = {tm, sp}; }
    }
  }
  return best;
}

// Forward products of at most 32 rows, few enough for a workgroup of 32 columns on every compute unit and up to 2 048 inputs have a kernel without LDS
// (fc_rows_short_kernel).  us, with the launch of a second pass, tiles / that: 512 -> 1 024, one row 10.6 / 5.0; 1 152 -> 512 of 18 versions 16 rows each 13 / 12; 1 536
// -> 64, 16 rows 10.8 / 7.4; 256 -> 4 096 of 7 versions 6.8 / 10.2; 1 024 -> 1 024 of 10, 32 rows 11.8 / 12.6; 4 096 -> 64, 16 rows 11.9 / 14.4.
inline bool fc_rows_short(int K, int N, int rows, int groups) { return rows <= 32 && K <= 2048 && (int64_t)((N + 31) / 32) * groups <= 256; }

// ---- first convolution and max pooling in one kernel
// Is it the faster way for a call of `images`?  Up to 1 024 of them a launch and its round trips are saved whatever the shapes.  Beyond, small images
// leave most of a workgroup's 256 positions empty (bf16, separate kernels / this, us: 96 filters 3 x 3 over 6 x 7 of 16 channels, 1 024 images 20 / 18, 2 048 24 / 31,
// 4 096 33 / 59; 128 over 10 x 7, 4 096 50 / 70; 64 over 8 x 10, 4 096 34 / 33), and many input channels behind few filters or large windows leave little
// but the patch's way to LDS (8 filters 2 x 2 over 16 x 16 of 64 channels, 7 680 images 120 / 151; 64 of 5 x 5 over 18 x 18 of 64 552 / 609; 16 of 3 x 3
// over 32 x 40 of 64, 2 048 images 220 / 182).  Of 302 such layers at 2 to 7 680 images, 4 are behind by more than 3 % now, 43 without the rule.
inline bool conv_pool_wins(int64_t images, int positions, int C, int Ncols, int ks) {
  if (images <= 1024) return true;
  if (positions <= 90) return false;
  return C < 64 || (ks < 5 && (Ncols > 32 || (positions > 128 && (ks > 2 || positions > 400))));
}

// Pooled rows of a workgroup, which walks down them `conv_rows` convolution rows at a time (one row more than two per pooled row), with
// `resident` workgroups on a compute unit, each of which slows the others by a quarter (CIFAR-shaped net, 256 / 576 / 1 152 / 2 304 images at one walk
// an image: 19 / 26 / 41 / 73 us): as little time as possible.
inline int conv_pool_rows(int pooled_rows, int conv_rows, int64_t images, int resident) {
  int best = pooled_rows;
  double least = 0.;
  for (int per = pooled_rows; per >= 1; per--) {
    const int64_t each = ((int64_t)((pooled_rows + per - 1) / per) * images + 255) / 256;
    const int left = (int)(each % resident);
    const double rounds = (double)(each / resident) * (0.75 + 0.25 * resident) + (left ? 0.75 + 0.25 * left : 0.);
    const double cost = rounds * ((2 * per + conv_rows) / conv_rows + 0.3);
    if (per == pooled_rows || cost < least) { best = per; least = cost; }
  }
  return best;
}

// ---- flattening in front of a fully connected layer
// A value a lane, straight from memory to memory, or tiles of 64 channels x 64 positions that a workgroup turns around in LDS.  The tiles' second step
// costs a call of few values 1 us; beyond half a million values the other one's scattered reads cost more (bf16, direct / tiles, forward in us: 64
// channels of 13 x 13, 16 images 3.4 / 5.3; 128 of 20 x 20, 16 images 6.2 / 3.7; 64 of 25 x 25, 16 images 5.6 / 5.5).  Tiles of few channels
// are small, and without whole 16-byte pieces of positions no faster at any size (8 of 45 x 45, 576 images 18.4 / 27.6; 16 of them 47.7 / 31.2).
constexpr int kFlat = 64;
// A tile's side of positions: of a channel one by one, in whole pieces, or all channels' in one run, where the tile holds the whole image; that of up to 128
// positions too, which as 64 and a rest of single ones are slower (9 x 9, 184 channels, 432 images 17 us backward, 13 so).
enum FlatRows { FLAT_ELEMENTS, FLAT_PIECES, FLAT_BLOCK, FLAT_BLOCK_128 };
constexpr int flat_positions_of(int rows) { return rows == FLAT_BLOCK_128 ? 128 : kFlat; }
struct FlattenPlan {
  bool direct;
  bool pieces;       // the tiles' side of channels in whole pieces
  int rows;          // FlatRows
  int64_t groups;    // workgroups of an image
};
inline FlattenPlan flatten_plan(int64_t images, int C, int HW, bool bf16) {
  const int v = bf16 ? 8 : 4;
  FlattenPlan p;
  p.pieces = C % v == 0;
  p.rows = p.pieces && HW <= kFlat ? FLAT_BLOCK : HW % v == 0 ? FLAT_PIECES : p.pieces && HW <= 2 * kFlat ? FLAT_BLOCK_128 : FLAT_ELEMENTS;
  p.direct = images * C * HW <= 1 << 19 || (C <= 8 && HW % v != 0);
  const int positions = flat_positions_of(p.rows);
  p.groups = p.direct ? ((int64_t)C * HW + 255) / 256 : (int64_t)((C + kFlat - 1) / kFlat) * ((HW + positions - 1) / positions);
  return p;
}

// ---- last layer, loss and its input gradient in one kernel
// A workgroup per image reads the layer's weights twice, so for few of them only, and walks the classes one after the other for the input gradient, a lane
// per four inputs: for few classes, or some more behind at least 64 inputs.  Against separate kernels for pooling, flattening, scores, loss,
// input gradient and its re-layout: 1 024 inputs, 10 classes, bf16, 64 / 256 / 2 304 images 9 / 10 / 29 us instead of 27 / 28 / 47 (2 304 in fp32 24
// instead of 41); 512 inputs, 50 classes behind a hidden layer, bf16, 2 304 images 33 instead of 48; whole heads, 1 024 inputs, 31 classes, 1 024 images 46
// instead of 91; 64 and 301, 64 images 50 instead of 55; 8 and 101, 64 images 32 and 32; 8 and 301 50 instead of 40; 32 and 1 001 122 instead of 69.
inline bool head_kernel_wins(int in, int classes) {
  return (int64_t)in * classes <= 32768 && (classes <= 128 || (in >= 64 && classes <= 320));
}

}  // namespace sasgd
