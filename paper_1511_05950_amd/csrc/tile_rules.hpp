// Which kernel and which tiles serve a layer, from its sizes.  No HIP types: host code and host tests include it alone.
#pragma once
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
// (3072 x 256 pixels, 4 learners x 2 images: 21 us; a lane per pixel takes 50).
inline int input_row_piece(int Wp) {
  const int pieces = (Wp + 639) / 640;
  return (Wp + pieces - 1) / pieces;
}
// Workgroups of the kPixels kernel a learner: 256 pixels each, counted through all images.
inline int64_t input_pixel_groups(int N, int Hp, int Wp) {
  const int64_t groups = ((int64_t)N * Hp * Wp + 255) / 256;
  return groups < 16384 ? groups : 16384;
}

}  // namespace sasgd
