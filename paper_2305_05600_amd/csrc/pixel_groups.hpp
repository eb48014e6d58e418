// Splitting of a batch of images into launches whose pixels are counted in 32
// bits.  Plain C++ (host only).
#pragma once

#include <stdint.h>

namespace hvpic {

// most pixels of a launch: the kernels form the index of a tile's last lane,
// and that of the pixels past the end, in 32 bits
constexpr int64_t kMaxLaunchPixels = int64_t(1) << 31;

// Calls f(first pixel, pixels) for groups of whole images of P pixels (at most
// kMaxLaunchPixels each) that make up the N pixels of a batch.
template <class F>
void for_pixel_groups(int64_t N, int64_t P, F f) {
  const int64_t images = kMaxLaunchPixels / P, step = (images > 0 ? images : 1) * P;
  for (int64_t p = 0; p < N; p += step) f(p, N - p < step ? N - p : step);
}

}  // namespace hvpic
