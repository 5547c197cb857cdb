// How many wavefronts take one work item, by what a launch has of items and an item of pixels.
//
// Several wavefronts per item shorten the item's latency, which is a launch's time while its
// items alone leave most of the chip idle; past that they cost: their per-lane sums pass from
// one to the next in turn, and a wavefront without pixels (an item of fewer groups than
// wavefronts) holds its place to the end of the item.  So the line lies the lower the fewer
// groups an item has, and items of one group keep one wavefront.  What an item has is the mean
// over the plan's, parts of groups counted whole.  Every choice gives the same sums, bit for bit.
//
// All times in us of the kernel, one wavefront per item / several; the pixel kernel's with the
// gradient.  Host code only.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace celmi {

// Groups of `group` pixels in a patch of n_pixels that is cut into items of item_pixels (the last
// one shorter): the passes that a wavefront makes, the partly filled ones counted whole.
inline int64_t patch_groups(int64_t n_pixels, int64_t item_pixels, int64_t group) {
  const auto up = [group](int64_t n) { return (n + group - 1) / group; };
  return n_pixels / item_pixels * up(item_pixels) + up(n_pixels % item_pixels);
}

// Pixel kernel: one wavefront, or kWideWaves.  groups: of as many pixels as a wavefront takes at a
// time.
//   float32   1 group: 870 items 11.3 / 11.8, 2495 items 13.9 / 20.8
//             1.9 groups: 645 items 19.4 / 13.1, 1300 21.1 / 16.4, 2670 25.0 / 26.9
//             2.6 groups: 1815 items 31.0 / 21.6, 3500 36.3 / 34.2, 7725 58.1 / 61.7
//             3.5 groups: 115 items 27.8 / 11.7, 3610 49.1 / 37.7, 10950 95.5 / 92.0 (2 pixels a
//             lane); 2670 items 30.0 / 22.0, 6995 43.4 / 46.9 (1 pixel a lane)
//   float64   1 group: 485 items 15.7 / 17.3, 955 15.6 / 29.9
//             1.9 groups: 250 items 25.5 / 16.9, 550 49.5 / 40.6, 1060 51.3 / 66.4
//             3.5 groups: 550 items 53.7 / 28.9, 1750 75.1 / 66.3, 2195 78.4 / 82.9
constexpr int kWideWaves = 4;
inline bool wide_pixels(bool fp64, double groups, int64_t n_items) {
  const double most = fp64 ? std::min(2048.0, 768.0 * (groups - 1.0)) : std::min(4096.0, 2048.0 * (groups - 1.0));
  return (double)n_items <= most;
}

// Map kernel: one wavefront with several pixels per lane, or as many wavefronts with one (no
// sums to hand on; a short item costs one wavefront as much as a whole group).
//   float32   20 items 11.9 / 9.1, 1065 15.9 / 14.6, 1895 18.8 / 19.4, 5850 31.7 / 38.0
//             (64-pixel items: 1070 9.8 / 8.6, 7735 20.3 / 27.3)
//   float64   465 items 27.6 / 21.5, 870 30.3 / 31.7, 1240 44.8 / 39.0, 2395 58.3 / 58.6
inline bool wide_maps(bool fp64, int64_t n_items) { return n_items <= (fp64 ? 512 : 1024); }

// Hessian kernel, float32 (the double form's sums alone fill a wavefront's registers): one, four
// or eight wavefronts.  passes: of 64 pixels.
//   1 pass:     870 items 14.2 / 19.2 / 40.0
//   1.9 passes: 440 items 21.6 / 18.2 / 22.9, 1265 24.8 / 28.5
//   2.8 passes: 1725 items 34.9 / 35.4
//   3.6 passes: 225 items 35.1 / 18.2 / 22.0, 1300 42.4 / 31.1, 2670 54.6 / 50.7, 5155 80.0 / 85.0
//   5.2 passes: 875 items 56.2 / 36.5 / 43.5, 1815 62.8 / 59.4, 3500 87.8 / 96.1
//   6.8 passes: 115 items 59.8 / 28.1 / 20.8, 425 70.2 / 30.7 / 26.7, 665 72.0 / 36.1 / 40.0,
//               1985 81.2 / 66.8, 4405 130 / 125, 7650 177 / 192
//   12 passes:  185 items 126 / 52 / 36, 725 141 / 59 / 69, 3110 187 / 154
inline int hessian_waves(double passes, int64_t n_items) {
  if (passes > 4.0 && n_items <= 512) return 8;
  return (double)n_items <= std::min(4608.0, 768.0 * (passes - 1.0)) ? 4 : 1;
}

}  // namespace celmi
