// How many wavefronts take one work item, by what a launch has of items and an item of pixels.
//
// Several wavefronts per item shorten the item's latency, which is a launch's time while its
// items alone leave most of the chip idle; past that they cost: their per-lane sums pass from
// one to the next in turn, and a wavefront without pixels (an item of fewer groups than
// wavefronts) holds its place to the end of the item.  So the line lies the lower the fewer
// groups an item has, and items of hardly more than one group keep one wavefront.  What an item
// has is the mean over the plan's.  Every choice gives the same sums, bit for bit.
//
// All times in us of the kernel, one wavefront per item / several; the pixel kernel's with the
// gradient.  Host code only.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace celmi {

// Pixel kernel: one wavefront, or kWideWaves.  groups: an item's pixels over those that a
// wavefront takes at a time.
//   float32   1 group and less: 870 items 11.9 / 12.7, 2495 items 13.9 / 22.4
//             1.7 groups: 645 items 19.8 / 14.7, 1300 21.1 / 16.8, 2670 25.5 / 28.9
//             2.5 groups: 1815 items 31.9 / 22.7, 3500 36.2 / 36.1, 7725 57.8 / 66.6
//             3.3 groups: 115 items 28.7 / 12.7, 3610 49.3 / 39.0, 10950 98 / 99 (2 pixels a lane);
//             2670 items 30.2 / 23.1, 6995 42.9 / 50.5 (1 pixel a lane)
//   float64   1 group and less: 485 items 15.8 / 17.9, 955 16.2 / 31.6
//             1.7 groups: 250 items 26.2 / 17.7, 550 50.1 / 43.0, 1060 52.7 / 72.2
//             3.3 groups: 550 items 53.9 / 30.2, 1750 75.1 / 68.9, 2195 80.3 / 85.8
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
// or eight wavefronts.  passes: an item's pixels over 64.
//   1 and less: 870 items 14.2 / 19.2 / 40.0
//   1.7 passes: 440 items 21.6 / 18.2 / 22.9, 1265 24.8 / 28.5
//   2.6 passes: 1725 items 34.9 / 35.4
//   3.4 passes: 225 items 35.1 / 18.2 / 22.0, 1300 42.4 / 31.1, 2670 54.6 / 50.7, 5155 80.0 / 85.0
//   5 passes:   875 items 56.2 / 36.5 / 43.5, 1815 62.8 / 59.4, 3500 87.8 / 96.1
//   6.5 passes: 115 items 59.8 / 28.1 / 20.8, 425 70.2 / 30.7 / 26.7, 665 72.0 / 36.1 / 40.0,
//               1985 81.2 / 66.8, 4405 130 / 125, 7650 177 / 192
//   12 passes:  185 items 126 / 52 / 36, 725 141 / 59 / 69, 3110 187 / 154
inline int hessian_waves(double passes, int64_t n_items) {
  if (passes > 4.0 && n_items <= 512) return 8;
  return (double)n_items <= std::min(4608.0, 768.0 * (passes - 1.0)) ? 4 : 1;
}

}  // namespace celmi
