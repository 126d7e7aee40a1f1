// Lines between two ways of doing the same work, measured.  Host code only.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace og {

// What a walk's cost per target depends on.  Of a batch: the smallest leaf_max,
// theta and alpha of its boxes.
struct WalkShape {
  bool fp64;      // FP64 pair terms, else mixed
  bool newton;    // no cutoff
  bool ext;       // spline softening, relative criterion or per-particle lengths
  bool relative;  // relative opening criterion: theta unused
  int leaf_max;
  double theta, alpha;
};

// Up to how many targets a walk takes eight lanes per target (k_walk8) instead of
// one (the 64-target walks).  Eight lanes are faster while the 64-target walks cannot fill the
// chip, and as long as their vector loads and per-target tests cost less than
// those walks' idle waves.  Measured, 64-target walk time / eight-lane time
// (mixed | FP64), theta 0.5, leaves of 8:
//   all of     1k      32k     65k     100k    132k    160k    200k     300k     400k targets
//   clustered  3.8|5.3 1.9|2.6 1.5|2.0 1.3|1.8 1.1     1.1|1.7 0.9|1.4  0.8|1.3  0.6|1.0
//   smooth             2.9|3.4 2.2     1.6|1.7 1.2     1.1     0.95|1.1 0.9|1.06
//   isolated   (20k) 2.3|4.7, (50k) 1.2|2.2, (70k) 1.0, (100k) 0.76|1.4, (200k) 0.5|0.9
//   list of 2M         21|27 (1k)  2.7|3.0 (100k) 1.5|1.9 (200k) 1.2|1.6 (300k)
//                      0.94|1.35 (400k) 0.7|1.0 (600k)
//   list of 1M isolated (70k) 1.4|2.0, (100k) 1.0|1.5, (150k) 0.75|1.1, (250k) -|0.75
// so the line lies at 160k (mixed) and 320k (FP64), lower without a cutoff (no
// node is pruned, so a 64-target wave's lanes mostly agree), and up to twice as
// high for lists of a quarter of the particles or less, whose targets lie apart.
// A small theta and small leaves lower it: targets open more nodes, and
// neighbours more of the same ones, which a 64-target wave reads once.  Targets
// at which both take the same time, all of a box in thousands (mixed | FP64):
//   theta            0.2       0.3       0.4       0.5
//   leaves of 1      33|125    75|265    145|280   160|290
//   leaves of 2      45|175    95|280    150|285   160|290
//   leaves of 4      82|285    105|295   155|300   160|308
//   leaves of 8      100|320   128|320   160|320   160|320
//   isolated, of 1   42|75     50|85               62|130
//   isolated, of 8   48|150    60|150              70|150
// and for lists of 300k | 700k | 3M, mixed: theta 0.2 leaves of 1 100|85|140,
// of 8 115|115|160; theta 0.3 150|110|260, 170|148|270.  Below theta 0.2 little
// changes.  Long pair terms weigh on both walks alike, so with spline softening
// or lengths theta matters less (0.2, leaves of 8: over 160; of 1: 50).
inline uint32_t eight_lane_line(const WalkShape &w, bool list, uint32_t n_particles) {
  const double k = w.leaf_max >= 8 ? 0.0 : std::log2(8.0 / std::max(w.leaf_max, 1));
  // how far theta lies below 0.45, up to where the line stops falling
  const double below = w.relative ? 0.0 : std::max(0.0, 0.45 - w.theta);
  const double d = std::min(below, w.fp64 ? 0.3 : 0.25);
  const double e = w.relative ? 0.0 : std::min(0.17, std::max(0.0, 0.4 - w.theta));  // mixed walks with a cutoff
  const double base = w.newton ? (w.fp64 ? 150e3 : 70e3) : (w.fp64 ? 320e3 : 160e3);
  // The line of a whole box as a share of `base`: straight lines through the times
  // above, in theta and in halvings of the leaf size (k).
  double f;
  if (w.relative && w.fp64) f = 1.0 - 0.015 * k;
  else if (w.relative) f = 1.0 - (w.alpha < 0.001 ? 0.18 : w.alpha < 0.005 ? 0.1 : 0.0) * std::max(0.0, k - 1.0);
  else if (w.newton && w.ext) f = 1.0 - (w.fp64 ? 0.27 : 0.3) * k * d;
  else if (w.ext) f = w.fp64 ? 1.0 - k * (0.01 + 0.2 * d) : 1.0 - k * d;
  else if (w.fp64) f = 1.0 - k * (w.newton ? 0.035 + 0.68 * d : 0.008 + 0.87 * d);
  else if (w.newton) f = w.leaf_max == 1 && w.theta < 0.15 ? 0.0 : 1.0 - d * (1.5 + 0.1 * k);
  else f = 1.0 - 0.004 * k - e * (2.0 + 0.9 * k);
  double line = base * f;
  if (list) {
    const double quarter = n_particles / 4;
    if (w.newton) {
      const double above = w.relative ? 0.0 : std::min(0.3, std::max(0.0, w.theta - 0.5));
      const double most = w.fp64 ? 150e3 * (1.0 - d * (1.8 + 0.25 * k) + 1.2 * above)
                                 : 100e3 * (1.0 - d * (1.5 + 0.2 * k) + 0.5 * above);
      line = std::min(most, std::max(line, quarter));
    } else if (w.fp64) {
      line = std::max(line, std::min(2.0 * base * (1.0 - d * (0.7 + 0.65 * k)), quarter * (1.0 - 0.6 * k * d)));
    } else {
      const double all = base * (1.0 - e * (1.4 + 0.45 * k));  // of a list whatever the box
      const double far = std::min(below, 0.3);
      line = std::max({line, all, std::min(2.0 * base * (1.0 - 8.5 * far * far), quarter * (1.0 - e * (1.9 + 0.55 * k)))});
    }
  }
  return (uint32_t)std::max(0.0, line);
}

// From how many caller-order particles the mesh deposit goes by blocks of 8^3
// cells (the particles' numbers sorted by block first) instead of eight atomics a
// particle, on a mesh of n^3 cells.  Measured, whole call, us, atomics|blocks:
// clustered particles in random order on 256^3 1117|1037 at 5e5, 1953|1347 at
// 2e6, on 128^3 522|309 at 4e5, 1046|404 at 1e6, on 512^3 8322|8642 at 1e6,
// 8939|8910 at 2e6, 9584|9194 at 3e6; grid order, whose atomics mostly hit one
// line per wave, on 256^3 946|980 at 5.1e5, 1032|1018 at 1e6, on 128^3 229|241
// at 5.1e5, 263|259 at 1e6, on 512^3 8123|8524 at 1e6, 8378|8682 at 2.1e6,
// 8666|8898 at 3.4e6.  A block's own cost (its nodes stored, its halo written and
// read) does not shrink with its particles, so a large mesh needs more of them.
inline uint64_t block_deposit_line(uint64_t n) { return std::max<uint64_t>(500000, n * n * n / 34); }

}  // namespace og
