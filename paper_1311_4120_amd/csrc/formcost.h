// Which form and chunk the sums of a tuned JGB_MIXED plan take.  Host code
// without device dependencies, so that the CPU tests cover it.
//
// In float32 the order of a sum decides its last digits: E moves by up to some
// 1e-7 from one form or chunk to another (its error against 64-bit sums is some
// 5e-7 in each), and a program's results should not move with the speed of a
// kernel or the noise of a timing.  Forms and chunks therefore follow from what
// the plan counts: the times below, in microseconds, are those of the kernels
// with which plans that timed their forms gave the results that programs know
// (the present gather, rings and tiles load a batch ahead and are faster),
// fitted to some 1950 3D node sets of 16^3 to 256^3 points, 64 to 4 million half-set
// nodes, 4 to 8 taps and the Gaussian's 12, each form and chunk of which was
// timed twice.  Where both timings of a node set took the same, the costs take
// it too for 95% of 1023 node sets of common sizes (94% of those that a fit to
// the others left out), all of 120 planar ones (not fitted), and 86% of a grid of
// 282 sparse, dense and elongated ones; where they do not, the choices lay within
// a few percent of each other, mostly the noise of a timing.
// The staged interpolation's chunk moves no result by more than the rounding of
// E's float64 sum and is still timed.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace jgb {
namespace formcost {

// The node set: half-set nodes, taps, entries of the gather's lists, and of
// the ring lists (node entries, rings).
struct Nodes {
  double nodes, width, entries, ring_entries, rings;
};

// A launch's work items: how many, the partial tiles among them, the most
// partial tiles of one tile, and the longest item's entries (rings: of one of
// its wavefronts).
struct Items {
  double count, slots, most, longest;
};

// A launch of independent items ends with the later of all its work and its
// longest item, and somewhat later where both take as long.
inline double either(double all, double longest, double p) {
  const double m = std::max(all, longest);
  return m * std::pow(std::pow(all / m, p) + std::pow(longest / m, p), 1.0 / p);
}

// The second launch, where tiles are split: all partial tiles, or one tile's
// one after the other.
inline double partials(const Items& it, double start, double slot, double chain) {
  return it.slots > 0 ? start + std::max(slot * it.slots, chain * it.most) : 0.0;
}

// 0 .. 1: how far the nodes' records (MB) outgrow a cache of `mb`; the larger
// `sharp`, the sharper the turn (4 MB of L2 per XCD for the gather and the rings).
inline double beyond(const Nodes& n, double mb, double sharp) {
  return 1.0 / (1.0 + std::pow(mb / (n.nodes * (3 * n.width + 3) * 4e-6), sharp));
}

// 16-byte pieces of a record that each lane of the gather and the rings copies,
// against the two of 5 to 10 taps.
inline double pieces(const Nodes& n) { return std::ceil(std::ceil((3 * n.width + 3) / 4) / 4) - 2; }

inline double gather(const Nodes& n, const Items& it) {
  const double f = 1 + 0.112 * pieces(n);
  return 7.71 + either(2.91e-5 * f * n.entries + 0.00175 * it.count, 0.01538 * f * (1 + 0.66 * beyond(n, 4.13, 5)) * it.longest, 4) +
         partials(it, 1.36, 0.00175, 0.111);
}
inline double rings(const Nodes& n, const Items& it) {
  const double f = 1 + 0.091 * pieces(n);
  return 8.77 + either(f * (2.23e-5 * n.ring_entries + 7.7e-5 * n.rings) + 0.00782 * it.count,
                       0.0483 * f * (1 + 0.086 * beyond(n, 3.7, 35)) * it.longest, 10) +
         partials(it, 1.8, 0.00812, 0.0936);
}
// it: the items of the untuned gather, whose lists the tiles then shared
inline double tiles(const Nodes& n, const Items& it) {
  const bool wide = n.width > 8;  // the twelve taps of the Gaussian
  return 7.78 + either(1.72e-6 * (wide ? 0.7 : 1.0) * n.entries * n.width + 0.00255 * it.count,
                       0.00348 * (wide ? 1.06 : 1.0) * (1 + 3.8 * beyond(n, 0.0106, 1)) * it.longest, 5) +
         std::max(2.3e-5 * n.nodes, 1.08e-5 * n.entries) + 0.125 * n.entries / n.nodes;
}
inline double staged(const Nodes& n, double count, double longest) {
  if (n.width > 8) return 10.4 + either(3.08e-4 * n.nodes + 0.0316 * count, 0.071 * longest, 5);
  return 8.18 + either(3.55e-5 * n.nodes * std::sqrt(n.width) + 0.0129 * count, 0.027 * longest, 5);
}

// Ring items from which on the two longest chunks cost the same: with 21 254 of
// them (256^3) they are 0.1 to 0.6% apart, and plans that timed them took
// either, the shorter 30 times of 61 -- the one taken here.  With 17 722 (240^3)
// the longer one was taken, 0.2 to 1.4% ahead.
constexpr double kManyItems = 20000;

}  // namespace formcost
}  // namespace jgb
