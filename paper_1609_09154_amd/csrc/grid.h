// Launch-size cap shared by the kernels whose grids grow with the data.
#pragma once

#include <stdint.h>

namespace nmfk {

// A dispatch counts the work-items of each grid dimension in 32 bits, so a
// grid that grows with the data (rows x KP copies, one wavefront per row of a
// 10^8-row factor) is capped at GRID_CAP blocks and its kernel strides over
// the remaining blocks; below the cap the grid is unchanged.
constexpr int64_t GRID_CAP = (int64_t)1 << 20;
inline unsigned capped_grid(int64_t blocks) {
  return (unsigned)(blocks < 1 ? 1 : (blocks > GRID_CAP ? GRID_CAP : blocks));
}

// How full the rounds of `slots` workgroups are with t slabs of wgs workgroups
// each, after what the slabs cost (`cost` of the product's time for each slab
// beyond none: the slab is written and read once more).
inline double round_score(int64_t wgs, int64_t t, int64_t slots, double cost) {
  const double rounds = (double)(wgs * t) / (double)slots;
  return rounds / (double)cdiv(wgs * t, slots) / (t > 1 ? 1.0 + cost * (double)t : 1.0);
}

// The slab count with the fullest rounds, of s and the counts above it that fit
// (ok, up to the first that does not).
template <typename Ok>
inline int64_t fullest_rounds(int64_t wgs, int64_t s, int64_t slots, double cost, Ok ok) {
  int64_t best = s;
  double top = round_score(wgs, s, slots, cost);
  for (int64_t t = s + 1; ok(t); ++t) {
    const double score = round_score(wgs, t, slots, cost);
    if (score > top) best = t, top = score;
  }
  return best;
}

// The slab count of a split reduction, from s (a grid of wgs workgroups per
// slab that fills `slots` of them at least once): where the last round of
// workgroups would be mostly empty, a count between s / 2 and 4 s that fits
// (ok) and whose rounds are fuller by a tenth after what its slabs cost. Rounds
// are an estimate, since workgroups do not end
// together, so a smaller gain is not taken.
template <typename Ok>
inline int64_t full_rounds(int64_t wgs, int64_t s, int64_t slots, double cost, Ok ok) {
  if (wgs * s <= slots) return s;
  auto score = [&](int64_t t) { return round_score(wgs, t, slots, cost); };
  int64_t best = s;
  double top = 1.1 * score(s);
  for (int64_t t = cdiv(s, 2); t <= 4 * s; ++t)
    if (ok(t) && score(t) > top) best = t, top = score(t);
  return best;
}

}  // namespace nmfk
