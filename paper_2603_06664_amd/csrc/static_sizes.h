// Which scratch a call is taken with.  Three estimates that once divided the calls and no longer do.  They stay as
// they were, so that what a program may rely on doesn't change whenever the division that is really made
// (choose_plan in attention.hip) is fitted to another kernel:
//   * chunk_attention_static takes a size if the partial results of the division that one of them or
//     choose_plan picks fit the built-in buffer;
//   * chunk_attention takes a workspace of the size that the second or third one asks for, though the fastest
//     division now wants more (1664x960, last chunk: none by the second, 234 MB for two splits now).
#pragma once
#include <algorithm>
#include <cmath>
#include <stddef.h>
#include <stdint.h>
#include "crope_internal.h"

namespace crope {
namespace {

constexpr int kCus = 256;
constexpr int kMaxSplits = 16;
constexpr int kUnitKeys = 64;   // granularity of a key split

size_t partial_bytes(int splits, int n_q, int n_heads) {
  return splits == 1 ? 0 : (size_t)splits * n_heads * n_q * (kHeadDim + 2) * sizeof(float);
}

// The first estimate: key tiles on the busiest work-group slot.
bool always_fitted_static(int n_q, int n_heads, int64_t n_keys) {
  const int n_tiles = (int)((n_keys + kUnitKeys - 1) / kUnitKeys);
  int best = 1;
  double best_cost = 1e30;
  for (int nw = 4; nw <= 8; nw += 4) {
    const int slots = kCus * (8 / nw);
    const int64_t units = (int64_t)((n_q + 32 * nw - 1) / (32 * nw)) * n_heads;
    for (int s = 1; s <= kMaxSplits && s <= n_tiles; ++s) {
      const int tiles_per = (n_tiles + s - 1) / s;
      if ((int64_t)(s - 1) * tiles_per >= n_tiles) continue;
      const double rounds = (double)((units * s + slots - 1) / slots);
      double cost = rounds * tiles_per * (nw == 8 ? 0.96 : 1.0);
      if (s > 1) cost = 1.05 * (cost + 2.0 + (double)s * n_q * n_heads * 1040.0 / 8.4e6);
      if (cost < best_cost - 1e-9) { best_cost = cost; best = s; }
    }
  }
  return partial_bytes(best, n_q, n_heads) <= (size_t)CROPE_STATIC_SCRATCH_BYTES;
}

// The second one: microseconds, with rates of the kernel of its day.  Returns its number of splits; `waves` pins
// the work-group's size where it isn't 0.
int second_splits(int n_q, int n_heads, int64_t n_keys, int waves) {
  const int n_tiles = (int)((n_keys + kUnitKeys - 1) / kUnitKeys);
  int best = 1;
  const bool huge = (int64_t)n_heads * n_keys > 3000000;
  const bool fitted = huge && always_fitted_static(n_q, n_heads, n_keys);
  const bool from_hbm = n_q <= 256 && (int64_t)n_heads * n_keys * 4 * kHeadDim > (32 << 20) && (!huge || fitted);
  double best_cost = 1e30;
  for (int nw = 4; nw <= 8; nw += 4) {
    if (waves && nw != waves) continue;
    const int bm = 32 * nw;
    const int64_t units = (int64_t)((n_q + bm - 1) / bm) * n_heads;
    for (int s = 1; s <= kMaxSplits && s <= n_tiles; ++s) {
      const int tiles_per = (n_tiles + s - 1) / s;
      if ((int64_t)(s - 1) * tiles_per >= n_tiles) continue;   // would leave an empty split
      const size_t bytes = partial_bytes(s, n_q, n_heads);
      if (huge && s > 1 && s < 8 && !(fitted && bytes <= (size_t)CROPE_STATIC_SCRATCH_BYTES)) continue;
      const double rounds = (double)((units * s + kCus - 1) / kCus);
      const double fill = (double)(units * s) / (rounds * kCus);
      double tile_us = nw == 8 ? std::max(1.15, 1.5 * fill) : std::max(0.62, 1.4 * fill);
      if (from_hbm) tile_us = nw == 8 ? 1.3 + 0.7 * fill : n_q <= bm ? 1.1 + 0.5 * fill : std::max(1.0, 1.4 * fill);
      double cost = rounds * (tiles_per * tile_us + (nw == 8 ? 9.0 : 6.0));
      if (s > 1) cost += 4.5 + 0.3 * s + 0.2e-6 * (double)s * n_q * n_heads * (kHeadDim + 2) * sizeof(float);
      if (cost < best_cost - 1e-9) { best_cost = cost; best = s; }
    }
  }
  return best;
}

// The third one, for the kernels of today: choose_plan before its corrections.
int third_splits(int n_q, int n_heads, int64_t n_keys, int waves) {
  const int n_tiles = (int)((n_keys + kUnitKeys - 1) / kUnitKeys);
  int best = 1;
  const bool huge = (int64_t)n_heads * n_keys > 3000000;
  const bool fitted = huge && always_fitted_static(n_q, n_heads, n_keys);
  const bool from_hbm = n_q <= 256 && (int64_t)n_heads * n_keys * 4 * kHeadDim > (200 << 20);
  double best_cost = 1e30;
  for (int nw = 4; nw <= 8; nw += 4) {
    if (waves && nw != waves) continue;
    const bool wide = nw == 8;
    const int bm = 32 * nw;
    double alone = wide ? 1.15 : 0.74, shared = wide ? 1.13 : 0.84;
    if (from_hbm) {
      alone = wide ? 1.20 : n_q <= bm ? 1.22 : 1.06;
      shared = wide ? 1.38 : n_q <= bm ? 1.36 : 1.06;
    }
    const int64_t units = (int64_t)((n_q + bm - 1) / bm) * n_heads;
    for (int s = 1; s <= kMaxSplits && s <= n_tiles; ++s) {
      int tiles_per = (n_tiles + s - 1) / s;
      if ((int64_t)(s - 1) * tiles_per >= n_tiles) continue;
      const size_t bytes = partial_bytes(s, n_q, n_heads);
      if (huge && s > 1 && s < 8 && !(fitted && bytes <= (size_t)CROPE_STATIC_SCRATCH_BYTES)) continue;
      if (wide) tiles_per = (tiles_per + 1) & ~1;
      const int64_t work_groups = units * s, rounds = (work_groups + kCus - 1) / kCus;
      const double p = shared * (double)work_groups / (double)(rounds * kCus);
      double tile_us = std::sqrt(std::sqrt(alone * alone * alone * alone + p * p * p * p));
      if (wide && s > 1) tile_us *= 1.05;
      double cost = (double)rounds * (tiles_per * tile_us + (wide ? 6.0 : 2.8));
      if (s == 1 && rounds > 1 && (work_groups - 1) % kCus < kCus / 6) cost *= 1.1;
      if (s > 1) cost += 2.9 + 0.48 * s + 0.28e-6 * (double)bytes;
      if (cost < best_cost - 1e-9) { best_cost = cost; best = s; }
    }
  }
  return best;
}

bool always_refused_static(int n_q, int n_heads, int64_t n_keys) {
  const size_t buffer = (size_t)CROPE_STATIC_SCRATCH_BYTES;
  return !always_fitted_static(n_q, n_heads, n_keys) &&
         partial_bytes(second_splits(n_q, n_heads, n_keys, 0), n_q, n_heads) > buffer &&
         partial_bytes(third_splits(n_q, n_heads, n_keys, 0), n_q, n_heads) > buffer;
}

}  // namespace
}  // namespace crope
