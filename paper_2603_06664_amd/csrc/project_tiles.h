// Work division of the projection: which work-group computes which tiles.  Host and device use the same code, and nothing
// here needs a GPU.
#pragma once
#include "fastdiv.h"

namespace crope {

constexpr int kProjXcds = 8, kProjCusPerXcd = 32;
constexpr int kTokGroup = 4;    // token tiles walked together with 8 pairs of heads by one XCD's CUs

// The output as tiles of one head of q, k or v ("channel tile") x tile_tokens tokens.  Four token tiles make a group, walked channels
// first, tokens within: 32 consecutive units (what an XCD's 32 CUs hold at a time) are 8 x 4 of them, whose W and x tiles
// stream through that XCD's L2 once; every XCD has a run of units.  With `doubles`, a unit is two neighbouring channel tiles; v
// starts at an even one, so that no unit holds k and v, and the odd last one (odd numbers of heads) is one tile.  The first
// `doubles` units of a run are one work-group's each, the others two's (of which the one for a missing tile leaves at once).
// Without, a unit is one tile: units of two gave 4346 tokens x 5 heads, c_in 4608, norm per head, 255 tiles, more than 256
// work-groups and so doubles, 95 us; 71 in one round.
struct ProjTiles {
  int ch_tiles, tok_tiles;
  int total, per_xcd, doubles;   // units
  int pairs;                     // 1: units of two tiles, 0: of one
  FastDiv div_group;             // by the units of a group
};

// What a work-group computes: `heads` (0, 1 or 2) neighbouring channel tiles from ch_tile on, of one token tile.
struct ProjWork {
  int heads, ch_tile, tok_tile;
};

CROPE_HD inline ProjWork project_work(const ProjTiles& pt, uint32_t block) {
  const int idx = (int)(block / kProjXcds), rest = idx - pt.doubles;
  const bool first = rest < 0;   // a whole unit
  const int unit = (int)(block % kProjXcds) * pt.per_xcd + (first ? idx : pt.doubles + (rest >> pt.pairs));
  const int group = (int)fastdiv((uint32_t)unit, pt.div_group), local = unit - group * (int)pt.div_group.d;
  const int left = pt.tok_tiles - kTokGroup * group, gs = left >= kTokGroup ? kTokGroup : left > 1 ? left : 1;
  const int ch = (int)((uint32_t)local * (gs == 3 ? 21846u : 65536u >> (gs >> 1)) >> 16);   // local / gs, local < 32768
  const int ch_tile = (ch << pt.pairs) + (first ? 0 : rest & pt.pairs);
  ProjWork w{1, ch_tile, kTokGroup * group + local - ch * gs};
  if (first && ch_tile + 1 < pt.ch_tiles) w.heads = 2;
  if (unit >= pt.total || ch_tile >= pt.ch_tiles) w.heads = 0;
  return w;
}

// Work-groups of the launch.
inline int project_blocks(const ProjTiles& pt) {
  return (pt.doubles + ((pt.per_xcd - pt.doubles) << pt.pairs)) * kProjXcds;
}

// A one-head work-group's time in two-head ones.
constexpr double kSingleCost = 0.58;

// Time of an XCD's doubles and singles in doubles, when its CUs take the doubles first.
inline double project_span(int doubles, int singles) {
  const int late = doubles % kProjCusPerXcd;   // CUs that are a double behind the others
  double t0 = doubles / kProjCusPerXcd, t1 = t0 + 1.0, end = late ? t1 : t0;
  while (singles > 0) {
    if (late && t0 > t1 && singles > 4 * kProjCusPerXcd) {   // from here on both kinds of CU take turns: whole turns at once
      const int turns = singles / kProjCusPerXcd - 2;
      singles -= turns * kProjCusPerXcd;
      t0 += turns * kSingleCost;
      t1 += turns * kSingleCost;
    }
    double& t = late == 0 || t0 <= t1 ? t0 : t1;
    const int cus = &t == &t0 ? kProjCusPerXcd - late : late;
    const int waves = late == 0 ? (singles + cus - 1) / cus : 1;
    singles -= waves * cus;
    t += waves * kSingleCost;
    end = t > end ? t : end;
  }
  return end;
}

// Two heads per work-group or one.  Two are cheaper per row, one fills the chip more evenly: whole rounds of doubles
// first, what is left in singles where that takes fewer rounds at 0.58 of a double's time (us, mixed / singles / doubles, norm per head, then
// row-wide: 4680 tokens x 12 heads, c_in 1536, 342 pairs on 256 CUs, 63 / 67 / 77, 82 / 87 / 98; 585 x 40, 5120, one round of doubles, 88 /
// 102 / 87, 97 / 114 / 97; 600 x 12, 1536, one round of singles, 19 / 19 / 27, 26 / 26 / 36).  An odd last tile is one tile, not two.
// Equal estimates: as many whole rounds as possible, which move fewer bytes (6241 x 5, c_in 640, 24.5 us with 32 of an XCD's 33
// units in doubles, 28.6 in singles).  340 sizes of odd numbers of heads: 0.2 % behind the fastest of all numbers of rounds on
// average, 11 % at worst; 1.5 and 43 while the odd tile counted as two.
inline ProjTiles make_tiles(int n_tokens, int n_heads, int tile_tokens) {
  ProjTiles pt;
  pt.ch_tiles = 3 * n_heads;
  pt.tok_tiles = (n_tokens + tile_tokens - 1) / tile_tokens;
  const int ch_pairs = pt.ch_tiles / 2, ch_units = pt.ch_tiles - ch_pairs, odd = ch_units - ch_pairs;
  const int all = ch_units * pt.tok_tiles, units = (all + kProjXcds - 1) / kProjXcds;   // per XCD
  const int tiles = (pt.ch_tiles * pt.tok_tiles + kProjXcds - 1) / kProjXcds;
  auto odd_before = [&](int unit) {   // units of one tile before this one
    if (!odd) return 0;
    const int group = unit / (kTokGroup * ch_units), local = unit - group * kTokGroup * ch_units;
    const int left = pt.tok_tiles - kTokGroup * group, in_pairs = (left < kTokGroup ? left : kTokGroup) * ch_pairs;
    return group * kTokGroup + (local > in_pairs ? local - in_pairs : 0);
  };
  pt.doubles = 0;
  double best = project_span(0, tiles);
  for (int r = 1; r <= (units + kProjCusPerXcd - 1) / kProjCusPerXcd; ++r) {   // whole rounds of doubles, the rest in singles
    const int d = r * kProjCusPerXcd < units ? r * kProjCusPerXcd : units;
    double cost = 0.0;
    for (int x = 0; x < (odd ? kProjXcds : 1); ++x) {   // the slowest run; without odd units the first one
      const int u0 = x * units, u1 = u0 + units < all ? u0 + units : all, u = u0 + d < u1 ? u0 + d : u1;
      if (u0 >= u1) break;
      const int lone = odd_before(u) - odd_before(u0), lone_rest = odd_before(u1) - odd_before(u);
      const double c = project_span(u - u0 - lone, lone + 2 * (u1 - u) - lone_rest);
      cost = c > cost ? c : cost;
    }
    if (cost < best - 1e-9 || (d % kProjCusPerXcd == 0 && cost < best + 1e-9)) { best = cost; pt.doubles = d; }
  }
  pt.pairs = pt.doubles > 0;
  pt.total = pt.pairs ? all : pt.ch_tiles * pt.tok_tiles;
  pt.per_xcd = pt.pairs ? units : tiles;
  pt.div_group = make_fastdiv((uint32_t)(kTokGroup * (pt.pairs ? ch_units : pt.ch_tiles)));
  return pt;
}

// Two token widths of a tile.  256 moves fewer bytes per product (18720 tokens x 12 heads, row-wide norm, 306 us, 321 in tiles of
// 192); 192 is taken where its rounds of one-head tiles over the 256 CUs, at 0.88 of the price, are fewer: calls whose rounds of
// 256-wide tiles end nearly empty or that fit one round in either (us, 192 / 256, norm per head, then row-wide: 585 x 40 heads, c_in 5120,
// 88 / 108, 97 / 115; 4680 x 5, 5120, 82 / 96, 93 / 106; 2340 x 12, 1536, 34 / 38, 46 / 51; 600 x 12, 1536, 19 / 22, 26 / 29; but 1560 x 12, 1536,
// 29 / 25, 39 / 34; 3000 x 24, 3072, 153 / 141, 177 / 164; 1000 x 40, 2560, 83 / 66, 99 / 81).
// At reductions of at most 512, 192 has to take fewer rounds at full price.  That line was fitted to a kernel with one head per
// work-group throughout and the epilogue through LDS, and wants a new fit: with this one 192 is the faster at most short reductions (norm
// per head: 200 x 2, 256, 8.3 / 9.5; 540 x 8, 512, 11.4 / 12.8; 4000 x 8, 512, 18.7 / 21.8; 540 x 40, 192, 14.3 / 17.1), though not at all of
// them (8000 x 6, 384, 24.7 / 24.7, row-wide 42.9 / 40.1).
constexpr double kMidCost = 0.88;
constexpr int kShortReduction = 512;

// rounds of a tile per CU
inline int project_rounds(int n_tokens, int n_heads, int tile_tokens) {
  const int total = 3 * n_heads * ((n_tokens + tile_tokens - 1) / tile_tokens);
  return ((total + kProjXcds - 1) / kProjXcds + kProjCusPerXcd - 1) / kProjCusPerXcd;
}

inline int project_tile_width(int n_tokens, int n_heads, int c_in) {
  const double mid_cost = c_in <= kShortReduction ? 1.0 : kMidCost;
  return project_rounds(n_tokens, n_heads, 256) <= project_rounds(n_tokens, n_heads, 192) * mid_cost ? 256 : 192;
}

}  // namespace crope
