// Which kernel and tile a sparse x sparse product runs on (library private; plain C++, also compiled
// on the host by the tests).
#ifndef BSP_SPGEMM_PICK_H
#define BSP_SPGEMM_PICK_H

#include <stdint.h>

#include <cmath>

// The tiled kernel's instances: block rows of A and B per workgroup, LDS buffers of a step (eight block
// columns), and what one of them takes, in us: rounds of `slots` workgroups times (fixed + per step).
struct SpTile {
  int32_t ra, rb, nbuf, slots;
  double fixed, step;
};
enum { SP_TILE_64, SP_TILE_128, SP_TILE_128W, SP_TILE_256, SP_TILES, SP_SELECT = SP_TILES };
constexpr SpTile kSpTile[SP_TILES] = {
    {8, 8, 4, 512, 3.0, 0.48}, {16, 16, 3, 256, 4.0, 0.62}, {16, 32, 3, 256, 5.0, 0.98}, {32, 32, 2, 256, 6.0, 1.8}};

// LDS of a tile: its buffers and a word per (step, block row).  The table of a long inner dimension does
// not fit beside the buffers of the large tiles (128 x 256: 5440 elements, 256 x 256: 8192, 128 x 128:
// 32768, 64 x 64: 98304).
inline int64_t sp_tile_lds(const SpTile& t, int64_t nsteps) { return (t.ra + t.rb) * (t.nbuf * 1024ll + nsteps * 4ll); }
constexpr int64_t kSpLds = 160 * 1024;

// Time by the model, from timings at 512 to 4096, inner dimensions to 16384 and ragged sizes; da, db:
// shares of the blocks that are kept.  For the kernel that selects columns it grows with the share of
// columns that both sides of a tile keep.  4096 x 4096 x 16384, tiled / selecting columns: a fifth kept
// 878 (64 x 64) / 470 us, half kept 608 (128 x 128) / 1343; x 8320, a quarter kept 319 (128 x 128) / 304.
inline double sp_time(int which, int64_t ra, int64_t rb, int64_t nsteps, double da, double db) {
  auto rounds = [&](int64_t tr, int64_t tc, int slots) { return std::ceil((double)((ra + tr - 1) / tr) * (double)((rb + tc - 1) / tc) / slots); };
  const double n = (double)nsteps;
  if (which == SP_SELECT) {
    const double both = (1 - (1 - da) * (1 - da)) * (1 - (1 - db) * (1 - db));
    return rounds(16, 16, 512) * (2 + n * (0.6 + both * (2.6 + 1.9 * both)));
  }
  const SpTile& t = kSpTile[which];
  if (which == SP_TILE_64 && rounds(8, 8, 256) <= 1) return 3.5 + n * 0.38;
  return rounds(t.ra, t.rb, t.slots) * (t.fixed + n * t.step);
}

// The fastest of those that fit.
inline int sp_pick(int64_t ra, int64_t rb, int64_t nsteps, double da, double db) {
  int best = SP_SELECT;
  for (int t = 0; t < SP_TILES; ++t)
    if (sp_tile_lds(kSpTile[t], nsteps) <= kSpLds && sp_time(t, ra, rb, nsteps, da, db) < sp_time(best, ra, rb, nsteps, da, db)) best = t;
  return best;
}

#endif
