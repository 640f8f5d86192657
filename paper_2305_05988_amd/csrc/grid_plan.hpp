// Which grids the plane sweep (grid.hpp) takes, and how it cuts them.  Host
// code without HIP.
#pragma once

#include <algorithm>
#include <cstdint>

namespace its {

constexpr int kGridThreads = 256;  // threads per block of the sweep

struct GridPlan {
  int32_t W, H, ntx, nty, zb, ncz;  // tile, tiles in x and y, planes per chunk, chunks
};

// Tiles that cover the grid with the least points loaded and thread slots
// spent, the ring at most one point per thread; then z chunks for about
// `blocks` blocks of at least 4 planes.  R: points per thread.
// lines: tiles of whole 128-byte lines (16 points).
inline GridPlan grid_plan(int32_t nx, int32_t ny, int32_t nz, int R, int blocks, bool lines) {
  GridPlan best{1, 1, 1, 1, 1, 1};
  double cost = 1e300;
  auto consider = [&](int32_t W) {
    int32_t H = std::min(kGridThreads * R / W, 126 - W);
    H = std::min(H, ny);
    if (H < 1) return;
    const int32_t ntx = (nx + W - 1) / W, nty = (ny + H - 1) / H;
    H = (ny + nty - 1) / nty;
    const double c = double(ntx) * nty * (0.5 * kGridThreads * R + double(W + 4) * (H + 2));
    if (c < cost) {
      cost = c;
      best = GridPlan{W, H, ntx, nty, 1, 1};
    }
  };
  if (lines) {
    for (int32_t W = 96; W >= 48; W -= 16) consider(W);  // the wider of equals
  } else {
    const int32_t least = (nx + 109) / 110;
    for (int32_t ntx = least; ntx <= least + 6 && ntx <= nx; ++ntx) consider((nx + ntx - 1) / ntx);
  }
  const int64_t tiles = int64_t(best.ntx) * best.nty;
  int64_t chunks = std::max<int64_t>(1, blocks / tiles);
  chunks = std::min<int64_t>(chunks, std::max(1, nz / 4));
  best.zb = int32_t((nz + chunks - 1) / chunks);
  best.ncz = (nz + best.zb - 1) / best.zb;
  return best;
}

// The share of its blocks' point slots that a plane of the grid fills: a block
// has no more than a column of planes, so on a long duct the others idle.
inline double grid_fill(int32_t nx, int32_t ny, const GridPlan &g, int R) {
  return double(nx) * ny / (double(g.ntx) * g.nty * kGridThreads * R);
}

struct GridShape {
  int points;  // per thread
  GridPlan plan;
  double fill;
};

// npts: 7, 27, or 1 for variable coefficients.
//
// By the size of the grid alone, as measured on 7 points in FP64 (27 points and
// the refinement's FP32 take the same).  Four points per thread in 512 blocks (two
// per CU, all resident) from 5 * 2^20 points on: CG 256^3 164 us an iteration, 174 with 1024 blocks, 179 with two
// points; below, two points in 768 blocks: BiCGStab 160x144x150 78.3 us against
// 82.4 with four, CG 150^3 42.2 against 43.1 with 1024 blocks.  Variable
// coefficients: two points in 512 blocks (four do not leave registers for two
// blocks on a CU; 128^3 42.9 us against 44.5 with 768).  Tiles that four points
// per thread would leave half empty take two: CG 16x16x31250 136 us and 100.
//
// From 2^23 points on, where the vectors stream past the caches (grid_run), a
// line of memory that two tiles share is moved twice and stored in two parts:
// tiles of whole lines there, where the grid's own lines start at even points
// and are long enough to cut.  CG 272^3 in tiles of 39 points 342 us an iteration
// (bricks 250), of 48 220; 400^3 1024 (841) and 688, 250^3 231 (208) and 186; one
// product of 800x800x100 291 (219) and 216.  Tiles of 32 lose to the ring.
inline GridShape grid_shape(int npts, int32_t nx, int32_t ny, int32_t nz) {
  const int64_t n = int64_t(nx) * ny * nz;
  const bool var = npts == 1, lines = !var && n >= (int64_t(1) << 23) && nx % 2 == 0 &&
                                     (nx >= 96 || (nx >= 64 && nx % 8 == 0));
  GridShape s;
  s.points = !var && n >= (5 << 20) ? 4 : 2;
  for (;;) {
    s.plan = grid_plan(nx, ny, nz, s.points, var || s.points == 4 ? 512 : 768, lines);
    s.fill = grid_fill(nx, ny, s.plan, s.points);
    if (s.points == 2 || s.fill >= 0.5) return s;
    s.points = 2;
  }
}

// The same share of the brick march's 64 x 4 tiles (brick.hpp).
inline double brick_fill(int32_t nx, int32_t ny) {
  return double(nx) * ny / (double((nx + 63) / 64) * ((ny + 3) / 4) * 256.0);
}

// Whether the sweep takes the grid of a matrix-free operator, or that of a
// packed matrix, which the pattern walk (pattern.hpp) would take otherwise.
//
// From 360,448 points on; per iteration, packed rows (or bricks) and planes:
// packed CG 64^3 13.2 and 16.1 us, 72^3 17.9 and 17.1, 88^3 22.4 and 19.4;
// matrix-free BiCGStab 72^3 35.6 and 28.9; packed 27-point Jacobi 72^3 14.6 and
// 10.4 (below, the chain of planes of a block costs more than the gathers).
//
// A thin grid's blocks are few and mostly idle, and each walks a long chain of
// planes, while the pattern walk has every lane busy on any shape and the
// bricks are many.  CG an iteration, the other route and planes, with the share
// of the slots filled: packed 4x4x187500 (0.03) 51 and 332 us, 10x10x30000
// (0.20) 51 and 68, 14x14x15306 (0.38) 50 and 45; matrix-free 4x4x187500 (0.03,
// of the bricks' slots 0.06) 139 and 331, 8x8x46875 (0.13, 0.13) 92 and 95,
// 10x10x30000 (0.20, 0.13) 89 and 68; 27 points 32x1x250000 (0.06, 0.13) 400 and
// 1034.
//
// Variable coefficients from 786,432 cells to 6 million: CG 80^3 25.0 us an
// iteration by bricks and 26.5 by planes, 131x118x107 46.1 and 38.2, 180^3 104
// and 98, but 256^3 254 and 275 (two passes form the faces, and there the bricks'
// one pass and the stored A p cost less); Jacobi 131x118x107 33.7 and 18.9,
// BiCGStab 93 and 67.  Their faces make the ring and a chunk's first plane dear:
// CG 300x3x1111 30 and 34, 1732x1733x1 62 and 73, 1000x1001x3 60 and 60,
// 12x12x20833 122 and 128.
//
// In-plane rows are 28-bit so that their byte offsets fit 32 bits.
inline bool grid_takes(int npts, int32_t nx, int32_t ny, int32_t nz, bool packed) {
  const int64_t nxy = int64_t(nx) * ny, n = nxy * nz;
  if (n < (int64_t(11) << 15) || nxy >= (int64_t(1) << 28)) return false;
  const GridShape s = grid_shape(npts, nx, ny, nz);
  const bool filled = s.fill >= 0.375;
  const double bricks = brick_fill(nx, ny);
  if (npts == 1) {
    if (n < (int64_t(3) << 18) || n >= (int64_t(6) << 20)) return false;
    return s.plan.H >= 4 && (s.fill >= 2.0 * bricks || (filled && nz >= 3));
  }
  if (packed) return filled;
  return filled || s.fill >= (npts == 27 ? 1.0 : 1.2) * bricks;
}

// Whether matrix-free CG, which forms A p twice in the sweep and once in the
// bricks, takes the sweep on a grid that it takes.  Not
// on large grids whose lines start at any point or whose planes are too few tiles
// for the chip: bricks and planes 401^3 905 and 1013 us an iteration, 350^3 594 and
// 739, 1581x1582x8 248 and 266, 720x360x100 (270 bricks) 321 and 391.
inline bool grid_takes_cg(int npts, int32_t nx, int32_t ny, int32_t nz) {
  if (npts != 7 || int64_t(nx) * ny * nz < (int64_t(1) << 24)) return true;
  const GridPlan g = grid_shape(npts, nx, ny, nz).plan;
  return nx % 4 == 0 && int64_t(g.ntx) * g.nty * g.ncz >= 320;
}

}  // namespace its
