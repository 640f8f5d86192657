// The plane sweep of constant stencils on large grids.
#pragma once

#include <algorithm>

#include "grid_passes.hpp"

namespace its {

// A block owns a W x H (x, y) tile of the grid, R points per thread (point k =
// thread + kBlock u of the tile in x-fastest order), and sweeps it through a
// chunk of zb planes.  Each plane of the tile and the ring of points around it
// are loaded once, one plane ahead of the arithmetic; the values go to one of
// two LDS planes for the neighbours in the plane, and a thread keeps its own
// points' values in registers for the neighbours above and below.  A row's
// chain is started when its plane arrives and finished when the next one does,
// in the stored order: one barrier a plane, five LDS reads a row for 7 points,
// and for 27 points nine, each value feeding the chains of three planes.
//
// Neighbours outside the grid are zeros in LDS that are never written, so the
// chain takes a term c * 0 where the CSR row has no entry; c is finite, so the
// term changes nothing.
//
// W need not be a multiple of a wave: a 160-point line is cut into two tiles
// of 80 with every lane at work.
// Tiles that cover the grid with the least points loaded and thread slots
// spent, the ring at most one point per thread; then z chunks for about
// `blocks` blocks of at least 4 planes.
inline GridPlan grid_plan(int32_t nx, int32_t ny, int32_t nz, int R, int blocks) {
  GridPlan best{1, 1, 1, 1, 1, 1};
  double cost = 1e300;
  for (int32_t ntx = (nx + 109) / 110; ntx <= (nx + 109) / 110 + 6 && ntx <= nx; ++ntx) {
    const int32_t W = (nx + ntx - 1) / ntx;
    int32_t H = std::min(kBlock * R / W, 126 - W);
    H = std::min(H, ny);
    if (H < 1) continue;
    const int32_t nty = (ny + H - 1) / H;
    H = (ny + nty - 1) / nty;
    const double c = double(ntx) * nty * (0.5 * kBlock * R + double(W + 4) * (H + 2));
    if (c < cost) {
      cost = c;
      best = GridPlan{W, H, (nx + W - 1) / W, nty, 1, 1};
    }
  }
  const int64_t tiles = int64_t(best.ntx) * best.nty;
  int64_t chunks = std::max<int64_t>(1, blocks / tiles);
  chunks = std::min<int64_t>(chunks, std::max(1, nz / 4));
  best.zb = int32_t((nz + chunks - 1) / chunks);
  best.ncz = (nz + best.zb - 1) / best.zb;
  return best;
}

// The plain chain of a row.
template <class T>
struct ChainSum {
  T s = T(0);
  __device__ __forceinline__ void add(T a, T v) { s = fmaT(a, v, s); }
  __device__ __forceinline__ void centre(T a, T v) { s = fmaT(a, v, s); }
};

// The chain and the chain without the diagonal.
struct ChainSplit {
  double s = 0.0, off = 0.0;
  __device__ __forceinline__ void add(double a, double v) {
    s = fma(a, v, s);
    off = fma(a, v, off);
  }
  __device__ __forceinline__ void centre(double a, double v) { s = fma(a, v, s); }
};

// The sweep's hooks, for plane z (uniform) and in-plane row `off` of a point:
//   load.at(nxy z, off)  what is loaded for a point, of any type
//   begin()              called once the first plane's loads are on their way
//                        and before anything else: false ends the sweep
//   value(raw)           the vector's value there
//   keep(raw, value)     what the body needs of the point's own load
//   side(i)              what the body loads for its own row besides
//   body(i, chain, kept, side)  for every row of the tile, in order of planes
template <int NPTS, class T, int R>
struct GridOp {
  int32_t nx, ny, nz, n;
  T c[NPTS];
  GridPlan g;

  static constexpr int kPts = kBlock * R + kBlock;  // tile and ring
  struct SweepSmem {
    T v[2][kPts + 1];  // the last is written by threads without a point
  };

  __device__ __forceinline__ double centre() const { return c[NPTS / 2]; }

  template <class Chain, class Load, class Begin, class Value, class Keep, class Side, class Body>
  __device__ __forceinline__ bool sweep(SweepSmem &sm, Load &&load, Begin &&begin, Value &&value, Keep &&keep,
                                        Side &&side, Body &&body) const {
    using Raw = decltype(load.at(0, 0u));
    using Extra = decltype(side(0));
    using Kept = decltype(keep(load.at(0, 0u), T(0)));
    const int t = threadIdx.x;
    const int32_t W = g.W, H = g.H, pitch = W + 2, ring = 2 * pitch + 2 * H;
    const int64_t nxy = int64_t(nx) * ny;
    const int64_t nbricks = int64_t(g.ntx) * g.nty * g.ncz;
    const Sched sc = my_tiles(nbricks);
    for (int64_t b = sc.begin; b < sc.end; b += sc.stride) {
      const int32_t bx = int32_t(b % g.ntx), by = int32_t((b / g.ntx) % g.nty);
      const int32_t bz = int32_t(b / (int64_t(g.ntx) * g.nty));
      const int32_t x0 = bx * W, y0 = by * H, z0 = bz * g.zb, z1 = min(nz, z0 + g.zb);
      // the thread's points: in-plane row (0 where it has none), LDS index to
      // write, LDS index to read around
      uint32_t off[R], ok = 0;
      int wr[R], rd[R];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int32_t k = t + u * kBlock;
        const int32_t y = k / W, x = k - y * W;
        const bool in = y < H && x0 + x < nx && y0 + y < ny;
        off[u] = in ? uint32_t(x0 + x + nx * (y0 + y)) : 0u;
        rd[u] = in ? (y + 1) * pitch + x + 1 : pitch + 1;
        wr[u] = in ? rd[u] : kPts;
        ok |= uint32_t(in) << u;
      }
      uint32_t hoff = 0;  // its point of the ring
      int hwr = kPts;
      if (t < ring) {
        const int32_t q = t - 2 * pitch;
        const int32_t y = t < pitch ? -1 : q < 0 ? H : q >> 1;
        const int32_t x = t < pitch ? t - 1 : q < 0 ? t - pitch - 1 : (q & 1) ? W : -1;
        const bool corner = (x < 0 || x == W) && (y < 0 || y == H);
        if (x0 + x >= 0 && x0 + x < nx && y0 + y >= 0 && y0 + y < ny && !(NPTS == 7 && corner)) {
          hoff = uint32_t(x0 + x + nx * (y0 + y));
          hwr = (y + 1) * pitch + x + 1;
        }
      }
      const int32_t zs = max(z0 - 1, 0), ze = min(z1, nz - 1);
      Raw raw[R], rawh;
      Extra ex[R];
      auto issue = [&](int32_t z) {
        const int64_t zo = nxy * z;
#pragma unroll
        for (int u = 0; u < R; ++u) raw[u] = load.at(zo, off[u]);
        rawh = load.at(zo, hoff);
      };
      auto issue_side = [&](int32_t z) {
        const int64_t zo = nxy * z;
#pragma unroll
        for (int u = 0; u < R; ++u) ex[u] = side(int32_t(zo) + int32_t(off[u]));
      };
      auto finish = [&](int32_t z, const Chain *ch, const Kept *own) {
        const int32_t zo = int32_t(nxy * z);
#pragma unroll
        for (int u = 0; u < R; ++u)
          if ((ok >> u) & 1u) body(zo + int32_t(off[u]), ch[u], own[u], ex[u]);
      };
      issue(zs);
      for (int k = t; k < 2 * (kPts + 1); k += kBlock) (&sm.v[0][0])[k] = T(0);
      if (b == sc.begin && !begin()) return false;
      __syncthreads();
      if constexpr (NPTS == 7) {
        Chain ch[R];
        T prev[R];
        Kept own[R];
#pragma unroll
        for (int u = 0; u < R; ++u) prev[u] = T(0);
        for (int32_t z = zs; z <= ze; ++z) {
          T *pl = sm.v[z & 1];
          T nv[R];
#pragma unroll
          for (int u = 0; u < R; ++u) {
            nv[u] = value(raw[u]);
            pl[wr[u]] = nv[u];
          }
          pl[hwr] = value(rawh);
          if (z > z0) {  // rows z - 1 are complete
#pragma unroll
            for (int u = 0; u < R; ++u) ch[u].add(c[6], nv[u]);
            finish(z - 1, ch, own);
          }
#pragma unroll
          for (int u = 0; u < R; ++u) own[u] = keep(raw[u], nv[u]);
          if (z < ze) issue(z + 1);
          if (z >= z0 && z < z1) {
            issue_side(z);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < R; ++u) {
              const T *p = pl + rd[u];
              Chain q;
              if (z > 0) q.add(c[0], prev[u]);
              q.add(c[1], p[-pitch]);
              q.add(c[2], p[-1]);
              q.centre(c[3], nv[u]);
              q.add(c[4], p[1]);
              q.add(c[5], p[pitch]);
              ch[u] = q;
            }
          }
#pragma unroll
          for (int u = 0; u < R; ++u) prev[u] = nv[u];
        }
        if (z1 == nz) finish(nz - 1, ch, own);
      } else {
        Chain lo[R], mid[R];  // rows z - 1 and z when plane z arrives
        Kept own[R];
        for (int32_t z = zs; z <= ze; ++z) {
          T *pl = sm.v[z & 1];
          T nv[R];
          Kept mine[R];
#pragma unroll
          for (int u = 0; u < R; ++u) {
            nv[u] = value(raw[u]);
            mine[u] = keep(raw[u], nv[u]);
            pl[wr[u]] = nv[u];
          }
          pl[hwr] = value(rawh);
          if (z < ze) issue(z + 1);
          __syncthreads();
#pragma unroll
          for (int u = 0; u < R; ++u) {
            const T *p = pl + rd[u];
            Chain hi;
#pragma unroll
            for (int q = 0; q < 9; ++q) {
              const T v = q == 4 ? nv[u] : p[(q / 3 - 1) * pitch + (q % 3 - 1)];
              lo[u].add(c[18 + q], v);
              if (q == 4)
                mid[u].centre(c[13], v);
              else
                mid[u].add(c[9 + q], v);
              hi.add(c[q], v);
            }
            if (z > z0 && ((ok >> u) & 1u)) body(int32_t(nxy * (z - 1)) + int32_t(off[u]), lo[u], own[u], ex[u]);
            lo[u] = mid[u];
            mid[u] = hi;
            own[u] = mine[u];
          }
          if (z >= z0 && z < z1) issue_side(z);
        }
        if (z1 == nz) finish(nz - 1, lo, own);
      }
      if (b + sc.stride < sc.end) __syncthreads();
    }
    return sc.begin < sc.end || begin();
  }
};

}  // namespace its
