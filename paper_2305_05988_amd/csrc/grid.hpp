// The plane sweep of constant stencils on large grids.
#pragma once

#include <type_traits>

#include "grid_passes.hpp"

namespace its {

// A block owns a W x H (x, y) tile of the grid, R points per thread (point k =
// thread + kBlock u of the tile in x-fastest order), and sweeps it through a
// chunk of zb planes.  Each plane of the tile and the ring of points around it
// are loaded once, one plane ahead of the arithmetic; the values go to one of
// two LDS planes for the neighbours in the plane, and a thread keeps its own
// points' values in registers for the neighbours above and below.  A row's
// chain is started when its plane arrives and finished when the next one does,
// in the stored order: one barrier a plane, four LDS reads a row for 7 points, and
// for 27 points eight, each value feeding the chains of three planes.
//
// Neighbours outside the grid are zeros in LDS that are never written, so the
// chain takes a term c * 0 where the CSR row has no entry; c is finite, so the
// term changes nothing.
//
// W need not be a multiple of a wave (grid_plan.hpp): a 160-point line is cut into
// five tiles of 32, a 146-point line into two of 73, with every lane at work.

// The plain chain of a row.  add: an entry below the diagonal; centre: the
// diagonal; above: an entry above it (the 7-point sweeps number theirs: at x +
// 1, y + 1 and z + 1).
template <class T>
struct ChainSum {
  T s = T(0);
  __device__ __forceinline__ void add(T a, T v) { s = fmaT(a, v, s); }
  __device__ __forceinline__ void centre(T a, T v) { s = fmaT(a, v, s); }
  template <int Q>
  __device__ __forceinline__ void above(T a, T v) { add(a, v); }
};

// The chain, the chain without the diagonal, and the diagonal.
struct ChainSplit {
  double s = 0.0, off = 0.0, d = 0.0;
  __device__ __forceinline__ void add(double a, double v) {
    s = fma(a, v, s);
    off = fma(a, v, off);
  }
  __device__ __forceinline__ void centre(double a, double v) {
    s = fma(a, v, s);
    d = a;
  }
  template <int Q>
  __device__ __forceinline__ void above(double a, double v) { add(a, v); }
};

// The chain without the diagonal, and what it takes to run the whole chain
// again with another value of the row itself (7 points).
struct ChainTwice {
  double low = 0.0, off = 0.0, v[3];
  __device__ __forceinline__ void add(double a, double x) {
    low = fma(a, x, low);
    off = fma(a, x, off);
  }
  __device__ __forceinline__ void centre(double, double) {}
  template <int Q>
  __device__ __forceinline__ void above(double a, double x) {
    off = fma(a, x, off);
    v[Q] = x;
  }
  // c: the stencil; last: the row has an entry at z + 1
  __device__ __forceinline__ double with(const double (&c)[7], double x, bool last) const {
    const double s = fma(c[5], v[1], fma(c[4], v[0], fma(c[3], x, low)));
    return last ? fma(c[6], v[2], s) : s;
  }
};

// A thread's points of a tile: in-plane row (0 where it has none), LDS index to
// write, LDS index to read around; and its point of the ring.
template <int R>
struct TilePoints {
  static constexpr int kPts = kBlock * R + kBlock;  // tile and ring
  uint32_t off[R], ok = 0, odd = 0, hoff = 0;  // odd: x + y
  int wr[R], rd[R], hwr = kPts;  // kPts: written by threads without a point
  __device__ __forceinline__ TilePoints(int32_t W, int32_t H, int32_t x0, int32_t y0, int32_t nx, int32_t ny,
                                        bool corners) {
    const int t = threadIdx.x;
    const int32_t pitch = W + 2;
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int32_t k = t + u * kBlock;
      const int32_t y = k / W, x = k - y * W;
      const bool in = y < H && x0 + x < nx && y0 + y < ny;
      off[u] = in ? uint32_t(x0 + x + nx * (y0 + y)) : 0u;
      rd[u] = in ? (y + 1) * pitch + x + 1 : pitch + 1;
      wr[u] = in ? rd[u] : kPts;
      ok |= uint32_t(in) << u;
      odd |= uint32_t((x0 + x + y0 + y) & 1) << u;
    }
    if (t < 2 * pitch + 2 * H) {
      const int32_t q = t - 2 * pitch;
      const int32_t y = t < pitch ? -1 : q < 0 ? H : q >> 1;
      const int32_t x = t < pitch ? t - 1 : q < 0 ? t - pitch - 1 : (q & 1) ? W : -1;
      const bool corner = (x < 0 || x == W) && (y < 0 || y == H);
      if (x0 + x >= 0 && x0 + x < nx && y0 + y >= 0 && y0 + y < ny && (corners || !corner)) {
        hoff = uint32_t(x0 + x + nx * (y0 + y));
        hwr = (y + 1) * pitch + x + 1;
      }
    }
  }
};

// The sweep's hooks, for plane z (uniform) and in-plane row `off` of a point:
//   load.at(nxy z, off)  what is loaded for a point, of any type
//   begin()              called once the first plane's loads are on their way
//                        and before anything else: false ends the sweep
//   value(raw)           the vector's value there
//   keep(raw, value)     what the body needs of the point's own load
//   side(i)              what the body loads for its own row besides
//   body(i, chain, kept, side)  for every row of the tile, in order of planes;
//                        a body of six arguments also gets the parity of x + y
//                        + z and whether the row has a row above it
template <class Body, class Chain, class Kept, class Extra>
__device__ __forceinline__ void call_body(Body &body, int32_t i, const Chain &ch, const Kept &own, const Extra &ex,
                                          uint32_t odd, bool last) {
  if constexpr (std::is_invocable_v<Body &, int32_t, const Chain &, const Kept &, const Extra &, uint32_t, bool>)
    body(i, ch, own, ex, odd, last);
  else
    body(i, ch, own, ex);
}

template <int NPTS, class T, int R>
struct GridOp {
  int32_t nx, ny, nz, n;
  T c[NPTS];
  GridPlan g;

  static constexpr int kPts = TilePoints<R>::kPts;
  struct SweepSmem {
    T v[2][kPts + 1];
  };

  template <class Chain>
  __device__ __forceinline__ T diagonal(const Chain &) const {
    return c[NPTS / 2];
  }


  template <class Chain, class Load, class Begin, class Value, class Keep, class Side, class Body>
  __device__ __forceinline__ bool sweep(SweepSmem &sm, Load &&load, Begin &&begin, Value &&value, Keep &&keep,
                                        Side &&side, Body &&body) const {
    using Raw = decltype(load.at(0, 0u));
    using Extra = decltype(side(0));
    using Kept = decltype(keep(load.at(0, 0u), T(0)));
    const int t = threadIdx.x;
    const int32_t W = g.W, H = g.H, pitch = W + 2;
    const int64_t nxy = int64_t(nx) * ny;
    const int64_t nbricks = int64_t(g.ntx) * g.nty * g.ncz;
    const Sched sc = my_tiles(nbricks);
    for (int64_t b = sc.begin; b < sc.end; b += sc.stride) {
      const int32_t bx = int32_t(b % g.ntx), by = int32_t((b / g.ntx) % g.nty);
      const int32_t bz = int32_t(b / (int64_t(g.ntx) * g.nty));
      const int32_t x0 = bx * W, y0 = by * H, z0 = bz * g.zb, z1 = min(nz, z0 + g.zb);
      const TilePoints<R> pt(W, H, x0, y0, nx, ny, NPTS == 27);
      const auto &off = pt.off;
      const auto &wr = pt.wr;
      const auto &rd = pt.rd;
      const uint32_t ok = pt.ok, hoff = pt.hoff;
      const int hwr = pt.hwr;

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
          if ((ok >> u) & 1u)
            call_body(body, zo + int32_t(off[u]), ch[u], own[u], ex[u], ((pt.odd >> u) ^ uint32_t(z)) & 1u, z < nz - 1);
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
            for (int u = 0; u < R; ++u) ch[u].template above<2>(c[6], nv[u]);
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
              q.template above<0>(c[4], p[1]);
              q.template above<1>(c[5], p[pitch]);
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

// The variable-coefficient diffusion operator (varcoef.hpp: its faces, their
// order and its roundings) in the same sweep: k lies beside the values in LDS.
// A row's lower chain, its in-plane faces and their sum wait in registers for
// the next plane, whose own k gives the face above -- and below the next row,
// so a row forms five faces instead of six.  A face across the boundary is the
// cell's own k and adds no term (its neighbour's value is a zero in LDS).
//
// Bound by the instructions of the faces, five divisions a row.  While every k
// a block has met lies in [2^-250, 2^250] nothing in a face can leave the
// normal range, and the quotient comes from the reciprocal, two Newton steps
// and one correction by the exact remainder (Markstein), without the scaling
// and the special cases of the general division: the same correctly rounded
// quotient.
template <int R>
struct VarGridOp {
  int32_t nx, ny, nz, n;
  const double *__restrict__ k;
  GridPlan g;

  static constexpr int kPts = TilePoints<R>::kPts;
  struct SweepSmem {
    double v[2][kPts + 1], k[2][kPts + 1];
    int wide;  // a k outside the range was met
  };

  __device__ __forceinline__ double diagonal(const ChainSplit &q) const { return q.d; }

  __device__ static __forceinline__ bool plain(double k) {
    const uint32_t e = uint32_t(__builtin_bit_cast(uint64_t, k) >> 52);
    return e - (1023u - 250u) < 500u;
  }
  template <bool Plain>
  __device__ static __forceinline__ double face(double a, double b) {
    const double q = 2.0 * a * b, s = a + b;
    if constexpr (!Plain) return q / s;
    double r = __builtin_amdgcn_rcp(s);
    r = fma(r, fma(-s, r, 1.0), r);
    r = fma(r, fma(-s, r, 1.0), r);
    const double f = q * r;
    return fma(fma(-s, f, q), r, f);
  }

  template <class Chain, class Load, class Begin, class Value, class Keep, class Side, class Body>
  __device__ __forceinline__ bool sweep(SweepSmem &sm, Load &&load, Begin &&begin, Value &&value, Keep &&keep,
                                        Side &&side, Body &&body) const {
    using Raw = decltype(load.at(0, 0u));
    using Extra = decltype(side(0));
    using Kept = decltype(keep(load.at(0, 0u), 0.0));
    const int t = threadIdx.x;
    const int32_t W = g.W, H = g.H, pitch = W + 2;
    const int64_t nxy = int64_t(nx) * ny;
    const int64_t nbricks = int64_t(g.ntx) * g.nty * g.ncz;
    const Sched sc = my_tiles(nbricks);
    for (int64_t b = sc.begin; b < sc.end; b += sc.stride) {
      const int32_t bx = int32_t(b % g.ntx), by = int32_t((b / g.ntx) % g.nty);
      const int32_t bz = int32_t(b / (int64_t(g.ntx) * g.nty));
      const int32_t x0 = bx * W, y0 = by * H, z0 = bz * g.zb, z1 = min(nz, z0 + g.zb);
      const TilePoints<R> pt(W, H, x0, y0, nx, ny, false);
      // the lanes whose in-plane neighbours lie inside the grid
      uint64_t in[R][4];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int32_t y = int32_t(pt.off[u]) / nx, x = int32_t(pt.off[u]) - y * nx;
        in[u][0] = __ballot(y > 0);
        in[u][1] = __ballot(x > 0);
        in[u][2] = __ballot(x < nx - 1);
        in[u][3] = __ballot(y < ny - 1);
      }
      const int32_t zs = max(z0 - 1, 0), ze = min(z1, nz - 1);
      Raw raw[R], rawh;
      double kraw[R], krawh;
      Extra ex[R];
      auto issue = [&](int32_t z) {
        const int64_t zo = nxy * z;
#pragma unroll
        for (int u = 0; u < R; ++u) {
          raw[u] = load.at(zo, pt.off[u]);
          kraw[u] = (k + zo)[pt.off[u]];
        }
        rawh = load.at(zo, pt.hoff);
        krawh = (k + zo)[pt.hoff];
      };
      issue(zs);
      for (int q = t; q < 2 * (kPts + 1); q += kBlock) {
        (&sm.v[0][0])[q] = 0.0;
        (&sm.k[0][0])[q] = 0.0;
      }
      if (t == 0) sm.wide = 0;
      if (b == sc.begin && !begin()) return false;
      __syncthreads();
      Chain ch[R];                                  // of row z - 1, up to its lower entries
      double pv[R], pk[R], fz[R], sum[R];           // value, k, face below the new plane, faces so far
      double fx[R], fy[R], vx[R], vy[R];            // faces and values at x + 1 and y + 1
      Kept own[R];
#pragma unroll
      for (int u = 0; u < R; ++u) pv[u] = pk[u] = fz[u] = sum[u] = fx[u] = fy[u] = vx[u] = vy[u] = 0.0;
      auto finish = [&](int u, double up) {  // the rest of the chain, without the entry above
        ch[u].centre(sum[u] + up, pv[u]);
        ch[u].add(-fx[u], vx[u]);
        ch[u].add(-fy[u], vy[u]);
      };
      bool was = true;  // the plane before: the thread's k in range
      for (int32_t z = zs; z <= ze; ++z) {
        double *pl = sm.v[z & 1], *kl = sm.k[z & 1];
        double nv[R], nk[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
          nv[u] = value(raw[u]);
          nk[u] = kraw[u];
          pl[pt.wr[u]] = nv[u];
          kl[pt.wr[u]] = nk[u];
        }
        pl[pt.hwr] = value(rawh);
        kl[pt.hwr] = krawh;
        bool fine = plain(krawh);
#pragma unroll
        for (int u = 0; u < R; ++u) fine = fine && plain(nk[u]);
        if (!fine) sm.wide = 1;
        if (z > zs) {
          const bool all = __all(fine && was);
#pragma unroll
          for (int u = 0; u < R; ++u) fz[u] = all ? face<true>(pk[u], nk[u]) : face<false>(pk[u], nk[u]);
        }
        was = fine;
        if (z > z0) {
          const int32_t zo = int32_t(nxy * (z - 1));
#pragma unroll
          for (int u = 0; u < R; ++u) {
            finish(u, fz[u]);
            ch[u].add(-fz[u], nv[u]);
            if ((pt.ok >> u) & 1u) body(zo + int32_t(pt.off[u]), ch[u], own[u], ex[u]);
          }
        }
#pragma unroll
        for (int u = 0; u < R; ++u) own[u] = keep(raw[u], nv[u]);
        if (z < ze) issue(z + 1);
        if (z >= z0 && z < z1) {
          const int32_t zo = int32_t(nxy * z);
#pragma unroll
          for (int u = 0; u < R; ++u) ex[u] = side(zo + int32_t(pt.off[u]));
          __syncthreads();
          auto start = [&](auto in_range) {
            constexpr bool P = decltype(in_range)::value;
#pragma unroll
            for (int u = 0; u < R; ++u) {
              const double *p = pl + pt.rd[u], *q = kl + pt.rd[u];
              const double kc = nk[u], below = z > 0 ? fz[u] : kc;
              auto pick = [&](int d, double f) { return __builtin_amdgcn_inverse_ballot_w64(in[u][d]) ? f : kc; };
              const double f1 = pick(0, face<P>(q[-pitch], kc)), f2 = pick(1, face<P>(q[-1], kc));
              fx[u] = pick(2, face<P>(kc, q[1]));
              fy[u] = pick(3, face<P>(kc, q[pitch]));
              sum[u] = ((((0.0 + below) + f1) + f2) + fx[u]) + fy[u];
              Chain c;
              if (z > 0) c.add(-below, pv[u]);
              c.add(-f1, p[-pitch]);
              c.add(-f2, p[-1]);
              ch[u] = c;
              vx[u] = p[1];
              vy[u] = p[pitch];
            }
          };
          if (sm.wide == 0)
            start(std::true_type());
          else
            start(std::false_type());
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
          pv[u] = nv[u];
          pk[u] = nk[u];
        }
      }
      if (z1 == nz) {
        const int32_t zo = int32_t(nxy * (nz - 1));
#pragma unroll
        for (int u = 0; u < R; ++u) {
          finish(u, pk[u]);
          if ((pt.ok >> u) & 1u) body(zo + int32_t(pt.off[u]), ch[u], own[u], ex[u]);
        }
      }
      if (b + sc.stride < sc.end) __syncthreads();
    }
    return sc.begin < sc.end || begin();
  }
};

}  // namespace its
