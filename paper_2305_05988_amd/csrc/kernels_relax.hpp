// Relaxation kernels: Jacobi sweep and colour-ordered symmetric Gauss-Seidel.
#pragma once

#include "common.hpp"
#include "fins.hpp"
#include "csr.hpp"
#include "sell.hpp"
#include "stencil.hpp"

namespace its {

// ------------------------------------------------------------------ Jacobi
// One fused sweep: the residual of x_k (full chain) and x_{k+1} = (b - off)/d.
// The test applies to x_k, so a converged solve returns x_k from xo.
template <class Op, class P>
__global__ void __launch_bounds__(kBlock) k_jacobi(Op A, const double *__restrict__ b,
                                                   const double *__restrict__ xo,
                                                   double *__restrict__ xn, P ps) {
  __shared__ typename Op::Smem sm;
  State ls;
  if (!pass_begin<1>(ps, ls, FinJacobi{})) return;
  const Gather<double> xj{xo};
  auto same = [](double v) { return v; };
  Dot2 a;
  A.rows(sm, xj, same, [&](int32_t i, bool valid, auto &&entries, auto &&) {
    double full = 0.0, off = 0.0, diag = 0.0;
    entries([&](int32_t j, double av, double v, bool has = true) {
      full = has ? fma(av, v, full) : full;
      diag = has && j == i ? av : diag;
      off = has && j != i ? fma(av, v, off) : off;
    });
    if (valid) {
      const double bi = ld_nt(b + i);
      const double ri = bi - full;
      a.add(ri, ri);
      st_pairs<GathersPairs<Op>::value>(xn + i, (bi - off) / diag);
    }
  });
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst, rev_of(A));
}

// ------------------------------------------------------------ Gauss-Seidel
// Half-sweep over the rows of one colour, in place.  Rows of one colour do
// not couple, so their updates are independent and the order within the
// colour does not change any bit.
//
// With two colours (red 0, black 1) on a CSR matrix an iteration after the
// first sweeps black then red, and the residual of the iterate it leaves
// comes from the sweeps themselves instead of a separate SpMV pass:
//   kGsFinal  (red sweep): after a row's update, its full chain again with
//             the new value -- the red residual of the new iterate (dot 0);
//   kGsLagged (next black sweep): before a row's update, the full chain over
//             the values it reads anyway -- the black residual of that same
//             iterate (dot 1) -- and the old value saved to xs, so a solve
//             that stops on this test can put the tested iterate back.
// Every chain is the SpMV chain (ascending columns, diagonal in place), so
// r.r equals the separate pass's bit for bit.  (The matrix-free sweeps keep
// the separate pass: its LDS-tiled stencil SpMV costs less than the extra
// chains in the sweeps.)

// A half-sweep's start: the first of an iteration applies the pending test
// (FinGs2 with two colours on CSR, FinGs elsewhere), the others have none.
template <bool Two, class P>
__device__ __forceinline__ bool gs_begin(const P &ps, State &ls) {
  if constexpr (Two)
    return pass_begin<2>(ps, ls, FinGs2{});
  else
    return pass_begin<1>(ps, ls, FinGs{});
}

template <int Mode, class P>
__global__ void __launch_bounds__(kBlock) k_gs_rows_csr(CsrOp<double, double> A,
                                                        const int32_t *__restrict__ rows,
                                                        int32_t count, const double *__restrict__ b,
                                                        double *x, double *__restrict__ xs,
                                                        P ps) {
  State ls;
  if (!gs_begin<Mode != kGsPlain>(ps, ls)) return;
  Dot2 a;
  for_rows(count, [&](int32_t t) {
    const int32_t i = rows[t];
    const double bi = b[i];
    double full, off, diag;
    A.relax(i, [&](int32_t j) { return x[j]; }, full, off, diag);
    if (Mode == kGsLagged) {
      const double ri = bi - full;
      a.add(ri, ri);
      xs[t] = x[i];
    }
    x[i] = (bi - off) / diag;
    if (Mode == kGsFinal) {
      A.relax(i, [&](int32_t j) { return x[j]; }, full, off, diag);
      const double ri = bi - full;
      a.add(ri, ri);
    }
  });
  if (Mode != kGsPlain) {
    DD v[1] = {a.get()};
    block_partial_to<1>(v, ps.dst);
  }
}

// The same half-sweep over a colour's rows in their own packed layout (row p
// of the layout is rows[p]), so the entries stream coalesced.
template <int Mode, class Op, class P>
__global__ void __launch_bounds__(kBlock) k_gs_rows_packed(Op A, const int32_t *__restrict__ rows,
                                                           const double *__restrict__ b, double *x,
                                                           double *__restrict__ xs,
                                                           P ps) {
  __shared__ typename Op::Smem sm;
  State ls;
  if (!gs_begin<Mode != kGsPlain>(ps, ls)) return;
  const Gather<double> xj{x};
  Dot2 a;
  for_tiles(A.n, [&](int32_t r0, int32_t r1) {
    const int32_t p = r0 + int32_t(threadIdx.x);
    const int32_t i = p < r1 ? rows[p] : -1;
    double full = 0.0, off = 0.0, diag = 0.0, xi = 0.0;
    A.tile_entries(r0, r1, sm, xj, [&](int32_t j, double av, double v, bool has = true) {
      if (Mode == kGsLagged) full = has ? fma(av, v, full) : full;
      const bool own_entry = has && j == i;
      off = has && j != i ? fma(av, v, off) : off;
      diag = own_entry ? av : diag;
      xi = own_entry ? v : xi;
    });
    const double bi = p < r1 ? b[i] : 0.0;
    if (p < r1) {
      if (Mode == kGsLagged) {
        const double ri = bi - full;
        a.add(ri, ri);
        xs[p] = xi;
      }
      x[i] = (bi - off) / diag;
    }
    if (Mode == kGsFinal) {
      double f2 = 0.0;
      A.tile_entries(r0, r1, sm, xj, [&](int32_t, double av, double v, bool has = true) {
        f2 = has ? fma(av, v, f2) : f2;
      });
      if (p < r1) {
        const double ri = bi - f2;
        a.add(ri, ri);
      }
    }
  }, rev_of(A));
  if (Mode != kGsPlain) {
    DD v[1] = {a.get()};
    block_partial_to<1>(v, ps.dst, rev_of(A));
  }
}

// Matrix-free half-sweep over one colour's cells, walked on a compact index
// so that every thread updates a cell: with two colours (7 points) every
// other cell of each x line, with eight (27 points) every other cell along
// each axis.
template <int NPTS>
__host__ __device__ inline int64_t gs_colour_cells(int32_t nx, int32_t ny, int32_t nz) {
  const int64_t hx = (nx + 1) / 2;
  return NPTS == 7 ? hx * ny * nz : hx * ((ny + 1) / 2) * ((nz + 1) / 2);
}

template <int NPTS, class P>
__global__ void __launch_bounds__(kBlock) k_gs_stencil(StencilOp<NPTS, double> A, int32_t color,
                                                       const double *__restrict__ b, double *x,
                                                       P ps) {
  State ls;
  if (!gs_begin<false>(ps, ls)) return;
  const int32_t hx = (A.nx + 1) / 2;
  const int32_t hy = NPTS == 7 ? A.ny : (A.ny + 1) / 2;
  const int32_t cells = int32_t(gs_colour_cells<NPTS>(A.nx, A.ny, A.nz));
  for_rows(cells, [&](int32_t t) {
    const int32_t line = t / hx, k = t - line * hx;
    const int32_t qz = line / hy, qy = line - qz * hy;
    int32_t ix, iy, iz;
    if (NPTS == 7) {
      iy = qy;
      iz = qz;
      ix = 2 * k + ((color + iy + iz) & 1);
    } else {
      ix = 2 * k + (color & 1);
      iy = 2 * qy + ((color >> 1) & 1);
      iz = 2 * qz + (color >> 2);
    }
    if (ix >= A.nx || iy >= A.ny || iz >= A.nz) return;
    const int32_t i = ix + A.nx * (iy + A.ny * iz);
    double off = 0.0;
    A.row_entries_at(i, ix, iy, iz, [&](int32_t j) { return x[j]; },
                     [&](int32_t j, double av, double v) {
                       if (j != i) off = fma(av, v, off);
                     });
    x[i] = (b[i] - off) / A.c[NPTS / 2];
  });
}

// Puts the black rows of the tested iterate back: x[rows[p]] = xs[p] over the
// black colour's row list.
__global__ void __launch_bounds__(kBlock) k_gs_restore_rows(const int32_t *__restrict__ rows,
                                                            int32_t count, const double *__restrict__ xs,
                                                            double *__restrict__ x) {
  for_rows(count, [&](int32_t p) { x[rows[p]] = xs[p]; });
}

// Residual of the iterate after a full symmetric iteration, and the test.
template <class Op, class P>
__global__ void __launch_bounds__(kBlock) k_gs_check(Op A, const double *__restrict__ b,
                                                     const double *__restrict__ x, P ps) {
  __shared__ typename Op::Smem sm;
  State ls;
  if (!gs_begin<false>(ps, ls)) return;
  const Gather<double> xj{x};
  auto same = [](double v) { return v; };
  Dot2 a;
  A.rows(sm, xj, same, [&](int32_t i, bool valid, auto &&entries, auto &&) {
    double acc = 0.0;
    entries([&](int32_t, double av, double v, bool has = true) { acc = has ? fma(av, v, acc) : acc; });
    if (valid) {
      const double ri = b[i] - acc;
      a.add(ri, ri);
    }
  });
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst, rev_of(A));
}

}  // namespace its
