// The passes of constant stencils on large grids (grid.hip), for the drivers.
#pragma once

#include "common.hpp"
#include "fins.hpp"
#include "grid_plan.hpp"

namespace its {

// A constant stencil on nx*ny*nz with neighbours outside the grid omitted -- a
// matrix-free operator, or a packed CSR matrix found to be one -- or the
// variable-coefficient diffusion operator.
struct GridStencil {
  int32_t npts = 0;  // 7 or 27; 1: variable coefficients; 0: none
  int32_t nx = 0, ny = 0, nz = 0, n = 0;
  double c[27] = {};    // ascending column order
  float lo[27] = {};    // the same for the refinement's inner solve
  const double *k = nullptr;  // variable coefficients: one per cell
};

// What every pass runs with.
struct GridRun {
  const GridStencil *a;
  GridPlan plan;
  int points;  // per thread
  int blocks;
  bool stream;  // the vectors do not fit the memory-side cache
  hipStream_t s;
};
// vector_bytes: of all vectors that an iteration touches.
GridRun grid_run(const GridStencil &a, int64_t vector_bytes, hipStream_t s);

// Each launches one kernel of g.blocks blocks; the block partials go to
// ps.dst.  The arithmetic of each is stated beside its kernel.  defer: an even
// iteration of CG, which leaves x alone.
hipError_t grid_spmv(const GridRun &g, const double *x, double *y);
hipError_t grid_residual(const GridRun &g, const double *b, const double *x, double *r, double *zero, DD *dst);
hipError_t grid_check(const GridRun &g, const double *b, const double *x, const PassPlain &ps);
hipError_t grid_jacobi(const GridRun &g, const double *b, const double *x, double *xn, const Pass &ps);
hipError_t grid_cg_a(const GridRun &g, const double *r, const double *p, double *pn, const Pass &ps);
hipError_t grid_cg_b(const GridRun &g, const double *pn, const double *p, double *r, double *x, bool defer,
                     const Pass &ps);
hipError_t grid_cg_a(const GridRun &g, const float *r, const float *p, float *pn, const Pass &ps);
hipError_t grid_cg_b(const GridRun &g, const float *pn, const float *p, float *r, float *x, bool defer,
                     const Pass &ps);
hipError_t grid_cgnb_x(const GridRun &g, const double2_t *ra, double *w, const Pass &ps);
hipError_t grid_bicg_a(const GridRun &g, const double *r, const double *u, double *rs, double *v, const FinBicgC &fin,
                       const Pass &ps);
hipError_t grid_bicg_b(const GridRun &g, const double *r, const double *v, const Pass &ps);
hipError_t grid_bicg_c(const GridRun &g, const double *r, double *rn, double *u, const double *v, const double *rs,
                       double *x, const Pass &ps);
// Half-sweeps of red-black Gauss-Seidel (7 points; modes of kernels_relax.hpp;
// xs: n / 2 rounded up values).
hipError_t grid_gs(const GridRun &g, int mode, int colour, const double *b, double *x, double *xs, const Pass &ps);
hipError_t grid_gs_restore(const GridRun &g, const double *xs, double *x);

}  // namespace its
