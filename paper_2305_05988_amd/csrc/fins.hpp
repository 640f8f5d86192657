// The scalar update that ends each pass (Fin): what the totals of the pass's
// partials do to the State.  Applied by a finishing kernel, at the start of the
// next pass (pass_begin) or by every block of a persistent kernel.
#pragma once

#include "common.hpp"

namespace its {

// -------------------------------------------------------------------- CG

// alpha = rho / (p.q); p.q = 0 or non-finite is a breakdown.
struct FinCg1 {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[1]) const {
    const double pq = dd_round(v[0]);
    if (pq == 0.0 || !finite(pq))
      st->flag = kBreakdown;
    else
      st->alpha = st->rho / pq;
  }
};

// rho' = r.r, one more iteration, beta = rho'/rho, convergence test.
struct FinCg2 {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[1]) const {
    const double rho_new = dd_round(v[0]);
    const int64_t k = st->k + 1;
    if (k & 1) st->alpha_x = st->alpha;  // iteration k - 1 (even) deferred its x update
    st->k = k;
    st->beta = rho_new / st->rho;
    st->rho = rho_new;
    if (rho_new <= st->thr2)
      st->flag = kConverged;
    else if (!finite(rho_new))
      st->flag = kBreakdown;
    else if (k >= st->max_iter)
      st->flag = kMaxIter;
  }
};

// ----------------------------------------------------------------- CG-NB

// alpha_n,j; beta and gamma for pass Y.
struct FinCgnbX {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[1]) const {
    const double an_new = dd_round(v[0]), an = st->rho;
    st->alpha_n = an_new;
    st->beta = an_new / an;
    st->gamma = (an * an) / (st->alpha_d * an_new);
  }
};

// alpha_d,j; one more iteration; the test on alpha_n,j (the residual of the
// x_j just formed); alpha_j for the next pass X.
struct FinCgnbY {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[1]) const {
    const double ad = dd_round(v[0]), an = st->alpha_n;
    const int64_t k = st->k + 1;
    st->k = k;
    st->rho = an;
    if (an <= st->thr2)
      st->flag = kConverged;
    else if (!finite(an))
      st->flag = kBreakdown;
    else if (k >= st->max_iter)
      st->flag = kMaxIter;
    else if (ad == 0.0 || !finite(ad))
      st->flag = kBreakdown;
    else {
      st->alpha_d = ad;
      st->alpha = an / ad;
    }
  }
};

// -------------------------------------------------------------- BiCGStab

// alpha_d = v.r', alpha = alpha_n / alpha_d; the restart (if any) is consumed.
struct FinBicgA {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[1]) const {
    const double ad = dd_round(v[0]);
    st->plain = st->k == 0 || st->restart;
    st->restart = 0;
    if (ad == 0.0 || !finite(ad)) {
      st->flag = kBreakdown;
    } else {
      st->alpha_d = ad;
      st->alpha = st->alpha_n / ad;
    }
  }
};

// omega = (t.s) / (t.t), 0 if t.t = 0.
struct FinBicgB {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&d)[2]) const {
    const double ts = dd_round(d[0]), tt = dd_round(d[1]);
    st->ts = ts;
    st->tt = tt;
    st->omega = (tt == 0.0) ? 0.0 : ts / tt;
  }
};

// alpha_n' = r.r', beta = r.r; the restart test, then the convergence test
// (in that order, as the restart count of the returned iterate includes a
// restart decided in its last iteration).
struct FinBicgC {
  State *st;
  double restart_tol2;
  int32_t paper_mode;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&d)[2]) const {
    const double om = st->omega;
    const bool half = (om == 0.0);
    const double an = dd_round(d[0]), beta = dd_round(d[1]);
    const int64_t k = st->k + 1;
    st->k = k;
    st->rho = beta;
    if (half) {
      st->flag = (beta <= st->thr2) ? kConverged : kBreakdown;
      return;
    }
    const bool want = paper_mode ? (__builtin_fabs(an) < restart_tol2)
                                 : (an * an < restart_tol2 * beta);
    if (want && beta > 0.0 && finite(beta)) {
      st->restart = 1;
      st->alpha_n = __builtin_sqrt(beta);
      st->restarts += 1;
    } else {
      st->beta = an / (st->alpha_d * om);
      st->alpha_n = an;
    }
    if (beta <= st->thr2)
      st->flag = kConverged;
    else if (!finite(beta))
      st->flag = kBreakdown;
    else if (k >= st->max_iter)
      st->flag = kMaxIter;
  }
};

// ----------------------------------------------- Jacobi and Gauss-Seidel

// The Jacobi sweep's residual belongs to x_k: test it; if it fails, x_{k+1} is the
// new iterate.
struct FinJacobi {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[1]) const {
    const double rr = dd_round(v[0]);
    const int64_t k = st->k;
    st->rho = rr;
    if (rr <= st->thr2)
      st->flag = kConverged;
    else if (!finite(rr))
      st->flag = kBreakdown;
    else if (k >= st->max_iter)
      st->flag = kMaxIter;
    else
      st->k = k + 1;
  }
};

// What a half-sweep of Gauss-Seidel with two colours does besides updating its
// rows (kernels_relax.hpp).
enum : int32_t { kGsPlain = 0, kGsFinal = 1, kGsLagged = 2 };

// The test after a lagged black sweep: r.r of the iterate = red part (dot 0,
// from the red sweep that made it) + black part (dot 1).
struct FinGs2 {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[2]) const {
    const double rr = dd_round(dd_add(v[0], v[1]));
    const int64_t k = st->k + 1;
    st->k = k;
    st->rho = rr;
    if (rr <= st->thr2)
      st->flag = kConverged;
    else if (!finite(rr))
      st->flag = kBreakdown;
    else if (k >= st->max_iter)
      st->flag = kMaxIter;
  }
};

// Residual of x_{k+1} after a symmetric iteration, and the test.
struct FinGs {
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[1]) const {
    const double rr = dd_round(v[0]);
    const int64_t k = st->k + 1;
    st->k = k;
    st->rho = rr;
    if (rr <= st->thr2)
      st->flag = kConverged;
    else if (!finite(rr))
      st->flag = kBreakdown;
    else if (k >= st->max_iter)
      st->flag = kMaxIter;
  }
};

}  // namespace its
