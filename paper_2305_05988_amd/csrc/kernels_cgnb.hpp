// CG-NB, the paper's nonblocking CG (Algorithm 1), in two fused passes per
// iteration.  The SpMV is applied to r; A p is carried by the recurrence
// A p_j = A r_j + beta_j A p_{j-1}; r and A p are stored interleaved as pairs
// {r_i, (Ap)_i} so the SpMV pass gathers both with one access.
//   pass X: r_j = r_{j-1} - alpha_{j-1} (Ap)_{j-1} formed on the fly for every
//           gathered column, w = A r_j, alpha_n,j = r_j.r_j
//   pass Y: r_j again (same fma), (Ap)_j = fma(beta, (Ap)_{j-1}, w),
//           p_j = fma(beta, p_{j-1}, r_j),
//           x_j = x_{j-1} + gamma (p_j - r_j) as the three-term update
//           fma(gamma, p_j, fma(-gamma, r_j, x_{j-1})),
//           alpha_d,j = (Ap)_j.p_j
// with beta = alpha_n,j / alpha_n,j-1 and
// gamma = alpha_n,j-1^2 / (alpha_d,j-1 alpha_n,j).  (Algorithm 1 prints the x
// update with a minus sign; gamma (p_j - r_j) = alpha_{j-1} p_{j-1}, so it is
// an addition.)  If alpha_n,j is exactly 0, gamma divides by zero and the
// update takes its exact value alpha_{j-1} p_{j-1}.
#pragma once

#include "common.hpp"
#include "fins.hpp"
#include "rowops.hpp"

namespace its {

// Start: w = A r0 (stored as (Ap)_0), p0 = r0, alpha_d,0 = (Ap)_0.p0.
template <class Op>
__global__ void __launch_bounds__(kBlock) k_cgnb_init(Op A, double2_t *__restrict__ ra,
                                                      double *__restrict__ p, Reduce *R) {
  __shared__ typename Op::Smem sm;
  auto rj = [&](int32_t j) -> double { return ra[j].x; };
  auto same = [](double v) { return v; };
  Dot2 a;
  A.rows(sm, rj, same, [&](int32_t i, bool valid, auto &&entries, auto &&) {
    double acc = 0.0;
    entries([&](int32_t, double av, double v, bool has = true) { acc = has ? fma(av, v, acc) : acc; });
    if (valid) {
      const double ri = ra[i].x;
      st_nt(p + i, ri);
      a.add(acc, ri);
      // own pair only: other rows gather the .x member, never .y
      ra[i].y = acc;
    }
  });
  DD v[1] = {a.get()};
  block_partial<1>(v, R, rev_of(A));
}

struct FinCgnbInit {  // alpha_d,0 and alpha_0
  State *st;
  __device__ bool active() const { return st->flag == kRunning; }
  __device__ void operator()(DD (&v)[1]) const {
    const double ad = dd_round(v[0]);
    if (ad == 0.0 || !finite(ad)) {
      st->flag = kBreakdown;
    } else {
      st->alpha_d = ad;
      st->alpha = st->rho / ad;
    }
  }
};

template <class Op, class P>
__global__ void __launch_bounds__(kBlock) k_cgnb_x(Op A, const double2_t *__restrict__ ra,
                                                   double *__restrict__ w, P ps) {
  __shared__ typename Op::Smem sm;
  State ls;
  if (!pass_begin<1>(ps, ls, FinCgnbY{})) return;
  const double alpha = ls.alpha;
  const Gather<double2_t> load{ra};
  auto rv = [&](const double2_t &v) -> double { return fma(-alpha, v.y, v.x); };
  Dot2 a;
  A.rows(sm, load, rv, [&](int32_t i, bool valid, auto &&entries, auto &&own) {
    double acc = 0.0, ri = 0.0;
    bool have = false;  // r_i taken from the row's diagonal entry
    entries([&](int32_t j, double av, double rj, bool has = true) {
      acc = has ? fma(av, rj, acc) : acc;
      const bool own_entry = has && j == i;
      ri = own_entry ? rj : ri;
      have = have || own_entry;
    });
    if (valid) {
      st_nt(w + i, acc);
      if (!have) ri = own();
      a.add(ri, ri);
    }
  });
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst, rev_of(A));
}

template <bool Keep, class P>
__global__ void __launch_bounds__(kBlock) k_cgnb_y(int32_t n, double *__restrict__ x,
                                                   double2_t *__restrict__ ra,
                                                   double *__restrict__ p,
                                                   const double *__restrict__ w, P ps) {
  State ls;
  if (!pass_begin<1>(ps, ls, FinCgnbX{})) return;
  const double alpha = ls.alpha, beta = ls.beta, gamma = ls.gamma;
  const bool exact = ls.alpha_n == 0.0;  // gamma = 1/0: use the limit alpha p_{j-1}
  Dot2 a;
  for_rows(n, [&](int32_t i) {
    const double2_t v = ld_nt(ra + i);
    const double ri = fma(-alpha, v.y, v.x);
    const double api = fma(beta, v.y, ld_nt(w + i));
    const double p_old = ld_nt(p + i);
    const double pi = fma(beta, p_old, ri);
    const double xi = ld_nt(x + i);
    st_nt(x + i, exact ? fma(alpha, p_old, xi) : fma(gamma, pi, fma(-gamma, ri, xi)));
    st_nt(p + i, pi);
    double2_t o;
    o.x = ri;
    o.y = api;
    st_pairs<Keep>(ra + i, o);
    a.add(api, pi);
  }, Keep);  // backwards with kept pairs: k_cgnb_x starts where this ends
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst, Keep);
}

}  // namespace its
