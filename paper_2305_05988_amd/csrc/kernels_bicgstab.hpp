// BiCGStab passes (arithmetic of the paper's Algorithm 2, with restart).
#pragma once

#include "common.hpp"
#include "fins.hpp"
#include "rowops.hpp"

namespace its {

// --------------------------------------------------------------- BiCGStab
// Algorithm 2's arithmetic in three fused passes per iteration:
//   A: p = r + beta u on the fly (p = r after a restart or at the start),
//      r' = r/||r|| after a restart, v = A p, alpha_d = v.r'
//   B: s = r - alpha v on the fly, t = A s, t.s, t.t, omega
//   C: x = (x + alpha p) + omega s, r = s - omega t, u = p - omega v,
//      alpha_n' = r.r', beta = r.r, restart test, convergence test
// u = p - omega v is formed in pass C, where omega is already known, so
// pass A forms p = fma(beta, u, r) -- the same roundings as forming
// fma(beta, fma(-omega, v, p), r) there.  What the SpMV passes gather is
// stored as interleaved pairs, one 16-byte access per column: {r, u} for
// pass A (written by pass C), {r, v} for pass B (written by pass A).

// r' = r / ||r||, alpha_n = r.r' (r: a vector, or with Stride 2 the first
// members of the {r, u} pairs)
template <int Stride>
__global__ void __launch_bounds__(kBlock) k_bicg_init(int32_t n, const double *__restrict__ r,
                                                      double *__restrict__ rs, Reduce *R,
                                                      double rnorm) {
  Dot2 a;
  for_rows(n, [&](int32_t i) {
    const double ri = r[int64_t(i) * Stride];
    const double rsi = ri / rnorm;
    rs[i] = rsi;
    a.add(ri, rsi);
  });
  DD v[1] = {a.get()};
  block_partial<1>(v, R);
}

struct FinBicgInit {  // alpha_n = r.r'
  State *st;
  __device__ bool active() const { return true; }
  __device__ void operator()(DD (&v)[1]) const { st->alpha_n = dd_round(v[0]); }
};

template <class Op, class P>
__global__ void __launch_bounds__(kBlock) k_bicg_a(Op A, const double2_t *__restrict__ ru,
                                                   double *__restrict__ rs, double *__restrict__ p,
                                                   double2_t *__restrict__ rv, FinBicgC fin,
                                                   P ps) {
  __shared__ typename Op::Smem sm;
  State ls;
  if (!pass_begin<2>(ps, ls, fin)) return;
  const bool plain = ls.k == 0 || ls.restart;
  const bool restart = ls.restart;
  const double bet = ls.beta;
  const double rn = restart ? __builtin_sqrt(ls.rho) : 1.0;
  const Gather<double2_t> load{ru};
  auto pv = [&](const double2_t &e) -> double { return plain ? e.x : fma(bet, e.y, e.x); };
  Dot2 a;
  A.rows(sm, load, pv, [&](int32_t i, bool valid, auto &&entries, auto &&own) {
    double acc = 0.0, pi = 0.0;
    bool have = false;  // p_i taken from the row's diagonal entry
    entries([&](int32_t j, double av, double pj, bool has = true) {
      acc = has ? fma(av, pj, acc) : acc;
      const bool own_entry = has && j == i;
      pi = own_entry ? pj : pi;
      have = have || own_entry;
    });
    if (valid) {
      if (!have) pi = own();
      const double ri = ru[i].x;
      st_nt(p + i, pi);
      double2_t o;
      o.x = ri;
      o.y = acc;
      st_pairs<GathersPairs<Op>::value>(rv + i, o);
      double rsi;
      if (restart) {
        rsi = ri / rn;
        rs[i] = rsi;
      } else {
        rsi = rs[i];
      }
      a.add(acc, rsi);
    }
  });
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst, rev_of(A));
}

template <class Op, class P>
__global__ void __launch_bounds__(kBlock) k_bicg_b(Op A, const double2_t *__restrict__ rv,
                                                   double *__restrict__ t, P ps) {
  __shared__ typename Op::Smem sm;
  State ls;
  if (!pass_begin<1>(ps, ls, FinBicgA{})) return;
  const double alpha = ls.alpha;
  const Gather<double2_t> load{rv};
  auto sv = [&](const double2_t &e) -> double { return fma(-alpha, e.y, e.x); };
  Dot2 a0, a1;
  A.rows(sm, load, sv, [&](int32_t i, bool valid, auto &&entries, auto &&own) {
    double acc = 0.0, si = 0.0;
    bool have = false;  // s_i taken from the row's diagonal entry
    entries([&](int32_t j, double av, double sv_j, bool has = true) {
      acc = has ? fma(av, sv_j, acc) : acc;
      const bool own_entry = has && j == i;
      si = own_entry ? sv_j : si;
      have = have || own_entry;
    });
    if (valid) {
      if (!have) si = own();
      st_nt(t + i, acc);
      a0.add(acc, si);
      a1.add(acc, acc);
    }
  });
  DD d[2] = {a0.get(), a1.get()};
  block_partial_to<2>(d, ps.dst, rev_of(A));
}

template <bool Keep, class P>
__global__ void __launch_bounds__(kBlock) k_bicg_c(int32_t n, double *__restrict__ x,
                                                   double2_t *__restrict__ ru,
                                                   const double *__restrict__ rs,
                                                   const double *__restrict__ p,
                                                   const double2_t *__restrict__ rv,
                                                   const double *__restrict__ t, P ps) {
  State ls;
  if (!pass_begin<2>(ps, ls, FinBicgB{})) return;
  const double alpha = ls.alpha, om = ls.omega;
  const bool half = (om == 0.0);
  Dot2 a0, a1;
  // rows i and i + kBlock of each tile of 2 kBlock rows, the loads of both in
  // flight together (a row past n re-reads row n - 1 and stores nothing)
  const int64_t ntiles = (int64_t(n) + 2 * kBlock - 1) / (2 * kBlock);
  const Sched sc = my_tiles(ntiles);
  for (int64_t k = sc.begin; k < sc.end; k += sc.stride) {
    int32_t i[2];
    i[0] = int32_t(k * 2 * kBlock + threadIdx.x);
    i[1] = i[0] + kBlock;
    double2_t e[2];
    double xi[2], pi[2], rsi[2], ti[2] = {0.0, 0.0};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int32_t j = min(i[h], n - 1);
      e[h] = ld_nt(rv + j);  // {r_j, v_j}
      xi[h] = ld_nt(x + j);
      pi[h] = ld_nt(p + j);
      rsi[h] = ld_nt(rs + j);
      if (!half) ti[h] = ld_nt(t + j);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (i[h] >= n) continue;
      const double si = fma(-alpha, e[h].y, e[h].x);
      double ri;
      if (half) {
        st_nt(x + i[h], fma(alpha, pi[h], xi[h]));
        ri = si;
      } else {
        st_nt(x + i[h], fma(om, si, fma(alpha, pi[h], xi[h])));
        ri = fma(-om, ti[h], si);
      }
      double2_t o;
      o.x = ri;
      o.y = fma(-om, e[h].y, pi[h]);  // u = p - omega v
      st_pairs<Keep>(ru + i[h], o);
      a0.add(ri, rsi[h]);
      a1.add(ri, ri);
    }
  }
  DD d[2] = {a0.get(), a1.get()};
  block_partial_to<2>(d, ps.dst);
}

}  // namespace its
