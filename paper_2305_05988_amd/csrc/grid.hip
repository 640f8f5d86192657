// The passes of constant stencils on large grids: kernels and launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "fins.hpp"
#include "grid.hpp"

namespace its {

struct None {};

// Accesses to a row's own entries, which no other block wants soon.  Stream:
// past the caches, for solves whose vectors do not fit the 256 MB memory-side
// cache (grid_run); the others keep what they store and find it there.
template <bool Stream, class T>
__device__ __forceinline__ T ld(const T *p) {
  if constexpr (Stream)
    return ld_nt(p);
  else
    return *p;
}
template <bool Stream, class T>
__device__ __forceinline__ void st(T *p, T v) {
  if constexpr (Stream)
    st_nt(p, v);
  else
    *p = v;
}

// Loads of one vector and of two.
template <class T>
struct One {
  const T *p;
  __device__ __forceinline__ T at(int64_t ub, uint32_t off) const { return (p + ub)[off]; }
};
template <class T>
struct Two {
  struct Raw {
    T a, b;
  };
  const T *a, *b;
  __device__ __forceinline__ Raw at(int64_t ub, uint32_t off) const { return {(a + ub)[off], (b + ub)[off]}; }
};

struct Always {
  __device__ __forceinline__ bool operator()() const { return true; }
};
struct Same {
  template <class T>
  __device__ __forceinline__ T operator()(T v) const { return v; }
};
struct KeepValue {
  template <class Raw, class T>
  __device__ __forceinline__ T operator()(const Raw &, T v) const { return v; }
};
struct KeepNone {
  template <class Raw, class T>
  __device__ __forceinline__ None operator()(const Raw &, T) const { return {}; }
};

// y = A x
template <class Op>
__global__ void __launch_bounds__(kBlock) k_grid_spmv(Op A, const double *__restrict__ x, double *__restrict__ y) {
  __shared__ typename Op::SweepSmem sm;
  A.template sweep<ChainSum<double>>(sm, One<double>{x}, Always{}, Same{}, KeepNone{}, [](int32_t) { return None{}; },
                                     [&](int32_t i, const ChainSum<double> &q, None, None) { st_nt(y + i, q.s); });
}

// r = b - A x (stored where r is not null, with zeros in `zero`) and r.r
template <class Op>
__global__ void __launch_bounds__(kBlock) k_grid_residual(Op A, const double *__restrict__ b,
                                                          const double *__restrict__ x, double *__restrict__ r,
                                                          double *__restrict__ zero, DD *dst) {
  __shared__ typename Op::SweepSmem sm;
  Dot2 a;
  A.template sweep<ChainSum<double>>(sm, One<double>{x}, Always{}, Same{}, KeepNone{}, [&](int32_t i) { return ld_nt(b + i); },
                                     [&](int32_t i, const ChainSum<double> &q, None, double bi) {
                                       const double ri = bi - q.s;
                                       if (r) st_nt(r + i, ri);
                                       if (zero) st_nt(zero + i, 0.0);
                                       a.add(ri, ri);
                                     });
  DD v[1] = {a.get()};
  DD *const to[kMaxDots] = {dst, nullptr};
  block_partial_to<1>(v, to);
}

// The same without r, for the test after a Gauss-Seidel iteration.
template <class Op>
__global__ void __launch_bounds__(kBlock) k_grid_check(Op A, const double *__restrict__ b,
                                                       const double *__restrict__ x, PassPlain ps) {
  __shared__ typename Op::SweepSmem sm;
  if (ps.in->flag != kRunning) return;
  Dot2 a;
  A.template sweep<ChainSum<double>>(sm, One<double>{x}, Always{}, Same{}, KeepNone{}, [&](int32_t i) { return b[i]; },
                                     [&](int32_t, const ChainSum<double> &q, None, double bi) {
                                       const double ri = bi - q.s;
                                       a.add(ri, ri);
                                     });
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst);
}

// A Jacobi sweep (k_jacobi): the residual of x, and xn = (b - off) / diag.
template <class Op, bool S, class P>
__global__ void __launch_bounds__(kBlock) k_grid_jacobi(Op A, const double *__restrict__ b,
                                                        const double *__restrict__ x, double *__restrict__ xn, P ps) {
  __shared__ typename Op::SweepSmem sm;
  State s;
  Dot2 a;
  const auto begin = [&] { return pass_begin<1>(ps, s, FinJacobi{}); };
  const bool on = A.template sweep<ChainSplit>(sm, One<double>{x}, begin, Same{}, KeepNone{}, [&](int32_t i) { return ld<S>(b + i); },
                               [&](int32_t i, const ChainSplit &q, None, double bi) {
                                 const double ri = bi - q.s;
                                 a.add(ri, ri);
                                 xn[i] = (bi - q.off) / A.diagonal(q);  // the next sweep's x
                               });
  if (!on) return;
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst);
}

// A red-black Gauss-Seidel half-sweep over the rows of one colour (the parity
// of x + y + z), in place, with the residual test riding on the sweeps as in
// k_gs_rows_packed (kGsFinal, kGsLagged).  A row reads only rows of the other
// colour, which no block writes.  xs: the old values of the black rows, row i at
// i / 2 (two neighbours in a line, or the last point of a line and the first
// of the next where they share a pair, have different colours).  Whole lines
// are stored, the other colour's values as they were.
template <class Op, int Mode, class P>
__global__ void __launch_bounds__(kBlock) k_grid_gs(Op A, uint32_t colour, const double *__restrict__ b, double *x,
                                                    double *__restrict__ xs, P ps) {
  __shared__ typename Op::SweepSmem sm;
  using Chain = std::conditional_t<Mode == kGsFinal, ChainTwice, ChainSplit>;
  State s;
  Dot2 a;
  const auto begin = [&] { return pass_begin<2>(ps, s, FinGs2{}); };
  const bool on = A.template sweep<Chain>(
      sm, One<double>{x}, begin, Same{}, KeepValue{}, [&](int32_t i) { return b[i]; },
      [&](int32_t i, const Chain &q, double xi, double bi, uint32_t odd, bool last) {
        double xn = xi;
        if (odd == colour) {
          xn = (bi - q.off) / A.diagonal(q);
          double ri = 0.0;
          if constexpr (Mode == kGsLagged) {
            ri = bi - q.s;
            xs[i >> 1] = xi;
          }
          if constexpr (Mode == kGsFinal) ri = bi - q.with(A.c, xn, last);
          if constexpr (Mode != kGsPlain) a.add(ri, ri);
        }
        x[i] = xn;
      });
  if (!on) return;
  if constexpr (Mode != kGsPlain) {
    DD v[1] = {a.get()};
    block_partial_to<1>(v, ps.dst);
  }
}

// The black rows of the tested iterate put back.
__global__ void __launch_bounds__(kBlock) k_grid_gs_restore(int32_t n, int32_t nx, int32_t ny,
                                                            const double *__restrict__ xs, double *__restrict__ x) {
  for_rows(n, [&](int32_t i) {
    const int32_t t = i / nx, ix = i - t * nx, iz = t / ny, iy = t - iz * ny;
    if ((ix + iy + iz) & 1) x[i] = xs[i >> 1];
  });
}

// CG in 7.5 vectors an iteration (the pair form of k_cg_pass1 and k_cg_pass2
// moves 9): with the operator for free, A p costs less to form twice than to
// store and load.
//   pass a: p' = r + beta p formed for every point loaded and stored for the
//           block's own, p'.(A p')
//   pass b: q = A p' again, r -= alpha q, r.r; every other iteration x with
//           both iterations' steps
// p and p' are two buffers: other blocks still load p while p' is stored.  The
// roundings are k_cg_pass1's and k_cg_pass2's.
template <class Op, class T, bool S, class P>
__global__ void __launch_bounds__(kBlock) k_grid_cg_a(Op A, const T *__restrict__ r, const T *__restrict__ p,
                                                      T *__restrict__ pn, P ps) {
  __shared__ typename Op::SweepSmem sm;
  State s;
  T beta = T(0);
  Dot2 a;
  const auto begin = [&] {
    const bool on = pass_begin<1>(ps, s, FinCg2{});
    beta = T(s.beta);
    return on;
  };
  const bool on = A.template sweep<ChainSum<T>>(sm, Two<T>{r, p}, begin, [&](const typename Two<T>::Raw &v) { return fmaT(beta, v.b, v.a); },
                                KeepValue{}, [](int32_t) { return None{}; },
                                [&](int32_t i, const ChainSum<T> &q, T pi, None) {
                                  st<S>(pn + i, pi);
                                  a.add(double(pi), double(q.s));
                                });
  if (!on) return;
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst);
}

template <class Op, class T, bool S, class P>
__global__ void __launch_bounds__(kBlock) k_grid_cg_b(Op A, const T *__restrict__ pn, const T *__restrict__ p,
                                                      T *__restrict__ r, T *__restrict__ x, bool defer, P ps) {
  __shared__ typename Op::SweepSmem sm;
  State s;
  T alpha = T(0), alpha_x = T(0);
  bool on = false;
  Dot2 a;
  const auto begin = [&] {
    const bool ok = pass_begin<1>(ps, s, FinCg1{});
    alpha = T(s.alpha);
    alpha_x = T(s.alpha_x);
    return ok;
  };
  struct Own {
    T r, x, p;
  };
  auto run = [&](auto later) {
    constexpr bool kLater = decltype(later)::value;
    on = A.template sweep<ChainSum<T>>(sm, One<T>{pn}, begin, Same{}, KeepValue{},
                                  [&](int32_t i) {
                                    if constexpr (kLater)
                                      return ld<S>(r + i);
                                    else
                                      return Own{ld<S>(r + i), ld<S>(x + i), ld<S>(p + i)};
                                  },
                                  [&](int32_t i, const ChainSum<T> &q, T pi, const auto &o) {
                                    T ri;
                                    if constexpr (kLater) {
                                      ri = fmaT(-alpha, q.s, o);
                                    } else {
                                      st<S>(x + i, fmaT(alpha, pi, fmaT(alpha_x, o.p, o.x)));
                                      ri = fmaT(-alpha, q.s, o.r);
                                    }
                                    st<S>(r + i, ri);
                                    a.add(double(ri), double(ri));
                                  });
  };
  if (defer)
    run(std::true_type());
  else
    run(std::false_type());
  if (!on) return;
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst);
}

// Pass X of CG-NB (k_cgnb_x).
template <class Op, class P>
__global__ void __launch_bounds__(kBlock) k_grid_cgnb_x(Op A, const double2_t *__restrict__ ra,
                                                        double *__restrict__ w, P ps) {
  __shared__ typename Op::SweepSmem sm;
  State s;
  double alpha = 0.0;
  Dot2 a;
  const auto begin = [&] {
    const bool ok = pass_begin<1>(ps, s, FinCgnbY{});
    alpha = s.alpha;
    return ok;
  };
  const bool on = A.template sweep<ChainSum<double>>(sm, One<double2_t>{ra}, begin, [&](const double2_t &v) { return fma(-alpha, v.y, v.x); },
                                     KeepValue{}, [](int32_t) { return None{}; },
                                     [&](int32_t i, const ChainSum<double> &q, double ri, None) {
                                       st_nt(w + i, q.s);
                                       a.add(ri, ri);
                                     });
  if (!on) return;
  DD v[1] = {a.get()};
  block_partial_to<1>(v, ps.dst);
}

// BiCGStab in 14 vectors an iteration (the pair form, kernels_bicgstab.hpp,
// moves 18): t = A s is formed twice instead of stored, and p, which is
// r + beta u, where it is needed.
//   pass a: p for every point loaded, v = A p, v.r'
//   pass b: s = r - alpha v for every point loaded, t = A s, t.s, t.t
//   pass c: s and t again, x, r, u = p - omega v, r.r', r.r
// r alternates between two buffers: pass c stores its own rows' new r while
// other blocks load the old one.  The roundings are the pair form's.
template <class Op, bool S, class P>
__global__ void __launch_bounds__(kBlock) k_grid_bicg_a(Op A, const double *__restrict__ r,
                                                        const double *__restrict__ u, double *__restrict__ rs,
                                                        double *__restrict__ v, FinBicgC fin, P ps) {
  __shared__ typename Op::SweepSmem sm;
  State s;
  bool restart = false, plain = false;
  double bet = 0.0, rn = 1.0;
  using Raw = Two<double>::Raw;
  Dot2 a;
  const auto begin = [&] {
    const bool ok = pass_begin<2>(ps, s, fin);
    restart = s.restart != 0;
    plain = s.k == 0 || restart;
    bet = s.beta;
    if (restart) rn = __builtin_sqrt(s.rho);
    return ok;
  };
  const bool on = A.template sweep<ChainSum<double>>(sm, Two<double>{r, u}, begin,
                                     [&](const Raw &e) { return plain ? e.a : fma(bet, e.b, e.a); },
                                     [](const Raw &e, double) { return e.a; }, [&](int32_t i) { return ld<S>(rs + i); },
                                     [&](int32_t i, const ChainSum<double> &q, double ri, double rsi) {
                                       st<S>(v + i, q.s);
                                       if (restart) {
                                         rsi = ri / rn;
                                         rs[i] = rsi;
                                       }
                                       a.add(q.s, rsi);
                                     });
  if (!on) return;
  DD d[1] = {a.get()};
  block_partial_to<1>(d, ps.dst);
}

template <class Op, class P>
__global__ void __launch_bounds__(kBlock) k_grid_bicg_b(Op A, const double *__restrict__ r,
                                                        const double *__restrict__ v, P ps) {
  __shared__ typename Op::SweepSmem sm;
  State s;
  double alpha = 0.0;
  Dot2 a0, a1;
  const auto begin = [&] {
    const bool ok = pass_begin<1>(ps, s, FinBicgA{});
    alpha = s.alpha;
    return ok;
  };
  const bool on = A.template sweep<ChainSum<double>>(sm, Two<double>{r, v}, begin,
                                     [&](const Two<double>::Raw &e) { return fma(-alpha, e.b, e.a); }, KeepValue{},
                                     [](int32_t) { return None{}; },
                                     [&](int32_t, const ChainSum<double> &q, double si, None) {
                                       a0.add(q.s, si);
                                       a1.add(q.s, q.s);
                                     });
  if (!on) return;
  DD d[2] = {a0.get(), a1.get()};
  block_partial_to<2>(d, ps.dst);
}

template <class Op, bool S, class P>
__global__ void __launch_bounds__(kBlock) k_grid_bicg_c(Op A, const double *__restrict__ r, double *__restrict__ rn,
                                                        double *__restrict__ u, const double *__restrict__ v,
                                                        const double *__restrict__ rs, double *__restrict__ x,
                                                        P ps) {
  __shared__ typename Op::SweepSmem sm;
  State s;
  double alpha = 0.0, om = 0.0, bet = 0.0;
  bool half = false, plain = false;
  const auto begin = [&] {
    const bool ok = pass_begin<2>(ps, s, FinBicgB{});
    alpha = s.alpha;
    om = s.omega;
    bet = s.beta;
    half = om == 0.0;
    plain = s.plain != 0;
    return ok;
  };
  using Raw = Two<double>::Raw;
  struct Own {
    double u, rs, x;
  };
  Dot2 a0, a1;
  const bool on = A.template sweep<ChainSum<double>>(sm, Two<double>{r, v}, begin, [&](const Raw &e) { return fma(-alpha, e.b, e.a); },
                                     [](const Raw &e, double) { return e; },
                                     [&](int32_t i) { return Own{ld<S>(u + i), ld<S>(rs + i), ld<S>(x + i)}; },
                                     [&](int32_t i, const ChainSum<double> &q, const Raw &e, const Own &o) {
                                       const double si = fma(-alpha, e.b, e.a);
                                       const double pi = plain ? e.a : fma(bet, o.u, e.a);
                                       const double xh = fma(alpha, pi, o.x);
                                       st<S>(x + i, half ? xh : fma(om, si, xh));
                                       const double ri = half ? si : fma(-om, q.s, si);
                                       st<S>(rn + i, ri);
                                       st<S>(u + i, fma(-om, e.b, pi));
                                       a0.add(ri, o.rs);
                                       a1.add(ri, ri);
                                     });
  if (!on) return;
  DD d[2] = {a0.get(), a1.get()};
  block_partial_to<2>(d, ps.dst);
}

// ------------------------------------------------------------------ launches

namespace {

template <int NPTS, class T, int R>
GridOp<NPTS, T, R> make(const GridRun &g) {
  GridOp<NPTS, T, R> op{g.a->nx, g.a->ny, g.a->nz, g.a->n, {}, g.plan};
  for (int q = 0; q < NPTS; ++q) op.c[q] = std::is_same<T, float>::value ? T(g.a->lo[q]) : T(g.a->c[q]);
  return op;
}


template <class T, class F>
hipError_t with(const GridRun &g, F &&f) {
  if constexpr (std::is_same<T, double>::value) {
    if (g.a->npts == 1) {
      f(VarGridOp<2>{g.a->nx, g.a->ny, g.a->nz, g.a->n, g.a->k, g.plan});
      return hipGetLastError();
    }
  }
  if (g.a->npts == 7)
    g.points == 4 ? f(make<7, T, 4>(g)) : f(make<7, T, 2>(g));
  else
    g.points == 4 ? f(make<27, T, 4>(g)) : f(make<27, T, 2>(g));
  return hipGetLastError();
}
template <class F>
void with_pass(const Pass &p, F &&f) {
  if (p.count > 0)
    f(p);
  else
    f(PassPlain{p.in, {p.dst[0], p.dst[1]}});
}
// f(op, whether the pass streams)
template <class F>
hipError_t with_stream(const GridRun &g, F &&f) {
  return with<double>(g, [&](auto op) { g.stream ? f(op, std::true_type()) : f(op, std::false_type()); });
}

}  // namespace

// Streaming from 256 MB of vectors on: CG 256^3 (512 MB) 164 us against 197
// with allocating accesses, 27-point 192^3 (226 MB) 79.6 against 73.3.  The
// refinement's FP32 CG never streams: 272^3 124 us against 145 streaming, 288^3
// 144 and 156, 400^3 405 and 421 (320^3 alone 201 and 177).
GridRun grid_run(const GridStencil &a, int64_t vector_bytes, hipStream_t s) {
  static_assert(kGridThreads == kBlock, "the plan's block size");
  if (a.npts == 1) vector_bytes += int64_t(8) * a.n;  // k
  const GridShape shape = grid_shape(a.npts, a.nx, a.ny, a.nz);
  GridRun g{&a, shape.plan, shape.points, 0, vector_bytes > (int64_t(256) << 20), s};
  const int64_t b = int64_t(g.plan.ntx) * g.plan.nty * g.plan.ncz;
  // one round for all: up to the next multiple of 8 (XCDs), not down (CG
  // 192x193x191, 507 bricks: 93 us with 504 blocks, 72 with 512; 272^3, 468: 297
  // and 220)
  g.blocks = int(std::min<int64_t>(b < 64 ? b : (b + kXcds - 1) / kXcds * kXcds, kFinishOne));
  return g;
}

#define GRID_LAUNCH(T, kernel, ...)                                                                 \
  return with<T>(g, [&](auto op) {                                                                  \
    using Op = decltype(op);                                                                        \
    hipLaunchKernelGGL((kernel), dim3(g.blocks), dim3(kBlock), 0, g.s, op, __VA_ARGS__);            \
  })

// The same with the pass as its type says: pending partials or none.
#define GRID_LAUNCH_PASS(T, pass, kernel, ...)                                                      \
  return with<T>(g, [&](auto op) {                                                                  \
    using Op = decltype(op);                                                                        \
    with_pass(pass, [&](auto ps) {                                                                  \
      using P = decltype(ps);                                                                       \
      hipLaunchKernelGGL((kernel), dim3(g.blocks), dim3(kBlock), 0, g.s, op, __VA_ARGS__, ps);      \
    });                                                                                             \
  })

#define GRID_LAUNCH_STREAM(pass, kernel, ...)                                                             \
  return with_stream(g, [&](auto op, auto stream) {                                                 \
    using Op = decltype(op);                                                                        \
    constexpr bool S = decltype(stream)::value;                                                     \
    with_pass(pass, [&](auto ps) {                                                                  \
      using P = decltype(ps);                                                                       \
      hipLaunchKernelGGL((kernel), dim3(g.blocks), dim3(kBlock), 0, g.s, op, __VA_ARGS__, ps);      \
    });                                                                                             \
  })

hipError_t grid_spmv(const GridRun &g, const double *x, double *y) { GRID_LAUNCH(double, k_grid_spmv<Op>, x, y); }
hipError_t grid_residual(const GridRun &g, const double *b, const double *x, double *r, double *zero, DD *dst) {
  GRID_LAUNCH(double, k_grid_residual<Op>, b, x, r, zero, dst);
}
hipError_t grid_check(const GridRun &g, const double *b, const double *x, const PassPlain &ps) {
  GRID_LAUNCH(double, k_grid_check<Op>, b, x, ps);
}
hipError_t grid_jacobi(const GridRun &g, const double *b, const double *x, double *xn, const Pass &ps) {
  GRID_LAUNCH_STREAM(ps, (k_grid_jacobi<Op, S, P>), b, x, xn);
}
hipError_t grid_cg_a(const GridRun &g, const double *r, const double *p, double *pn, const Pass &ps) {
  GRID_LAUNCH_STREAM(ps, (k_grid_cg_a<Op, double, S, P>), r, p, pn);
}
hipError_t grid_cg_b(const GridRun &g, const double *pn, const double *p, double *r, double *x, bool defer,
                     const Pass &ps) {
  GRID_LAUNCH_STREAM(ps, (k_grid_cg_b<Op, double, S, P>), pn, p, r, x, defer);
}
hipError_t grid_cg_a(const GridRun &g, const float *r, const float *p, float *pn, const Pass &ps) {
  GRID_LAUNCH_PASS(float, ps, (k_grid_cg_a<Op, float, false, P>), r, p, pn);
}
hipError_t grid_cg_b(const GridRun &g, const float *pn, const float *p, float *r, float *x, bool defer,
                     const Pass &ps) {
  GRID_LAUNCH_PASS(float, ps, (k_grid_cg_b<Op, float, false, P>), pn, p, r, x, defer);
}
hipError_t grid_cgnb_x(const GridRun &g, const double2_t *ra, double *w, const Pass &ps) {
  GRID_LAUNCH_PASS(double, ps, (k_grid_cgnb_x<Op, P>), ra, w);
}
hipError_t grid_bicg_a(const GridRun &g, const double *r, const double *u, double *rs, double *v, const FinBicgC &fin,
                       const Pass &ps) {
  GRID_LAUNCH_STREAM(ps, (k_grid_bicg_a<Op, S, P>), r, u, rs, v, fin);
}
hipError_t grid_bicg_b(const GridRun &g, const double *r, const double *v, const Pass &ps) {
  GRID_LAUNCH_PASS(double, ps, (k_grid_bicg_b<Op, P>), r, v);
}
hipError_t grid_bicg_c(const GridRun &g, const double *r, double *rn, double *u, const double *v, const double *rs,
                       double *x, const Pass &ps) {
  GRID_LAUNCH_STREAM(ps, (k_grid_bicg_c<Op, S, P>), r, rn, u, v, rs, x);
}

hipError_t grid_gs(const GridRun &g, int mode, int colour, const double *b, double *x, double *xs, const Pass &ps) {
  auto go = [&](auto op, auto m) {
    using Op = decltype(op);
    constexpr int M = decltype(m)::value;
    with_pass(ps, [&](auto p) {
      hipLaunchKernelGGL((k_grid_gs<Op, M, decltype(p)>), dim3(g.blocks), dim3(kBlock), 0, g.s, op, uint32_t(colour), b,
                         x, xs, p);
    });
  };
  auto modes = [&](auto op) {
    if (mode == kGsPlain) go(op, std::integral_constant<int, kGsPlain>());
    if (mode == kGsFinal) go(op, std::integral_constant<int, kGsFinal>());
    if (mode == kGsLagged) go(op, std::integral_constant<int, kGsLagged>());
  };
  g.points == 4 ? modes(make<7, double, 4>(g)) : modes(make<7, double, 2>(g));
  return hipGetLastError();
}
hipError_t grid_gs_restore(const GridRun &g, const double *xs, double *x) {
  hipLaunchKernelGGL(k_grid_gs_restore, dim3(grid_for(g.a->n, kFinishOne)), dim3(kBlock), 0, g.s, g.a->n, g.a->nx,
                     g.a->ny, xs, x);
  return hipGetLastError();
}

}  // namespace its
