// Sums of unevaluated pairs of doubles (error-free transformations).  Plain
// arithmetic behind HIP's qualifiers, so that a host compiler takes it as well.
#pragma once

namespace its {

struct DD {  // unevaluated sum hi + lo, |lo| <= ulp(hi)/2 when normalised
  double hi, lo;
};

__device__ __forceinline__ DD two_sum(double a, double b) {
  const double s = a + b;
  const double bp = s - a;
  const double e = (a - (s - bp)) + (b - bp);
  return {s, e};
}

__device__ __forceinline__ DD fast_two_sum(double a, double b) {  // |a| >= |b|
  const double s = a + b;
  return {s, b - (s - a)};
}

// Accurate double-double addition (of normalised pairs: relative error at most 3 * 2^-106).
__device__ __forceinline__ DD dd_add(DD a, DD b) {
  DD s = two_sum(a.hi, b.hi);
  const DD t = two_sum(a.lo, b.lo);
  s.lo += t.hi;
  s = fast_two_sum(s.hi, s.lo);
  s.lo += t.lo;
  return fast_two_sum(s.hi, s.lo);
}

// Cascaded sum of unevaluated pairs (the Sum2 step of Ogita-Rump-Oishi):
// the high parts are added error-free, their error joins the low parts.
// The result is the sum of the operands' values up to an error of about
// 2^-106 times the sum of their magnitudes, the accuracy class of Dot2
// itself, so a reduction of Dot2 partials through it keeps Dot2's bound; it
// costs 8 additions instead of dd_add's 20.
__device__ __forceinline__ DD dd_cascade(DD a, DD b) {
  const DD s = two_sum(a.hi, b.hi);
  return {s.hi, (a.lo + b.lo) + s.lo};
}

__device__ __forceinline__ double dd_round(DD v) { return v.hi + v.lo; }

// A running sum of such pairs with the errors of the low parts kept as well:
// more accurate than a chain of dd_add, whose every addition waits for the one
// before it to renormalise, where here each accumulator waits for one addition.
struct DDSum {
  double s = 0.0, c = 0.0, e = 0.0;
  __device__ __forceinline__ void add(DD v) {
    const DD h = two_sum(s, v.hi), l = two_sum(c, v.lo);
    const DD m = two_sum(l.hi, h.lo);
    s = h.hi;
    c = m.hi;
    e += l.lo + m.lo;
  }
  __device__ __forceinline__ DD get() const {
    const DD t = two_sum(s, c);
    return fast_two_sum(t.hi, t.lo + e);
  }
};

// v[d] = the partials first, first + step, ... below count of src[d], added in
// that order, four of them in flight at a time: the serial part of the sums over
// a grid's blocks.  Its error follows the running sum; with dd_cascade, which
// takes 8 operations instead of 20, it would follow the magnitudes of all partials.
template <int ND>
__device__ __forceinline__ void dd_sum(const DD *const *src, int first, int step, int count, DD (&v)[ND]) {
  constexpr int kU = 4;
  DDSum sum[ND];
  for (int at = 0; at < count; at += kU * step) {  // at: the same for all first < step
    DD t[kU][ND];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int j = first + at + u * step;
#pragma unroll
      for (int d = 0; d < ND; ++d) t[u][d] = j < count ? src[d][j] : DD{0.0, 0.0};
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      if (at + u * step >= count) break;
#pragma unroll
      for (int d = 0; d < ND; ++d) sum[d].add(t[u][d]);
    }
  }
#pragma unroll
  for (int d = 0; d < ND; ++d) v[d] = sum[d].get();
}

}  // namespace its
