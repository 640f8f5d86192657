// How many iterations the host launches between two reads of the State.  Host
// code without HIP.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace its {

struct Batches {
  int least, most;  // equal: every batch has this length
};

// A read idles the GPU for ~20 us; an iteration launched after the solve has
// stopped costs 4-10 us, and 40 with eight Gauss-Seidel colours.  Systems of
// 2^20 rows and more start with 8 iterations and go to 32 while the end is far:
// in batches of 32 from the start CG on 128^3 varying values that stops after one
// iteration takes 531 us instead of 267, 27-point Gauss-Seidel on 104^3 1320
// instead of 400, and in batches of 8 throughout 40 Jacobi sweeps of 120x110x96
// take 720 us instead of 676.  Below, 32: 64 loses where a solve has few hundred
// iterations (45x38x41 1.74 -> 2.06 ms).
inline Batches batches(int check_every, int64_t n) {
  if (check_every > 0) return {check_every, check_every};
  return {n >= (int64_t(1) << 20) ? 8 : 32, 32};
}

// The next batch, after `done` iterations that took r.r from rho0 to rho1: half
// of what is left to the threshold at the mean rate so far.
inline int next_batch(const Batches &b, double rho0, double rho1, int64_t done, double thr2) {
  if (b.least == b.most) return b.least;
  if (!(rho1 > thr2) || !std::isfinite(rho1) || !(rho0 > 0.0) || done < 1) return b.least;
  if (thr2 <= 0.0 || rho1 >= rho0) return b.most;
  const double left = std::log(rho1 / thr2) * double(done) / std::log(rho0 / rho1);
  return int(std::min<double>(b.most, std::max<double>(b.least, 0.5 * left)));
}

}  // namespace its
