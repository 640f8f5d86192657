// Packed CSR whose slices repeat: a table of slice patterns and one pattern
// number per 64-row slice (see rowops.hpp for the row-walk contract).
#pragma once

#include "sell.hpp"

namespace its {

// A slice (64 consecutive rows of the layout, sell.hpp) has a pattern when
// its rows are strictly ascending, take their column offsets (column minus
// row) from one list of at most kPatMax offsets and, per offset, hold one
// value, bit for bit the same in every row that has the entry.  The pattern
// is the ascending list of {offset, 64-bit mask of the lanes that have the
// entry, value}.  Matrices of constant-coefficient operators on structured
// grids consist of a few patterns (one per kind of boundary and per phase of
// the grid line within a slice), so the matrix costs a pass 4 bytes per 64
// rows instead of 8 per entry, and a row's entries, their presence and their
// values are wave-uniform: the table is read through the scalar cache, the
// masks become exec masks and the gathers of a wave are contiguous runs at
// uniform bases, with no address arithmetic per lane.  A row's entries are
// consumed in ascending offset, which is its stored order, so the chain is
// the CSR chain bit for bit.
//
// Bound by the gathers through L1 and L2 (seven 16-byte ones per row for the
// 7-point CG pass), not by HBM.  Measured against the layout with a value per
// entry, on a duct of 8x8x125000 points that the plane sweep (grid.hpp) leaves to
// this walk: one product 91 -> 37 us, an iteration of CG 167 -> 117, of Jacobi
// 118 -> 71 and of red-black Gauss-Seidel 191 -> 90.  Blocks walk several tiles: the
// CG pass alone on 16.8 million rows takes 103 us with at most 4096 blocks, 124
// with 8192 and 137 with one tile per block.
constexpr int kPatMax = 32;            // positions per pattern
static_assert(kPatMax == kMaxOffsetWidth, "the scan of a slice serves both forms");
constexpr int kPatTable = 1 << 15;     // hash slots of the search for patterns
constexpr int kPatLimit = 1 << 13;     // most patterns a layout may have

struct alignas(16) PatHead {
  int32_t w;           // positions
  int32_t dmin, dmax;  // first and last offset
  int32_t full;        // every lane has every entry
};

// Pattern q's entries sit at positions kPatMax q + j.
struct PatTable {
  const PatHead *head;
  const int32_t *off;
  const uint64_t *mask;
  const double *val;
};

// Wave-uniform reads that the compiler turns into scalar loads.
template <class X>
using const_ptr = const __attribute__((address_space(4))) X *;
template <class X>
__device__ __forceinline__ const_ptr<X> as_const(const X *p) {
  return (const_ptr<X>)(reinterpret_cast<uintptr_t>(p));
}

// A gather functor's load of element ub + lane, ub wave-uniform.
template <class L>
__device__ __forceinline__ auto load_at(const L &load, int64_t ub, uint32_t lane, int)
    -> decltype(load.at(ub, lane)) {
  return load.at(ub, lane);
}
template <class L>
__device__ __forceinline__ auto load_at(const L &load, int64_t ub, uint32_t lane, long)
    -> decltype(load(0)) {
  return load(int32_t(ub + lane));
}

// T: the arithmetic type (double, or float for the refinement's inner solve,
// whose table holds the FP32 or FP16 values widened exactly to float).
template <class T>
struct PatOp {
  using value_type = T;
  const int32_t *__restrict__ pid;  // pattern of each slice
  const PatHead *__restrict__ head;
  const int32_t *__restrict__ off;
  const uint64_t *__restrict__ mask;
  const T *__restrict__ val;
  int32_t n;
  const int32_t *__restrict__ row_of;  // layout row p is matrix row row_of[p] (null: p)

  struct Smem {};

  int grid() const { return grid_for(n, kFinishOne); }
  template <class Load, class Value, class Body>
  __device__ __forceinline__ void rows(Smem &sm, Load &&load, Value &&value, Body &&body) const {
    tiled_rows(*this, sm, load, value, body);
  }
  template <class Body>
  __device__ __forceinline__ void own_rows(Body &&body) const {
    tiled_own_rows(*this, body);
  }

  // Entries g .. g + W - 1 of the pattern at table position k.  Inside: every
  // row + offset of the slice is a row of the matrix, so the gathers need no
  // per-lane check (a lane without the entry loads some row's value and does
  // not consume it).  Full: every lane has every entry.
  template <int W, bool Inside, bool Full, class Fetch, class Consume>
  __device__ __forceinline__ void group(int32_t k, int32_t ub, uint32_t lane, int32_t row, int32_t standin,
                                        Fetch &&fetch, Consume &&consume) const {
    int32_t d[W];
    uint64_t m[W];
    T a[W];
#pragma unroll
    for (int u = 0; u < W; ++u) {
      d[u] = as_const(off)[k + u];
      if (!Full) m[u] = as_const(mask)[k + u];
      a[u] = as_const(val)[k + u];
    }
    bool has[W];
#pragma unroll
    for (int u = 0; u < W; ++u) has[u] = Full || __builtin_amdgcn_inverse_ballot_w64(m[u]);
    decltype(fetch(0)) x[W];
#pragma unroll
    for (int u = 0; u < W; ++u) {
      if constexpr (Inside)
        x[u] = load_at(fetch, int64_t(ub) + d[u], lane, 0);
      else
        x[u] = fetch(has[u] ? row + d[u] : standin);
    }
#pragma unroll
    for (int u = 0; u < W; ++u) consume(row + d[u], a[u], x[u], has[u]);
  }

  template <bool Inside, bool Full, class Fetch, class Consume>
  __device__ __forceinline__ void walk(int32_t k, int32_t w, int32_t ub, uint32_t lane, int32_t row,
                                       int32_t standin, Fetch &&fetch, Consume &&consume) const {
    int32_t g = 0;
    for (; w - g >= 9; g += 9) group<9, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume);
    switch (w - g) {  // wave-uniform
      case 1: group<1, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume); break;
      case 2: group<2, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume); break;
      case 3: group<3, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume); break;
      case 4: group<4, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume); break;
      case 5: group<5, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume); break;
      case 6: group<6, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume); break;
      case 7: group<7, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume); break;
      case 8: group<8, Inside, Full>(k + g, ub, lane, row, standin, fetch, consume); break;
      default: break;
    }
  }

  template <class Fetch, class Consume>
  __device__ __forceinline__ void tile_entries(int32_t r0, int32_t r1, Smem &, Fetch &&fetch,
                                               Consume &&consume) const {
    const int32_t s = __builtin_amdgcn_readfirstlane((r0 >> 6) + (int32_t(threadIdx.x) >> 6));
    if (s * kSlice >= r1) return;
    const uint32_t lane = threadIdx.x & 63u;
    const int32_t q = as_const(pid)[s];
    const int32_t k = q * kPatMax;
    const auto *h = as_const(head) + q;
    const int32_t w = h->w, dmin = h->dmin, dmax = h->dmax, full = h->full;
    const int32_t ub = s * kSlice;
    if (!row_of && int64_t(ub) + dmin >= 0 && int64_t(ub) + (kSlice - 1) + dmax < n) {
      // the row as the kernels form it, so that their tests for the diagonal
      // entry (column == row) become tests of the uniform offset
      const int32_t row = r0 + int32_t(threadIdx.x);
      if (full)
        walk<true, true>(k, w, ub, lane, row, ub, fetch, consume);
      else
        walk<true, false>(k, w, ub, lane, row, ub, fetch, consume);
    } else {
      const int32_t p = ub + int32_t(lane);
      const int32_t row = p < n ? (row_of ? row_of[p] : p) : ub;
      walk<false, false>(k, w, ub, lane, row, row_of ? row_of[ub] : ub, fetch, consume);
    }
  }
};

// ------------------------------------------------------------------ packing

// What a wave finds out about one slice: lane j < w holds position j.
struct SlicePattern {
  int32_t d;      // offset
  uint64_t m;     // lanes with the entry
  uint64_t v, v32, v16;  // bits of the values
  int32_t w;      // positions (wave-uniform, as the rest)
  int32_t wmax;   // the slice's longest row
  bool ascending; // every row strictly ascending, at most kPatMax offsets
  bool constant;  // one value per offset, in every precision
};

__device__ __forceinline__ int32_t wave_min(int32_t v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}

// Row p of the layout is matrix row rows[p] (p when rows is null); every lane
// of the wave calls it for the same slice.  val32 and val16 may be null.  tight:
// only an offset slice is looked for, which has no more offsets than its longest
// row has entries.
__device__ __forceinline__ SlicePattern slice_pattern(int64_t s, int32_t count, const int32_t *rp, const int32_t *rows,
                                                      const int32_t *col, const double *val, const float *val32,
                                                      const __half *val16, bool tight = false) {
  const int lane = threadIdx.x & 63;
  const int64_t p = s * kSlice + lane;
  int32_t i = 0, e = 0, end = 0;
  if (p < count) {
    i = rows ? rows[p] : int32_t(p);
    e = rp[i];
    end = rp[i + 1];
  }
  SlicePattern r{0, 0, 0, 0, 0, 0, -wave_min(-(end - e)), true, true};
  const int32_t most = tight ? min(kPatMax, r.wmax) : kPatMax;
  if (r.wmax > most) {
    r.ascending = false;
    return r;
  }
  for (;;) {
    const int32_t c = e < end ? col[e] : 0;
    const int32_t mine = e < end ? c - i : INT32_MAX;
    const int32_t d = wave_min(mine);
    if (d == INT32_MAX) break;
    if (r.w == most) {
      r.ascending = false;
      break;
    }
    const bool has = mine == d;
    const uint64_t m = __ballot(has);
    const int first = __ffsll(static_cast<unsigned long long>(m)) - 1;
    const uint64_t v = has ? __builtin_bit_cast(uint64_t, val[e]) : 0;
    const uint64_t v32 = has && val32 ? __builtin_bit_cast(uint32_t, val32[e]) : 0;
    const uint64_t v16 = has && val16 ? __builtin_bit_cast(unsigned short, val16[e]) : 0;
    const uint64_t u = __shfl(static_cast<unsigned long long>(v), first);
    const uint64_t u32 = __shfl(static_cast<unsigned long long>(v32), first);
    const uint64_t u16 = __shfl(static_cast<unsigned long long>(v16), first);
    if (__any(has && (v != u || v32 != u32 || v16 != u16))) r.constant = false;
    if (lane == r.w) {
      r.d = d;
      r.m = m;
      r.v = u;
      r.v32 = u32;
      r.v16 = u16;
    }
    bool order = true;
    if (has) {
      ++e;
      order = e >= end || col[e] > c;
    }
    ++r.w;
    if (__any(!order)) {
      r.ascending = false;
      break;
    }
  }
  return r;
}

__device__ __forceinline__ uint64_t mix64(uint64_t h) {  // the finaliser of SplitMix64
  h = (h ^ (h >> 30)) * 0xbf58476d1ce4e5b9ull;
  h = (h ^ (h >> 27)) * 0x94d049bb133111ebull;
  return h ^ (h >> 31);
}

__device__ __forceinline__ bool is_set(unsigned long long *flag) {
  return __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
// Sets a flag that many may set: only the first few write.
__device__ __forceinline__ void set_once(unsigned long long *flag) {
  if (!is_set(flag)) atomicAdd(flag, 1ull);
}

// One wave per slice.  Slices whose offsets make an offset slice (sell.hpp:
// as many offsets as the longest row has entries) get their descriptors and
// their flag in sp; the slots of the others are added to *col_slots.  The
// slices that have a pattern enter its hash into the table (hkey, with the
// lowest slice of each hash in hrep) and keep its slot in pid; *odd becomes
// nonzero where one has none (or the table is full), and then the rest enter
// nothing: the layout keeps its values.
__global__ void __launch_bounds__(kBlock) k_slice_scan(int32_t count, const int32_t *__restrict__ rp,
                                                       const int32_t *__restrict__ rows,
                                                       const int32_t *__restrict__ col, const double *val,
                                                       const float *val32, const __half *val16, int64_t *sp,
                                                       int32_t *__restrict__ soff, uint64_t *__restrict__ smask,
                                                       int32_t *__restrict__ pid, unsigned long long *hkey,
                                                       unsigned int *hrep, unsigned long long *col_slots,
                                                       unsigned long long *odd) {
  const int64_t ns = (int64_t(count) + kSlice - 1) / kSlice;
  const int lane = threadIdx.x & 63;
  for (int64_t s = int64_t(blockIdx.x) * kWaves + (threadIdx.x >> 6); s < ns; s += int64_t(gridDim.x) * kWaves) {
    // whether the layout keeps its values already (the same for the whole wave)
    const bool lost = __builtin_amdgcn_readfirstlane(is_set(odd)) != 0;
    const SlicePattern r = slice_pattern(s, count, rp, rows, col, val, val32, val16, lost);
    if (r.wmax > 0) {
      if (r.ascending && r.w == r.wmax) {
        const int64_t base = sp[s];
        if (lane < r.w) {
          soff[(base >> 6) + lane] = r.d;
          smask[(base >> 6) + lane] = r.m;
        }
        if (lane == 0) sp[s] = base | kOffsetSlice;
      } else if (lane == 0) {
        atomicAdd(col_slots, static_cast<unsigned long long>(kSlice) * unsigned(r.wmax));
      }
    }
    if (!r.ascending || !r.constant) {
      if (lane == 0) set_once(odd);
      continue;
    }
    if (lost) continue;
    uint64_t h = 0;
    if (lane < r.w) {
      h = mix64(uint64_t(lane + 1) * 0x9e3779b97f4a7c15ull ^ uint32_t(r.d));
      h = mix64(h ^ r.m);
      h = mix64(h ^ r.v);
      h = mix64(h ^ (r.v32 << 16) ^ r.v16);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) h += __shfl_xor(static_cast<unsigned long long>(h), o);
    if (lane != 0) continue;
    h |= 1;  // 0 marks a free slot
    int at = -1;
    for (int t = 0; t < 256; ++t) {
      const int q = int((h >> 20) + t) & (kPatTable - 1);
      unsigned long long seen = __hip_atomic_load(hkey + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (seen == 0) seen = atomicCAS(hkey + q, 0ull, static_cast<unsigned long long>(h));
      if (seen == 0 || seen == h) {
        at = q;
        break;
      }
    }
    if (at < 0) {
      set_once(odd);
      continue;
    }
    if (__hip_atomic_load(hrep + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > uint32_t(s))
      atomicMin(hrep + at, uint32_t(s));
    pid[s] = at;
  }
}

// Writes pattern q (one wave each) from its first slice, rep[q].
__global__ void __launch_bounds__(kBlock) k_pattern_emit(int32_t patterns, int32_t count,
                                                         const int32_t *__restrict__ rp,
                                                         const int32_t *__restrict__ rows,
                                                         const int32_t *__restrict__ col, const double *val,
                                                         const float *val32, const __half *val16,
                                                         const int32_t *__restrict__ rep, PatHead *head, int32_t *off,
                                                         uint64_t *mask, double *pval, float *pval32, float *pval16) {
  const int lane = threadIdx.x & 63;
  for (int32_t q = int32_t(blockIdx.x) * kWaves + int32_t(threadIdx.x >> 6); q < patterns;
       q += int32_t(gridDim.x) * kWaves) {
    const SlicePattern r = slice_pattern(rep[q], count, rp, rows, col, val, val32, val16);
    const int32_t last = __shfl(r.d, max(r.w - 1, 0)), first = __shfl(r.d, 0);
    const int32_t full = __all(lane >= r.w || r.m == ~uint64_t(0));
    if (lane == 0) head[q] = PatHead{r.w, r.w ? first : 0, r.w ? last : 0, full};
    if (lane < kPatMax) {
      const int64_t k = int64_t(q) * kPatMax + lane;
      const bool in = lane < r.w;
      off[k] = in ? r.d : 0;
      mask[k] = in ? r.m : 0;
      pval[k] = in ? __builtin_bit_cast(double, r.v) : 0.0;
      if (pval32) pval32[k] = in ? __builtin_bit_cast(float, uint32_t(r.v32)) : 0.0f;
      if (pval16)
        pval16[k] = in ? __half2float(__builtin_bit_cast(__half, static_cast<unsigned short>(r.v16))) : 0.0f;
    }
  }
}

// Replaces each slice's hash slot by its pattern's number and compares the
// slice with the pattern bit for bit: *odd becomes nonzero where one differs (two
// patterns with one hash).
__global__ void __launch_bounds__(kBlock) k_pattern_check(int32_t count, const int32_t *__restrict__ rp,
                                                          const int32_t *__restrict__ rows,
                                                          const int32_t *__restrict__ col, const double *val,
                                                          const float *val32, const __half *val16,
                                                          const int32_t *__restrict__ number, const PatHead *head,
                                                          const int32_t *off, const uint64_t *mask,
                                                          const double *pval, const float *pval32,
                                                          const float *pval16, int32_t *pid,
                                                          unsigned long long *odd) {
  const int64_t ns = (int64_t(count) + kSlice - 1) / kSlice;
  const int lane = threadIdx.x & 63;
  for (int64_t s = int64_t(blockIdx.x) * kWaves + (threadIdx.x >> 6); s < ns; s += int64_t(gridDim.x) * kWaves) {
    const SlicePattern r = slice_pattern(s, count, rp, rows, col, val, val32, val16);
    const int32_t q = number[pid[s]];
    bool same = r.w == head[q].w;
    if (lane < r.w) {
      const int64_t k = int64_t(q) * kPatMax + lane;
      same = same && off[k] == r.d && mask[k] == r.m && __builtin_bit_cast(uint64_t, pval[k]) == r.v;
      if (pval32) same = same && __builtin_bit_cast(uint32_t, pval32[k]) == uint32_t(r.v32);
      if (pval16)
        same = same && __builtin_bit_cast(uint32_t, pval16[k]) ==
                           __builtin_bit_cast(uint32_t, __half2float(__builtin_bit_cast(
                                                            __half, static_cast<unsigned short>(r.v16))));
    }
    const bool all = __all(same);
    if (lane == 0) {
      pid[s] = q;
      if (!all) set_once(odd);
    }
  }
}

// Ascending column offsets of a 7- or 27-point stencil.
struct GridOffsets {
  int32_t d[27];
};

// Compares every slice's pattern with the entries that the stencil of np
// offsets has on an nx*ny*nz grid, neighbours outside it omitted; *bad counts
// the slices that differ.  n = nx ny nz.
__global__ void __launch_bounds__(kBlock) k_grid_match(int32_t n, int32_t nx, int32_t ny, int32_t nz, int32_t np,
                                                       GridOffsets d, const int32_t *__restrict__ pid,
                                                       const PatHead *__restrict__ head,
                                                       const int32_t *__restrict__ off,
                                                       const uint64_t *__restrict__ mask, uint32_t *bad) {
  const int64_t ns = (int64_t(n) + kSlice - 1) / kSlice;
  const int lane = threadIdx.x & 63;
  for (int64_t s = int64_t(blockIdx.x) * kWaves + (threadIdx.x >> 6); s < ns; s += int64_t(gridDim.x) * kWaves) {
    const int64_t p = s * kSlice + lane;
    const int32_t i = int32_t(min(p, int64_t(n) - 1));
    const int32_t t = i / nx, ix = i - t * nx, iz = t / ny, iy = t - iz * ny;
    const int32_t q = pid[s], w = head[q].w;
    int32_t j = 0;
    bool same = true;
    for (int dk = -1, u = 0; dk <= 1; ++dk)
      for (int dj = -1; dj <= 1; ++dj)
        for (int di = -1; di <= 1; ++di) {
          if (np == 7 && (dk != 0) + (dj != 0) + (di != 0) > 1) continue;
          const uint64_t m = __ballot(p < n && iz + dk >= 0 && iz + dk < nz && iy + dj >= 0 && iy + dj < ny &&
                                      ix + di >= 0 && ix + di < nx);
          if (m != 0) {
            const int64_t k = int64_t(q) * kPatMax + j;
            same = same && j < w && off[k] == d.d[u] && mask[k] == m;
            ++j;
          }
          ++u;
        }
    if (lane == 0 && (!same || j != w)) atomicAdd(bad, 1u);
  }
}

// Counts into *bad the rows rows[0 .. count) of an nx*ny grid whose parity of
// x + y + z is not `colour`.
__global__ void __launch_bounds__(kBlock) k_colour_parity(int32_t count, const int32_t *__restrict__ rows, int32_t nx,
                                                          int32_t ny, int32_t colour, uint32_t *bad) {
  for_rows(count, [&](int32_t p) {
    const int32_t i = rows[p], t = i / nx, ix = i - t * nx, iz = t / ny, iy = t - iz * ny;
    if (((ix + iy + iz) & 1) != colour) atomicAdd(bad, 1u);
  });
}

}  // namespace its
