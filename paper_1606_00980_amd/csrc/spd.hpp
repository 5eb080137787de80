// Inverse of a small symmetric positive definite block held packed (lower
// triangle, row-major) in registers: Cholesky A = L L', then
// A^{-1} = L^{-T} L^{-1}, every step in place.
#pragma once
#include "common.hpp"

namespace gp {

// v / l from inv = 1 / l correctly rounded: the product's exact remainder times
// inv corrects it to the rounding of the division itself (Markstein 1990), in
// five instructions instead of a dozen.  v * inv alone is up to an ulp off:
// the factors were 10 to 17 % further from 64-bit exact ones, their inverses
// 8 to 22 %.  An overflowed product or an infinite l (inv = 0) has no finite
// remainder and gives v * inv, which is v / l there.
__device__ __forceinline__ double div_by(double v, double l, double inv) {
  const double q = v * inv, rem = __builtin_fma(-q, l, v);
  return __builtin_isfinite(rem) ? __builtin_fma(rem, inv, q) : q;
}

// Replaces the packed SPD block a by its inverse and returns whether every
// pivot was positive and finite.  A failed pivot is replaced by one so that
// the arithmetic stays finite.  A row or column divides by one pivot, so that
// a block costs 2 K divisions (separate arrays for L, its inverse and the
// result and a division per entry: the red set-up took 34 us at K = 15,
// N = 52,740; 29 so).
template <int K>
__device__ inline bool spd_inverse(double (&a)[K * (K + 1) / 2]) {
  bool ok = true;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    double dj = a[pk(j, j)];
#pragma unroll
    for (int l = 0; l < j; ++l) dj -= a[pk(j, l)] * a[pk(j, l)];
    ok = ok && (dj > 0.0) && (dj == dj);
    const double ljj = sqrt(dj > 0.0 ? dj : 1.0), inv = 1.0 / ljj;
    a[pk(j, j)] = ljj;
#pragma unroll
    for (int i = j + 1; i < K; ++i) {
      double v = a[pk(i, j)];
#pragma unroll
      for (int l = 0; l < j; ++l) v -= a[pk(i, l)] * a[pk(j, l)];
      a[pk(i, j)] = div_by(v, ljj, inv);
    }
  }
  // L^{-1}, row by row (row i from row i of L and the rows of L^{-1} above it)
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const double lii = a[pk(i, i)], inv = 1.0 / lii;
#pragma unroll
    for (int j = 0; j < i; ++j) {
      double v = 0.0;
#pragma unroll
      for (int l = j; l < i; ++l) v -= a[pk(i, l)] * a[pk(l, j)];
      a[pk(i, j)] = div_by(v, lii, inv);
    }
    a[pk(i, i)] = inv;
  }
  // L^{-T} L^{-1}, row i from rows i and below
#pragma unroll
  for (int i = 0; i < K; ++i) {
#pragma unroll
    for (int j = 0; j <= i; ++j) {
      double v = 0.0;
#pragma unroll
      for (int l = i; l < K; ++l) v += a[pk(l, i)] * a[pk(l, j)];
      a[pk(i, j)] = v;
    }
  }
  return ok;
}

// Blocks above this K are factored by the rolled routines below (runtime K,
// arrays in scratch memory): the set-up kernels run once per change of the
// blocks or alpha, and fully unrolled O(K^3) code for larger K would take
// minutes to compile.
constexpr int KREG = 16;

// In-place lower Cholesky factor of the packed SPD block a (runtime K); a
// failed pivot is replaced by one.  Returns whether every pivot was positive.
__device__ inline bool cholesky_dyn(int K, double* a) {
  bool ok = true;
#pragma unroll 1
  for (int j = 0; j < K; ++j) {
    double dj = a[pk(j, j)];
#pragma unroll 1
    for (int l = 0; l < j; ++l) dj -= a[pk(j, l)] * a[pk(j, l)];
    ok = ok && (dj > 0.0) && (dj == dj);
    const double ljj = sqrt(dj > 0.0 ? dj : 1.0);
    a[pk(j, j)] = ljj;
#pragma unroll 1
    for (int i = j + 1; i < K; ++i) {
      double v = a[pk(i, j)];
#pragma unroll 1
      for (int l = 0; l < j; ++l) v -= a[pk(i, l)] * a[pk(j, l)];
      a[pk(i, j)] = v / ljj;
    }
  }
  return ok;
}

// Replaces the packed SPD block a (runtime K) by its inverse; inv is scratch.
__device__ inline bool spd_inverse_dyn(int K, double* a, double* inv) {
  const bool ok = cholesky_dyn(K, a);
  // L^{-1} into inv, column by column by forward substitution
#pragma unroll 1
  for (int c = 0; c < K; ++c) {
#pragma unroll 1
    for (int i = c; i < K; ++i) {
      double v = (i == c) ? 1.0 : 0.0;
#pragma unroll 1
      for (int l = c; l < i; ++l) v -= a[pk(i, l)] * inv[pk(l, c)];
      inv[pk(i, c)] = v / a[pk(i, i)];
    }
  }
  // A^{-1} = L^{-T} L^{-1} back into a
#pragma unroll 1
  for (int i = 0; i < K; ++i) {
#pragma unroll 1
    for (int j = 0; j <= i; ++j) {
      double v = 0.0;
#pragma unroll 1
      for (int l = i; l < K; ++l) v += inv[pk(l, i)] * inv[pk(l, j)];
      a[pk(i, j)] = v;
    }
  }
  return ok;
}

// Replaces a packed SPD block by its inverse: unrolled up to K = KREG, through
// the rolled routine above beyond.
template <int K>
__device__ inline bool spd_inverse_any(double (&a)[K * (K + 1) / 2]) {
  if constexpr (K <= KREG) {
    return spd_inverse<K>(a);
  } else {
    double inv[K * (K + 1) / 2];
    return spd_inverse_dyn(K, a, inv);
  }
}

// Stores the packed block a of voxel n in FP64 and FP32 (entry i at i * N + n),
// factors it in place and stores the factor; a block that is not positive
// definite lowers *bad to n.
template <int K>
__device__ inline void pack_factor(int N, int n, double (&a)[K * (K + 1) / 2], double* __restrict__ B64,
                                   float* __restrict__ B32, double* __restrict__ L64, int* __restrict__ bad) {
  constexpr int NB = K * (K + 1) / 2;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    B64[(size_t)i * N + n] = a[i];
    B32[(size_t)i * N + n] = (float)a[i];
  }
  bool ok = true;
  if constexpr (K <= KREG) {
#pragma unroll
    for (int j = 0; j < K; ++j) {
      double dj = a[pk(j, j)];
#pragma unroll
      for (int l = 0; l < j; ++l) dj -= a[pk(j, l)] * a[pk(j, l)];
      ok = ok && (dj > 0.0) && (dj == dj);
      const double ljj = sqrt(dj > 0.0 ? dj : 1.0), inv = 1.0 / ljj;
      a[pk(j, j)] = ljj;
#pragma unroll
      for (int i = j + 1; i < K; ++i) {
        double v = a[pk(i, j)];
#pragma unroll
        for (int l = 0; l < j; ++l) v -= a[pk(i, l)] * a[pk(j, l)];
        a[pk(i, j)] = div_by(v, ljj, inv);
      }
    }
  } else {
    ok = cholesky_dyn(K, a);
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) L64[(size_t)i * N + n] = a[i];
  if (!ok) atomicMin(bad, n);
}

}  // namespace gp
