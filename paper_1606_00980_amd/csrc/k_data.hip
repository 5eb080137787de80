// Data term of the AR(P) likelihood on the device (Appendix A.2).
//
// Time-summed tensors, conditional on the first P scans (scans t = P..T-1,
// lagged design X~[t] with row p = X[t-1-p], lagged data d_t with entry
// p = y[t-1-p]):
//   global    XX = X'X (K x K), R = X'X~ (K x K x P), S = X~X~ (P x K x K x P)
//   per voxel YX_n = Y_n'X (K), Bt_n = Y_n'X~ + d_n X (P x K), Dt_n = d_n X~ (P x K x P)
// and, for noise precisions lambda and Ns draws A^j of the AR coefficients
// (the full conditional of W for Ns = 1, its SVB expectation for Ns > 1,
// Appendix B),
//   B_n = lambda_n (XX - mean_j [R a + (R a)' - a' S a]),  a = A^j_n
//   b_n = lambda_n (YX_n - mean_j [a' Bt_n - a' Dt_n a]).
// The lambda full conditional also needs YY_n = y'y, dY_n[p] = sum_t y[t-1-p] y[t]
// and dd_n[p][q] = sum_t y[t-1-p] y[t-1-q]; its bracket is the whitened
// residual sum of squares
//   rss_n = YY - 2 YX'w + w'XXw - 2 dY'a + a'dd a + 2 a'Bt w - 2 w'(R a)w
//           - 2 a'(Dt w)a + w'(a'S a)w.
// Layouts (device, voxel fastest): Y [T][N]; YX [K][N]; Bt [P][K][N];
// Dt [P][K][P][N]; YY [N]; dY [P][N]; dd [P][P][N]; globals [XX | R | S] with
// R[k][l][p], S[p][k][l][q]; A [Ns][P][N]; W [Ns][K][N]; output blocks
// [N][K][K] (both triangles) and b_w [K][N].
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "launch.hpp"
#include "pcg.hpp"
#include "spd.hpp"

namespace gp {

namespace {

constexpr int DT = 256;   // threads per workgroup

constexpr int PMAX = 4;   // largest AR order
constexpr int GSCANS = 128;   // scans of the design staged at a time

// Every sum over scans of this file (globals and tensors) is one chain of fused
// multiply-adds over t = P .. T - 1, an entry of its own, as the definitions
// above read: the same data give the same bits in whatever kernel forms them.
// (Sums shared by the lag pairs, or added in parts, are as good or better
// against exact values, but a last bit moved in the data moves the FP32 inner
// solves to another path: draws 1e-11 and noise precisions up to 1e-9 away.)

// One lane per global tensor entry, the design staged in LDS GSCANS scans at a
// time (with the P before them).
// A thread per entry reading it from memory walked T dependent loads in turn
// (85 us at K = 15, T = 200; 12 us so).
__global__ __launch_bounds__(DT) void k_data_globals(int T, int K, int Ks, int P, const double* __restrict__ X,
                                                     double* __restrict__ G) {
  __shared__ double sX[(PMAX + GSCANS) * KMAX];
  const int e = blockIdx.x * DT + threadIdx.x;
  const int nXX = K * K, nR = K * K * P, nS = P * K * K * P;
  int k = 0, l = 0, a = 0, b = 0;   // sum over scans of X[t - a][k] X[t - b][l]
  if (e < nXX) {
    k = e / K;
    l = e % K;
  } else if (e < nXX + nR) {
    const int i = e - nXX;
    k = i / (K * P);
    l = (i / P) % K;
    b = 1 + i % P;
  } else if (e < nXX + nR + nS) {
    const int i = e - nXX - nR;
    a = 1 + i / (K * K * P);
    k = (i / (K * P)) % K;
    l = (i / P) % K;
    b = 1 + i % P;
  }
  const double *xa = sX + (P - a) * K + k, *xb = sX + (P - b) * K + l;
  double s = 0.0;
  for (int t0 = P; t0 < T; t0 += GSCANS) {
    const int nt = min(GSCANS, T - t0);
    __syncthreads();
    for (int i = threadIdx.x; i < (P + nt) * K; i += DT) sX[i] = X[(size_t)(t0 - P + i / K) * Ks + i % K];
    __syncthreads();
#pragma unroll 8
    for (int t = 0; t < nt; ++t) s = __builtin_fma(xa[t * K], xb[t * K], s);
  }
  if (e < nXX + nR + nS) G[e] = s;
}

// Coefficient table of the voxel blocks, [K(K+1)/2][TAB]: packed entry (k, l) of
// XX - [R a + (R a)'] + a'S a as a polynomial in a: the constant, the
// coefficients of a_p (PMAX slots), then those of a_p a_q, p <= q (packed by
// tab_pair(p, q, PMAX)); slots past P are zero.
constexpr int TAB = 16;
// Table of the assembly behind it, [K(K+1)/2][BTAB]: XX_kl, R_klp + R_lkp (PMAX
// slots), S_pklq (PMAX x PMAX slots); zero past P.
constexpr int BTAB = 1 + PMAX + PMAX * PMAX;

__host__ __device__ constexpr int tab_pair(int p, int q, int P) { return p * P - p * (p - 1) / 2 + q - p; }   // p <= q < P

__global__ __launch_bounds__(DT) void k_data_table(int K, int P, const double* __restrict__ G,
                                                   double* __restrict__ Tab) {
  const int i = blockIdx.x * DT + threadIdx.x;
  const int e = i / TAB, c = i % TAB;
  if (e >= K * (K + 1) / 2) return;
  int k = 0;
  while ((k + 1) * (k + 2) / 2 <= e) ++k;
  const int l = e - k * (k + 1) / 2;
  const double* R = G + K * K;
  const double* S = R + K * K * P;
  double v = 0.0;
  if (c == 0) {
    v = G[k * K + l];
  } else if (c <= PMAX) {
    const int p = c - 1;
    if (p < P) v = -(R[(k * K + l) * P + p] + R[(l * K + k) * P + p]);
  } else {
    for (int p = 0; p < P; ++p)
      for (int q = p; q < P; ++q)
        if (1 + PMAX + tab_pair(p, q, PMAX) == c) {
          v = S[((p * K + k) * K + l) * P + q];
          if (q != p) v += S[((q * K + k) * K + l) * P + p];
        }
  }
  Tab[i] = v;
  // and the entry's own parts for the assembly, in the order it adds them
  if (c == 0) {
    double* t = Tab + (size_t)K * (K + 1) / 2 * TAB + (size_t)e * BTAB;
    t[0] = G[k * K + l];
    for (int p = 0; p < PMAX; ++p) t[1 + p] = p < P ? R[(k * K + l) * P + p] + R[(l * K + k) * P + p] : 0.0;
    for (int p = 0; p < PMAX; ++p)
      for (int q = 0; q < PMAX; ++q)
        t[1 + PMAX + p * PMAX + q] = p < P && q < P ? S[((p * K + k) * K + l) * P + q] : 0.0;
  }
}

// Per voxel and regressor, YX, Bt and Dt, and per voxel YY, dY and dd, in one
// pass over Y per chunk of KC regressors.  A lane holds one voxel, the last
// P + 1 values of y in a ring of registers (loaded once per scan, coalesced) and
// the (P + 1)^2 sums of KC regressors; the design's rows (padded to whole
// chunks) are wave-uniform: one scalar load of KC doubles per scan.
// Bound: the FP64 operations, (1 + 3 P + P^2) K T per voxel, and the scalar loads
// of the design in front of them.  163 us at N = 52,740, K = 15, T = 200,
// P = 3 (K = 6: 97); a workgroup per output entry, which read Y once per entry (208
// passes), took 2,427.
// blockIdx.y = regressor chunk; the last one forms YY, dY and dd.
// KC = 4, or less where such a launch leaves SIMDs idle: a wavefront's chain over
// the scans is then shorter (KC = 1, 2, 4 at P = 3, T = 200, us: N = 900, K = 6 29, 46
// and 69; N = 5,000, K = 6 57, 51, 69; N = 10,000, K = 10 63, 60, 58; N = 20,000,
// K = 6 77, 69, 77; N = 20,000, K = 15 109, 85, 76).
constexpr int TENSOR_KC = 4;
constexpr int TENSOR_WG = 64;

template <int P, int KC>
__device__ __forceinline__ void tensor_cross(int T, int K, int Ks, int N, int n, int k0, const double* __restrict__ X,
                                             const double* __restrict__ Y, double* __restrict__ YX,
                                             double* __restrict__ Bt, double* __restrict__ Dt) {
  // scans GS at a time, their data loaded while the last GS are used: the fewer
  // the sums, the more scans it takes to cover a load from memory
  constexpr int W = P + 1, P1 = P > 0 ? P : 1, GS = W * (KC == 1 ? 16 / W : KC == 2 ? 8 / W : 1);
  const double* y = Y + n;
  double yx[KC], bt[P1][KC], dt[P1][P1][KC], yr[W], xr[W][KC], nxt[GS];
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    yx[c] = 0.0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      bt[p][c] = 0.0;
#pragma unroll
      for (int q = 0; q < P; ++q) dt[p][q][c] = 0.0;
    }
  }
  // scan m sits in slot m % W of both rings
#pragma unroll
  for (int m = 0; m < P; ++m) {
    yr[m] = y[(size_t)m * N];
#pragma unroll
    for (int c = 0; c < KC; ++c) xr[m][c] = X[(size_t)m * Ks + k0 + c];
  }
#pragma unroll
  for (int i = 0; i < GS; ++i) nxt[i] = y[(size_t)min(P + i, T - 1) * N];
  // scan t + i of a group of GS, t = P (mod W)
  auto scan = [&](int t, int i, double yn) {
#pragma clang fp contract(off)
    const int s0 = (P + i) % W;
    yr[s0] = yn;
    const double* x = X + (size_t)(t + i) * Ks + k0;
#pragma unroll
    for (int c = 0; c < KC; ++c) xr[s0][c] = x[c];
#pragma unroll
    for (int c = 0; c < KC; ++c) yx[c] = __builtin_fma(yr[s0], xr[s0][c], yx[c]);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int sp = (P + i - 1 - p) % W;
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        const double m = yr[sp] * xr[s0][c];
        bt[p][c] += __builtin_fma(yr[s0], xr[sp][c], m);
      }
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const int sq = (P + i - 1 - q) % W;
#pragma unroll
        for (int c = 0; c < KC; ++c) dt[p][q][c] = __builtin_fma(yr[sp], xr[sq][c], dt[p][q][c]);
      }
    }
  };
  int t = P;
#pragma unroll 1
  for (; t + GS <= T; t += GS) {
    double cur[GS];
#pragma unroll
    for (int i = 0; i < GS; ++i) cur[i] = nxt[i];
    // the next group's are loaded while these are used
#pragma unroll
    for (int i = 0; i < GS; ++i) nxt[i] = y[(size_t)min(t + GS + i, T - 1) * N];
#pragma unroll
    for (int i = 0; i < GS; ++i) scan(t, i, cur[i]);
  }
#pragma unroll
  for (int i = 0; i < GS - 1; ++i)
    if (t + i < T) scan(t, i, nxt[i]);
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const int k = k0 + c;
    if (k >= K) break;
    YX[(size_t)k * N + n] = yx[c];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      Bt[((size_t)p * K + k) * N + n] = bt[p][c];
#pragma unroll
      for (int q = 0; q < P; ++q) Dt[(((size_t)p * K + k) * P + q) * N + n] = dt[p][q][c];
    }
  }
}

template <int P>
__device__ __forceinline__ void tensor_auto(int T, int N, int n, const double* __restrict__ Y, double* __restrict__ YY,
                                            double* __restrict__ dY, double* __restrict__ dd) {
  constexpr int W = P + 1;
  const double* y = Y + n;
  double acc[W][W], ring[W];   // acc[a][b], a <= b: sum_t y[t - a] y[t - b]
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int b = 0; b < W; ++b) acc[a][b] = 0.0;
#pragma unroll
  for (int m = 0; m < P; ++m) ring[m] = y[(size_t)m * N];
  for (int t = P; t < T; t += W) {
    double cur[W];
#pragma unroll
    for (int i = 0; i < W; ++i) cur[i] = y[(size_t)min(t + i, T - 1) * N];
#pragma unroll
    for (int i = 0; i < W; ++i) {
      if (t + i >= T) break;
      ring[(P + i) % W] = cur[i];
#pragma unroll
      for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = a; b < W; ++b)
          acc[a][b] = __builtin_fma(ring[(P + i - a + W) % W], ring[(P + i - b + W) % W], acc[a][b]);
    }
  }
  YY[n] = acc[0][0];
#pragma unroll
  for (int p = 0; p < P; ++p) dY[(size_t)p * N + n] = acc[0][p + 1];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int q = 0; q < P; ++q) dd[((size_t)p * P + q) * N + n] = acc[(p < q ? p : q) + 1][(p < q ? q : p) + 1];
}

template <int P, int KC>
__global__ __launch_bounds__(TENSOR_WG) void k_data_tensors(int T, int K, int Ks, int N, const double* __restrict__ X,
                                                            const double* __restrict__ Y, double* __restrict__ YX,
                                                            double* __restrict__ Bt, double* __restrict__ Dt,
                                                            double* __restrict__ YY, double* __restrict__ dY,
                                                            double* __restrict__ dd) {
  const int n = blockIdx.x * TENSOR_WG + threadIdx.x;
  if (n >= N) return;
  const int k0 = blockIdx.y * KC;
  if (k0 < K)
    tensor_cross<P, KC>(T, K, Ks, N, n, k0, X, Y, YX, Bt, Dt);
  else
    tensor_auto<P>(T, N, n, Y, YY, dY, dd);
}

// One lane per voxel: the packed block B_n, stored as the operator holds it and
// factored in place (B_n = L_n L_n'), and b_n.  The draws enter through
// their first two moments at the voxel, m1 = mean_j a and m2 = mean_j a a'
// (both brackets are linear in them):
//   B_kl = lambda (XX_kl - sum_p (R_klp + R_lkp) m1_p + sum_pq S_pklq m2_pq)
//   b_k  = lambda (YX_k - sum_p Bt_pk m1_p + sum_pq Dt_pkq m2_pq).
// blockIdx.y = 0: the block; the others, if any, b_n, ASM_KC regressors each.
// From K = 14 on the block's registers leave one wavefront a SIMD, which b_n's
// loads then wait in: there it has a kernel of its own (N = 52,740; two kernels
// against one, us: K = 6 12 + 11 and 15, K = 10 27 + 13 and 32, K = 11 29 + 14 and
// 35, K = 13 38 + 16 and 43, K = 15 53 + 18 and 78, K = 16 63 + 19 and 86), unless
// the launch leaves SIMDs empty anyway (at most ASM_FEW workgroups; K = 16,
// N = 908: 35 + 5 and 37).
// Bound: the tensors read for b_n and the three packed arrays written, all
// coalesced (at K = 15, P = 3, N = 52,740: 225 MB, 45 us at 5 TB/s).
// Measured there 81 us; the rows of [N][K][K] blocks written by one kernel
// and gathered again by the packing kernel, a lane's rows K*K*8 bytes apart,
// took 112 + 57 us (K = 6: 29 + 9 to 16 us).
constexpr int ASM_WG = 64;
constexpr int ASM_KC = 3;   // regressors of b_w per lane
template <int K> constexpr bool ASM_FUSED = K <= 13;
constexpr unsigned ASM_FEW = 1024;

constexpr int ASM_NQ = PMAX * (PMAX + 1) / 2;

// m1 = mean_j a and m2 = mean_j a a' (packed by tab_pair) at voxel n
__device__ __forceinline__ void draw_moments(int P, int N, int n, int Ns, const double* __restrict__ A,
                                             double (&m1)[PMAX], double (&m2)[ASM_NQ]) {
#pragma unroll
  for (int p = 0; p < PMAX; ++p) m1[p] = 0.0;
#pragma unroll
  for (int i = 0; i < ASM_NQ; ++i) m2[i] = 0.0;
  for (int j = 0; j < Ns; ++j) {
    double a[PMAX];
#pragma unroll
    for (int p = 0; p < PMAX; ++p) a[p] = p < P ? A[((size_t)j * P + p) * N + n] : 0.0;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
      m1[p] += a[p];
#pragma unroll
      for (int q = p; q < PMAX; ++q) m2[tab_pair(p, q, PMAX)] += a[p] * a[q];
    }
  }
  const double inv = 1.0 / Ns;
#pragma unroll
  for (int p = 0; p < PMAX; ++p) m1[p] *= inv;
#pragma unroll
  for (int i = 0; i < ASM_NQ; ++i) m2[i] *= inv;
}

// Entries k0 .. k0 + ASM_KC - 1 of b_n at voxel n.
__device__ __forceinline__ void rhs_entries(int K, int P, int N, int n, int k0, double lam, const double (&m1)[PMAX],
                                            const double (&m2)[ASM_NQ], const double* __restrict__ YX,
                                            const double* __restrict__ Bt, const double* __restrict__ Dt,
                                            double* __restrict__ bw) {
#pragma unroll
  for (int c = 0; c < ASM_KC; ++c) {
    const int k = k0 + c;
    if (k >= K) break;
    double acc = 0.0;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
      if (p < P) {
        acc = __builtin_fma(Bt[((size_t)p * K + k) * N + n], m1[p], acc);
#pragma unroll
        for (int q = 0; q < PMAX; ++q)
          if (q < P)
            acc = __builtin_fma(-Dt[(((size_t)p * K + k) * P + q) * N + n],
                                m2[p <= q ? tab_pair(p, q, PMAX) : tab_pair(q, p, PMAX)], acc);
      }
    }
    bw[(size_t)k * N + n] = lam * (YX[(size_t)k * N + n] - acc);
  }
}

template <int K>
__global__ __launch_bounds__(ASM_WG) void k_data_assemble(int P, int N, int Ns, const double* __restrict__ Tab,
                                                          const double* __restrict__ YX,
                                                          const double* __restrict__ Bt,
                                                          const double* __restrict__ Dt,
                                                          const double* __restrict__ lambda,
                                                          const double* __restrict__ A, double* __restrict__ B64,
                                                          float* __restrict__ B32, double* __restrict__ L64,
                                                          int* __restrict__ bad, double* __restrict__ bw) {
  // the coefficient table in LDS (every lane reads the same entry)
  constexpr int NB = K * (K + 1) / 2;
  __shared__ double tab[NB * BTAB];
  const bool rhs = blockIdx.y > 0;
  if (!rhs)
    for (int i = threadIdx.x; i < NB * BTAB; i += ASM_WG) tab[i] = Tab[i];
  __syncthreads();
  const int n = blockIdx.x * ASM_WG + threadIdx.x;
  if (n >= N) return;
  const double lam = lambda[n];
  double m1[PMAX], m2[ASM_NQ], a[NB];
  draw_moments(P, N, n, Ns, A, m1, m2);
  if (rhs) {
    rhs_entries(K, P, N, n, ((int)blockIdx.y - 1) * ASM_KC, lam, m1, m2, YX, Bt, Dt, bw);
    return;
  }
  // B_kl and B_lk, each in the order of its own terms (S_plkq = S_qklp), averaged;
  // terms past P add zero
  auto entry = [&](int e) {
#pragma clang fp contract(off)
    const double* t = tab + e * BTAB;
    double u = 0.0, v = 0.0;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
      u = __builtin_fma(t[1 + p], m1[p], u);
      v = __builtin_fma(t[1 + p], m1[p], v);
#pragma unroll
      for (int q = 0; q < PMAX; ++q) {
        const double m = m2[p <= q ? tab_pair(p, q, PMAX) : tab_pair(q, p, PMAX)];
        u = __builtin_fma(-t[1 + PMAX + p * PMAX + q], m, u);
        v = __builtin_fma(-t[1 + PMAX + q * PMAX + p], m, v);
      }
    }
    return 0.5 * (lam * (t[0] - u) + lam * (t[0] - v));
  };
  if constexpr (K <= KREG) {
#pragma unroll
    for (int e = 0; e < NB; ++e) {
      a[e] = entry(e);
      // (or the compiler loads the table of many entries at once and spills)
      if (e % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
  } else {
#pragma unroll 1
    for (int e = 0; e < NB; ++e) a[e] = entry(e);
  }
  pack_factor<K>(N, n, a, B64, B32, L64, bad);
}

// b_n alone, ASM_KC regressors per blockIdx.y (K where the assembly leaves it out)
__global__ __launch_bounds__(ASM_WG) void k_data_rhs(int K, int P, int N, int Ns, const double* __restrict__ YX,
                                                     const double* __restrict__ Bt, const double* __restrict__ Dt,
                                                     const double* __restrict__ lambda, const double* __restrict__ A,
                                                     double* __restrict__ bw) {
  const int n = blockIdx.x * ASM_WG + threadIdx.x;
  if (n >= N) return;
  double m1[PMAX], m2[ASM_NQ];
  draw_moments(P, N, n, Ns, A, m1, m2);
  rhs_entries(K, P, N, n, (int)blockIdx.y * ASM_KC, lambda[n], m1, m2, YX, Bt, Dt, bw);
}

// The Monte Carlo mean over the Ns pairs (W^j, A^j) of the residual quadratic
// form, then the Gamma posterior of lambda_n: 1/u1t = rss/2 + 1/u1, mean =
// u1t * u2t (u2t = (T-P)/2 + u2).  A workgroup holds 64 voxels; its four
// wavefronts take every fourth regressor row k each and are added in order.
// Per draw, the quadratic part w'(XX - 2 R a + a'S a)w runs over the lower
// triangle with the wave-uniform coefficient table (scalar loads) and the
// lane's monomials of a, w in an LDS column of the lane; the parts linear in w
// come from the draws' sums of w_k {1, a_p, a_p a_q}, so each tensor entry is
// loaded once for all draws (ahead of their loop: 64 us, behind it 77).  The
// terms nearly cancel (Y'Y is 10^4 times the residual sum), so the additions'
// rounding errors are summed beside them.
// Bound: FP64 multiply-adds, K(K+1)/2 (P+1)(P+2)/2 per draw and voxel (about
// 15 us at N = 52,740, K = 15, P = 3, five draws).  Measured there 64 us; one
// thread per voxel over both triangles and all lag pairs, with w and a in
// scratch memory (run-time K), took 1,541 us (K = 6, one draw: 68 to 12 us).
constexpr int RSS_WAVES = 4;

template <int P>
__global__ __launch_bounds__(64 * RSS_WAVES) void k_data_rss(int K, int N, int Ns, const double* __restrict__ Tab,
                                                             const double* __restrict__ YX,
                                                             const double* __restrict__ Bt,
                                                             const double* __restrict__ Dt,
                                                             const double* __restrict__ YY,
                                                             const double* __restrict__ dY,
                                                             const double* __restrict__ dd,
                                                             const double* __restrict__ W,
                                                             const double* __restrict__ A, double u1, double u2t,
                                                             double* __restrict__ rss_out, double* __restrict__ scale,
                                                             double* __restrict__ mean) {
  extern __shared__ double sw[];   // [K, at least 2][64 * RSS_WAVES]: w of the lane, at the end its sum
  constexpr int P1 = P > 0 ? P : 1, NQ = P * (P + 1) / 2, Q1 = NQ > 0 ? NQ : 1, LDW = 64 * RSS_WAVES;
  const int lane = threadIdx.x % 64, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const int n = blockIdx.x * 64 + lane;
  const int nn = n < N ? n : N - 1;   // lanes past the end compute on the last voxel and store nothing
  double* w = sw + threadIdx.x;
  // tot + lo: what an addition to tot rounds away goes to lo
  double tot = 0.0, lo = 0.0;
  auto add = [&](double v) {
#pragma clang fp contract(off)
    const double t = tot + v, b = t - tot;
    lo += (tot - (t - b)) + (v - b);
    tot = t;
  };
  for (int j = 0; j < Ns; ++j) {
    double a[P1], aa[Q1];
#pragma unroll
    for (int p = 0; p < P; ++p) a[p] = A[((size_t)j * P + p) * N + nn];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int q = p; q < P; ++q) aa[tab_pair(p, q, P)] = a[p] * a[q];
#pragma unroll 4
    for (int k = 0; k < K; ++k) w[k * LDW] = W[((size_t)j * K + k) * N + nn];
    // coefficient of w_k w_l for packed entry e
    auto coef = [&](int e) {
      const double* t = Tab + (size_t)e * TAB;
      double g = 0.0;
#pragma unroll
      for (int p = 0; p < P; ++p) g += t[1 + p] * a[p];
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int q = p; q < P; ++q) g += t[1 + PMAX + tab_pair(p, q, PMAX)] * aa[tab_pair(p, q, P)];
      return t[0] + g;
    };
    for (int k = wv; k < K; k += RSS_WAVES) {
      const double wk = w[k * LDW];
      const int e0 = k * (k + 1) / 2;
      double s = 0.0;
#pragma unroll 4
      for (int l = 0; l < k; ++l) s += coef(e0 + l) * w[l * LDW];
      add(wk * (2.0 * s + coef(e0 + k) * wk));
    }
    if (wv == 0) {
      double v = 0.0;
#pragma unroll
      for (int p = 0; p < P; ++p) {
        v -= 2.0 * dY[(size_t)p * N + nn] * a[p];
#pragma unroll
        for (int q = p; q < P; ++q)
          v += (p == q ? 1.0 : 2.0) * dd[((size_t)p * P + q) * N + nn] * aa[tab_pair(p, q, P)];
      }
      add(YY[nn]);
      add(v);
    }
  }
  for (int k = wv; k < K; k += RSS_WAVES) {
    const double yx = YX[(size_t)k * N + nn];
    double bt[P1], dt[Q1];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      bt[p] = Bt[((size_t)p * K + k) * N + nn];
#pragma unroll
      for (int q = p; q < P; ++q) {
        dt[tab_pair(p, q, P)] = Dt[(((size_t)p * K + k) * P + q) * N + nn];
        if (q != p) dt[tab_pair(p, q, P)] += Dt[(((size_t)q * K + k) * P + p) * N + nn];
      }
    }
    double m0 = 0.0, m1[P1] = {0.0}, m2[Q1] = {0.0};
#pragma unroll 2
    for (int j = 0; j < Ns; ++j) {
      const double wk = W[((size_t)j * K + k) * N + nn];
      double a[P1];
#pragma unroll
      for (int p = 0; p < P; ++p) a[p] = A[((size_t)j * P + p) * N + nn];
      m0 += wk;
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const double wa = wk * a[p];
        m1[p] += wa;
#pragma unroll
        for (int q = p; q < P; ++q) m2[tab_pair(p, q, P)] += wa * a[q];
      }
    }
    double v = 0.0;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      v += bt[p] * m1[p];
#pragma unroll
      for (int q = p; q < P; ++q) v -= dt[tab_pair(p, q, P)] * m2[tab_pair(p, q, P)];
    }
    add(-2.0 * yx * m0);
    add(2.0 * v);
  }
  w[0] = tot;
  w[LDW] = lo;
  __syncthreads();
  if (wv != 0 || n >= N) return;
#pragma unroll
  for (int i = 1; i < RSS_WAVES; ++i) {
    add(w[i * 64]);
    lo += w[LDW + i * 64];
  }
  const double rss = (__builtin_isfinite(lo) ? tot + lo : tot) / Ns;   // (an infinite sum leaves no remainder)
  const double u1t = 1.0 / (0.5 * rss + 1.0 / u1);
  if (rss_out) rss_out[n] = rss;
  if (scale) scale[n] = u1t;
  if (mean) mean[n] = u1t * u2t;
}

// The AR-coefficient system (full conditional of A, Appendix A.2; its SVB
// expectation over Ns draws W^j for Ns > 1): blockIdx.y = output entry,
// packed (p, q), q <= p, of
//   J_n = lambda_n (dd_n - mean_j [D_n w + (D_n w)' - w' S w]),
// then p of
//   b_n = lambda_n (dY_n - mean_j [Bt_n w - w' R w]),          w = W^j_n,
// with (D_n w)[p][q] = sum_k Dt[p][k][q] w_k, (w'Sw)[p][q] = sum_kl w_k S[p][k][l][q] w_l,
// (Bt w)[p] = sum_k Bt[p][k] w_k, (w'Rw)[p] = sum_kl w_k R[k][l][p] w_l.  Globals in LDS.
__global__ __launch_bounds__(DT) void k_data_assemble_ar(int K, int P, int N, int Ns, const double* __restrict__ G,
                                                         const double* __restrict__ Bt, const double* __restrict__ Dt,
                                                         const double* __restrict__ dY,
                                                         const double* __restrict__ dd,
                                                         const double* __restrict__ lambda,
                                                         const double* __restrict__ W, double* __restrict__ Jout,
                                                         double* __restrict__ ba) {
  extern __shared__ double sG[];
  const int nG = K * K + K * K * P + P * K * K * P;
  for (int i = threadIdx.x; i < nG; i += DT) sG[i] = G[i];
  __syncthreads();
  const int n = blockIdx.x * DT + threadIdx.x;
  if (n >= N) return;
  const double* R = sG + K * K;
  const double* S = R + K * K * P;
  const int e = blockIdx.y, NBp = P * (P + 1) / 2;
  const double lam = lambda[n];
  double acc = 0.0;   // sum over draws of the W-dependent part
  if (e < NBp) {
    int p = 0;
    while ((p + 1) * (p + 2) / 2 <= e) ++p;
    const int q = e - p * (p + 1) / 2;
    for (int j = 0; j < Ns; ++j) {
      double dw = 0.0, wsw = 0.0;
      for (int k = 0; k < K; ++k) {
        const double wk = W[((size_t)j * K + k) * N + n];
        dw += (Dt[(((size_t)p * K + k) * P + q) * N + n] + Dt[(((size_t)q * K + k) * P + p) * N + n]) * wk;
        double sw = 0.0;
        for (int l = 0; l < K; ++l) sw += S[((p * K + k) * K + l) * P + q] * W[((size_t)j * K + l) * N + n];
        wsw += wk * sw;
      }
      acc += dw - wsw;
    }
    const double v = lam * (dd[((size_t)p * P + q) * N + n] - acc / Ns);
    Jout[((size_t)n * P + p) * P + q] = v;
    Jout[((size_t)n * P + q) * P + p] = v;
  } else {
    const int p = e - NBp;
    for (int j = 0; j < Ns; ++j) {
      double bw = 0.0, wrw = 0.0;
      for (int k = 0; k < K; ++k) {
        const double wk = W[((size_t)j * K + k) * N + n];
        bw += Bt[((size_t)p * K + k) * N + n] * wk;
        double rw = 0.0;
        for (int l = 0; l < K; ++l) rw += R[(k * K + l) * P + p] * W[((size_t)j * K + l) * N + n];
        wrw += wk * rw;
      }
      acc += bw - wrw;
    }
    if (ba) ba[(size_t)p * N + n] = lam * (dY[(size_t)p * N + n] - acc / Ns);
  }
}

// Per (sample r, regressor k, tile): sum over the tile's voxels of the squared
// differences to the in-mask +x, +y, +z neighbours (one term per adjacent
// pair, so the total is W_k D_w W_k').  A workgroup takes QK regressors of one
// sample (blockIdx.y), whose lanes share the neighbour indices; fixed-order
// workgroup reduction.  One regressor per workgroup, the indices read for each:
// 25 us for five samples at K = 15, N = 52,740 (15 so).
constexpr int QK = 4;

__global__ __launch_bounds__(DT) void k_quadform_partials(OpDev op, const double* __restrict__ W,
                                                          double* __restrict__ part) {
  __shared__ double s_red[QK * (DT / 64)];
  const int N = op.N, K = op.K, nk = (K + QK - 1) / QK;
  const int tile = blockIdx.x, r = blockIdx.y / nk, k0 = (int)blockIdx.y % nk * QK;
  const int n = tile * DT + threadIdx.x;
  const bool valid = n < N;
  const int nn = valid ? n : N - 1;
  const double* w = W + ((size_t)r * K + k0) * N;
  int m[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) m[d] = d < op.dirs ? op.nbr[(size_t)(2 * d + 1) * N + nn] : nn;
  double v[QK];
#pragma unroll
  for (int c = 0; c < QK; ++c) {
    v[c] = 0.0;
    if (k0 + c < K) {
      const double* wk = w + (size_t)c * N;
      const double x = wk[nn];
#pragma unroll
      for (int d = 0; d < 3; ++d) {   // an absent neighbour is the voxel itself
        const double e = x - wk[m[d]];
        v[c] += m[d] != nn ? e * e : 0.0;
      }
    }
    if (!valid) v[c] = 0.0;
  }
  wave_deposit<QK>(s_red, 0, v);
  __syncthreads();
  if (threadIdx.x < QK && k0 + (int)threadIdx.x < K) {
    double t = 0.0;
    for (int i = 0; i < DT / 64; ++i) t += s_red[threadIdx.x * (DT / 64) + i];
    part[((size_t)r * K + k0 + threadIdx.x) * gridDim.x + tile] = t;
  }
}

// One wavefront per (r, k): the tile partials in a fixed order.
__global__ __launch_bounds__(64) void k_quadform_final(int nrk, int ntiles, const double* __restrict__ part,
                                                       double* __restrict__ out) {
  const int rk = blockIdx.x;
  if (rk >= nrk) return;
  double v = 0.0;
  for (int t = threadIdx.x; t < ntiles; t += 64) v += part[(size_t)rk * ntiles + t];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if (threadIdx.x == 0) out[rk] = v;
}

}  // namespace

size_t data_table_at(int K, int P) {
  const size_t n = (size_t)K * K + (size_t)K * K * P + (size_t)P * K * K * P;
  return (n + TAB - 1) / TAB * TAB;
}

size_t data_globals_size(int K, int P) { return data_table_at(K, P) + (size_t)(K * (K + 1) / 2) * (TAB + BTAB); }

int data_design_stride(int K) { return (K + TENSOR_KC - 1) / TENSOR_KC * TENSOR_KC; }

hipError_t launch_data_tensors(hipStream_t s, int T, int K, int P, int N, const double* X, const double* Y,
                               double* G, double* YX, double* Bt, double* Dt, double* YY, double* dY, double* dd) {
  const int nG = K * K + K * K * P + P * K * K * P, Ks = data_design_stride(K);
  GP_LAUNCH(k_data_globals, dim3((nG + DT - 1) / DT), dim3(DT), 0, s, T, K, Ks, P, X, G);
  if (hipError_t e = hipGetLastError()) return e;
  const int nT = K * (K + 1) / 2 * TAB;
  GP_LAUNCH(k_data_table, dim3((nT + DT - 1) / DT), dim3(DT), 0, s, K, P, G, G + data_table_at(K, P));
  if (hipError_t e = hipGetLastError()) return e;
  const unsigned nb = (N + TENSOR_WG - 1) / TENSOR_WG;
  const int kc = nb * K <= 400 ? 1 : nb * ((K + TENSOR_KC - 1) / TENSOR_KC) <= 800 ? 2 : TENSOR_KC;
  const dim3 g(nb, (K + kc - 1) / kc + 1), b(TENSOR_WG);
  switch (P * 8 + kc) {
#define X_PC(PP, CC)                                                                                     \
  case PP * 8 + CC:                                                                                      \
    GP_LAUNCH((k_data_tensors<PP, CC>), g, b, 0, s, T, K, Ks, N, X, Y, YX, Bt, Dt, YY, dY, dd);           \
    break;
#define X_P(PP) X_PC(PP, 1) X_PC(PP, 2) X_PC(PP, TENSOR_KC)
    X_P(0) X_P(1) X_P(2) X_P(3) X_P(4)
#undef X_P
#undef X_PC
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_data_rss(hipStream_t s, int K, int P, int N, int Ns, const double* G, const double* YX,
                           const double* Bt, const double* Dt, const double* YY, const double* dY, const double* dd,
                           const double* W, const double* A, double u1, double u2t, double* rss, double* scale,
                           double* mean) {
  const double* tab = G + data_table_at(K, P);
  const dim3 g((N + 63) / 64), b(64 * RSS_WAVES);
  const size_t lds = (size_t)std::max(K, 2) * 64 * RSS_WAVES * sizeof(double);
  switch (P) {
#define X_P(PP)                                                                                                  \
  case PP:                                                                                                       \
    GP_LAUNCH(k_data_rss<PP>, g, b, lds, s, K, N, Ns, tab, YX, Bt, Dt, YY, dY, dd, W, A, u1, u2t, rss, scale,    \
              mean);                                                                                             \
    break;
    X_P(0) X_P(1) X_P(2) X_P(3) X_P(4)
#undef X_P
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int quadform_tiles(int N) { return (N + DT - 1) / DT; }

hipError_t launch_quadform(hipStream_t s, const OpDev& op, int R, const double* W, double* part, double* out) {
  const int nt = quadform_tiles(op.N), nrk = R * op.K;
  GP_LAUNCH(k_quadform_partials, dim3(nt, R * ((op.K + QK - 1) / QK)), dim3(DT), 0, s, op, W, part);
  if (hipError_t e = hipGetLastError()) return e;
  GP_LAUNCH(k_quadform_final, dim3(nrk), dim3(64), 0, s, nrk, nt, part, out);
  return hipGetLastError();
}

hipError_t launch_data_assemble(hipStream_t s, int K, int P, int N, int Ns, const double* G, const double* YX,
                                const double* Bt, const double* Dt, const double* lambda, const double* A,
                                double* B64, float* B32, double* L64, int* bad, double* bw) {
  if (P > PMAX) return hipErrorInvalidValue;
  const double* tab = G + data_table_at(K, P) + (size_t)(K * (K + 1) / 2) * TAB;
  const dim3 g((N + ASM_WG - 1) / ASM_WG), b(ASM_WG);
  const unsigned nrhs = bw ? (K + ASM_KC - 1) / ASM_KC : 0;
  bool fused;
  switch (K) {
#define X(KK)                                                                                                      \
  case KK:                                                                                                         \
    fused = ASM_FUSED<KK> || g.x * (1 + nrhs) <= ASM_FEW;                                                          \
    if (!fused && bw) GP_LAUNCH(k_data_rhs, dim3(g.x, nrhs), b, 0, s, K, P, N, Ns, YX, Bt, Dt, lambda, A, bw);     \
    GP_LAUNCH(k_data_assemble<KK>, dim3(g.x, fused ? 1 + nrhs : 1), b, 0, s, P, N, Ns, tab, YX, Bt, Dt,             \
              lambda, A, B64, B32, L64, bad, bw);                                                                  \
    break;
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) X(20)
    X(21) X(22) X(23) X(24)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_data_assemble_ar(hipStream_t s, int K, int P, int N, int Ns, const double* G, const double* Bt,
                                   const double* Dt, const double* dY, const double* dd, const double* lambda,
                                   const double* W, double* Jout, double* ba) {
  const int nG = K * K + K * K * P + P * K * K * P;
  const int entries = P * (P + 1) / 2 + P;
  GP_LAUNCH(k_data_assemble_ar, dim3((N + DT - 1) / DT, entries), dim3(DT), (size_t)nG * sizeof(double), s,
                     K, P, N, Ns, G, Bt, Dt, dY, dd, lambda, W, Jout, ba);
  return hipGetLastError();
}

}  // namespace gp
