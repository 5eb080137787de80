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

#include "common.hpp"
#include "launch.hpp"

namespace gp {

namespace {

constexpr int DT = 256;   // threads per workgroup

// Compile-time lags: for_lags<P>(f) calls f(Lag<0>), .., f(Lag<P - 1>).
template <int V> struct Lag { static constexpr int v = V; };
template <int P, int I = 0, typename F>
__device__ __forceinline__ void for_lags(const F& f) {
  if constexpr (I < P) {
    f(Lag<I>{});
    for_lags<P, I + 1>(f);
  }
}

constexpr int PMAX = 4;   // largest AR order

// One wavefront per global tensor entry, the scans dealt to the lanes.  A
// thread per entry walked T dependent loads in turn (85 us at K = 15, T = 200;
// 8 us with the wavefront).
__global__ __launch_bounds__(DT) void k_data_globals(int T, int K, int Ks, int P, const double* __restrict__ X,
                                                     double* __restrict__ G) {
  const int e = (blockIdx.x * DT + threadIdx.x) / 64, lane = threadIdx.x % 64;
  const int nXX = K * K, nR = K * K * P, nS = P * K * K * P;
  if (e >= nXX + nR + nS) return;
  int k, l, a = 0, b = 0;   // sum over scans of X[t - a][k] X[t - b][l]
  if (e < nXX) {
    k = e / K;
    l = e % K;
  } else if (e < nXX + nR) {
    const int i = e - nXX;
    k = i / (K * P);
    l = (i / P) % K;
    b = 1 + i % P;
  } else {
    const int i = e - nXX - nR;
    a = 1 + i / (K * K * P);
    k = (i / (K * P)) % K;
    l = (i / P) % K;
    b = 1 + i % P;
  }
  double s = 0.0;
  for (int t = P + lane; t < T; t += 64) s += X[(t - a) * Ks + k] * X[(t - b) * Ks + l];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) G[e] = s;
}

// Per voxel, the sums C(a, b)[k] = sum_{t=P}^{T-1} y[t - a] X[t - b][k], a, b = 0..P,
// that YX = C(0, 0), Bt = C(0, p + 1) + C(p + 1, 0) and Dt = C(p + 1, q + 1)
// are made of, and the products of y with itself (YY, dY, dd).
//
// With j = t - b, C(a, b) runs over j = P - b .. T - 1 - b of y[j - d] X[j][k],
// d = a - b: the scans j = P .. T - 1 - P belong to every pair of a lag d, so
// 2P + 1 running sums serve all (P + 1)^2 pairs and the at most P scans at
// either end are added per pair.  A lane holds one voxel, a window of 2P + 1
// values of y in a ring of registers (loaded once per scan, coalesced) and the
// sums of KC regressors; the design's rows (padded to whole chunks) are
// wave-uniform: one 32-byte scalar load per scan.
// Bound: the FP64 multiply-adds, (2P + 1) K T per voxel (about 30 us at
// N = 52,740, K = 15, T = 200, P = 3), and the scalar loads of the design in
// front of them.  120 us there; a workgroup per output entry, which read Y
// once per entry (208 passes), took 2,427 us.
// blockIdx.y = regressor chunk; the last one forms YY, dY and dd.
constexpr int TENSOR_KC = 4;
constexpr int TENSOR_WG = 64;

template <int P>
__device__ __forceinline__ void tensor_cross(int T, int K, int Ks, int N, int n, int k0, const double* __restrict__ X,
                                             const double* __restrict__ Y, double* __restrict__ YX,
                                             double* __restrict__ Bt, double* __restrict__ Dt) {
  constexpr int W = 2 * P + 1, KC = TENSOR_KC;
  const double* y = Y + n;
  double acc[W][KC];   // acc[d + P][c] = sum_j y[j - d] X[j][k0 + c]
#pragma unroll
  for (int d = 0; d < W; ++d)
#pragma unroll
    for (int c = 0; c < KC; ++c) acc[d][c] = 0.0;
  const int jend = T - 1 - P;
  if (jend >= P) {
    // y[m] of the window sits in ring[m % W]
    double ring[W], nxt[W];
#pragma unroll
    for (int m = 0; m < 2 * P; ++m) ring[m] = y[(size_t)m * N];
#pragma unroll
    for (int i = 0; i < W; ++i) nxt[i] = y[(size_t)min(2 * P + i, T - 1) * N];
    // scan j + i of a block: y[j + i + P] enters the ring
    auto scan = [&](int j, int i, double yn) {
      ring[(2 * P + i) % W] = yn;
      const double* xr = X + (size_t)(j + i) * Ks + k0;
      double x[KC];
#pragma unroll
      for (int c = 0; c < KC; ++c) x[c] = xr[c];
#pragma unroll
      for (int d = -P; d <= P; ++d) {
        const double yv = ring[(P + i - d + W) % W];
#pragma unroll
        for (int c = 0; c < KC; ++c) acc[d + P][c] += yv * x[c];
      }
    };
    int j = P;
#pragma unroll 1
    for (; j + W - 1 <= jend; j += W) {
      double cur[W];
#pragma unroll
      for (int i = 0; i < W; ++i) cur[i] = nxt[i];
      // the next W scans are loaded while these are used
#pragma unroll
      for (int i = 0; i < W; ++i) nxt[i] = y[(size_t)min(j + W + P + i, T - 1) * N];
#pragma unroll
      for (int i = 0; i < W; ++i) scan(j, i, cur[i]);
    }
#pragma unroll
    for (int i = 0; i < W - 1; ++i)
      if (j + i <= jend) scan(j, i, nxt[i]);
  }
  // the scans at the ends: y[0 .. 2P) and y[T - 2P .. T), where they exist
  constexpr int P2 = P > 0 ? 2 * P : 1, P1 = P > 0 ? P : 1;
  double yl[P2], yh[P2], xl[P1][KC], xh[P1][KC];
#pragma unroll
  for (int m = 0; m < 2 * P; ++m) {
    yl[m] = y[(size_t)min(m, T - 1) * N];
    yh[m] = y[(size_t)max(T - 1 - m, 0) * N];
  }
#pragma unroll
  for (int i = 0; i < P; ++i)
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      xl[i][c] = X[(size_t)min(i, T - 1) * Ks + k0 + c];
      xh[i][c] = X[(size_t)max(T - 1 - i, 0) * Ks + k0 + c];
    }
  auto sum = [&](auto A, auto B, int c) {
    constexpr int a = decltype(A)::v, b = decltype(B)::v;
    double s = acc[a - b + P][c];
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (i >= P - b && i <= T - 1 - b) s += yl[i + b - a >= 0 ? i + b - a : 0] * xl[i][c];
      if (i >= b && T - 1 - i >= P) s += yh[i - b + a >= 0 ? i - b + a : 0] * xh[i][c];
    }
    return s;
  };
#pragma unroll
  for (int c = 0; c < KC; ++c) {
    const int k = k0 + c;
    if (k >= K) break;
    YX[(size_t)k * N + n] = sum(Lag<0>{}, Lag<0>{}, c);
    for_lags<P>([&](auto Pp) {
      constexpr int p = decltype(Pp)::v;
      Bt[((size_t)p * K + k) * N + n] = sum(Lag<0>{}, Lag<p + 1>{}, c) + sum(Lag<p + 1>{}, Lag<0>{}, c);
      for_lags<P>([&](auto Q) {
        constexpr int q = decltype(Q)::v;
        Dt[(((size_t)p * K + k) * P + q) * N + n] = sum(Lag<p + 1>{}, Lag<q + 1>{}, c);
      });
    });
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
        for (int b = a; b < W; ++b) acc[a][b] += ring[(P + i - a + W) % W] * ring[(P + i - b + W) % W];
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

template <int P>
__global__ __launch_bounds__(TENSOR_WG) void k_data_tensors(int T, int K, int Ks, int N, const double* __restrict__ X,
                                                            const double* __restrict__ Y, double* __restrict__ YX,
                                                            double* __restrict__ Bt, double* __restrict__ Dt,
                                                            double* __restrict__ YY, double* __restrict__ dY,
                                                            double* __restrict__ dd) {
  const int n = blockIdx.x * TENSOR_WG + threadIdx.x;
  if (n >= N) return;
  const int k0 = blockIdx.y * TENSOR_KC;
  if (k0 < K)
    tensor_cross<P>(T, K, Ks, N, n, k0, X, Y, YX, Bt, Dt);
  else
    tensor_auto<P>(T, N, n, Y, YY, dY, dd);
}

// One thread per (voxel, row k): row k of B_n and entry k of b_n.  The draws
// enter through their first two moments at the voxel, m1 = mean_j a and
// m2 = mean_j a a' (both brackets are linear in them):
//   B_kl = lambda (XX_kl - sum_p (R_klp + R_lkp) m1_p + sum_pq S_pklq m2_pq)
//   b_k  = lambda (YX_k - sum_p Bt_pk m1_p + sum_pq Dt_pkq m2_pq).
__global__ __launch_bounds__(DT) void k_data_assemble(int K, int P, int N, int Ns, const double* __restrict__ G,
                                                      const double* __restrict__ YX, const double* __restrict__ Bt,
                                                      const double* __restrict__ Dt,
                                                      const double* __restrict__ lambda,
                                                      const double* __restrict__ A, double* __restrict__ Bout,
                                                      double* __restrict__ bw) {
  extern __shared__ double sG[];
  const int nG = K * K + K * K * P + P * K * K * P;
  for (int i = threadIdx.x; i < nG; i += DT) sG[i] = G[i];
  __syncthreads();
  const int n = blockIdx.x * DT + threadIdx.x;
  if (n >= N) return;
  const double* XX = sG;
  const double* R = sG + K * K;
  const double* S = R + K * K * P;
  const int k = blockIdx.y;
  const double lam = lambda[n];
  double m1[PMAX] = {0.0, 0.0, 0.0, 0.0}, m2[PMAX][PMAX] = {};
  for (int j = 0; j < Ns; ++j) {
    double a[PMAX];
#pragma unroll
    for (int p = 0; p < PMAX; ++p) a[p] = p < P ? A[((size_t)j * P + p) * N + n] : 0.0;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
      m1[p] += a[p];
#pragma unroll
      for (int q = 0; q < PMAX; ++q) m2[p][q] += a[p] * a[q];
    }
  }
  const double inv = Ns > 0 ? 1.0 / Ns : 0.0;
#pragma unroll
  for (int p = 0; p < PMAX; ++p) {
    m1[p] *= inv;
#pragma unroll
    for (int q = 0; q < PMAX; ++q) m2[p][q] *= inv;
  }
  // b_k first: its loads are independent of each other
  if (bw) {
    double bt[PMAX], dt[PMAX][PMAX];
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
      bt[p] = p < P ? Bt[((size_t)p * K + k) * N + n] : 0.0;
#pragma unroll
      for (int q = 0; q < PMAX; ++q) dt[p][q] = p < P && q < P ? Dt[(((size_t)p * K + k) * P + q) * N + n] : 0.0;
    }
    double acc = 0.0;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
      acc += bt[p] * m1[p];
#pragma unroll
      for (int q = 0; q < PMAX; ++q) acc -= dt[p][q] * m2[p][q];
    }
    bw[(size_t)k * N + n] = lam * (YX[(size_t)k * N + n] - acc);
  }
  double* row = Bout + ((size_t)n * K + k) * K;
  for (int l = 0; l < K; ++l) {
    double acc = 0.0;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
      if (p < P) {
        acc += (R[(k * K + l) * P + p] + R[(l * K + k) * P + p]) * m1[p];
#pragma unroll
        for (int q = 0; q < PMAX; ++q)
          if (q < P) acc -= S[((p * K + k) * K + l) * P + q] * m2[p][q];
      }
    }
    row[l] = lam * (XX[k * K + l] - acc);
  }
}

// One thread per voxel: the Monte Carlo mean over the Ns pairs (W^j, A^j) of
// the residual quadratic form, then the Gamma posterior of lambda_n:
// 1/u1t = rss/2 + 1/u1, mean = u1t * u2t (u2t = (T-P)/2 + u2).
__global__ __launch_bounds__(DT) void k_data_rss(int K, int P, int N, int Ns, const double* __restrict__ G,
                                                 const double* __restrict__ YX, const double* __restrict__ Bt,
                                                 const double* __restrict__ Dt, const double* __restrict__ YY,
                                                 const double* __restrict__ dY, const double* __restrict__ dd,
                                                 const double* __restrict__ Wall, const double* __restrict__ A,
                                                 double u1, double u2t, double* __restrict__ rss_out,
                                                 double* __restrict__ scale, double* __restrict__ mean) {
  extern __shared__ double sG[];
  const int nG = K * K + K * K * P + P * K * K * P;
  for (int i = threadIdx.x; i < nG; i += DT) sG[i] = G[i];
  __syncthreads();
  const int n = blockIdx.x * DT + threadIdx.x;
  if (n >= N) return;
  const double* XX = sG;
  const double* R = sG + K * K;
  const double* S = R + K * K * P;
  double w[KMAX], a[4];
  double tot = 0.0;
  for (int j = 0; j < Ns; ++j) {
    for (int k = 0; k < K; ++k) w[k] = Wall[((size_t)j * K + k) * N + n];
    for (int p = 0; p < P; ++p) a[p] = A[((size_t)j * P + p) * N + n];
    double v = YY[n];
    for (int k = 0; k < K; ++k) {
      double xw = 0.0;
      for (int l = 0; l < K; ++l) xw += XX[k * K + l] * w[l];
      v += w[k] * xw - 2.0 * YX[(size_t)k * N + n] * w[k];
    }
    for (int p = 0; p < P; ++p) {
      v -= 2.0 * dY[(size_t)p * N + n] * a[p];
      for (int q = 0; q < P; ++q) v += a[p] * dd[((size_t)p * P + q) * N + n] * a[q];
      for (int k = 0; k < K; ++k) {
        v += 2.0 * a[p] * Bt[((size_t)p * K + k) * N + n] * w[k];
        for (int q = 0; q < P; ++q) v -= 2.0 * a[p] * Dt[(((size_t)p * K + k) * P + q) * N + n] * w[k] * a[q];
      }
    }
    for (int k = 0; k < K; ++k) {
      for (int l = 0; l < K; ++l) {
        double ra = 0.0, asa = 0.0;
        for (int p = 0; p < P; ++p) {
          ra += R[(k * K + l) * P + p] * a[p];
          for (int q = 0; q < P; ++q) asa += a[p] * S[((p * K + k) * K + l) * P + q] * a[q];
        }
        v += w[k] * (asa - 2.0 * ra) * w[l];
      }
    }
    tot += v;
  }
  const double rss = tot / Ns;
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
// pair, so the total is W_k D_w W_k').  Fixed-order workgroup reduction.
__global__ __launch_bounds__(DT) void k_quadform_partials(OpDev op, const double* __restrict__ W,
                                                          double* __restrict__ part) {
  __shared__ double s_red[DT / 64];
  const int N = op.N;
  const int tile = blockIdx.x, rk = blockIdx.y;
  const int n = tile * DT + threadIdx.x;
  double v = 0.0;
  if (n < N) {
    const double* w = W + (size_t)rk * N;
    const double c = w[n];
    for (int d = 0; d < op.dirs; ++d) {
      const int m = op.nbr[(size_t)(2 * d + 1) * N + n];
      if (m != n) {
        const double e = c - w[m];
        v += e * e;
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x / 64] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < DT / 64; ++i) t += s_red[i];
    part[(size_t)rk * gridDim.x + tile] = t;
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

int data_design_stride(int K) { return (K + TENSOR_KC - 1) / TENSOR_KC * TENSOR_KC; }

hipError_t launch_data_tensors(hipStream_t s, int T, int K, int P, int N, const double* X, const double* Y,
                               double* G, double* YX, double* Bt, double* Dt, double* YY, double* dY, double* dd) {
  const int nG = K * K + K * K * P + P * K * K * P, Ks = data_design_stride(K);
  GP_LAUNCH(k_data_globals, dim3((nG + DT / 64 - 1) / (DT / 64)), dim3(DT), 0, s, T, K, Ks, P, X, G);
  if (hipError_t e = hipGetLastError()) return e;
  const dim3 g((N + TENSOR_WG - 1) / TENSOR_WG, (K + TENSOR_KC - 1) / TENSOR_KC + 1), b(TENSOR_WG);
  switch (P) {
#define X_P(PP) \
  case PP: GP_LAUNCH(k_data_tensors<PP>, g, b, 0, s, T, K, Ks, N, X, Y, YX, Bt, Dt, YY, dY, dd); break;
    X_P(0) X_P(1) X_P(2) X_P(3) X_P(4)
#undef X_P
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_data_rss(hipStream_t s, int K, int P, int N, int Ns, const double* G, const double* YX,
                           const double* Bt, const double* Dt, const double* YY, const double* dY, const double* dd,
                           const double* W, const double* A, double u1, double u2t, double* rss, double* scale,
                           double* mean) {
  const int nG = K * K + K * K * P + P * K * K * P;
  GP_LAUNCH(k_data_rss, dim3((N + DT - 1) / DT), dim3(DT), (size_t)nG * sizeof(double), s, K, P, N, Ns, G, YX,
                     Bt, Dt, YY, dY, dd, W, A, u1, u2t, rss, scale, mean);
  return hipGetLastError();
}

int quadform_tiles(int N) { return (N + DT - 1) / DT; }

hipError_t launch_quadform(hipStream_t s, const OpDev& op, int R, const double* W, double* part, double* out) {
  const int nt = quadform_tiles(op.N), nrk = R * op.K;
  GP_LAUNCH(k_quadform_partials, dim3(nt, nrk), dim3(DT), 0, s, op, W, part);
  if (hipError_t e = hipGetLastError()) return e;
  GP_LAUNCH(k_quadform_final, dim3(nrk), dim3(64), 0, s, nrk, nt, part, out);
  return hipGetLastError();
}

hipError_t launch_data_assemble(hipStream_t s, int K, int P, int N, int Ns, const double* G, const double* YX,
                                const double* Bt, const double* Dt, const double* lambda, const double* A,
                                double* Bout, double* bw) {
  const int nG = K * K + K * K * P + P * K * K * P;
  if (P > PMAX) return hipErrorInvalidValue;
  GP_LAUNCH(k_data_assemble, dim3((N + DT - 1) / DT, K), dim3(DT), (size_t)nG * sizeof(double), s, K,
                     P, N, Ns, G, YX, Bt, Dt, lambda, A, Bout, bw);
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
