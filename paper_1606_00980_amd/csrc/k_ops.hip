// Operator construction and the non-iterative operations:
//   * mask -> compact voxel numbering and 6-neighbour table (Section 2, the
//     unweighted graph Laplacian over in-mask neighbours; Section 3.1, one
//     incidence row per adjacent pair)
//   * packing and Cholesky factorisation of the data blocks B_n (the L_data of
//     Algorithm 2, step 1)
//   * Jacobi / block-Jacobi preconditioner set-up from the voxel blocks of Q
//   * FP64 operator application y = Q x (Section 3)
//   * perturbed right-hand sides of Algorithm 2, step 4
//   * Hutchinson reductions for tr(Q^{-1}), tr([Q^{-1}]_kk), tr(D_w [Q^{-1}]_kk)
//     (the trace inside E[W_k D_w W_k'], Section 3.3)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "launch.hpp"
#include "pcg.hpp"
#include "spd.hpp"

namespace gp {

// ------------------------------------------------------------------ grid
constexpr int SCAN_BLOCK = 256;
constexpr int CELLS_PER_THREAD = 4;
constexpr int CELLS_PER_BLOCK = SCAN_BLOCK * CELLS_PER_THREAD;

__device__ inline int block_exclusive_scan(int v, int* s_tmp /*[SCAN_BLOCK]*/, int* total) {
  const int t = threadIdx.x;
  s_tmp[t] = v;
  __syncthreads();
  for (int off = 1; off < SCAN_BLOCK; off <<= 1) {
    const int add = t >= off ? s_tmp[t - off] : 0;
    __syncthreads();
    s_tmp[t] += add;
    __syncthreads();
  }
  const int incl = s_tmp[t];
  if (total) *total = s_tmp[SCAN_BLOCK - 1];
  __syncthreads();
  return incl - v;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_mask_count(const uint8_t* __restrict__ mask,
                                                           long ncell, int* __restrict__ counts) {
  __shared__ int s_tmp[SCAN_BLOCK];
  const long base = (long)blockIdx.x * CELLS_PER_BLOCK + (long)threadIdx.x * CELLS_PER_THREAD;
  int c = 0;
  for (int i = 0; i < CELLS_PER_THREAD; ++i) c += (base + i < ncell && mask[base + i] != 0) ? 1 : 0;
  int total;
  block_exclusive_scan(c, s_tmp, &total);
  if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// Exclusive scan of nb block counts in one workgroup; offsets[nb] = total.
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_counts(const int* __restrict__ counts, int nb,
                                                            int* __restrict__ offsets) {
  __shared__ int s_tmp[SCAN_BLOCK];
  const int per = (nb + SCAN_BLOCK - 1) / SCAN_BLOCK;
  const int lo = threadIdx.x * per;
  int sum = 0;
  for (int i = lo; i < lo + per && i < nb; ++i) sum += counts[i];
  int total;
  int run = block_exclusive_scan(sum, s_tmp, &total);
  for (int i = lo; i < lo + per && i < nb; ++i) {
    offsets[i] = run;
    run += counts[i];
  }
  if (threadIdx.x == 0) offsets[nb] = total;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_mask_index(const uint8_t* __restrict__ mask, long ncell,
                                                           const int* __restrict__ offsets,
                                                           int* __restrict__ gridmap,
                                                           int* __restrict__ lin) {
  __shared__ int s_tmp[SCAN_BLOCK];
  const long base = (long)blockIdx.x * CELLS_PER_BLOCK + (long)threadIdx.x * CELLS_PER_THREAD;
  int c = 0;
  for (int i = 0; i < CELLS_PER_THREAD; ++i) c += (base + i < ncell && mask[base + i] != 0) ? 1 : 0;
  int n = offsets[blockIdx.x] + block_exclusive_scan(c, s_tmp, nullptr);
  for (int i = 0; i < CELLS_PER_THREAD; ++i) {
    const long l = base + i;
    if (l >= ncell) break;
    if (mask[l] != 0) {
      gridmap[l] = n;
      lin[n] = (int)l;
      ++n;
    } else {
      gridmap[l] = -1;
    }
  }
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_neighbours(int N, const int* __restrict__ lin,
                                                           const int* __restrict__ gridmap, int nx,
                                                           int ny, int nz, int conn,
                                                           int* __restrict__ nbr,
                                                           unsigned long long* __restrict__ edges) {
  __shared__ int s_tmp[SCAN_BLOCK];
  const int n = blockIdx.x * SCAN_BLOCK + threadIdx.x;
  int e = 0;
  if (n < N) {
    const long l = lin[n];
    const int x = (int)(l % nx);
    const int y = (int)((l / nx) % ny);
    const int z = (int)(l / ((long)nx * ny));
    const long sx = 1, sy = nx, sz = (long)nx * ny;
    int m[6];
    m[0] = x > 0 ? gridmap[l - sx] : -1;
    m[1] = x < nx - 1 ? gridmap[l + sx] : -1;
    m[2] = y > 0 ? gridmap[l - sy] : -1;
    m[3] = y < ny - 1 ? gridmap[l + sy] : -1;
    m[4] = (conn == 6 && z > 0) ? gridmap[l - sz] : -1;
    m[5] = (conn == 6 && z < nz - 1) ? gridmap[l + sz] : -1;
    for (int d = 0; d < 6; ++d) nbr[(size_t)d * N + n] = m[d] >= 0 ? m[d] : n;
    e = (m[1] >= 0) + (m[3] >= 0) + (m[5] >= 0);
  }
  int total;
  block_exclusive_scan(e, s_tmp, &total);
  if (threadIdx.x == 0 && total > 0) atomicAdd(edges, (unsigned long long)total);
}

hipError_t launch_grid_build(hipStream_t s, const uint8_t* mask, long ncell, int* counts, int* offsets,
                             int nblocks) {
  GP_LAUNCH(k_mask_count, dim3(nblocks), dim3(SCAN_BLOCK), 0, s, mask, ncell, counts);
  GP_LAUNCH(k_scan_counts, dim3(1), dim3(SCAN_BLOCK), 0, s, counts, nblocks, offsets);
  return hipGetLastError();
}

hipError_t launch_grid_index(hipStream_t s, const uint8_t* mask, long ncell, const int* offsets,
                             int nblocks, int* gridmap, int* lin, int N, int nx, int ny, int nz, int conn,
                             int* nbr, unsigned long long* edges) {
  GP_LAUNCH(k_mask_index, dim3(nblocks), dim3(SCAN_BLOCK), 0, s, mask, ncell, offsets, gridmap,
                     lin);
  GP_LAUNCH(k_neighbours, dim3((N + SCAN_BLOCK - 1) / SCAN_BLOCK), dim3(SCAN_BLOCK), 0, s, N, lin,
                     gridmap, nx, ny, nz, conn, nbr, edges);
  return hipGetLastError();
}

int grid_cells_per_block() { return CELLS_PER_BLOCK; }

// ---------------------------------------------------------------- blocks
// Symmetrise B_n, store it packed in FP64 and FP32, and factor B_n = L L'.
template <int K>
__global__ __launch_bounds__(TILE) void k_pack_blocks(int N, const double* __restrict__ B,
                                                      double* __restrict__ B64, float* __restrict__ B32,
                                                      double* __restrict__ L64, int* __restrict__ bad) {
  constexpr int NB = Tri<K>::NB;
  const int n = blockIdx.x * TILE + threadIdx.x;
  if (n >= N) return;
  const double* Bn = B + (size_t)n * K * K;
  double a[NB];
#pragma unroll
  for (int k = 0; k < K; ++k) {
#pragma unroll
    for (int j = 0; j <= k; ++j) a[pk(k, j)] = 0.5 * (Bn[k * K + j] + Bn[j * K + k]);
  }
  pack_factor<K>(N, n, a, B64, B32, L64, bad);
}

// Preconditioner from the voxel block of Q, M_n = B_n + diag_k(alpha_k deg_n):
// the inverse diagonal (Jacobi) or the inverse of the whole block (block Jacobi).
template <int K>
__global__ __launch_bounds__(TILE) void k_precond(OpDev op, int pc, double* __restrict__ P64,
                                                  float* __restrict__ P32, int* __restrict__ bad) {
  constexpr int NB = Tri<K>::NB;
  const int n = blockIdx.x * TILE + threadIdx.x;
  const int N = op.N;
  if (n >= N) return;
  int deg = 0;
  for (int d = 0; d < 6; ++d) deg += op.nbr[(size_t)d * N + n] != n;
  double a[NB];
  load_soa(op.B64, N, n, a);
#pragma unroll
  for (int k = 0; k < K; ++k) a[pk(k, k)] += op.alpha64[k] * (double)deg;
  if (pc == PC_JACOBI) {
    bool ok = true;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double dk = a[pk(k, k)];
      ok = ok && dk > 0.0;
      const double inv = 1.0 / dk;
      P64[(size_t)k * N + n] = inv;
      P32[(size_t)k * N + n] = (float)inv;
    }
    if (!ok) atomicMin(bad, n);
    return;
  }
  // Cholesky M = L L', then M^{-1} = L^{-T} L^{-1}.
  const bool ok = spd_inverse_any<K>(a);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    P64[(size_t)i * N + n] = a[i];
    P32[(size_t)i * N + n] = (float)a[i];
  }
  if (!ok) atomicMin(bad, n);
}

// ----------------------------------------------------------------- apply
// RC = 0: one right-hand side per workgroup on a two-dimensional grid.
// RC = 1: the same, the right-hand sides of a tile side by side and the items
// dealt to the XCDs in contiguous ranges, so that the readers of a block and of
// a vector's neighbours share an L2.  RC = 2: rc right-hand sides per workgroup,
// their voxels' blocks held; items by blocks of tb tiles, every chunk of
// right-hand sides over a block's tiles before the next block.
// The vectors are read through buffer descriptors, the neighbours of all
// regressors (four with RC = 2) together: with a 64-bit address per gather, or
// left to the compiler's order, few loads were in flight at a time (K = 5: one).
// Beyond K = KREG, and in launches that leave most wavefronts empty, the
// compiler's order is the better one.
// Measured (us; one right-hand side per workgroup with 64-bit addresses and no
// mapping of items, then so):
//   N = 52,740, K = 6, R = 8    25.1   17.9  (2.7 TB/s of its 49 MB)
//   N = 85,936, K = 5, R = 8    22.0   19.4    K = 10, R = 8   77    41
//               K = 15, R = 8    200     67    K = 15, R = 1   35    23
//               K = 20, R = 4    194     74    K = 24, R = 4  546   120
//   N = 12,704, K = 9, R = 2     8.2    6.2    N = 2,620, K = 5, R = 2   3.8   3.8
template <int K, int RC>
__global__ __launch_bounds__(TILE) void k_apply(OpDev op, const double* __restrict__ x, double* __restrict__ y, int R,
                                                int rc, int tb) {
  constexpr int NB = Tri<K>::NB;
  constexpr bool MANY = RC == 2, TOGETHER = RC > 0 && K <= KREG;
  constexpr int G = !TOGETHER ? 1 : MANY && K > 4 ? 4 : K;
  const int N = op.N;
  int tile = blockIdx.x, r0 = blockIdx.y;
  if constexpr (MANY) {
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    const int per = tb * ((R + rc - 1) / rc), blk = item / per, rem = item - blk * per;
    const int len = min(tb, op.ntiles - blk * tb);
    r0 = rem / len * rc;
    tile = blk * tb + rem % len;
  } else if constexpr (RC == 1) {
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    tile = item / R;
    r0 = item - tile * R;
  }
  const int r1 = MANY ? min(R, r0 + rc) : r0 + 1;
  const int n = tile * TILE + threadIdx.x;
  if (n >= N) return;
  const unsigned o = (unsigned)n * 8u;
  unsigned nb[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) nb[d] = (unsigned)op.nbr[(size_t)d * N + n] * 8u;
  const Slab<double> Bs(op.B64, NB, N);
  double B[NB];
  auto load_block = [&]() {
#pragma unroll
    for (int e = 0; e < NB; ++e) B[e] = Bs.ld(e, o);
  };
  if constexpr (MANY) load_block();
#pragma unroll 1
  for (int r = r0; r < r1; ++r) {
    const Slab<double> xs(x + (size_t)r * K * N, K, N), ys(y + (size_t)r * K * N, K, N);
    double xo[K], s6[K];
#pragma unroll
    for (int k = 0; k < K; ++k) xo[k] = xs.ld(k, o);
    if constexpr (!MANY) load_block();
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += G) {
      double t[G][6];
#pragma unroll
      for (int c = 0; c < G; ++c)
#pragma unroll
        for (int d = 0; d < 6; ++d)
          if (k0 + c < K) t[c][d] = xs.ld(k0 + c, nb[d]);
      if constexpr (TOGETHER) __builtin_amdgcn_sched_barrier(0);   // none waits for another
#pragma unroll
      for (int c = 0; c < G; ++c)
        if (k0 + c < K) {
          s6[k0 + c] = 0.0;
#pragma unroll
          for (int d = 0; d < 6; ++d) s6[k0 + c] += xo[k0 + c] - t[c][d];
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double v = op.alpha64[k] * s6[k];
#pragma unroll
      for (int j = 0; j < K; ++j) v += B[pk(k, j)] * xo[j];
      ys.st(k, o, v);
    }
  }
}

// -------------------------------------------------------------- perturb
// b_r = b_w + (blkdiag_k sqrt(alpha_k) G_w)' z1_r + H' L_data H z2_r
// Row (n, n+e_d) of G_w has +1 at n and -1 at n+e_d; its z1 entry sits in slot
// (k, d, n).  So (G_w' z1)_n = sum_d [z1(d, n) if n+e_d in mask]
//                              - [z1(d, n-e_d) if n-e_d in mask].
template <int K>
__global__ __launch_bounds__(TILE) void k_perturb(OpDev op, const double* __restrict__ bw,
                                                  const double* __restrict__ z1,
                                                  const double* __restrict__ z2,
                                                  double* __restrict__ b, int R, int tb) {
  const int N = op.N, dirs = op.dirs;
  // items (right-hand side, tile) by blocks of tb tiles: every right-hand
  // side sweeps a block's tiles before the next one starts, and the items go
  // to the XCDs in contiguous ranges, so that the block's Cholesky factors and
  // neighbour table stay in the XCD's L2 across the right-hand sides and the
  // lower neighbours' z1 values (a plane back) were just read for the same
  // right-hand side
  const int W = gridDim.x;
  const int item = xcd_remap(blockIdx.x, W);
  const int per = tb * R;
  const int blk = item / per, rem = item - blk * per;
  const int len = min(tb, op.ntiles - blk * tb);
  const int r = rem / len, tile = blk * tb + rem % len;
  const int n = tile * TILE + threadIdx.x;
  if (n >= N) return;
  int nb[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) nb[d] = op.nbr[(size_t)d * N + n];
  double zz[K];
#pragma unroll
  for (int j = 0; j < K; ++j) zz[j] = z2[((size_t)r * K + j) * N + n];
  // KG regressors at a time, all of them up to K = 9: their factor rows and z1
  // entries are loaded together before any use (a missing neighbour is the
  // voxel itself, so each address is valid; its term is dropped by a select).
  // From K = 10 on the loads of all take the registers of most wavefronts of a
  // SIMD (K = 15, five right-hand sides: 100 us, by groups 72; K = 10 127 and
  // 113); at K = 9 the one group is faster (86 against 91).
  constexpr int NG = K <= 9 ? 1 : (K + 5) / 6, KG = (K + NG - 1) / NG;
  double Lh[NG == 1 ? Tri<K>::NB : 1];
  if constexpr (NG == 1) load_soa(op.L64, N, n, Lh);
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (g > 0) __builtin_amdgcn_sched_barrier(0);
    const int k0 = g * KG;
    double hv[KG][3], lv[KG][3], L[NG > 1 ? KG : 1][K], bwv[KG];
#pragma unroll
    for (int c = 0; c < KG; ++c) {
      const int k = k0 + c;
      if (k < K) {
        const double* zk = z1 + ((size_t)r * K + k) * dirs * N;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int dd = d < dirs ? d : 0;
          hv[c][d] = zk[(size_t)dd * N + n];
          lv[c][d] = zk[(size_t)dd * N + nb[2 * dd]];
        }
        if constexpr (NG > 1) {
#pragma unroll
          for (int j = 0; j <= k; ++j) L[c][j] = op.L64[(size_t)pk(k, j) * N + n];
          bwv[c] = bw[(size_t)k * N + n];
        }
      }
    }
#pragma unroll
    for (int c = 0; c < KG; ++c) {
      const int k = k0 + c;
      if (k < K) {
        double pr = 0.0, dt = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          pr += d < dirs && nb[2 * d + 1] != n ? hv[c][d] : 0.0;
          pr -= d < dirs && nb[2 * d] != n ? lv[c][d] : 0.0;
        }
#pragma unroll
        for (int j = 0; j <= k; ++j) dt += (NG == 1 ? Lh[NG == 1 ? pk(k, j) : 0] : L[NG > 1 ? c : 0][j]) * zz[j];
        b[((size_t)r * K + k) * N + n] = (NG > 1 ? bwv[c] : bw[(size_t)k * N + n]) + sqrt(op.alpha64[k]) * pr + dt;
      }
    }
  }
}

// b[r][i] += bw[i] for R right-hand sides of length kn.
__global__ void k_add_broadcast(long total, long kn, const double* __restrict__ bw, double* __restrict__ b) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) b[i] += bw[i % kn];
}

__global__ void k_probe_rhs(long total, const int8_t* __restrict__ v, double* __restrict__ b) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) b[i] = (double)v[i];
}

// ----------------------------------------------------------------- trace
// Per (probe i, regressor k, tile): sum_n v u and sum_n (D_w v)_n u, where
// (D_w v)_n = sum_d (v_n - v_nb_d(n)).  Partials laid out [2][m][K][ntiles].
template <int K>
__global__ __launch_bounds__(TILE) void k_trace_partials(OpDev op, const int8_t* __restrict__ v,
                                                         const double* __restrict__ u,
                                                         double* __restrict__ part, int m) {
  // per-thread terms, then block reductions of them through LDS, G terms at a
  // time (24 KB of LDS)
  constexpr int NV = 2 * K, G = NV < 12 ? NV : 12;
  __shared__ double s_val[G][TILE];
  __shared__ double s_mid[G][TILE / 16];
  const int N = op.N, nt = op.ntiles;
  const int tile = blockIdx.x, i = blockIdx.y;
  const int n = tile * TILE + threadIdx.x;
  const bool valid = n < N;
  const int nn = valid ? n : N - 1;
  int nb[6];
#pragma unroll
  for (int d = 0; d < 6; ++d) nb[d] = op.nbr[(size_t)d * N + nn];
  // every load of the voxel issued before any use
  int vv[K][7];
  double un[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const size_t off = ((size_t)i * K + k) * N;
    vv[k][6] = v[off + nn];
#pragma unroll
    for (int d = 0; d < 6; ++d) vv[k][d] = v[off + nb[d]];
    un[k] = u[off + nn];
  }
  double val[NV];   // [0, K): v_k u_k, [K, 2K): (G v)_k u_k
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double gv = 0.0;
#pragma unroll
    for (int d = 0; d < 6; ++d) gv += (double)(vv[k][6] - vv[k][d]);
    val[k] = valid ? (double)vv[k][6] * un[k] : 0.0;
    val[K + k] = valid ? gv * un[k] : 0.0;
  }
#pragma unroll
  for (int g0 = 0; g0 < NV; g0 += G) {
    const int ng = NV - g0 < G ? NV - g0 : G;
#pragma unroll
    for (int j = 0; j < G; ++j)
      if (j < ng) s_val[j][threadIdx.x] = val[g0 + j];
    __syncthreads();
    // ng x 16 partial sums of 16 terms, then ng sums of 16 partials, each in
    // a fixed order
    for (int t = threadIdx.x; t < ng * (TILE / 16); t += TILE) {
      const int q = t / (TILE / 16), c = t % (TILE / 16);
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < 16; ++j) acc += s_val[q][c * 16 + j];
      s_mid[q][c] = acc;
    }
    __syncthreads();
    if (threadIdx.x < ng) {
      const int e = g0 + threadIdx.x, which = e / K, k = e % K;
      double t = 0.0;
#pragma unroll
      for (int c = 0; c < TILE / 16; ++c) t += s_mid[threadIdx.x][c];
      part[(((size_t)which * m + i) * K + k) * nt + tile] = t;
    }
    __syncthreads();
  }
}

// Sums over tiles, one wavefront per (which, probe, regressor) pair:
// pairbuf[q] = sum_t part[q][t] in a fixed order.
__global__ __launch_bounds__(TILE) void k_trace_pairs(const double* __restrict__ part, int pairs, int nt,
                                                      double* __restrict__ pairbuf) {
  const int q = blockIdx.x * (TILE / WAVE) + (int)(threadIdx.x / WAVE);
  if (q >= pairs) return;
  const int lane = threadIdx.x % WAVE;
  double s = 0.0;
  for (int t = lane; t < nt; t += WAVE) s += part[(size_t)q * nt + t];
  s = wave_sum(s);
  if (lane == 0) pairbuf[q] = s;
}

// out[0] = (1/m) sum_{i,k} vu, out[1+k] = (1/m) sum_i vu_k,
// out[1+K+k] = (1/m) sum_i (Gv)u_k, each sum over probes in a fixed order.
__global__ __launch_bounds__(WAVE) void k_trace_final(const double* __restrict__ pairbuf, int m, int K,
                                                      double* __restrict__ out) {
  const int k = threadIdx.x;
  double a = 0.0, g = 0.0;
  if (k < K) {
    for (int i = 0; i < m; ++i) {
      a += pairbuf[(0 * (size_t)m + i) * K + k];
      g += pairbuf[(1 * (size_t)m + i) * K + k];
    }
    out[1 + k] = a / m;
    out[1 + K + k] = g / m;
  }
  // total over regressors in order k = 0..K-1
  double tot = 0.0;
  for (int j = 0; j < K; ++j) tot += __shfl(a, j, WAVE);
  if (k == 0) out[0] = tot / m;
}

// --------------------------------------------------------------- launchers
#define GP_K_CASES(X)                                                                                  \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) \
      X(20) X(21) X(22) X(23) X(24)

hipError_t launch_pack_blocks(hipStream_t s, int K, int N, const double* B, double* B64, float* B32,
                              double* L64, int* bad) {
  const dim3 g((N + TILE - 1) / TILE), b(TILE);
  switch (K) {
#define X(KK) case KK: GP_LAUNCH(k_pack_blocks<KK>, g, b, 0, s, N, B, B64, B32, L64, bad); break;
    GP_K_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_precond(hipStream_t s, const OpDev& op, int pc, double* P64, float* P32, int* bad) {
  const dim3 g((op.N + TILE - 1) / TILE), b(TILE);
  switch (op.K) {
#define X(KK) case KK: GP_LAUNCH(k_precond<KK>, g, b, 0, s, op, pc, P64, P32, bad); break;
    GP_K_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Tiles per block of an item order: two planes of voxels and two tiles, the
// block's packed matrices at most 1.5 MB.
static int tiles_per_block(const OpDev& op) {
  const long reach = ((long)op.N / (op.nz > 0 ? op.nz : 1) + TILE - 1) / TILE;
  const long cap = std::max(4L, (long)(1536 << 10) / ((long)(op.K * (op.K + 1) / 2) * TILE * 8));
  return (int)std::max(1L, std::min({2 * reach + 2, cap, (long)op.ntiles}));
}

hipError_t launch_apply(hipStream_t s, const OpDev& op, int R, const double* x, double* y) {
  if (op.ntiles == 0 || R == 0) return hipSuccess;
  // right-hand sides per workgroup (their block read once): the largest of 4, 2
  // that leaves 640 workgroups (8 right-hand sides at N = 85,936, 672 of them:
  // 23.2 us at K = 6 against 27.6 at one each, 12.1 against 12.6 at K = 3; 24 at
  // N = 12,704, K = 4, 600 of them: 10.0 against 8.8), else one; more where a
  // launch could not hold the workgroups (2^32 lanes).  Beyond K = KREG a block
  // does not stay in registers (K = 20, N = 85,936, R = 4: 73 us at 1, 217 at
  // 2).  0: one on a two-dimensional grid, where few workgroups make the
  // mapping's divisions cost more than it gives (K = 10, N = 20,848, R = 4, 328
  // of them: 12.6 us unmapped, 10.0 mapped; K = 7, N = 9,048, R = 3, 108: 4.7
  // and 5.2).
  int rc = (long)op.ntiles * R >= 320 ? 1 : 0;
  if (op.K <= KREG)
    for (int cand : {4, 2})
      if ((long)op.ntiles * ((R + cand - 1) / cand) >= 640) {
        rc = cand;
        break;
      }
  const auto blocks = [&]() { return (long)op.ntiles * ((R + std::max(rc, 1) - 1) / std::max(rc, 1)); };
  while (blocks() * TILE >= 1L << 32) rc *= 2;
  const dim3 g = rc ? dim3((unsigned)blocks()) : dim3(op.ntiles, R), b(TILE);
  const int tb = tiles_per_block(op);
  switch (op.K) {
#define X(KK)                                                                          \
  case KK:                                                                             \
    if (rc > 1)                                                                        \
      GP_LAUNCH((k_apply<KK, 2>), g, b, 0, s, op, x, y, R, rc, tb);                    \
    else if (rc == 1)                                                                  \
      GP_LAUNCH((k_apply<KK, 1>), g, b, 0, s, op, x, y, R, rc, tb);                    \
    else                                                                               \
      GP_LAUNCH((k_apply<KK, 0>), g, b, 0, s, op, x, y, R, rc, tb);                    \
    break;
    GP_K_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_perturb(hipStream_t s, const OpDev& op, int R, const double* bw, const double* z1,
                          const double* z2, double* b) {
  if (op.ntiles == 0 || R == 0) return hipSuccess;
  const dim3 g((unsigned)((long)op.ntiles * R)), bl(TILE);
  const int tb = tiles_per_block(op);
  switch (op.K) {
#define X(KK) case KK: GP_LAUNCH(k_perturb<KK>, g, bl, 0, s, op, bw, z1, z2, b, R, tb); break;
    GP_K_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_add_broadcast(hipStream_t s, int R, long kn, const double* bw, double* b) {
  const long total = (long)R * kn;
  const int bs = 256;
  GP_LAUNCH(k_add_broadcast, dim3((unsigned)((total + bs - 1) / bs)), dim3(bs), 0, s, total, kn, bw, b);
  return hipGetLastError();
}

hipError_t launch_probe_rhs(hipStream_t s, long total, const int8_t* v, double* b) {
  const int bs = 256;
  GP_LAUNCH(k_probe_rhs, dim3((unsigned)((total + bs - 1) / bs)), dim3(bs), 0, s, total, v, b);
  return hipGetLastError();
}

hipError_t launch_finalize(hipStream_t s, int kind, const Prob* probs, int nprob, int nblocks) {
  const dim3 g(nblocks), b(FIN_WAVES * WAVE);
  switch (kind) {
    case 0: GP_LAUNCH(k_finalize<0>, g, b, 0, s, probs, nprob); break;
    case 1: GP_LAUNCH(k_finalize<1>, g, b, 0, s, probs, nprob); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int finalize_rhs_per_block() { return FIN_WAVES; }

hipError_t launch_trace(hipStream_t s, const OpDev& op, int m, const int8_t* v, const double* u,
                        double* part, double* pairbuf, double* out) {
  const dim3 g(op.ntiles, m), b(TILE);
  switch (op.K) {
#define X(KK) case KK: GP_LAUNCH(k_trace_partials<KK>, g, b, 0, s, op, v, u, part, m); break;
    GP_K_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
  }
  const int pairs = 2 * m * op.K;
  GP_LAUNCH(k_trace_pairs, dim3((pairs + TILE / WAVE - 1) / (TILE / WAVE)), dim3(TILE), 0, s, part, pairs,
                     op.ntiles, pairbuf);
  GP_LAUNCH(k_trace_final, dim3(1), dim3(WAVE), 0, s, pairbuf, m, op.K, out);
  return hipGetLastError();
}

}  // namespace gp
