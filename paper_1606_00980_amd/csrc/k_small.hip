// FP64 PCG solves of small operators (a 2D slice), one workgroup per
// right-hand side carrying the whole solve: the same iteration, refinement
// and stopping rules as the grouped kernels of pcg.hpp.
//
// Such a solve is bound by launches: an iteration of the grouped kernels is
// three of them, 3 to 4 us each at N = 2,472, K = 2, for 0.3 MB of vectors.
// Here a lane owns V voxels and keeps their r, d and q in registers; the
// direction p, which the stencil gathers, is in LDS; the blocks and the
// preconditioner are held in registers or come from L2.  An iteration is two barriers: after p is
// written, and in the reduction, whose seven sums every wavefront finishes by
// itself from the eight per-wavefront partials in a fixed order, so that all
// lanes advance the same state without a further exchange.  x and b are
// touched only by the refinement.
// Measured on that slice (36 iterations of Jacobi to 1e-10): 3.4 us an
// iteration against 8.7 in the grouped kernels; a solve and a sample 264 us
// against 675 (with replayed rounds; 16 wavefronts a workgroup instead of
// eight, with spills and the blocks read per use, 360 us).
#include <utility>

#include "launch.hpp"
#include "pcg.hpp"

namespace gp {
namespace {

constexpr int SM_WG = 512, SM_NW = SM_WG / WAVE;

// NV per-lane values summed over the workgroup, every lane receiving the
// totals.  The caller has a barrier between two calls.
template <int NV>
__device__ __forceinline__ void group_sums(double* s_red, const double (&acc)[NV], double (&tot)[NV]) {
  static_assert(NV <= 8 && SM_NW == 8, "eight lanes per value, a partial each");
  wave_deposit<NV>(s_red, 0, acc);   // s_red[v * SM_NW + wavefront]
  __syncthreads();
  const int lane = threadIdx.x % WAVE, v = lane / 8, c = lane % 8;
  double e = v < NV ? s_red[v * SM_NW + c] : 0.0;
#pragma unroll
  for (int dist = 4; dist > 0; dist >>= 1) e += __shfl_xor(e, dist, WAVE);
  const long long eb = __builtin_bit_cast(long long, e);
  const int lo = (int)eb, hi = (int)(eb >> 32);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const unsigned l = (unsigned)__builtin_amdgcn_readlane(lo, i * 8);
    const unsigned h = (unsigned)__builtin_amdgcn_readlane(hi, i * 8);
    tot[i] = __builtin_bit_cast(double, ((unsigned long long)h << 32) | l);
  }
}

template <int PC, int K, int V>
__global__ __launch_bounds__(SM_WG) void k_small(const Prob* __restrict__ probs, int nprob) {
  constexpr int NB = Tri<K>::NB, NP = PSize<PC, K>::n, NV = V * SM_WG;
  __shared__ double sp[K * NV];
  __shared__ double s_red[8 * SM_NW];
  int pi = 0;
  while (pi + 1 < nprob && (int)blockIdx.x >= probs[pi + 1].sm_begin) ++pi;
  const Prob& pr = probs[pi];
  const OpDev& op = pr.op;
  const int R = (int)blockIdx.x - pr.sm_begin, N = op.N;
  const SolveCfg& cfg = pr.cfg;
  const Slab<double> Bs(op.B64, NB, N), Ps(op.P64, NP, N);
  const Slab<double> bs(pr.b + (size_t)R * K * N, K, N), xs(pr.x + (size_t)R * K * N, K, N);
  // lanes past the end work on the last voxel and contribute and store nothing
  int nn[V];
  bool ok[V];
  unsigned nb[V][3];   // six neighbours (the voxel itself where absent), two to a word
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int n = v * SM_WG + (int)threadIdx.x;
    ok[v] = n < N;
    nn[v] = ok[v] ? n : N - 1;
    const Slab<int> nbr(op.nbr, 6, N);
#pragma unroll
    for (int w = 0; w < 3; ++w)
      nb[v][w] = (unsigned)nbr.ld(2 * w, (unsigned)nn[v] * 4u) | ((unsigned)nbr.ld(2 * w + 1, (unsigned)nn[v] * 4u) << 16);
  }
  auto neighbour = [&](int v, int d) { return (int)((nb[v][d / 2] >> (16 * (d % 2))) & 0xFFFFu); };
  double r[V][K], d[V][K], q[V][K];
  RhsState s{};
  long long* prof = threadIdx.x == 0 ? pr.prof : nullptr;   // the finalisers count for the profiler on one lane
  if (prof) {
    atomicAdd((unsigned long long*)&pr.prof[PF_REFINE_ACT], 1ull);
    atomicAdd((unsigned long long*)&pr.prof[PF_MATVEC_ACT], 1ull);
    atomicAdd((unsigned long long*)&pr.prof[PF_UPDATE_ACT], 1ull);
  }
  // the voxels' blocks and preconditioner, in registers where they fit beside
  // the vectors, else read (L2) where they are used
  constexpr bool HOLD = V * (NB + NP + 3 * K) <= 72;
  double Bh[HOLD ? V : 1][NB], Ph[HOLD ? V : 1][NP];
  if constexpr (HOLD) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      load_soa(Bs, (unsigned)nn[v] * 8u, Bh[v]);
      load_soa(Ps, (unsigned)nn[v] * 8u, Ph[v]);
    }
  }
  auto block = [&](int v, const double (&x)[K], double (&y)[K]) {   // y += B x
    if constexpr (HOLD)
      sym_apply<K>([&](int i) { return Bh[v][i]; }, x, y);
    else
      sym_apply<K>([&](int i) { return Bs.ld(i, (unsigned)nn[v] * 8u); }, x, y);
  };
  auto precond = [&](int v, const double (&y)[K], double (&z)[K]) {   // z = M^{-1} y
    auto get = [&](int i) {
      if constexpr (HOLD)
        return Ph[v][i];
      else
        return Ps.ld(i, (unsigned)nn[v] * 8u);
    };
#pragma unroll
    for (int k = 0; k < K; ++k) z[k] = 0.0;
    if constexpr (PC == PC_JACOBI) {
#pragma unroll
      for (int k = 0; k < K; ++k) z[k] = get(k) * y[k];
    } else {
      sym_apply<K>(get, y, z);
    }
  };
  while (s.phase != PH_DONE) {
    if (s.phase == PH_OUTER) {
      // x += d (+ a p of a stopping step), then r = b - Q x, p = M^{-1} r
      const bool fresh = cfg.zero_guess && s.outer == 1, x0 = cfg.zero_guess && s.outer == 0;
      if (s.has_d || s.pend || fresh) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const unsigned o = (unsigned)nn[v] * 8u;
          double xv[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            xv[k] = fresh ? 0.0 : xs.ld(k, o);
            if (s.has_d) xv[k] += d[v][k];
            if (s.pend) xv[k] += s.a * sp[k * NV + nn[v]];
          }
          if (ok[v]) {
#pragma unroll
            for (int k = 0; k < K; ++k) xs.st(k, o, xv[k]);
          }
        }
      }
      __syncthreads();
      double acc[3] = {0.0, 0.0, 0.0}, z[V][K];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const unsigned o = (unsigned)nn[v] * 8u;
        double y[K];
#pragma unroll
        for (int k = 0; k < K; ++k) y[k] = 0.0;
        if (!x0) {
          double xo[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            xo[k] = xs.ld(k, o);
            double s6 = 0.0;
#pragma unroll
            for (int e = 0; e < 6; ++e) s6 += xo[k] - xs.ld(k, (unsigned)neighbour(v, e) * 8u);
            y[k] = op.alpha64[k] * s6;
          }
          block(v, xo, y);
        }
        double bb = 0.0, rr = 0.0, rz = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const double bk = bs.ld(k, o);
          r[v][k] = bk - y[k];
          rr += r[v][k] * r[v][k];
          bb += bk * bk;
        }
        precond(v, r[v], z[v]);
#pragma unroll
        for (int k = 0; k < K; ++k) rz += r[v][k] * z[v][k];
        acc[0] += ok[v] ? rr : 0.0;
        acc[1] += ok[v] ? bb : 0.0;
        acc[2] += ok[v] ? rz : 0.0;
      }
      double tot[3];
      group_sums<3>(s_red, acc, tot);
      finalize_refine(cfg, prof, s, tot);
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (ok[v]) {
#pragma unroll
          for (int k = 0; k < K; ++k) sp[k * NV + nn[v]] = z[v][k];
        }
    } else {
      double acc[NPART] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int v = 0; v < V; ++v) {
        double p[K], z[K], t[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
          p[k] = sp[k * NV + nn[v]];
          double s6 = 0.0;
#pragma unroll
          for (int e = 0; e < 6; ++e) s6 += p[k] - sp[k * NV + neighbour(v, e)];
          q[v][k] = op.alpha64[k] * s6;
        }
        block(v, p, q[v]);
        precond(v, r[v], z);
        precond(v, q[v], t);
        double a[NPART] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < K; ++k) {
          a[0] += p[k] * q[v][k];
          a[1] += r[v][k] * z[k];
          a[2] += q[v][k] * z[k];
          a[3] += q[v][k] * t[k];
          a[4] += r[v][k] * r[v][k];
          a[5] += q[v][k] * r[v][k];
          a[6] += q[v][k] * q[v][k];
        }
#pragma unroll
        for (int e = 0; e < NPART; ++e) acc[e] += ok[v] ? a[e] : 0.0;
      }
      double tot[NPART];
      group_sums<NPART>(s_red, acc, tot);
      finalize_matvec(cfg, prof, s, tot);
      if (s.phase == PH_INNER) {
        // d += a p, r -= a q, p = M^{-1} r + beta p
        const bool first = s.inner_it == 1;
#pragma unroll
        for (int v = 0; v < V; ++v) {
          double p[K], z[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            p[k] = sp[k * NV + nn[v]];
            d[v][k] = (first ? 0.0 : d[v][k]) + s.a * p[k];
            r[v][k] -= s.a * q[v][k];
          }
          precond(v, r[v], z);
          if (ok[v]) {
#pragma unroll
            for (int k = 0; k < K; ++k) sp[k * NV + nn[v]] = z[k] + s.beta * p[k];
          }
        }
      }
    }
    __syncthreads();   // p is written, the partials are read
  }
  if (threadIdx.x == 0) pr.st[R] = s;
}

}  // namespace

// Doubles a lane handles per iteration: V voxels' block, preconditioner, r, d
// and q.  Up to SM_MOST the one-workgroup solve is the faster one also for a
// single right-hand side (block Jacobi, small against grouped: K = 2, N = 4,060,
// 96 doubles, 203 against 308 us; K = 6, N = 1,020, 120 doubles, 276 against
// 440 us), beyond it the blocks, then read from L2 by one compute unit, cost
// more than the launches (K = 8, N = 820, 192 doubles, 632 against 554 us).
constexpr int SM_MOST = 128;
constexpr int SM_KMOST = 10;   // largest K with a kernel
constexpr int SM_V[] = {1, 2, 3, 4, 5, 6, 8, 12};   // voxels per lane with a kernel
constexpr int lane_doubles(int pc, int K, int V) {
  return V * (K * (K + 1) / 2 + (pc == PC_BLOCK ? K * (K + 1) / 2 : K) + 3 * K);
}

// What the rule may return and the launcher can run, for V out of SM_V.  (Up
// to 512 voxels Jacobi stays within SM_MOST at K = 11 and 12 too: those have no
// kernel and take the grouped ones.)
constexpr bool small_kernel(int pc, int K, int V) { return K <= SM_KMOST && lane_doubles(pc, K, V) <= SM_MOST; }

// Voxels per lane, 0 where the grouped kernels take the solve.
int small_lane_voxels(int pc, int N, int K) {
  for (int v : SM_V)
    if (N <= v * SM_WG) return small_kernel(pc, K, v) ? v : 0;
  return 0;
}

namespace {
template <int PC, int K, int V>
bool try_small(hipStream_t s, int pc, int k, int v, const Prob* probs, int nprob, int nrhs) {
  if constexpr (small_kernel(PC, K, V)) {
    if (pc == PC && k == K && v == V) {
      GP_LAUNCH((k_small<PC, K, V>), dim3(nrhs), dim3(SM_WG), 0, s, probs, nprob);
      return true;
    }
  }
  return false;
}
template <int K, int... I>
bool try_small_k(std::integer_sequence<int, I...>, hipStream_t s, int pc, int k, int v, const Prob* probs, int nprob,
                 int nrhs) {
  return (try_small<PC_BLOCK, K, SM_V[I]>(s, pc, k, v, probs, nprob, nrhs) || ...) ||
         (try_small<PC_JACOBI, K, SM_V[I]>(s, pc, k, v, probs, nprob, nrhs) || ...);
}
// every K up to SM_KMOST with every V
template <int... I>
bool try_small_all(std::integer_sequence<int, I...>, hipStream_t s, int pc, int k, int v, const Prob* probs, int nprob,
                   int nrhs) {
  constexpr int NV = sizeof(SM_V) / sizeof(SM_V[0]);
  return (try_small_k<I + 1>(std::make_integer_sequence<int, NV>{}, s, pc, k, v, probs, nprob, nrhs) || ...);
}
}  // namespace

hipError_t launch_small(hipStream_t s, int pc, int K, int V, const Prob* probs, int nprob, int nrhs) {
  if (!try_small_all(std::make_integer_sequence<int, SM_KMOST>{}, s, pc, K, V, probs, nprob, nrhs))
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace gp
