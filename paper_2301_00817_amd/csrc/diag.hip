// Diagnostics of a state: conservation totals and azimuthal statistics.
//
//   totals[c] = sum over the interior of J^-1 Q_c   (c = rho, rho u, rho v,
//               rho w, E): the discrete conserved quantities, constant in
//               time on a periodic mesh because every face flux enters its
//               two cells with opposite signs;
//   sum1[c](i, j) += sum_k phi_c,  sum2[c](i, j) += sum_k phi_c^2  with
//               phi = (rho, u, v, w, p): accumulators of the azimuthal (and,
//               over calls, temporal) mean and rms fields.
//
// Both reductions run in a fixed order (totals: per-block tree, then one block
// over the partials in block order; statistics: every eighth plane per thread,
// the eight sums in order), so repeated runs are bitwise identical, and the
// totals are the same with and without the statistics.  FP64 throughout.
#include "launch.hpp"
#include "physics.hpp"

namespace lesjet {

constexpr int DIAG_BS = 256;

// One pass over Q for both.  A block takes groups of DG_I consecutive (i, j)
// columns; its eight rows of threads share the planes k of a group (one thread
// per column left 46,000 threads for 5.9 M points: the statistics took 72 us, the
// totals in a second pass 48 us and their last sums 14 us; now 58 + 5 us, 4.1 TB/s
// of the state).  The eight partial sums of a column are added in order through
// LDS; the totals stay in the threads' registers to the end.  PROD: J^-1 of a
// product mesh from its tables.
// CUT: few columns give few blocks, however many planes there are.  The totals then
// cut the azimuth into chunks of planes, a block each (alone, 64 x 64 x 1440: 123 us
// in 128 blocks, now 60; 16 x 16 x 4096: 207 us in eight, now 19).  The statistics
// keep one block per group, as each column is added up by one, with four planes
// in flight; asked for together, both kinds of blocks are in one launch (107 and
// 130 us; 129 and 230 by blocks of one kind).
constexpr int DG_I = 32, DG_K = DIAG_BS / DG_I;

struct DiagPlan {
  int groups;         // column groups
  int chunks, kc;     // chunks of planes of the totals and their length
};

template <typename TM, bool PROD, bool CUT>
__global__ __launch_bounds__(DIAG_BS) void k_diag(const double* __restrict__ Q,
                                                  const TM* __restrict__ M, Grid g,
                                                  Phys<double> ph, ProdTab pt, DiagPlan pl,
                                                  double* __restrict__ part,
                                                  double* __restrict__ s1, double* __restrict__ s2) {
  __shared__ double red[10][DG_K][DG_I];
  const int li = threadIdx.x % DG_I, lk = threadIdx.x / DG_I;
  const int ncol = g.nx * g.nr;
  constexpr int U = CUT ? 4 : 1;      // planes loaded together
  bool stats = s1 || s2;
  int b = blockIdx.x, np = gridDim.x, g0 = b, gs = np, k0 = 0, k1 = g.nth;
  if (CUT) {                 // the first blocks the statistics, the others a chunk each
    const int ns = stats ? pl.groups : 0;
    gs = pl.groups;
    if (b < ns) {
      part = nullptr;
    } else {
      stats = false;
      b -= ns;
      np -= ns;
      g0 = b / pl.chunks;
      k0 = (b - g0 * pl.chunks) * pl.kc;
      k1 = min(k0 + pl.kc, g.nth);
    }
  }
  double tot[5] = {0, 0, 0, 0, 0};
  for (int gp = g0; gp < pl.groups; gp += gs) {
    const int t = gp * DG_I + li;
    double a[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (t < ncol) {
      const int j = t / g.nx, i = t - j * g.nx;
      const double xx = PROD ? pt.x[(i + NG) * PX_N] : 0.0;
#pragma unroll CUT ? 1 : 2
      for (int k = k0 + lk; k < k1; k += U * DG_K) {
        double q[U][5];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int o = g.at(i, j, U == 1 ? k : min(k + u * DG_K, k1 - 1));
          for (int c = 0; c < 5; ++c) q[u][c] = Q[(long long)c * g.vs + o];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int ku = k + u * DG_K;
          if (U > 1 && ku >= k1) break;
          if (part) {
            double V;
            if (PROD) {      // the stored value is of the storage type
              double m[10];
              product_terms(xx, pt.yz + (long long)(ku + NG) * prod_plane(g) + (j + NG) * PT_N, m);
              V = (double)(TM)m[9];
            } else {
              V = (double)M[9LL * g.vs + g.at(i, j, ku)];
            }
            for (int c = 0; c < 5; ++c) tot[c] += V * q[u][c];
          }
          if (stats) {
            const Prim<double> s = primitives(q[u], ph);
            const double f[5] = {s.rho, s.u, s.v, s.w, s.p};
            for (int c = 0; c < 5; ++c) { a[c] += f[c]; a[5 + c] += f[c] * f[c]; }
          }
        }
      }
    }
    if (stats) {
      for (int c = 0; c < 10; ++c) red[c][lk][li] = a[c];
      __syncthreads();
      const long long sp = (long long)ncol;
      for (int e = threadIdx.x; e < 10 * DG_I; e += DIAG_BS) {
        const int c = e / DG_I, tc = gp * DG_I + e % DG_I;
        double* dst = c < 5 ? s1 : s2;
        if (tc < ncol && dst) {
          double v = 0.0;
          for (int r = 0; r < DG_K; ++r) v += red[c][r][e % DG_I];
          dst[(c % 5) * sp + tc] += v;
        }
      }
      __syncthreads();
    }
  }
  if (!part) return;
  double* rt = &red[0][0][0];
  for (int c = 0; c < 5; ++c) rt[c * DIAG_BS + threadIdx.x] = tot[c];
  __syncthreads();
  for (int w = DIAG_BS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int c = 0; c < 5; ++c) rt[c * DIAG_BS + threadIdx.x] += rt[c * DIAG_BS + threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 5) part[(long long)threadIdx.x * np + b] = rt[threadIdx.x * DIAG_BS];
}

// One block per total.
__global__ __launch_bounds__(DIAG_BS) void k_totals_final(const double* __restrict__ part, int nparts,
                                                          double* __restrict__ totals) {
  __shared__ double red[DIAG_BS];
  const double* p = part + (long long)blockIdx.x * nparts;
  double a = 0.0;
  for (int b = threadIdx.x; b < nparts; b += DIAG_BS) a += p[b];
  red[threadIdx.x] = a;
  __syncthreads();
  for (int w = DIAG_BS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = red[0];
}

// The totals are cut where the column groups leave half of the device idle (128
// blocks; 100 x 50 x 100, 157 groups: 11.5 us uncut): chunks of at least 32 planes,
// four per thread, a multiple of the rows, and no more than 512 blocks.
static DiagPlan diag_plan(const Grid& g) {
  DiagPlan pl = {(g.nx * g.nr + DG_I - 1) / DG_I, 1, g.nth};
  const int n = (g.nth + 31) / 32;
  if (pl.groups <= 128 && n > 1) {
    const int fit = 512 / pl.groups, c = n < fit ? n : fit;
    pl.kc = ((g.nth + c - 1) / c + DG_K - 1) / DG_K * DG_K;
    pl.chunks = (g.nth + pl.kc - 1) / pl.kc;
  }
  return pl;
}

int diag_partials(const Grid& g) {
  const DiagPlan pl = diag_plan(g);
  const int n = pl.groups * pl.chunks;
  return n > DIAG_MAX_PARTIALS ? DIAG_MAX_PARTIALS : n;
}

template <typename TM>
hipError_t launch_diagnostics(const double* Q, const TM* M, const Grid& g,
                              const Phys<double>& ph, double* part, double* totals, double* s1,
                              double* s2, const ProdTab& pt, hipStream_t s) {
  const DiagPlan pl = diag_plan(g);
  const int np = diag_partials(g);
  const bool stats = s1 || s2, cut = pl.chunks > 1;
  const int nb = cut ? (totals ? np : 0) + (stats ? pl.groups : 0) : np;
  if (!totals) part = nullptr;
#define LESJET_DIAG(P, C) \
  hipLaunchKernelGGL((k_diag<TM, P, C>), dim3(nb), dim3(DIAG_BS), 0, s, Q, M, g, ph, pt, pl, part, s1, s2)
  if (totals || stats) {
    if (pt.x) {
      if (cut) LESJET_DIAG(true, true);
      else LESJET_DIAG(true, false);
    } else {
      if (cut) LESJET_DIAG(false, true);
      else LESJET_DIAG(false, false);
    }
  }
#undef LESJET_DIAG
  if (totals) hipLaunchKernelGGL(k_totals_final, dim3(5), dim3(DIAG_BS), 0, s, part, np, totals);
  return hipGetLastError();
}

template hipError_t launch_diagnostics<double>(const double*, const double*, const Grid&,
                                               const Phys<double>&, double*, double*, double*,
                                               double*, const ProdTab&, hipStream_t);
template hipError_t launch_diagnostics<float>(const double*, const float*, const Grid&,
                                              const Phys<double>&, double*, double*, double*,
                                              double*, const ProdTab&, hipStream_t);

}  // namespace lesjet
