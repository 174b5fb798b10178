// Time-step reduction of Runge-Kutta steps (section "Time Marching Method", eq.
// localdt): one global dt = CFL / max over the interior of (lambda_xi +
// lambda_eta + lambda_zeta); the stage update is the stage kernel's epilogue.  The
// maximum is taken with an integer atomic on the bit
// pattern of non-negative doubles, which orders like the values and makes
// the result independent of scheduling; a NaN sorts above every number so a
// diverged state cannot hide.
#include "launch.hpp"
#include "physics.hpp"

namespace lesjet {

// First pass of a call over Q^n: the maximum over the interior of the
// spectral-radius sum (LAM) and, in the FP32-storage form, the FP32 copy of the
// interior that the first stage reads (Q32; the ghosts are filled from it).
// One thread per column (i, j) of a chunk of kc planes: the state is read once for
// both (0.37 ms on 23.6 M points, bound by memory; two passes, each with 64-bit
// index divisions per point, took 0.66 ms), a product mesh's metric terms come from its tables, and a
// block reduces to one atomic.
constexpr int LM_BS = 256;
template <typename TM, bool PROD, bool LAM>
__global__ __launch_bounds__(LM_BS) void k_first_pass(const double* __restrict__ Q,
                                                      const TM* __restrict__ M, Grid g,
                                                      Phys<double> ph, ProdTab pt, int kc,
                                                      unsigned long long* __restrict__ maxbits,
                                                      float* __restrict__ Q32) {
  __shared__ double red[LM_BS / 64];
  const int t = blockIdx.x * LM_BS + (int)threadIdx.x;
  double local = 0.0;
  if (t < g.nx * g.nr) {
    const int j = t / g.nx, i = t - j * g.nx;
    const int k0 = (int)blockIdx.y * kc, k1 = min(k0 + kc, g.nth);
    const double xx = LAM && PROD ? pt.x[(i + NG) * PX_N] : 0.0;
    const bool skip = ph.axis_node && j == 0;      // centerline row is not advanced
#pragma unroll 2
    for (int k = k0; k < k1; ++k) {
      const int o = g.at(i, j, k);
      double q[5];
      for (int c = 0; c < 5; ++c) q[c] = Q[(long long)c * g.vs + o];
      if (Q32)
        for (int c = 0; c < 5; ++c) Q32[(long long)c * g.vs + o] = (float)q[c];
      if (LAM && !skip) {
        double S[3][3], V;
        if (PROD) {     // the stored terms are those of the storage type
          double m[10];
          product_terms(xx, pt.yz + (long long)(k + NG) * prod_plane(g) + (j + NG) * PT_N, m);
          for (int d = 0; d < 3; ++d)
            for (int c = 0; c < 3; ++c) S[d][c] = (double)(TM)m[3 * d + c];
          V = (double)(TM)m[9];
        } else {
          for (int d = 0; d < 3; ++d)
            for (int c = 0; c < 3; ++c) S[d][c] = (double)M[(long long)(3 * d + c) * g.vs + o];
          V = (double)M[9LL * g.vs + o];
        }
        const double x = lambda_sum<PROD>(q, S, V, ph);
        if (x != x || x > local) local = x;      // keeps a NaN once seen
      }
    }
  }
  if (!LAM) return;
  for (int off = 32; off > 0; off >>= 1) {
    const double b = __shfl_xor(local, off, 64);
    if (b != b || b > local) local = b;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = local;
  __syncthreads();
  if (threadIdx.x == 0) {
    double b = red[0];
    for (int w = 1; w < LM_BS / 64; ++w)
      if (red[w] != red[w] || red[w] > b) b = red[w];
    atomicMax(maxbits, (unsigned long long)__double_as_longlong(b));
  }
}

// dt for one step; resets the reduction slot for the next step.
__global__ void k_dt_finalize(unsigned long long* maxbits, double cfl, double dt_fixed,
                              double* dt, double* dt_out, int* flag) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double h;
  if (dt_fixed > 0.0) {
    h = dt_fixed;
  } else {
    const double m = __longlong_as_double((long long)*maxbits);
    h = cfl / m;
    if (!(m > 0.0) || !isfinite(h)) *flag = 1;
  }
  *maxbits = 0ull;
  *dt = h;
  if (dt_out) *dt_out = h;
}

__global__ void k_reset(unsigned long long* maxbits, int* flag) {
  if (threadIdx.x == 0 && blockIdx.x == 0) { *maxbits = 0ull; *flag = 0; }
}

template <typename TM>
hipError_t launch_first_pass(const double* Q, const TM* M, const Grid& g, const Phys<double>& ph,
                             bool lambda, unsigned long long* maxbits, float* Q32,
                             const ProdTab& pt, hipStream_t s) {
  // chunks of up to 16 planes (one atomic per block), shorter while the mesh
  // gives fewer than eight blocks per CU or so
  const int nb = (int)blocks_for((long long)g.nx * g.nr, LM_BS);
  int kc = 16;
  while (kc > 1 && (long long)nb * ((g.nth + kc - 1) / kc) < 2048) kc /= 2;
  while ((g.nth + kc - 1) / kc > 65535) kc *= 2;
  const dim3 grid((unsigned)nb, (unsigned)((g.nth + kc - 1) / kc));
  if (!lambda)
    hipLaunchKernelGGL((k_first_pass<TM, false, false>), grid, dim3(LM_BS), 0, s, Q, M, g, ph, pt, kc,
                       maxbits, Q32);
  else if (pt.x)
    hipLaunchKernelGGL((k_first_pass<TM, true, true>), grid, dim3(LM_BS), 0, s, Q, M, g, ph, pt, kc,
                       maxbits, Q32);
  else
    hipLaunchKernelGGL((k_first_pass<TM, false, true>), grid, dim3(LM_BS), 0, s, Q, M, g, ph, pt, kc,
                       maxbits, Q32);
  return hipGetLastError();
}

hipError_t launch_dt_finalize(unsigned long long* maxbits, double cfl, double dt_fixed,
                              double* dt, double* dt_out, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_dt_finalize, dim3(1), dim3(64), 0, s, maxbits, cfl, dt_fixed, dt, dt_out,
                     flag);
  return hipGetLastError();
}

hipError_t launch_reset(unsigned long long* maxbits, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, s, maxbits, flag);
  return hipGetLastError();
}

template hipError_t launch_first_pass<double>(const double*, const double*, const Grid&,
                                              const Phys<double>&, bool, unsigned long long*,
                                              float*, const ProdTab&, hipStream_t);
template hipError_t launch_first_pass<float>(const double*, const float*, const Grid&,
                                             const Phys<double>&, bool, unsigned long long*,
                                             float*, const ProdTab&, hipStream_t);

}  // namespace lesjet
