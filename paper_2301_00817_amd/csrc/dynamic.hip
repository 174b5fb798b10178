// Coefficients of the dynamic Smagorinsky model (subsection "Dynamic
// Smagorinsky Model"): C_I of the isotropic SGS stress, C_ds of the eddy
// viscosity and the SGS Prandtl number, each a ratio of two volume averages
// over the interior.  Test filter: the separable three-point filter
// (1/4, 1/2, 1/4) along each index direction, test width 2 Delta; Delta =
// |J^-1|^(1/3) stays outside the hats (the local width at the averaging
// point).  Computed in FP64 from the state of the storage type; the sums are
// fixed-order trees (reproducible).
//
// The separable filter is applied one direction at a time:
//   k_dyn_hat     points of [-1, n]^3: the state fields rho, rho u_i, rho T
//                 filtered along j (LDS), i (lane moves) and k (registers,
//                 marching over planes) -> hat(rho), hat(rho u_i), hat(rho T);
//   k_dyn_terms   the stage kernel's march: per plane each ring-1 column forms
//                 rho |S| S_ij, rho |S|^2, rho |S| dT/dx_j, rho u_i u_j and
//                 rho u_i T, filters them along i (lane moves), j (LDS) and k
//                 (registers); with the strain of u_hat = hat(rho u)/hat(rho) and
//                 the gradient of T_hat = hat(rho T)/hat(rho) the J^-1-weighted
//                 numerator and denominator terms of the plane before are
//                 added up in registers, one set of seven sums per block (two
//                 launches, one per group of fields);
//   k_dyn_final   the sums, the coefficients, clipping.
// Only the five filtered state fields pass through memory.  (Filtering along
// i and j in one pass, 24 fields stored, and along k in two more took 0.48 ms
// on 2.05 M points, bound by those fields' 440 MB written and re-read at
// three planes; these passes take 0.044 + 0.098 + 0.068 ms.)
#include "launch.hpp"
#include "physics.hpp"
#include "tiles.hpp"

namespace lesjet {

// Scratch variables: the filtered state on [-1, n]^3.
enum { DY_HR = 0, DY_HRU = 1, DY_HRT = 4, DY_N = 5 };
static_assert(DY_N == DYN_SCRATCH_VARS, "dynamic-model scratch size");

// Fields of a plane: rho |S| S_ij, rho |S|^2, rho |S| dT/dx_j, rho u_i u_j,
// rho u_i T (ij = 00 11 22 01 02 12)
enum { DF_S = 0, DF_S2 = 6, DF_T = 7, DF_UU = 10, DF_UT = 16, DF_N = 19 };

constexpr int DY_BS = 256;
constexpr int DY_NSUM = 7;   // N_I, D_I, A, B, D_d, N_P, D_P
static_assert(DY_NSUM + 6 + 3 <= DYN_COEF_DOUBLES, "coefficient buffer size");

// Test filter (1/4, 1/2, 1/4) of three neighbouring values.
__device__ __forceinline__ double filt(double l, double c, double r) {
  return fma(0.25, l + r, 0.5 * c);
}

template <typename T>
__device__ __forceinline__ void load5(const T* __restrict__ Q, const Grid& g, unsigned col, int k,
                                      double q[5]) {
#pragma unroll
  for (int c = 0; c < 5; ++c) q[c] = (double)gld(Q, g, c, k, col);
}

// rho, u, v, w, T of a state.
__device__ __forceinline__ void prim_t(const double q[5], double gamma, double p[5]) {
  const double ir = trcp(q[0]);
  p[0] = q[0];
  p[1] = q[1] * ir;
  p[2] = q[2] * ir;
  p[3] = q[3] * ir;
  p[4] = gamma * ((gamma - 1.0) * (q[4] - 0.5 * q[0] * (p[1] * p[1] + p[2] * p[2] + p[3] * p[3]))) * ir;
}

// The chunks of planes: (rounds of resident blocks) x (planes per block).
static int dyn_chunk(long long tiles, int nth, int resident, int extra) {
  int best = nth;
  double best_cost = 1e300;
  for (int kc = 1; kc <= 64 && kc <= nth; ++kc) {
    const long long nb = tiles * ((nth + kc - 1) / kc);
    const double cost = (double)((nb + resident - 1) / resident) * (kc + extra);
    if (cost < best_cost) { best_cost = cost; best = kc; }
  }
  return best;
}

// Filtered state.  A block's rows of 32 threads hold the columns of 30
// outputs and one neighbour on each side; the rows above and below the tile
// are loaded by its first wave.
constexpr int DH_X = 32, DH_Y = 8;
template <typename T>
__global__ __launch_bounds__(DH_X * DH_Y) void k_dyn_hat(const T* __restrict__ Q, Grid g,
                                                         double gamma, int kc, TileMap tm,
                                                         double* __restrict__ SC) {
  __shared__ double sF[2][5][DH_Y + 2][DH_X];
  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * DH_X + tx;
  int bx, by, bz;
  if (!tile_of_block(tm, bx, by, bz)) return;
  // outputs i0 .. i0 + 29, j0 .. j0 + 7 of [-1, n]
  const int i0 = bx * (DH_X - 2) - 1, j0 = by * DH_Y - 1;
  const int k0 = bz * kc - 1, k1 = min(k0 + kc, g.nth + 1);
  const int i = i0 - 1 + tx, j = j0 + ty;
  const bool out = tx >= 1 && tx <= DH_X - 2 && i <= g.nx && j <= g.nr;
  const bool has_b = tid < 2 * DH_X;
  const int bry = tid < DH_X ? 0 : DH_Y + 1;
  const unsigned oq = q_col<T>(g, i, j), oob = q_col<T>(g, i0 - 1 + (tid & (DH_X - 1)), j0 - 1 + bry);
  const unsigned o64 = q_col<double>(g, i, j);
  // rho, rho u_i and rho T = gamma p of a state
  auto fields = [&](double q[5]) {
    q[4] = gamma * ((gamma - 1.0) *
                    (q[4] - 0.5 * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) * trcp(q[0])));
  };
  double q[5], b[5], fm[5] = {0, 0, 0, 0, 0}, fc[5] = {0, 0, 0, 0, 0};
  load5(Q, g, oq, k0 - 1, q);
  if (has_b) load5(Q, g, oob, k0 - 1, b);
  for (int kk = k0 - 1, buf = 0; kk <= k1; ++kk, buf ^= 1) {
    fields(q);
#pragma unroll
    for (int c = 0; c < 5; ++c) sF[buf][c][ty + 1][tx] = q[c];
    if (has_b) {
      fields(b);
#pragma unroll
      for (int c = 0; c < 5; ++c) sF[buf][c][bry][tid & (DH_X - 1)] = b[c];
    }
    double f[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) f[c] = q[c];
    if (kk < k1) {
      load5(Q, g, oq, kk + 1, q);
      if (has_b) load5(Q, g, oob, kk + 1, b);
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      f[c] = filt(sF[buf][c][ty][tx], f[c], sF[buf][c][ty + 2][tx]);
      f[c] = filt(from_left<DH_X>(f[c]), f[c], from_right<DH_X>(f[c]));
    }
    if (out && kk > k0) {
#pragma unroll
      for (int c = 0; c < 5; ++c) gst(SC, g, DY_HR + c, kk - 1, o64, filt(fm[c], fc[c], f[c]));
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) { fm[c] = fc[c]; fc[c] = f[c]; }
  }
}

// Gradients of (u, v, w, T) from the undivided central differences dl[d], by
// the chain rule with the metric terms m and hiV = 1 / (2 J^-1).
template <bool PROD>
__device__ __forceinline__ void chain_rule(const double dl[3][4], const double m[10], double hiV,
                                           double g[4][3]) {
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      if (!PROD) g[f][x] = (m[x] * dl[0][f] + m[3 + x] * dl[1][f] + m[6 + x] * dl[2][f]) * hiV;
      else if (x == 0) g[f][x] = m[0] * dl[0][f] * hiV;
      else g[f][x] = (m[3 + x] * dl[1][f] + m[6 + x] * dl[2][f]) * hiV;
    }
}

// S_ij (00 11 22 01 02 12) and |S| = sqrt(2 S_ij S_ij).
__device__ __forceinline__ void strain6(const double g[4][3], double S[6], double& Smag) {
  S[0] = g[0][0];
  S[1] = g[1][1];
  S[2] = g[2][2];
  S[3] = 0.5 * (g[0][1] + g[1][0]);
  S[4] = 0.5 * (g[0][2] + g[2][0]);
  S[5] = 0.5 * (g[1][2] + g[2][1]);
  Smag = tsqrt(2.0 * (S[0] * S[0] + S[1] * S[1] + S[2] * S[2] +
                      2.0 * (S[3] * S[3] + S[4] * S[4] + S[5] * S[5])));
}

// Whether sum q is of this part of k_dyn_terms.
__device__ __forceinline__ bool part_sum(int part, int q) {
  return (q == 0 || q == 2 || q == 6) == (part == 1);
}

constexpr int DT_X = 16, DT_Y = 16, DT_RX = DT_X + 2, DT_RY = DT_Y + 2;
constexpr int DT_BORDER = DT_RX * DT_RY - DT_X * DT_Y;

// PART 0: the strain fields (DF_S .. DF_T) and the terms of u_hat and T_hat
// -> D_I, B, D_d, N_P; PART 1: the products (DF_UU, DF_UT) -> N_I, A, D_P.  One
// pass over all 19 fields needs more than an FP64 wave's 256 registers (78 spilled:
// 0.35 ms on 2.05 M points against 0.17 ms for the two parts, which form the
// resolved strain twice; at three waves per SIMD they spill again, 0.65 ms).
template <typename T, bool PROD, int PART>
__global__ __launch_bounds__(DT_X * DT_Y, 2) void k_dyn_terms(
    const T* __restrict__ Q, const T* __restrict__ M, Grid g, double gamma, int kc, TileMap tm,
    ProdTab pt, const double* __restrict__ SC, double* __restrict__ part) {
  __shared__ double sP[4][DT_RY][DT_RX];       // u, v, w, T of plane kk
  constexpr int F0 = PART == 0 ? DF_S : DF_UU, FN = PART == 0 ? DF_UU - DF_S : DF_N - DF_UU;
  __shared__ double sF[FN][DT_Y][DT_X];        // fields of plane kk filtered along i
  __shared__ double sU[PART == 0 ? 4 : 1][DT_Y][DT_X];   // u_hat, T_hat of plane kk - 1
  const int tx = threadIdx.x, ty = threadIdx.y, tid = ty * DT_X + tx;
  int bx, by, bz;
  if (!tile_of_block(tm, bx, by, bz)) {        // fills up the last XCD's share
    if (tid < DY_NSUM && part_sum(PART, tid)) part[(long long)blockIdx.x * DY_NSUM + tid] = 0.0;
    return;
  }
  const int i0 = bx * (DT_X - 2), j0 = by * (DT_Y - 2);
  const int k0 = bz * kc, k1 = min(k0 + kc, g.nth);
  const int i = i0 - 1 + tx, j = j0 - 1 + ty;
  const bool inner = tx >= 1 && tx <= DT_X - 2 && ty >= 1 && ty <= DT_Y - 2 && i < g.nx && j < g.nr;
  const bool has_b = tid < DT_BORDER;
  int brx = 0, bry = 0;
  if (tid < DT_RX) { bry = 0; brx = tid; }
  else if (tid < 2 * DT_RX) { bry = DT_RY - 1; brx = tid - DT_RX; }
  else { const int r = tid - 2 * DT_RX; bry = 1 + (r >> 1); brx = (r & 1) ? DT_RX - 1 : 0; }
  const unsigned oq = q_col<T>(g, i, j), oob = q_col<T>(g, i0 - 2 + brx, j0 - 2 + bry);
  // filtered state and metrics: columns beyond [-1, n] take the nearest one
  const int ic = min(max(i, -1), g.nx), jc = min(max(j, -1), g.nr);
  const unsigned o64 = q_col<double>(g, ic, jc), om = q_col<T>(g, ic, jc);
  const double* px = PROD ? pt.x + (ic + NG) * PX_N : nullptr;
  const double xx = PROD ? px[0] : 0.0, rx = PROD ? px[1] : 0.0, d2x = PROD ? px[2] : 0.0;
  // metric terms, 1 / J^-1 and (d2) |J^-1|^(2/3) of the column at plane k
  auto metrics = [&](int k, double m[10], double& iV) {
    if (PROD) {      // the stored terms are those of the storage type
      const double* t = pt.yz + (long long)(k + NG) * prod_plane(g) + (jc + NG) * PT_N;
      product_terms(xx, t, m);
      if (sizeof(T) == 8) {
        iV = rx * t[6];
      } else {
#pragma unroll
        for (int c = 0; c < 10; ++c) m[c] = (double)(T)m[c];
        iV = trcp(m[9]);
      }
    } else {
#pragma unroll
      for (int c = 0; c < 10; ++c) m[c] = (double)gld(M, g, c, k, om);
      iV = trcp(m[9]);
    }
  };

  double Pm[4], Pc[5], Pp[5];                  // u, v, w, T at kk-1; rho, u, v, w, T at kk, kk+1
  double uhm[4], uhc[4];                       // u_hat, T_hat at kk-2, kk-1
  double fa[FN], fb[FN];                       // fields at kk-2 and kk-1, filtered in the plane
  double S[6], gT[3];                          // resolved strain, temperature gradient at kk-1
  double acc[DY_NSUM] = {0, 0, 0, 0, 0, 0, 0};
  {
    double q[5], p[5];
    load5(Q, g, oq, k0 - 2, q);
    prim_t(q, gamma, p);
#pragma unroll
    for (int c = 0; c < 4; ++c) Pm[c] = p[1 + c];
    load5(Q, g, oq, k0 - 1, q);
    prim_t(q, gamma, Pc);
    load5(Q, g, oq, k0, q);
    prim_t(q, gamma, Pp);
    if (has_b) {
      double b[5];
      load5(Q, g, oob, k0 - 1, b);
      prim_t(b, gamma, p);
#pragma unroll
      for (int c = 0; c < 4; ++c) sP[c][bry][brx] = p[1 + c];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) { sP[c][ty + 1][tx + 1] = Pc[1 + c]; uhm[c] = uhc[c] = 0.0; }
#pragma unroll
    for (int c = 0; c < FN; ++c) fa[c] = fb[c] = 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) S[c] = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) gT[c] = 0.0;
  }
  __syncthreads();

  for (int kk = k0 - 1; kk <= k1; ++kk) {
    const bool more = kk < k1;
    // gradients at (i, j, kk)
    double Sn[6], gTn[3];
    {
      double dl[3][4], m[10], iV, gu[4][3], Smag;
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        dl[0][f] = sP[f][ty + 1][tx + 2] - sP[f][ty + 1][tx];
        dl[1][f] = sP[f][ty + 2][tx + 1] - sP[f][ty][tx + 1];
        dl[2][f] = Pp[1 + f] - Pm[f];
      }
      metrics(kk, m, iV);
      chain_rule<PROD>(dl, m, 0.5 * iV, gu);
      strain6(gu, Sn, Smag);
      // field f filtered along i
      auto put = [&](int f, double v) {
        sF[f - F0][ty][tx] = filt(from_left<DT_X>(v), v, from_right<DT_X>(v));
      };
      const double rho = Pc[0], rS = rho * Smag;
#pragma unroll
      for (int x = 0; x < 3; ++x) gTn[x] = gu[3][x];
      if constexpr (PART == 0) {
#pragma unroll
        for (int q = 0; q < 6; ++q) put(DF_S + q, rS * Sn[q]);
        put(DF_S2, rS * Smag);
#pragma unroll
        for (int x = 0; x < 3; ++x) put(DF_T + x, rS * gTn[x]);
#pragma unroll
        for (int c = 0; c < 4; ++c) sU[c][ty][tx] = uhc[c];
      } else {
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          const double ru = rho * Pc[1 + x];
          put(DF_UU + x, ru * Pc[1 + x]);
          put(DF_UT + x, ru * Pc[4]);
        }
        put(DF_UU + 3, rho * Pc[1] * Pc[2]);
        put(DF_UU + 4, rho * Pc[1] * Pc[3]);
        put(DF_UU + 5, rho * Pc[2] * Pc[3]);
      }
    }
    // u_hat, T_hat of plane kk, hats of plane kk-1; own column two planes ahead
    // and border of the next plane (kk + 2 <= nth + 1 where used)
    double uhn[4], hn[5], hc[5], qn[5], bn[5];
    if (PART == 0) {
#pragma unroll
      for (int c = 0; c < 5; ++c) hn[c] = gld(SC, g, DY_HR + c, kk, o64);
    }
#pragma unroll
    for (int c = 0; c < (PART == 0 ? 1 : 5); ++c) hc[c] = gld(SC, g, DY_HR + c, max(kk - 1, -1), o64);
    if (more) {
      load5(Q, g, oq, kk + 2, qn);
      if (has_b) load5(Q, g, oob, kk + 1, bn);
    }
    double du[4];   // their differences along i at plane kk-1 (every lane takes part)
    if (PART == 0) {
      const double ihr = trcp(hn[0]);
#pragma unroll
      for (int c = 0; c < 4; ++c) uhn[c] = hn[1 + c] * ihr;
#pragma unroll
      for (int c = 0; c < 4; ++c) du[c] = from_right<DT_X>(uhc[c]) - from_left<DT_X>(uhc[c]);
    }
    __syncthreads();
    const int tym = max(ty - 1, 0), typ = min(ty + 1, DT_Y - 1);
    // field f filtered: along j now, along k with the two planes before
    auto hat = [&](int f) {
      f -= F0;
      const double F2 = filt(sF[f][tym][tx], sF[f][ty][tx], sF[f][typ][tx]);
      const double h = filt(fa[f], fb[f], F2);
      fa[f] = fb[f];
      fb[f] = F2;
      return h;
    };
    // terms of the output point (i, j, kk-1), formed by every thread and added
    // by those that hold one
    const bool emit = inner && kk > k0;
    const double trS = S[0] + S[1] + S[2];
    double m[10], iV;
    metrics(kk - 1, m, iV);
    const double V = m[9];
    if constexpr (PART == 0) {
      double guh[4][3], Sh[6], dl[3][4], Shmag, ShS = 0.0, gTT = 0.0, D2;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        dl[0][c] = du[c];
        dl[1][c] = sU[c][typ][tx] - sU[c][tym][tx];
        dl[2][c] = uhn[c] - uhm[c];
      }
      chain_rule<PROD>(dl, m, 0.5 * iV, guh);
      strain6(guh, Sh, Shmag);
      const double trSh = Sh[0] + Sh[1] + Sh[2];
#pragma unroll
      for (int q = 0; q < 6; ++q) ShS += (q < 3 ? 1.0 : 2.0) * Sh[q] * S[q];
#pragma unroll
      for (int x = 0; x < 3; ++x) gTT += guh[3][x] * gT[x];
      if (PROD && sizeof(T) == 8) {                  // Delta^2 = |J^-1|^(2/3)
        D2 = d2x * pt.yz[(long long)(kk - 1 + NG) * prod_plane(g) + (jc + NG) * PT_N + 7];
      } else {
        const double cV = cbrt(fabs(V));
        D2 = cV * cV;
      }
      const double hrSh = hc[0] * Shmag, Dh2 = 4.0 * D2;
      double hSS = 0.0, hSmm = 0.0, hTT = 0.0;
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        const double h = hat(DF_S + q);
        if (q < 3) hSmm += h;
        hSS += (q < 3 ? 1.0 : 2.0) * h * S[q];       // symmetric: off-diagonals twice
      }
      const double hS2 = hat(DF_S2);
#pragma unroll
      for (int x = 0; x < 3; ++x) hTT += hat(DF_T + x) * gT[x];
      if (emit) {
        acc[1] += V * (2.0 * Dh2 * hrSh * Shmag - 2.0 * D2 * hS2);              // D_I
        acc[3] += V * (trS * 2.0 * D2 * hS2 / 3.0);                             // B
        acc[4] += V * (2.0 * D2 * (hSS - hSmm * trS / 3.0) -
                       2.0 * Dh2 * hrSh * (ShS - trSh * trS / 3.0));            // D_d
        acc[5] += V * (D2 * hTT - Dh2 * hrSh * gTT);                            // N_P
      }
    } else {
      const double i_hr = trcp(hc[0]);
      double Lll = 0.0, LS = 0.0, DP = 0.0;
      constexpr int IA[6] = {0, 1, 2, 0, 0, 1}, IB[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        const double L = hat(DF_UU + q) - hc[1 + IA[q]] * hc[1 + IB[q]] * i_hr;
        if (q < 3) Lll += L;
        LS += (q < 3 ? 1.0 : 2.0) * L * S[q];
      }
#pragma unroll
      for (int x = 0; x < 3; ++x) DP += (hat(DF_UT + x) - hc[1 + x] * hc[4] * i_hr) * gT[x];
      if (emit) {
        acc[0] += V * Lll;                                                      // N_I
        acc[2] += V * (LS - trS * Lll / 3.0);                                   // A
        acc[6] += V * DP;                                                       // D_P
      }
    }
    // roll the window; plane kk+1 goes to LDS
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (PART == 0) { uhm[c] = uhc[c]; uhc[c] = uhn[c]; }
      Pm[c] = Pc[1 + c];
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) S[c] = Sn[c];
#pragma unroll
    for (int c = 0; c < 3; ++c) gT[c] = gTn[c];
#pragma unroll
    for (int c = 0; c < 5; ++c) Pc[c] = Pp[c];
    if (more) {
#pragma unroll
      for (int c = 0; c < 4; ++c) sP[c][ty + 1][tx + 1] = Pc[1 + c];
      prim_t(qn, gamma, Pp);
      if (has_b) {
        double p[5];
        prim_t(bn, gamma, p);
#pragma unroll
        for (int c = 0; c < 4; ++c) sP[c][bry][brx] = p[1 + c];
      }
    }
    __syncthreads();
  }

  double* red = &sF[0][0][0];
  for (int q = 0; q < DY_NSUM; ++q) red[q * DY_BS + tid] = acc[q];
  __syncthreads();
  for (int w = DY_BS / 2; w > 0; w >>= 1) {
    if (tid < w)
      for (int q = 0; q < DY_NSUM; ++q) red[q * DY_BS + tid] += red[q * DY_BS + tid + w];
    __syncthreads();
  }
  if (tid < DY_NSUM && part_sum(PART, tid)) part[(long long)blockIdx.x * DY_NSUM + tid] = red[tid * DY_BS];
}

// dyn[0] = C_ds+ / Cv (eddy-viscosity coefficient in jet-viscosity units),
// dyn[1] = 1 / Pr_sgs used, dyn[2] = (2/3) C_I+, dyn[3..5] = C_I, C_ds,
// Pr_sgs as computed, dyn[6..12] = the seven sums.
__global__ __launch_bounds__(DY_BS) void k_dyn_final(const double* __restrict__ part, int nblk,
                                                     double Cv, double Pr_static,
                                                     double* __restrict__ dyn) {
  __shared__ double red[DY_NSUM][DY_BS];
  double acc[DY_NSUM] = {0, 0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.x; b < nblk; b += DY_BS)
    for (int q = 0; q < DY_NSUM; ++q) acc[q] += part[(long long)b * DY_NSUM + q];
  for (int q = 0; q < DY_NSUM; ++q) red[q][threadIdx.x] = acc[q];
  __syncthreads();
  for (int w = DY_BS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int q = 0; q < DY_NSUM; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  const double N_I = red[0][0], D_I = red[1][0], A = red[2][0], B = red[3][0],
               D_d = red[4][0], N_P = red[5][0], D_P = red[6][0];
  const double C_I = D_I != 0.0 ? N_I / D_I : 0.0;
  const double C_Ip = fmax(C_I, 0.0);
  const double C_ds = D_d != 0.0 ? (A + C_Ip * B) / D_d : 0.0;
  const double C_dsp = fmax(C_ds, 0.0);
  const double Pr = D_P != 0.0 ? C_dsp * N_P / D_P : NAN;
  const double Pr_used = isfinite(Pr) && Pr > 0.0 ? Pr : Pr_static;
  dyn[0] = C_dsp / Cv;
  dyn[1] = 1.0 / Pr_used;
  dyn[2] = (2.0 / 3.0) * C_Ip;
  dyn[3] = C_I;
  dyn[4] = C_ds;
  dyn[5] = Pr;
  for (int q = 0; q < DY_NSUM; ++q) dyn[6 + q] = red[q][0];
}

static int dyn_terms_map(const Grid& g, int num_cu, TileMap& tm) {
  const int gx = (g.nx + DT_X - 3) / (DT_X - 2), gy = (g.nr + DT_Y - 3) / (DT_Y - 2);
  const int kc = dyn_chunk((long long)gx * gy, g.nth, 2 * num_cu, 3);
  tm = tile_map(gx, gy, (g.nth + kc - 1) / kc);
  return kc;
}

int dyn_blocks(const Grid& g, int num_cu) {
  TileMap tm;
  dyn_terms_map(g, num_cu, tm);
  return tm.per_xcd * NXCD;
}

template <typename T>
hipError_t launch_dynamic(const T* Q, const T* M, const Grid& g, double gamma, double Cv,
                          double Pr_static, double* SC, double* part, double* dyn, int num_cu,
                          const ProdTab& pt, hipStream_t s) {
  {
    const int gx = (g.nx + 2 + DH_X - 3) / (DH_X - 2), gy = (g.nr + 2 + DH_Y - 1) / DH_Y;
    const int kc = dyn_chunk((long long)gx * gy, g.nth + 2, 8 * num_cu, 3);
    const TileMap tm = tile_map(gx, gy, (g.nth + 2 + kc - 1) / kc);
    hipLaunchKernelGGL(k_dyn_hat<T>, dim3(tm.per_xcd * NXCD), dim3(DH_X, DH_Y), 0, s, Q, g, gamma, kc,
                       tm, SC);
  }
  TileMap tm;
  const int kc = dyn_terms_map(g, num_cu, tm);
  const int nb = tm.per_xcd * NXCD;
#define LESJET_DYN_TERMS(P, PART)                                                               \
  hipLaunchKernelGGL((k_dyn_terms<T, P, PART>), dim3(nb), dim3(DT_X, DT_Y), 0, s, Q, M, g, gamma, \
                     kc, tm, pt, (const double*)SC, part)
  if (pt.x) {
    LESJET_DYN_TERMS(true, 0);
    LESJET_DYN_TERMS(true, 1);
  } else {
    LESJET_DYN_TERMS(false, 0);
    LESJET_DYN_TERMS(false, 1);
  }
#undef LESJET_DYN_TERMS
  hipLaunchKernelGGL(k_dyn_final, dim3(1), dim3(DY_BS), 0, s, (const double*)part, nb, Cv,
                     Pr_static, dyn);
  return hipGetLastError();
}

template hipError_t launch_dynamic<double>(const double*, const double*, const Grid&, double,
                                           double, double, double*, double*, double*, int,
                                           const ProdTab&, hipStream_t);
template hipError_t launch_dynamic<float>(const float*, const float*, const Grid&, double, double,
                                          double, double*, double*, double*, int, const ProdTab&,
                                          hipStream_t);

}  // namespace lesjet
