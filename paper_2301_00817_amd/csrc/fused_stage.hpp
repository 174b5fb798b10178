// Fused residual / Runge-Kutta stage kernel (section "Spatial
// Discretization" with the stage update of eq. localdt as an epilogue).
//
// Work decomposition (2.5-D): a block of Tile::X x Tile::Y threads
// owns a ring-1 tile of (i, j) columns and marches along k over a chunk of
// planes.  For each plane kk it
//   (a) writes the state and primitives of the plane (ring-2 tile, two-point
//       halo for the fourth differences) to LDS,
//   (b) computes the point quantities G^d, lambda_bar^d, nu^d of every
//       ring-1 column, with in-plane neighbours from LDS and the kk-1, kk+1
//       neighbours from the thread's own registers, and publishes the eta
//       ones in LDS (the xi ones go to the neighbouring lane),
//   (c) evaluates the in-plane faces i - 1/2 and j - 1/2 of each column and
//       publishes the eta fluxes; after a barrier each interior column
//       takes its flux differences and forms the zeta face kk-1/2
//       from registers (point quantities of plane kk-1 are kept from the
//       previous iteration), which completes R at plane kk-1.
// Every point quantity of a ring-1 column is computed once per plane, every
// face flux once.  HBM traffic per interior point and stage: Q (in), the 10
// metric arrays (none on a product mesh), Q^(0) and the output, the halos
// coming from L2.
//
// Epilogues: EPI_R writes R; EPI_RK writes Q^(l) = Q^(0) - alpha dt R
// (accumulated in FP64, stored in the stage type); EPI_RK_LAST also writes
// Q^(n+1) in FP64 and reduces max(lambda_xi + lambda_eta + lambda_zeta) of
// the new state for the next step's dt.
#pragma once

#include "launch.hpp"
#include "physics.hpp"
#include "tiles.hpp"

namespace lesjet {

// Tile shapes (threads along i and j of a ring-1 tile): FP64 16 x 16 (LDS 57
// KB, two blocks per CU) or, WIDE, 32 x 16 (LDS 107 KB, one block of eight
// waves), FP32 32 x 8 (LDS 29 KB, four blocks per CU) or, WIDE, 32 x 16 (55
// KB, two blocks).  In FP64 the wide tile computes
// 512 ring-1 columns for 420 outputs, the narrow one 256 for 196 (7 % more):
// 21.3 against 23.4 ms a step on 102 M points, 440 against 495 us a residual
// of a 200^3 curvilinear mesh (while the xi faces went through LDS the two were
// within 1 %).  fused_plan picks the tile that a mesh's extents waste less of.
template <typename T, bool WIDE> struct Tile;
template <> struct Tile<double, false> { static constexpr int X = 16, Y = 16, PER_CU = 2; };
template <> struct Tile<double, true> { static constexpr int X = 32, Y = 16, PER_CU = 1; };
template <> struct Tile<float, false> { static constexpr int X = 32, Y = 8, PER_CU = 4; };
template <> struct Tile<float, true> { static constexpr int X = 32, Y = 16, PER_CU = 2; };

constexpr int NPQ = 8;                // G(5), lambda_bar, nu, V per direction

enum { EPI_R = 0, EPI_RK = 1, EPI_RK_LAST = 2 };

// Global memory is addressed plane by plane (plane_io.hpp): one 32-bit
// offset register per column serves every variable and plane of the march.

template <typename T>
__device__ __forceinline__ void load_q(const T* Q, const Grid& g, unsigned col, int k, T q[5]) {
#pragma unroll
  for (int c = 0; c < 5; ++c) q[c] = gld(Q, g, c, k, col);
}

template <typename T>
__device__ __forceinline__ void load_metrics(const T* M, const Grid& g, unsigned col, int k,
                                             T m[10]) {
#pragma unroll
  for (int c = 0; c < 10; ++c) m[c] = gld(M, g, c, k, col);
}

// s_waitcnt operand: no vector memory access outstanding (LDS and scalar
// counters not waited for).  The compiler places its waits for the fewest
// accesses issued on any path; the loads of the march sit in branches, so a
// wait of its own for an older load also drains every newer one.  Waiting
// where nothing young is in flight (before the march, and ahead of the
// epilogue's stores) clears its record: the loads at the top of an iteration
// then stay in flight through the point phase, and no load is waited for
// behind a store.  8 % of the FP64 step with held viscosities on 1.0 M points,
// 3-4 % of the steps on 102 M (FP64) and 23.6 M points (FP32).
constexpr int WAIT_VMEM = 0x0F70;

// On product meshes the FP64 kernel has registers left at two waves per SIMD: it
// loads Q^(0) of the output point an iteration ahead (FP32 at 128 VGPRs does not;
// nor do general meshes, whose registers hold two planes of metric terms: with it
// their stages spilled four to eight VGPRs, a step of a 200^3 curvilinear mesh took
// 2.79 against 2.70 ms, of 95^3 401 against 388 us).
template <typename T> struct PrefetchQ0 { static constexpr bool on = sizeof(T) == 8; };

// The last stage of a step evaluates the next step's CFL sum at its output
// point, which needs that point's metric terms, loaded two planes earlier
// and no longer in L2 (reloading them cost the FP64 kernel 10 ms, a sixth
// of the stage, on 1e9 points).  On a product mesh they come from the table
// rows in LDS; else the stage carries them from the previous plane in
// registers: FP64 frees the registers by loading Q^(0) and the next plane's
// border where they are used rather than ahead; FP32 runs that stage at three
// waves per SIMD (at four it spills; product meshes fit four, 1 % faster).

// Wave priority: the FP64 kernel (two waves per SIMD, bound by latency)
// raises its waves' issue priority from the face phase to the end of the
// epilogue, so that a wave that has its plane in LDS finishes the plane and
// reaches the next plane's loads ahead of the waves still in the point
// phase.  Measured on MI355X: 10 % less time per launch on the 5.9 M-point
// jet (one round of blocks, two per CU for the whole launch), about 2 % on
// meshes of 0.1 to 1 billion points; the FP32 kernel, bound by its ALUs,
// gains nothing from it.
template <typename T> struct WavePrio { static constexpr bool on = sizeof(T) == 8; };

// Register budget: FP64 two waves per SIMD (up to 256 VGPRs), FP32 four
// (128), three (168) in the last stage of general meshes.  The FP32 last stage of a
// product mesh spills one VGPR with held viscosities and up to four with the dynamic
// model, and is still 2-4 % of a step faster than at three waves (256 x 256 x 360,
// held: 4.28 against 4.36 ms).
template <typename T> struct FusedOcc;
template <> struct FusedOcc<double> { static constexpr int waves = 2; };
template <> struct FusedOcc<float> { static constexpr int waves = 4; };
template <typename T, int EPI, bool PROD> struct FusedOccE { static constexpr int waves = FusedOcc<T>::waves; };
template <> struct FusedOccE<float, EPI_RK_LAST, false> { static constexpr int waves = 3; };

// AXIS: the eta- face is a centerline through mesh nodes (row j = 0 on the
// axis); a separate instance so that the common case carries none of it.
// LAG: viscosity schedule (LAG_NONE; LAG_WRITE also stores mu + mu_sgs and
// the conductivity of every point the block evaluates into `visc`, two
// padded variables; LAG_READ takes them from there).  The tiling is the same
// in every stage, so the points read are those written; points shared by
// two blocks are written twice with the same value.
// PROD: product mesh.  The ten metric terms, the reciprocal of J^-1, the lengths
// of the area vectors and the filter width are formed from tables (eight FP64
// values per (j, k), staged in LDS once per plane and tile row by threads that
// hold no border point, three per i), which spares 80 of the 200 bytes per
// point and stage (FP32: 40 of 128), the registers of two planes of metric
// terms, and the arithmetic on the four terms that are zero.  The terms are bitwise those
// stored, the derived values within two ulps of those computed from them.  The same
// meshes with the terms read against the tables: a step of 102 M points 31.5 / 21.2
// ms, two of 5.9 M 3.71 / 2.66 ms, FP32 on 23.6 M 5.59 / 4.00 ms.  The derived values
// (FP64 only: the FP32 hardware reciprocal, root and logarithm cost no more than
// the products) spare a reciprocal, two roots and a cube root of the 850 vector
// operations per point and plane: 4 % of that (22.1 and 2.75 ms without them).
template <typename T, bool WIDE, int EPI, bool AXIS, int LAG, bool DYN, bool PROD>
__global__ void __launch_bounds__((Tile<T, WIDE>::X * Tile<T, WIDE>::Y), (FusedOccE<T, EPI, PROD>::waves))
k_fused(const T* __restrict__ Qin, const T* __restrict__ M, Grid g, Phys<T> ph_arg, int kc,
        TileMap tm, T* out, const double* Q0, double* Q64, double alpha,
        const double* __restrict__ dtp, Phys<double> ph64, unsigned long long* __restrict__ maxbits,
        T* __restrict__ visc, const double* __restrict__ dyn, ProdTab ptab) {
  Phys<T> ph = ph_arg;
  if (DYN) {   // dynamic model: coefficients of this state, from the device
    ph.sgs_coef = (T)dyn[0];
    ph.Prs_inv = (T)dyn[1];
    ph.iso_coef = (T)dyn[2];
  }
  constexpr int FB_X = Tile<T, WIDE>::X;        // threads along i (ring-1 columns)
  constexpr int FB_Y = Tile<T, WIDE>::Y;        // threads along j
  constexpr int FT_X = FB_X - 2;                // interior outputs along i
  constexpr int FT_Y = FB_Y - 2;                // interior outputs along j
  constexpr int FR_X = FB_X + 2;                // ring-2 tile
  constexpr int FR_Y = FB_Y + 2;
  constexpr int NBORDER = FR_X * FR_Y - FB_X * FB_Y;   // ring-2 points without a thread
  // plane state and primitives (one buffer: a second would save a barrier
  // per plane but costs a resident block per CU in either precision)
  __shared__ T sQ[5][FR_Y][FR_X];     // W = (rho, rho u, rho v, rho w, E + p)
  __shared__ T sP[5][FR_Y][FR_X];
  __shared__ T sE[NPQ][FB_Y][FB_X];
  // fluxes of the faces i - 1/2 (xi) and j - 1/2 (eta) of each column: each
  // in-plane face is evaluated once, by the column on its + side, and used
  // by both neighbours (evaluating it from both sides cost 11-14 % more time
  // in FP64 and the registers of a fourth FP32 block per CU).  Point
  // quantities and fluxes cross the xi faces by lane moves, the eta faces
  // through LDS: LDS was busy 45 % of the FP64 kernel's time when it carried
  // both (and the thread's own values back to it), a moved double costs two
  // vector moves on one of the four SIMDs against eight cycles of the CU's
  // LDS.  When the xi faces left it: LDS 6.2 -> 3.5 M cycles per CU and launch on
  // 102 M points, the stage 8 % shorter, a residual of a 95^3 mesh 8 %, an FP32
  // step on 23.6 M points 6 %.
  __shared__ T sFe[5][FB_Y][FB_X];
  __shared__ double sRed[(FB_X * FB_Y + 63) / 64];
  // product mesh: table rows of the planes kk-1 .. kk+1 (slot = plane mod 4)
  __shared__ __align__(16) double sM[PROD ? 4 : 1][FB_Y][PT_N];

  const int tx = threadIdx.x, ty = threadIdx.y;
  const int tid = ty * FB_X + tx;
  int bx, by, bz;
  if (!tile_of_block(tm, bx, by, bz)) return;         // uniform for the block
  const int i0 = bx * FT_X, j0 = by * FT_Y;
  const int k0 = bz * kc;
  const int k1 = min(k0 + kc, g.nth);
  const int i = i0 - 1 + tx, j = j0 - 1 + ty;
  const bool col_ok = i >= -1 && i <= g.nx && j >= -1 && j <= g.nr;   // needed ring-1 column
  const bool interior = tx >= 1 && tx <= FT_X && ty >= 1 && ty <= FT_Y && i < g.nx && j < g.nr;
  // columns that evaluate their xi face i - 1/2 / eta face j - 1/2
  const bool xface = tx >= 1 && ty >= 1 && ty <= FT_Y && i <= g.nx && j < g.nr;
  const bool eface = ty >= 1 && tx >= 1 && tx <= FT_X && j <= g.nr && i < g.nx;

  // ring-2 border point handled by this thread (if tid < NBORDER)
  const bool has_b = tid < NBORDER;
  int brx = 0, bry = 0;
  if (tid < FR_X) { bry = 0; brx = tid; }
  else if (tid < 2 * FR_X) { bry = FR_Y - 1; brx = tid - FR_X; }
  else { const int r = tid - 2 * FR_X; bry = 1 + (r >> 1); brx = (r & 1) ? FR_X - 1 : 0; }
  const int bi = i0 - 2 + brx, bj = j0 - 2 + bry;
  // Byte offsets within a plane of the own column and of the border point.
  // Every column that produces or feeds an output lies in the padded box,
  // where the clamp is the identity, so oq is also the offset of the output
  // point; the columns beyond [-1, n] read metrics and held viscosities of
  // ghost columns, whose point quantities no face uses.  oq64: the same
  // column in the FP64 arrays (Q^(0), Q^(n+1)).
  const unsigned oq = q_col<T>(g, i, j), oob = q_col<T>(g, bi, bj);
  const unsigned oq64 = sizeof(T) == 8 ? oq : 2u * oq;

  const bool axis_row = AXIS && j == 0;      // centerline row (not advanced)
  const bool axis_face = AXIS && j == 1;     // face j - 1/2 is the axis face
  // physical-boundary faces i - 1/2 and j - 1/2 of this column (the face
  // i - 1/2 of column i = nx is the face nx - 1/2)
  const bool phys_xf = (i == 0 && ph.phys_face[0][0]) || (i == g.nx && ph.phys_face[0][1]);
  const bool phys_ef = (j == 0 && ph.phys_face[1][0]) || (j == g.nr && ph.phys_face[1][1]);

  // ---- rolling column state ------------------------------------------------
  // The state and primitives of the current plane kk live in LDS once phase
  // (a) has written them; registers carry only what the march needs next.
  T Wa[5], Wb[5];        // W at kk-2, kk-1 (zeta fourth difference)
  T Qd[5], Pd[5];        // W and (u, v, w, T, p) at kk+1
  T Pb[5];               // (u, v, w, T, p) at kk-1
  T Qn[5];               // Q at kk+2, in flight
  T met[10], metn[10];   // general mesh: metrics at (i, j, kk), prefetch for kk+1
  T lag[2], lagn[2];     // held (mu + mu_sgs, conductivity), same planes (LAG_READ)
  // the last stage of a general mesh carries the metric terms of plane kk-1 (Sp)
  // and gives up the border loads ahead for them (and still spills 4 VGPRs, 9 with
  // held viscosities); a product mesh has the terms in LDS and keeps the loads (the
  // last stage of 5.9 M points 311 -> 280 us)
  constexpr bool CS = EPI == EPI_RK_LAST && !PROD;
  constexpr bool DEFER = CS && sizeof(T) == 8;    // loads deferred to free registers
  constexpr bool PQ0 = EPI != EPI_R && PROD && PrefetchQ0<T>::on;
  // the own column two planes ahead is loaded after the point phase in FP64
  // (2-4 % faster than at the top of the iteration; with held viscosities
  // 2 % slower) and on general FP32 meshes, at the top otherwise (FP32
  // product meshes: 2 % faster)
  constexpr bool LATE_QN = sizeof(T) == 8 ? LAG == LAG_NONE || CS : !PROD;
  // general FP32 meshes: the metric terms of the next plane are loaded after the
  // point phase too where the registers of the early loads would spill (a stage,
  // two to nine VGPRs: a step of 128^3 598 -> 590 us, with held viscosities 650 ->
  // 633; a dynamic residual, four: 297 -> 291 us); a residual, which does not spill,
  // keeps them early (200^3: 252 against 257 us)
  constexpr bool LATE_MET = !PROD && sizeof(T) == 4 && (EPI == EPI_RK || (EPI == EPI_R && DYN));
  double q0p[5];         // Q^(0) at (i, j, kk-1), loaded at the top of iteration kk
  const double ad_pre = PQ0 ? alpha * (*dtp) : 0.0;
  auto load_lag = [&](int kk, T v[2]) {
    // columns beyond [-1, n] lie among the ghosts, where stage 1 writes nothing
    // (it writes [-1, n]^3): what they read is not defined, and no face uses it
    v[0] = gld(visc, g, 0, kk, oq);
    v[1] = gld(visc, g, 1, kk, oq);
  };
  // zeta-face state of plane kk-1 (interior columns)
  T Gz[5], lbz = 0, nuz = 0, Vz = 0, hiVz = 0;   // hiVz = 1 / (2 Vz)
  T acc[5];              // twice the RHS at kk-1 without its zeta face kk-1/2:
                         // in-plane faces minus the zeta face kk-3/2
  double lmax = 0.0;
  T Sp[9];               // the same, last stage: metric terms of plane kk-1
  // product mesh: the column's values of the x table; the table value this
  // thread stages (columns and rows beyond the padded box take the nearest
  // point's, as for the state)
  constexpr int TAB0 = 128;
  static_assert(NBORDER <= TAB0 && TAB0 + FB_Y * PT_N <= FB_X * FB_Y, "threads of the table rows");
  double xx = 0, rx = 0, d2x = 0, mt = 0;
  const int tr = (tid - TAB0) / PT_N, tc = (tid - TAB0) % PT_N;
  const bool has_t = PROD && tid >= TAB0 && tr < FB_Y;
  const int trow = (min(max(j0 - 1 + tr, -NG), g.nr + NG - 1) + NG) * PT_N + tc;
  auto tab = [&](int k) { return ptab.yz[(long long)(k + NG) * prod_plane(g) + trow]; };
  if (PROD) {
    const double* px = ptab.x + (min(max(i, -NG), g.nx + NG - 1) + NG) * PX_N;
    xx = px[0];
    rx = px[1];
    d2x = px[2];
    if (has_t) sM[0][tr][tc] = tab(k0 - 1);
  }

  {
    T q[5], pc[5];
    load_q(Qin, g, oq, k0 - 2, q);
    prim5(q, ph, Pb);                    // primitives at kk-1 = k0-2
#pragma unroll
    for (int c = 0; c < 5; ++c) Wa[c] = q[c];
    Wa[4] += Pb[4];
    load_q(Qin, g, oq, k0 - 1, q);       // plane kk = k0-1 of the own column
    prim5(q, ph, pc);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      sQ[c][ty + 1][tx + 1] = c == 4 ? radd(q[c], pc[c]) : q[c];
      sP[c][ty + 1][tx + 1] = pc[c];
    }
    load_q(Qin, g, oq, k0, Qd);
    prim5(Qd, ph, Pd);
    Qd[4] = radd(Qd[4], Pd[4]);
    if (!PROD) load_metrics(M, g, oq, k0 - 1, met);
    if (LAG == LAG_READ) load_lag(k0 - 1, lag);
  }
#pragma unroll
  for (int c = 0; c < 5; ++c) { Wb[c] = Wa[c]; Gz[c] = 0; acc[c] = 0; }

  if (has_b) {                           // border of the first plane
    T bq[5], bp[5];
    load_q(Qin, g, oob, k0 - 1, bq);
    prim5(bq, ph, bp);
    bq[4] = radd(bq[4], bp[4]);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      sQ[c][bry][brx] = bq[c];
      sP[c][bry][brx] = bp[c];
    }
  }

  __builtin_amdgcn_s_waitcnt(WAIT_VMEM);
  for (int kk = k0 - 1, slot = 0; kk <= k1; ++kk, slot = (slot + 1) & 3) {
    const bool more = kk < k1;
    // metric loads of the next plane (and, early, the own column two planes
    // ahead), in flight during (b)
    if (more) {
      if (!LATE_QN && kk + 2 <= k1 + 1) load_q(Qin, g, oq, kk + 2, Qn);
      if (!PROD && !LATE_MET) load_metrics(M, g, oq, kk + 1, metn);
      else if (has_t) mt = tab(kk + 1);
      if (LAG == LAG_READ) load_lag(kk + 1, lagn);
    }
    if (PQ0 && interior && kk - 1 >= k0) {
#pragma unroll
      for (int c = 0; c < 5; ++c) q0p[c] = gld(Q0, g, c, kk - 1, oq64);
    }
    // (a) plane kk is in LDS (written before the loop or at the end of the
    // previous iteration)
    __syncthreads();

    // (b) point quantities at (i, j, kk)
    PointIn<T> in;
    PointOut<T> po;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      in.q[c] = sQ[c][ty + 1][tx + 1];
      in.pr[c] = sP[c][ty + 1][tx + 1];
    }
    {
      T m[5], pl[5];
#pragma unroll
      for (int f = 0; f < 5; ++f) { m[f] = sP[f][ty + 1][tx]; pl[f] = sP[f][ty + 1][tx + 2]; }
      neighbour_terms<true>(m, pl, in.pr[4], in.dl[0], in.nu[0]);
#pragma unroll
      for (int f = 0; f < 5; ++f) { m[f] = sP[f][ty][tx + 1]; pl[f] = sP[f][ty + 2][tx + 1]; }
      neighbour_terms<true>(m, pl, in.pr[4], in.dl[1], in.nu[1]);
      neighbour_terms<true>(Pb, Pd, in.pr[4], in.dl[2], in.nu[2]);
    }
    {
      T m[10];
      if constexpr (PROD) {
        double w[10];
        const double* t = sM[slot][ty];
        product_terms(xx, t, w);
#pragma unroll
        for (int c = 0; c < 10; ++c) m[c] = (T)w[c];
        if (sizeof(T) == 8) {      // in FP32 the hardware functions cost no more
          in.iV = rx * t[6];
          in.len[0] = tabs(m[0]);
          in.len[1] = fabs(xx) * t[4];
          in.len[2] = fabs(xx) * t[5];
          in.d2 = d2x * t[7];
        }
      } else {
#pragma unroll
        for (int c = 0; c < 10; ++c) m[c] = met[c];
      }
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int c = 0; c < 3; ++c) in.S[d][c] = m[3 * d + c];
      in.V = m[9];
    }
    if (LAG == LAG_READ) { in.mt = lag[0]; in.kap = lag[1]; }
    point_quantities<T, LAG, DYN, PROD, true>(in, ph, po);
    if (LAG == LAG_WRITE && col_ok && ph.viscous) {
      gst(visc, g, 0, kk, oq, po.mt);
      gst(visc, g, 1, kk, oq, po.kap);
    }
    if (AXIS && axis_row) {
      // centerline through the nodes: S^eta = 0 on the axis, so the eta
      // point flux vanishes (its viscous part, singular at V = 0, is not used)
#pragma unroll
      for (int c = 0; c < 5; ++c) po.G[1][c] = T(0);
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) sE[c][ty][tx] = po.G[1][c];
    sE[5][ty][tx] = po.lb[1];
    sE[6][ty][tx] = po.nu[1];
    sE[7][ty][tx] = in.V;
    // border of the next plane, in flight during the face phase
    T Bn[5];
    if (!DEFER && more && has_b) load_q(Qin, g, oob, kk + 1, Bn);
    if (LATE_MET && more) load_metrics(M, g, oq, kk + 1, metn);
    if (LATE_QN && more && kk + 2 <= k1 + 1) load_q(Qin, g, oq, kk + 2, Qn);
    __syncthreads();

    // (c) faces
    if (WavePrio<T>::on) __builtin_amdgcn_s_setprio(1);
    auto wload = [&](int yy, int xx, T w[5]) {
#pragma unroll
      for (int c = 0; c < 5; ++c) w[c] = sQ[c][yy][xx];
    };
    const T (&Wc)[5] = in.q;                        // W of the point itself
    // In-plane faces of the output planes, one per column and direction.
    // Threads without a face keep values that no output uses: the point
    // fluxes, whose registers the face fluxes take over (zeros would be
    // moved in for every plane).  rhs: flux differences (of doubled fluxes),
    // the eta face j + 1/2 added after the barrier.
    T rhs[5], Fe[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) { rhs[c] = po.G[0][c]; Fe[c] = po.G[1][c]; }
    const bool planes = kk >= k0 && kk < k1;
    if (planes) {
      T Wm[5], Wl[5], Wp[5], GA[5], (&F)[5] = rhs;
#pragma unroll
      for (int c = 0; c < 5; ++c) GA[c] = from_left<FB_X>(po.G[0][c]);
      const T lbA = from_left<FB_X>(po.lb[0]), nuA = from_left<FB_X>(po.nu[0]),
              VA = from_left<FB_X>(in.V);
      if (xface) {
        wload(ty + 1, tx - 1, Wm); wload(ty + 1, tx, Wl); wload(ty + 1, tx + 2, Wp);
        face_flux2(GA, po.G[0], lbA, po.lb[0], nuA, po.nu[0], VA, in.V, Wm, Wl, Wc, Wp, phys_xf, ph,
                   F);
      }
#pragma unroll
      for (int c = 0; c < 5; ++c) rhs[c] = from_right<FB_X>(F[c]) - F[c];
      if (eface) {
        // axis face: lambda_bar of row 1 and the three-point fourth
        // difference W(2) - 4 W(1) + 3 W(0), i.e. the standard formula with
        // W(-1) replaced by W(1); done by choosing the rows read
        const int rm = AXIS && axis_face ? ty + 1 : ty - 1;
        wload(rm, tx + 1, Wm); wload(ty, tx + 1, Wl); wload(ty + 2, tx + 1, Wp);
#pragma unroll
        for (int c = 0; c < 5; ++c) GA[c] = sE[c][ty - 1][tx];
        const T lbE = AXIS && axis_face ? po.lb[1] : sE[5][ty - 1][tx];
        face_flux2(GA, po.G[1], lbE, po.lb[1], sE[6][ty - 1][tx], po.nu[1], sE[7][ty - 1][tx], in.V,
                   Wm, Wl, Wc, Wp, phys_ef, ph, Fe);
#pragma unroll
        for (int c = 0; c < 5; ++c) sFe[c][ty][tx] = Fe[c];
      }
    }
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(WAIT_VMEM);
    if (interior && kk >= k0) {
      const bool emit = kk - 1 >= k0;       // R at (i, j, kk-1) completes here
      // zeta face kk-1/2: L = kk-1 (registers), R = kk
      T Fk[5];
      face_flux2(Gz, po.G[2], lbz, po.lb[2], nuz, po.nu[2], Vz, in.V, Wa, Wb, Wc, Qd, false, ph, Fk);
      if (emit) {
        // the epilogue's loads ahead of its stores (the compiler cannot order
        // buffer accesses of different arrays by itself): Q^(0) of the output
        // point (loaded an iteration ahead where registers allow) and, at the
        // last stage, its metric terms for the next step's dt (carried in
        // registers from the previous plane)
        double q0[5], S[3][3];
        if (EPI != EPI_R) {
#pragma unroll
          for (int c = 0; c < 5; ++c) q0[c] = PQ0 ? q0p[c] : gld(Q0, g, c, kk - 1, oq64);
        }
        if (EPI == EPI_RK_LAST) {
          double w[10];
          if constexpr (PROD) product_terms(xx, sM[(slot + 3) & 3][ty], w);
#pragma unroll
          for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int c = 0; c < 3; ++c)
              S[d][c] = PROD ? (double)(T)w[3 * d + c] : (double)Sp[3 * d + c];
        }
        // (general FP64 instances have no registers left to carry it)
        const T hiV = PROD || sizeof(T) == 4 ? hiVz : T(0.5) * trcp(Vz);
        T R[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) R[c] = AXIS && axis_row ? T(0) : (acc[c] + Fk[c]) * hiV;
        if (EPI == EPI_R) {
#pragma unroll
          for (int c = 0; c < 5; ++c) gst(out, g, c, kk - 1, oq, R[c]);
        } else {
          const double ad = PQ0 ? ad_pre : alpha * (*dtp);
          double qn[5];
#pragma unroll
          for (int c = 0; c < 5; ++c) {
            qn[c] = q0[c] - ad * (double)R[c];
            gst(out, g, c, kk - 1, oq, (T)qn[c]);
            if (EPI == EPI_RK_LAST && Q64) gst(Q64, g, c, kk - 1, oq64, qn[c]);
          }
          if (EPI == EPI_RK_LAST) {
            const double x = lambda_sum<PROD>(qn, S, (double)Vz, ph64);
            if (!(AXIS && axis_row) && (x != x || x > lmax)) lmax = x;
          }
        }
      }
      if (planes) {
#pragma unroll
        for (int c = 0; c < 5; ++c) acc[c] = rhs[c] + sFe[c][ty + 1][tx] - Fe[c] - Fk[c];
      }
    }
    if (WavePrio<T>::on) __builtin_amdgcn_s_setprio(0);
    // keep the zeta-direction point quantities of plane kk, roll the window
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      Gz[c] = po.G[2][c];
      Wa[c] = Wb[c];
      Wb[c] = Wc[c];
      Pb[c] = sP[c][ty + 1][tx + 1];     // re-read from LDS
    }
    lbz = po.lb[2];
    nuz = po.nu[2];
    Vz = in.V;
    hiVz = po.hiV;
    // plane kk is read by other threads until the barrier after the face
    // fluxes; what follows reads only the thread's own column, which the
    // next plane's border writes never touch
    if (more) {
      // plane kk+1 goes to LDS: own column and ring-2 border
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        sQ[c][ty + 1][tx + 1] = Qd[c];
        sP[c][ty + 1][tx + 1] = Pd[c];
        Qd[c] = Qn[c];
      }
      if (has_b) {
        if (DEFER) load_q(Qin, g, oob, kk + 1, Bn);
        T bp[5];
        prim5(Bn, ph, bp);
        Bn[4] = radd(Bn[4], bp[4]);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          sQ[c][bry][brx] = Bn[c];
          sP[c][bry][brx] = bp[c];
        }
      }
      prim5(Qd, ph, Pd);
      Qd[4] = radd(Qd[4], Pd[4]);
      if (PROD) {
        if (has_t) sM[(slot + 1) & 3][tr][tc] = mt;
      } else {
        if (CS) {
#pragma unroll
          for (int c = 0; c < 9; ++c) Sp[c] = met[c];
        }
#pragma unroll
        for (int c = 0; c < 10; ++c) met[c] = metn[c];
      }
      if (LAG == LAG_READ) { lag[0] = lagn[0]; lag[1] = lagn[1]; }
    }
  }

  if (EPI == EPI_RK_LAST) {
    // block max of the lambda sums, then one integer atomic per block
    double v = lmax;
    for (int off = 32; off > 0; off >>= 1) {
      const double o = __shfl_xor(v, off, 64);
      if (o != o || o > v) v = o;
    }
    if ((tid & 63) == 0) sRed[tid >> 6] = v;
    __syncthreads();
    if (tid == 0) {
      double b = sRed[0];
      for (int w = 1; w < (FB_X * FB_Y + 63) / 64; ++w)
        if (sRed[w] != sRed[w] || sRed[w] > b) b = sRed[w];
      atomicMax(maxbits, (unsigned long long)__double_as_longlong(b));
    }
  }
}

// Chunk length that minimises (rounds of resident blocks) x (planes per block),
// over every length up to the cap (a mesh that fits one round takes the
// shortest chunks that still do: 32^3, single planes, three iterations per
// block, 15.8 us a residual on the narrow tile against 20.1 us with four; FP32 keeps at least
// four, as its states depend on the chunk length by up to 6e-8, the rounding of
// a chunk's first planes in its prologue; lengths that divide the azimuth
// leave no short last chunk: against powers of two only, 5.6 % on the 128 x
// 128 x 360 mesh and 3.1 % on 1700 x 1700 x 360 in FP64, 1.4-1.6 % in FP32,
// 0.5 % on 1250 x 640 x 1250).
// FP32 (four waves per SIMD; the last stage, at three on general meshes, takes
// the same length) stops at 16 planes: longer chunks measured slower on large
// meshes (4 % at 1e8 points, 8 % at 1e9), the resident blocks of a round
// drifting apart in k and sharing fewer halo lines in L2.  FP64 takes 64 planes
// when that fits one round (the 5.9 M-point mesh: 4 % faster than 32) and at
// most 32 otherwise: the same time within 1 % on 1e8 and 1e9 points, with 12 %
// (32) to 21 % (16) fewer bytes crossing the L2 boundary than with 64.
template <typename T, bool WIDE>
FusedPlan tile_plan(const Grid& g, int num_cu, double* cost_out) {
  using TL = Tile<T, WIDE>;
  const long long tiles = (long long)((g.nx + TL::X - 3) / (TL::X - 2)) *
                          ((g.nr + TL::Y - 3) / (TL::Y - 2));
  const long long resident = (long long)num_cu * TL::PER_CU;
  FusedPlan best = {g.nth, WIDE};
  long long best_blocks = 0;
  const auto choose = [&](int kc_max) {
    *cost_out = 1e300;
    for (int kc = sizeof(T) == 8 ? 1 : 4; kc <= kc_max; ++kc) {
      const long long nb = tiles * ((g.nth + kc - 1) / kc);
      const double cost = (double)((nb + resident - 1) / resident) * (kc + 2);
      if (cost < *cost_out) { *cost_out = cost; best.kc = kc; best_blocks = nb; }
    }
  };
  if (sizeof(T) == 4) {
    choose(16);
    return best;
  }
  choose(64);
  if (best_blocks > resident) choose(32);
  // four waves alone on a CU take a plane in about 0.8 of the time of eight (12
  // meshes of 9^3 to 60 x 14 x 14 whose narrow blocks are each alone on a CU: a step
  // 6-11 % shorter with the narrow tile on every one, at equal rounds and planes;
  // eight of 32^3 to 48^3 with 288 to 384 narrow blocks: 0.5-4 % longer)
  if (!WIDE && best_blocks <= num_cu) *cost_out *= 0.8;
  return best;
}

template <typename T, bool WIDE>
hipError_t launch_fused_tile(const T* Q, const T* M, const Grid& g, const Phys<T>& ph, int kc, int epi,
                        T* out, const double* Q0, double* Q64, double alpha, const double* dt,
                        const Phys<double>& ph64, unsigned long long* maxbits, int lag, T* visc,
                        const double* dyn, const ProdTab& pt, hipStream_t s) {
  if (ph.sgs == 3 && !dyn) return hipErrorInvalidValue;
  // instances: LAG_NONE with every epilogue, LAG_WRITE with EPI_RK (stage 1),
  // LAG_READ with EPI_RK and EPI_RK_LAST (stages 2-5)
  if (lag != LAG_NONE && (!visc || epi == EPI_R || (lag == LAG_WRITE && epi != EPI_RK)))
    return hipErrorInvalidValue;
  using TL = Tile<T, WIDE>;
  constexpr int FT_X = TL::X - 2, FT_Y = TL::Y - 2;
  const TileMap tm = tile_map((g.nx + FT_X - 1) / FT_X, (g.nr + FT_Y - 1) / FT_Y,
                              (g.nth + kc - 1) / kc);
  const dim3 grid((unsigned)(tm.per_xcd * NXCD));
  const dim3 block(TL::X, TL::Y, 1);
#define LESJET_FUSED_P(E, A, L, D, P)                                                  \
  hipLaunchKernelGGL((k_fused<T, WIDE, E, A, L, D, P>), grid, block, 0, s, Q, M, g, ph, kc, tm, \
                     out, Q0, Q64, alpha, dt, ph64, maxbits, visc, dyn, pt)
#define LESJET_FUSED(E, A, L)                                                          \
  do {                                                                                 \
    if (ph.sgs == 3) {                                                                 \
      if (pt.x) LESJET_FUSED_P(E, A, L, true, true);                                   \
      else LESJET_FUSED_P(E, A, L, true, false);                                       \
    } else {                                                                           \
      if (pt.x) LESJET_FUSED_P(E, A, L, false, true);                                  \
      else LESJET_FUSED_P(E, A, L, false, false);                                      \
    }                                                                                  \
  } while (0)
#define LESJET_FUSED_EPI(A)                                                        \
  if (lag == LAG_WRITE) LESJET_FUSED(EPI_RK, A, LAG_WRITE);                        \
  else if (lag == LAG_READ) {                                                      \
    if (epi == EPI_RK) LESJET_FUSED(EPI_RK, A, LAG_READ);                          \
    else LESJET_FUSED(EPI_RK_LAST, A, LAG_READ);                                   \
  } else if (epi == EPI_R) LESJET_FUSED(EPI_R, A, LAG_NONE);                       \
  else if (epi == EPI_RK) LESJET_FUSED(EPI_RK, A, LAG_NONE);                       \
  else LESJET_FUSED(EPI_RK_LAST, A, LAG_NONE);
  if (ph.axis_node) {
    LESJET_FUSED_EPI(true)
  } else {
    LESJET_FUSED_EPI(false)
  }
#undef LESJET_FUSED_EPI
#undef LESJET_FUSED
#undef LESJET_FUSED_P
  return hipGetLastError();
}

}  // namespace lesjet
