// HIP kernels of the adjoint (vector-Jacobian product) of the semi-discrete
// right-hand side and of the SSP-RK3 stage map, FP64.
//
//   adj_emf_kernel       cotangent of the face-b right-hand side -> cotangents
//                        of the six transport fluxes (transposes of the b
//                        equations of Sect. 2.3 and of eq. ox1-ox3)
//   adj_sweep_kernel     one direction: recomputes the tile's forward data,
//                        runs the per-face reverse (adjoint_device.hpp) and
//                        the per-zone prologue reverse, and adds the zone
//                        cotangents of every zone its faces touch (own zones
//                        and the halo zones of the neighbouring tiles); the
//                        tiles of one launch touch disjoint zones
//   adj_bcell_kernel     face-b cotangent += transpose of the fourth-order
//                        zone interpolation
//   adj_collect_kernel   that, and the sum of the sweeps' own arrays, where one
//                        launch holds the sweeps of the three axes
//   adj_glue kernels     the RK3 stage combinations
//   init_adj kernels     transpose of the initial-state map (curl_h A, m, E)
// Accumulation orders are fixed, so results are bitwise reproducible: none of the
// additions in memory are atomic, and those in LDS (by the LDS unit) meet at one address
// in rounds, separated by barriers or issued in turn by one wave.
#pragma once
#include <hip/hip_runtime.h>

#include "adjoint_device.hpp"
#include "kernels.hpp"

namespace wm {

// ---------------------------------------------------------------------------
// b equations and corner fluxes, transposed
// ---------------------------------------------------------------------------
// Forward (update_kernel): rhs_bx = -(Ez - Ez[j-1])/h + (Ey - Ey[k-1])/h,
// rhs_by = -(Ex - Ex[k-1])/h + (Ez - Ez[i-1])/h, rhs_bz = -(Ey - Ey[i-1])/h +
// (Ex - Ex[j-1])/h with Ez = (Tyx + Tyx[i+1])/2 - (Txy + Txy[j+1])/2,
// Ex = (Tzy + Tzy[j+1])/2 - (Tyz + Tyz[k+1])/2, Ey = (Txz + Txz[k+1])/2 - (Tzx + Tzx[i+1])/2.
// It also clears zero3 ([3][N], the zone-B cotangent that the sweeps then add into)
// and, with FIELD, forms the zone field B of the face field b that they read.
template <bool FIELD>
__global__ __launch_bounds__(256) void adj_emf_kernel(Grid g, double inv_h, double inv_nx, double inv_ny,
                                                      const double* lam_k, double* lam_T, const double* b, double* B,
                                                      double* zero3) {
  int i, j, k;
  if (!bcell_zone(g, inv_nx, inv_ny, i, j, k)) return;
  const size_t N = g.N;
  if (FIELD) zone_field(g, b, B, i, j, k);
  {
    const size_t c = g.at(i, j, k);
    zero3[c] = 0.0;
    zero3[N + c] = 0.0;
    zero3[2 * N + c] = 0.0;
  }
  const double* lbx = lam_k + 5 * N;
  const double* lby = lam_k + 6 * N;
  const double* lbz = lam_k + 7 * N;
  const int im = wrap(i - 1, g.nx), ip = wrap(i + 1, g.nx);
  const int jm = wrap(j - 1, g.ny), jp = wrap(j + 1, g.ny);
  const int km = wrap(k - 1, g.nz), kp = wrap(k + 1, g.nz);
  // cotangents of the corner fluxes at edge index (ii, jj, kk)
  auto lEz = [&](int ii, int jj, int kk) {
    const int jjp = wrap(jj + 1, g.ny), iip = wrap(ii + 1, g.nx);
    return (-lbx[g.at(ii, jj, kk)] + lbx[g.at(ii, jjp, kk)] + lby[g.at(ii, jj, kk)] - lby[g.at(iip, jj, kk)]) * inv_h;
  };
  auto lEx = [&](int ii, int jj, int kk) {
    const int kkp = wrap(kk + 1, g.nz), jjp = wrap(jj + 1, g.ny);
    return (-lby[g.at(ii, jj, kk)] + lby[g.at(ii, jj, kkp)] + lbz[g.at(ii, jj, kk)] - lbz[g.at(ii, jjp, kk)]) * inv_h;
  };
  auto lEy = [&](int ii, int jj, int kk) {
    const int kkp = wrap(kk + 1, g.nz), iip = wrap(ii + 1, g.nx);
    return (lbx[g.at(ii, jj, kk)] - lbx[g.at(ii, jj, kkp)] - lbz[g.at(ii, jj, kk)] + lbz[g.at(iip, jj, kk)]) * inv_h;
  };
  (void)ip; (void)jp; (void)kp;
  const size_t c0 = g.at(i, j, k);
  const double ez = lEz(i, j, k), ex = lEx(i, j, k), ey = lEy(i, j, k);
  // T layout: [0] Txy, [1] Txz, [2] Tyz, [3] Tyx, [4] Tzx, [5] Tzy
  lam_T[0 * N + c0] = -0.5 * (ez + lEz(i, jm, k));   // Txy feeds Ez(j) and Ez(j-1)
  lam_T[1 * N + c0] = 0.5 * (ey + lEy(i, j, km));    // Txz feeds Ey(k) and Ey(k-1)
  lam_T[2 * N + c0] = -0.5 * (ex + lEx(i, j, km));   // Tyz feeds Ex(k) and Ex(k-1)
  lam_T[3 * N + c0] = 0.5 * (ez + lEz(im, j, k));    // Tyx feeds Ez(i) and Ez(i-1)
  lam_T[4 * N + c0] = -0.5 * (ey + lEy(im, j, k));   // Tzx feeds Ey(i) and Ey(i-1)
  lam_T[5 * N + c0] = 0.5 * (ex + lEx(i, jm, k));    // Tzy feeds Ex(j) and Ex(j-1)
}

// ---------------------------------------------------------------------------
// adjoint of one directional sweep
// ---------------------------------------------------------------------------
struct AdjSweepArgs {
  Grid g;
  Phys ph;
  double inv_h;
  const double* hydro;   // forward state [5][N]
  const double* bcell;   // its zone B [3][N]
  const double* lam_k;   // [8][N] cotangent of the right-hand side (hydro part used)
  const double* lam_T;   // [6][N] cotangents of the transport fluxes T^n_t1, T^n_t2 of x, y, z
  // per axis: the zone cotangents of rho, m_x, m_y, m_z, E and of the zone field, which
  // are added to, or stored if `store` (an axis of its own arrays, whose tiles span it)
  double* lam_h[3];      // [5][N]
  double* lam_Bz[3];     // [3][N]
  int store[3];
  SweepAxis ax[3];       // tile; ntile: the tiles of this launch; blk0
  int tile0[3];          // tile index along the axis of block 0 of this launch
  int tstride[3];        // tile index step between consecutive blocks along the axis
  unsigned nblk, per_xcd;   // blocks of this launch, an eighth of them rounded up
  double inv_nx;
};

// x += v in LDS by the LDS unit (no value returns to the lane)
__device__ __forceinline__ void lds_add(double* x, double v) {
  __hip_atomic_fetch_add(x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

constexpr int ADJ_NP = 11;   // cotangents of zone primitives and speeds (P_* order)
constexpr int ADJ_NR = ADJ_NP + 7;   // and of the flux components
constexpr int ADJ_THREADS = 256;
// Zones and interfaces a tile may hold: 80 KB of LDS for the values, so that two
// blocks of 256 faces share a CU (two waves per SIMD).
constexpr int ADJ_ZONES = 280, ADJ_FACES = 276;

// One block: ta x tb faces of one axis, numbered like the forward sweep's.  Every
// zone that a face of the tile touches (positions 0 .. tav+4 along the axis) gets
// its cotangent added to lam_h / lam_Bz by exactly one thread of the block;
// positions that wrap onto the same zone (a tile that spans the whole axis) are
// summed first.  Blocks of one launch touch disjoint zones (the host launches the
// tiles of an axis in conflict-free classes) or, with the three axes in one launch,
// the arrays of their axis, so the additions need no atomics in memory and the order
// of accumulation is fixed.
//
// Bound by latency: dependent FP64 chains and LDS round trips between barriers.
// One pair at a time and thirteen eigen cotangents instead of twenty-three bring a
// lane under 256 registers, and the zone cotangents take the place of the zone
// values and differences once those are spent, so that 80 KB of LDS hold a tile
// and a second wave per SIMD fills the waits: at 128^3 an axis took 744-790 us with
// one wave per SIMD (147 KB, 446 registers, two pairs at once), 505-550 with two,
// and 445-495 with columns of 64 faces to a wave, one reciprocal for a weight's
// value and gradient, and the entropy row's additions carried by the Alfven
// pair's; at 48^3 73-78, 37-39 and 35-37, where one tile spans the axis and the two
// or three launches of its classes become one.
constexpr int ADJ_LDS = (SW_NQ + SW_NPF) * ADJ_ZONES + SW_NQ * ADJ_FACES;   // doubles
template <int AXIS, int W>
__device__ __forceinline__ void adj_sweep_tile(const AdjSweepArgs& a, unsigned blk, double* lds) {
  constexpr int NC = ADJ_ZONES, ND = ADJ_FACES;
  // LDS: zone q/F, then the differences (14 rows) | zone primitives and speeds (8) |
  //      interface-difference cotangents (14); the zone cotangents of the face
  //      state, speeds and flux means (18 rows) over the first two at the end
  double* Q = lds;
  double* Pz = lds + SW_NQ * NC;
  double* LD = lds + (SW_NQ + SW_NPF) * NC;
  double* PB = lds;
  static_assert(ADJ_NR <= SW_NQ + SW_NPF && ND <= NC, "aliases fit");
  const Grid& g = a.g;
  const SweepAxis& ax = a.ax[AXIS];
  const int nA = AXIS == 0 ? g.nx : (AXIS == 1 ? g.ny : g.nz);
  const int TA = ax.ta, TB = ax.tb, NA = TA + SW_HL + SW_HR, NI = TA + 4;
  const int ncell = NA * TB;
  constexpr int CN = AXIS, CT1 = (AXIS + 1) % 3, CT2 = (AXIS + 2) % 3;
  auto mul = [](int x, int y) { return (int)__umul24((unsigned)x, (unsigned)y); };
  // In LDS a column's values are neighbours, and so are its faces among the
  // lanes; only the zones' accesses to memory follow the rows across y and z.
  auto cidx = [&](int aa, int bb) { return mul(bb, NA) + aa; };
  auto iidx = [&](int ia, int bb) { return mul(bb, NI) + ia; };
  auto quot = [](int n, unsigned div) { return (int)(__umul24((unsigned)n, div) >> SW_DIV_SHIFT); };
  auto split_cell = [&](int cell, int& aa, int& bb) {
    if (AXIS == 0) { bb = quot(cell, ax.div_na); aa = cell - mul(bb, NA); }
    else           { aa = quot(cell, ax.div_tb); bb = cell - mul(aa, TB); }
  };
  const unsigned grp = (unsigned)__builtin_amdgcn_readfirstlane((int)quot_by(blk, ax.inv_ntile));
  const int a0 = (a.tile0[AXIS] + (int)(blk - grp * (unsigned)ax.ntile) * a.tstride[AXIS]) * TA;
  const int b0 = (int)grp * TB;
  const int tav = min(TA, nA - a0);            // valid faces (and own zones) along the axis
  const unsigned plane = (unsigned)g.nx * (unsigned)g.ny;
  auto zone_at = [&](int q, int ia) -> size_t {
    if (AXIS == 0) return (unsigned)q * (unsigned)g.nx + (unsigned)ia;
    if (AXIS == 2) return (unsigned)q + (unsigned)ia * plane;
    const unsigned z = quot_by((unsigned)q, a.inv_nx);
    return (unsigned)q + z * (plane - (unsigned)g.nx) + (unsigned)mul(ia, g.nx);
  };
  // sweep frame: rho, m_n, m_t1, m_t2, E, B_n, B_t1, B_t2
  auto load_zone = [&](size_t gi, double u[8]) {
    u[0] = a.hydro[gi];
    u[1] = a.hydro[(1 + CN) * g.N + gi];
    u[2] = a.hydro[(1 + CT1) * g.N + gi];
    u[3] = a.hydro[(1 + CT2) * g.N + gi];
    u[4] = a.hydro[4 * g.N + gi];
    u[5] = a.bcell[CN * g.N + gi];
    u[6] = a.bcell[CT1 * g.N + gi];
    u[7] = a.bcell[CT2 * g.N + gi];
  };

  // ---- (1) forward zone prologue into LDS, with the cotangents that arrive at the
  // zone (7 rows, in the place of the difference cotangents)
  double* stage = LD;
  static_assert(7 * NC <= SW_NQ * ND, "the staged cotangents fit");
  for (int cell = threadIdx.x; cell < ncell; cell += ADJ_THREADS) {
    int aa, bb;
    split_cell(cell, aa, bb);
    const int cz = cidx(aa, bb);
    double u[8], z[Z_NVAR], lk[7];
    const size_t gi = zone_at(min(b0 + bb, ax.ncol - 1), wrap_near(a0 - SW_HL + aa, nA));
    load_zone(gi, u);
#pragma unroll
    for (int v = 0; v < 7; ++v) lk[v] = (v < 5 ? a.lam_k : a.lam_T + (2 * AXIS - 5) * (ptrdiff_t)g.N)[v * g.N + gi];
    zone_prologue(u[0], u[1], u[2], u[3], u[4], u[5], u[6], u[7], a.ph.gamma, z);
#pragma unroll
    for (int v = 0; v < SW_NQ; ++v) Q[v * NC + cz] = z[v];
    const int pv[SW_NPF] = {Z_VN, Z_VT1, Z_VT2, Z_BN, Z_P, Z_CF, Z_CA, Z_CS};
#pragma unroll
    for (int v = 0; v < SW_NPF; ++v) Pz[v * NC + cz] = z[pv[v]];
#pragma unroll
    for (int v = 0; v < 7; ++v) stage[v * NC + cz] = lk[v];
  }
  // the face of this thread; threads past the tile's faces repeat face 0 and add nothing
  const bool active = (int)threadIdx.x < TA * TB;
  int fa, fb;
  {
    const int t = active ? threadIdx.x : 0;
    fb = quot(t, ax.div_ta);
    fa = t - mul(fb, TA);
  }
  __syncthreads();

  // ---- (2) the difference of the face's own interface and of the four of a
  // column beyond its faces' own (lanes fa < 4), as in the forward sweep
  const int cL = cidx(fa + 2, fb), cR = cL + 1;
  double f_rho, f_bt1, f_bt2, lam[7];
  {
    // incoming cotangents: flux divergence transposed, lam_F_v(face i+1/2) =
    // (lam_k_v(i+1) - lam_k_v(i))/h, in the sweep frame; the B_t components carry the
    // transport-flux cotangents
    const double msk = active && fa < tav && b0 + fb < ax.ncol ? 1.0 : 0.0, mh = msk * a.inv_h;
    auto lF = [&](int v) { return mh * (stage[v * NC + cR] - stage[v * NC + cL]); };
    lam[0] = lF(0);
    lam[1] = lF(1 + CN);
    lam[2] = lF(1 + CT1);
    lam[3] = lF(1 + CT2);
    lam[4] = msk * stage[5 * NC + cL];
    lam[5] = msk * stage[6 * NC + cL];
    lam[6] = lF(4);
  }
  {
    double d0[SW_NQ], d1[SW_NQ], f_q[7];
#pragma unroll
    for (int v = 0; v < SW_NQ; ++v) {
      const double L = Q[v * NC + cL], R = Q[v * NC + cR];
      d0[v] = R - L;
      if (v < 7) f_q[v] = 0.5 * (L + R);
    }
    f_rho = f_q[Z_RHO]; f_bt1 = f_q[Z_BT1]; f_bt2 = f_q[Z_BT2];
    const int ie = fa < 2 ? fa : TA + fa;
    if (fa < 4) {
      const int c2 = cidx(ie, fb), c3 = cidx(ie + 1, fb);
#pragma unroll
      for (int v = 0; v < SW_NQ; ++v) d1[v] = Q[v * NC + c3] - Q[v * NC + c2];
    }
    __syncthreads();
    // stored as (Delta F, Delta q): rows 0..6 flux, 7..13 state
#pragma unroll
    for (int v = 0; v < SW_NQ; ++v) Q[(v < 7 ? v + 7 : v - 7) * ND + iidx(fa + 2, fb)] = d0[v];
    if (fa < 4) {
#pragma unroll
      for (int v = 0; v < SW_NQ; ++v) Q[(v < 7 ? v + 7 : v - 7) * ND + iidx(ie, fb)] = d1[v];
    }
  }
  for (int t = threadIdx.x; t < SW_NQ * ND; t += ADJ_THREADS) LD[t] = 0.0;
  __syncthreads();

  // ---- (3) per-face reverse; interface cotangents in barrier-separated sub-rounds
  // LF speed of field m: max(|v_L + sg c_L|, |v_R + sg c_R|); c index: fast 0, Alfven 1, slow 2, none (entropy)
  // sign and speed index of field m: m < 3 minus, m = 3 none, m > 3 plus
  auto sgm = [](int m) { return m < 3 ? -1 : (m == 3 ? 0 : 1); };
  auto spi = [](int m) { return (m == 0 || m == 6) ? 0 : ((m == 1 || m == 5) ? 1 : 2); };
  auto xarg = [&](int m, int cz) {
    const double v = Pz[FP_VN * NC + cz];
    return sgm(m) == 0 ? v : v + sgm(m) * Pz[(FP_CF + spi(m)) * NC + cz];
  };
  auto alf = [&](int m) { return fmax(fabs(xarg(m, cL)), fabs(xarg(m, cR))); };
  auto mean = [&](int v) { return 0.5 * (Pz[v * NC + cL] + Pz[v * NC + cR]); };
  const double* dl0 = Q + iidx(fa, fb);
  double* ld0 = LD + iidx(fa, fb);
  auto row = [&](int k) -> const double* { return dl0 + k; };
  // round k: every face adds its cotangent of interface difference fa + k.  A
  // barrier before each fixes the order of the additions to an interface; where a
  // wave's 64 faces are whole columns (of 64, 32, 16 or 8) no other wave adds to its
  // interfaces, and its own additions keep their order (the barriers cost 8% of an
  // axis at 128^3, 3-4% of a step's cotangents in 16^3 and 32^3).
  const bool own_columns = TA <= 64 && (TA & (TA - 1)) == 0;
  auto in_order = [&]() {
    if (own_columns) { reload_fence(); sched_fence(); }
    else __syncthreads();
  };
  auto emit = [&](int k, const double* v) {
    in_order();
    if (active) {
      double* l = ld0 + k;
#pragma unroll
      for (int j = 0; j < SW_NQ; ++j) lds_add(l + j * ND, v[j]);
    }
  };
  double pl[ADJ_NP], pr[ADJ_NP];
  {
    const double fp[8] = {f_rho, mean(FP_VN), mean(FP_VT1), mean(FP_VT2), mean(FP_BN), f_bt1, f_bt2, mean(FP_P)};
    FaceEig e;
    face_eig(fp[0], fp[1], fp[2], fp[3], fp[4], fp[5], fp[6], fp[7], a.ph, e);
    EigCot eb;
    double lal[7], lfp[8];
    face_corr_vjp<W, ND>(e, alf, lam, row, a.ph, eb, lal, emit);
    {
      pin(f_rho); pin(f_bt1); pin(f_bt2);   // nothing of face_eig is held for its reverse
      const double fq[8] = {f_rho, mean(FP_VN), mean(FP_VT1), mean(FP_VT2), mean(FP_BN), f_bt1, f_bt2, mean(FP_P)};
      face_eig_vjp(fq, a.ph, e, eb, lfp);
    }
    // zone-primitive cotangents of zones L (i) and R (i+1): face-state means,
    // LF speeds (branch of the larger argument; ties -> L) and transport-flux means
#pragma unroll
    for (int v = 0; v < ADJ_NP; ++v) { pl[v] = v < 8 ? 0.5 * lfp[v] : 0.0; pr[v] = pl[v]; }
#pragma unroll
    for (int m = 0; m < 7; ++m) {
      const double xl = xarg(m, cL), xr = xarg(m, cR);
      const bool left = fabs(xl) >= fabs(xr);
      const double x = left ? xl : xr;
      const double sx = x > 0.0 ? 1.0 : (x < 0.0 ? -1.0 : 0.0);
      // to the zone of the larger argument (weights instead of a pointer select,
      // which would move pl, pr to scratch memory)
      const double gl = left ? lal[m] * sx : 0.0, gr = left ? 0.0 : lal[m] * sx;
      pl[P_VN] += gl;
      pr[P_VN] += gr;
      if (sgm(m) != 0) {
        pl[P_CF + spi(m)] += gl * sgm(m);
        pr[P_CF + spi(m)] += gr * sgm(m);
      }
    }
    const double BnL = Pz[FP_BN * NC + cL], BnR = Pz[FP_BN * NC + cR];
    pl[P_BN] += 0.5 * (lam[4] * Pz[FP_VT1 * NC + cL] + lam[5] * Pz[FP_VT2 * NC + cL]);
    pr[P_BN] += 0.5 * (lam[4] * Pz[FP_VT1 * NC + cR] + lam[5] * Pz[FP_VT2 * NC + cR]);
    pl[P_VT1] += 0.5 * lam[4] * BnL; pr[P_VT1] += 0.5 * lam[4] * BnR;
    pl[P_VT2] += 0.5 * lam[5] * BnL; pr[P_VT2] += 0.5 * lam[5] * BnR;
  }
  // zone sums, over the spent zone values: zone L's part is stored (position fa + 2
  // of face fa; the five positions that are no face's zone L are cleared), then
  // zone R's added.  The central term gives half of lam to both zones.
  __syncthreads();
  if (active) {
#pragma unroll
    for (int v = 0; v < ADJ_NP; ++v) PB[v * NC + cL] = pl[v];
#pragma unroll
    for (int j = 0; j < 7; ++j) PB[(ADJ_NP + j) * NC + cL] = 0.5 * lam[j];
    if (fa < 5) {
      const int cz = cidx(fa < 2 ? fa : TA + fa, fb);
#pragma unroll
      for (int v = 0; v < ADJ_NR; ++v) PB[v * NC + cz] = 0.0;
    }
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int v = 0; v < ADJ_NP; ++v) PB[v * NC + cR] += pr[v];
#pragma unroll
    for (int j = 0; j < 7; ++j) PB[(ADJ_NP + j) * NC + cR] += 0.5 * lam[j];
  }
  __syncthreads();

  // ---- (4) per zone: gather, prologue reverse, add
  const int span = tav + SW_HL + SW_HR;          // positions touched by the valid faces
  const int nz_own = min(span, nA);              // distinct zones among them
  // cotangents of the prologue outputs at tile position aa (lz += ...)
  auto gather = [&](int aa, int bb, double* lz) {
    const int ii = iidx(aa, bb), cz = cidx(aa, bb);
    // interface differences: D(ia) = X(ia+1) - X(ia)
    if (aa >= 1) {
#pragma unroll
      for (int j = 0; j < 7; ++j) {
        lz[Z_F0 + j] += LD[j * ND + ii - 1];
        lz[Z_RHO + j] += LD[(7 + j) * ND + ii - 1];
      }
    }
    if (aa < NI) {
#pragma unroll
      for (int j = 0; j < 7; ++j) {
        lz[Z_F0 + j] -= LD[j * ND + ii];
        lz[Z_RHO + j] -= LD[(7 + j) * ND + ii];
      }
    }
#pragma unroll
    for (int j = 0; j < 7; ++j) lz[Z_F0 + j] += PB[(ADJ_NP + j) * NC + cz];
    const int zv[ADJ_NP] = {Z_RHO, Z_VN, Z_VT1, Z_VT2, Z_BN, Z_BT1, Z_BT2, Z_P, Z_CF, Z_CA, Z_CS};
#pragma unroll
    for (int v = 0; v < ADJ_NP; ++v) lz[zv[v]] += PB[v * NC + cz];
  };
  for (int cell = threadIdx.x; cell < ncell; cell += ADJ_THREADS) {
    int aa, bb;
    split_cell(cell, aa, bb);
    if (aa >= nz_own || b0 + bb >= ax.ncol) continue;
    const size_t gi = zone_at(b0 + bb, wrap_near(a0 - SW_HL + aa, nA));
    double u[8], lm[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    load_zone(gi, u);
    double* const lh = a.lam_h[AXIS];
    double* const lB = a.lam_Bz[AXIS];
    if (!a.store[AXIS]) {
#pragma unroll
      for (int v = 0; v < 8; ++v) lm[v] = v < 5 ? lh[v * g.N + gi] : lB[(v - 5) * g.N + gi];
    }
    double lz[Z_NVAR];
#pragma unroll
    for (int v = 0; v < Z_NVAR; ++v) lz[v] = 0.0;
    gather(aa, bb, lz);
    if (span > nA)   // a tile that wraps onto itself: other positions of the same zone
      for (int q = aa + nA; q < span; q += nA) gather(q, bb, lz);
    double lu[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    zone_prologue_vjp(u, a.ph.gamma, lz, lu);
    double out[8];
    out[0] = lu[0];
    out[1 + CN] = lu[1]; out[1 + CT1] = lu[2]; out[1 + CT2] = lu[3];
    out[4] = lu[4];
    out[5 + CN] = lu[5]; out[5 + CT1] = lu[6]; out[5 + CT2] = lu[7];
#pragma unroll
    for (int v = 0; v < 8; ++v) (v < 5 ? lh + v * g.N : lB + (v - 5) * g.N)[gi] = lm[v] + out[v];
  }
}

// Blocks go to the 8 XCDs in turn:
// each XCD takes a run of neighbouring column groups, whose lines of memory its L2
// then fetches once (a group of 4 columns uses 32 of a line's 128 bytes).
// AXIS 3: the three axes in one launch, x first.
template <int AXIS, int W>
__global__ __launch_bounds__(ADJ_THREADS, 2) void adj_sweep_kernel(AdjSweepArgs a) {
  __shared__ double lds[ADJ_LDS];
  const unsigned blk = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
  if (blk >= a.nblk) return;
  if constexpr (AXIS < 3) adj_sweep_tile<AXIS, W>(a, blk, lds);
  else if (blk < a.ax[1].blk0) adj_sweep_tile<0, W>(a, blk, lds);
  else if (blk < a.ax[2].blk0) adj_sweep_tile<1, W>(a, blk - a.ax[1].blk0, lds);
  else adj_sweep_tile<2, W>(a, blk - a.ax[2].blk0, lds);
}

// The sweeps of a small box in one launch: acc_h += the y and z sweeps' parts, and
// the zone-field cotangents of the three sweeps (x, y, z) through the transpose of
// the zone interpolation into acc_b.
__global__ __launch_bounds__(256) void adj_collect_kernel(Grid g, double inv_nx, double inv_ny, const double* y,
                                                          const double* z, const double* Bx, double* acc_h,
                                                          double* acc_b) {
  const unsigned t = blockIdx.x * 256u + threadIdx.x;
  if (t >= g.N) return;
  int i, j, k;
  thread_zone(t, inv_nx, g.nx, inv_ny, g.ny, i, j, k);
  const size_t N = g.N, c0 = t;
#pragma unroll
  for (int v = 0; v < 5; ++v) acc_h[v * N + c0] += y[v * N + c0] + z[v * N + c0];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double *p0 = Bx + d * N, *p1 = y + (5 + d) * N, *p2 = z + (5 + d) * N;
    double L[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int o = q - 1;   // j-1, j, j+1, j+2
      const size_t c = d == 0 ? g.at(wrap(i + o, g.nx), j, k)
                              : (d == 1 ? g.at(i, wrap(j + o, g.ny), k) : g.at(i, j, wrap(k + o, g.nz)));
      L[q] = p0[c] + p1[c] + p2[c];
    }
    acc_b[d * N + c0] += (-L[3] + 9.0 * L[2] + 9.0 * L[1] - L[0]) * (1.0 / 16.0);
  }
}

// face b cotangent += transpose of B_i = (-b_{i-2} + 9 b_{i-1} + 9 b_i - b_{i+1})/16:
// lam_b_j += (-lam_B_{j+2} + 9 lam_B_{j+1} + 9 lam_B_j - lam_B_{j-1})/16
__global__ __launch_bounds__(256) void adj_bcell_kernel(Grid g, const double* lam_B, double* lam_b) {
  const int i = blockIdx.x * 64 + (threadIdx.x & 63);
  const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
  const int k = blockIdx.z;
  if (i >= g.nx || j >= g.ny) return;
  const size_t N = g.N, c0 = g.at(i, j, k);
  const double* Lx = lam_B;
  const double* Ly = lam_B + N;
  const double* Lz = lam_B + 2 * N;
  lam_b[c0] += (-Lx[g.at(wrap(i + 2, g.nx), j, k)] + 9.0 * Lx[g.at(wrap(i + 1, g.nx), j, k)] + 9.0 * Lx[c0] -
                Lx[g.at(wrap(i - 1, g.nx), j, k)]) * (1.0 / 16.0);
  lam_b[N + c0] += (-Ly[g.at(i, wrap(j + 2, g.ny), k)] + 9.0 * Ly[g.at(i, wrap(j + 1, g.ny), k)] + 9.0 * Ly[c0] -
                    Ly[g.at(i, wrap(j - 1, g.ny), k)]) * (1.0 / 16.0);
  lam_b[2 * N + c0] += (-Lz[g.at(i, j, wrap(k + 2, g.nz))] + 9.0 * Lz[g.at(i, j, wrap(k + 1, g.nz))] + 9.0 * Lz[c0] -
                        Lz[g.at(i, j, wrap(k - 1, g.nz))]) * (1.0 / 16.0);
}

// y = a x (n doubles)
__global__ __launch_bounds__(256) void scale_kernel(size_t n, double a, const double* x, double* y) {
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (c < n) y[c] = a * x[c];
}
__global__ __launch_bounds__(256) void fill_kernel(size_t n, double v, double* y) {
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (c < n) y[c] = v;
}
// y = x widened from float (n values): FP32 states enter the FP64 adjoint
__global__ __launch_bounds__(256) void widen_kernel(size_t n, const float* x, double* y) {
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (c < n) y[c] = double(x[c]);
}

// The stage combinations of the adjoint step over the 8N cotangent entries
// (hydro [5][N] then face b [3][N]).  lam3, the incoming cotangent, is read in
// place from (lh, lb), which keep it until the last combination overwrites them:
//   glue_a: lk = c lam3, z = 0
//   glue_b: lk = a lam3 + b x, z = 0
//   glue_c: lk = a lam3 + b x + c y, (lh, lb) = lam3 + x + y
//   glue_d: lk = a lam3 + b x, (lh, lb) = lam3 + x + y + z (the four-stage sum of RK4)
__device__ __forceinline__ double lam3_at(size_t i, size_t N, const double* lh, const double* lb) {
  return i < 5 * N ? lh[i] : lb[i - 5 * N];
}
__global__ __launch_bounds__(256) void adj_glue_a_kernel(size_t N, double c, const double* lh, const double* lb,
                                                         double* lk, double* z) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 8 * N) return;
  lk[i] = c * lam3_at(i, N, lh, lb);
  z[i] = 0.0;
}
__global__ __launch_bounds__(256) void adj_glue_b_kernel(size_t N, double a, const double* lh, const double* lb,
                                                         double b, const double* x, double* lk, double* z) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 8 * N) return;
  lk[i] = a * lam3_at(i, N, lh, lb) + b * x[i];
  z[i] = 0.0;
}
__global__ __launch_bounds__(256) void adj_glue_c_kernel(size_t N, double a, double b, const double* x, double c,
                                                         const double* y, double* lk, double* lh, double* lb) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 8 * N) return;
  const double wi = lam3_at(i, N, lh, lb), xi = x[i], yi = y[i];
  lk[i] = a * wi + b * xi + c * yi;
  const double s = wi + xi + yi;
  if (i < 5 * N) lh[i] = s;
  else lb[i - 5 * N] = s;
}
__global__ __launch_bounds__(256) void adj_glue_d_kernel(size_t N, double a, double b, const double* x,
                                                         const double* y, const double* z, double* lk, double* lh,
                                                         double* lb) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 8 * N) return;
  const double wi = lam3_at(i, N, lh, lb), xi = x[i];
  lk[i] = a * wi + b * xi;
  const double s = wi + xi + y[i] + z[i];
  if (i < 5 * N) lh[i] = s;
  else lb[i - 5 * N] = s;
}

// Initial-state map transposed, per zone: m = rho v, E = P0/(gamma-1) + (rho v^2 + B^2)/2
// with B the zone interpolation of b:  lam_v = rho lam_m + rho v lam_E,  lam_B = B lam_E.
__global__ __launch_bounds__(256) void init_adj_zone_kernel(size_t N, const double* rho, const double* v,
                                                            const double* B, const double* lam_h, double* g_v,
                                                            double* lam_B) {
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (c >= N) return;
  const double r = rho[c], lE = lam_h[4 * N + c];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    g_v[d * N + c] = r * lam_h[(1 + d) * N + c] + r * v[d * N + c] * lE;
    lam_B[d * N + c] = B[d * N + c] * lE;
  }
}

// curl_h transposed: b_x = (Az - Az[j-1] - Ay + Ay[k-1])/h, b_y = (Ax - Ax[k-1] - Az + Az[i-1])/h,
// b_z = (Ay - Ay[i-1] - Ax + Ax[j-1])/h  =>  per edge value of A:
// g_Ax = (lby - lby[k+1] - lbz + lbz[j+1])/h, g_Ay = (lbz - lbz[i+1] - lbx + lbx[k+1])/h,
// g_Az = (lbx - lbx[j+1] - lby + lby[i+1])/h
__global__ __launch_bounds__(256) void curl_adj_kernel(Grid g, double inv_h, const double* lam_b, double* g_A) {
  const int i = blockIdx.x * 64 + (threadIdx.x & 63);
  const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
  const int k = blockIdx.z;
  if (i >= g.nx || j >= g.ny) return;
  const size_t N = g.N, c0 = g.at(i, j, k);
  const double* lbx = lam_b;
  const double* lby = lam_b + N;
  const double* lbz = lam_b + 2 * N;
  const int ip = wrap(i + 1, g.nx), jp = wrap(j + 1, g.ny), kp = wrap(k + 1, g.nz);
  g_A[c0] = (lby[c0] - lby[g.at(i, j, kp)] - lbz[c0] + lbz[g.at(i, jp, k)]) * inv_h;
  g_A[N + c0] = (lbz[c0] - lbz[g.at(ip, j, k)] - lbx[c0] + lbx[g.at(i, j, kp)]) * inv_h;
  g_A[2 * N + c0] = (lbx[c0] - lbx[g.at(i, jp, k)] - lby[c0] + lby[g.at(ip, j, k)]) * inv_h;
}

}  // namespace wm
