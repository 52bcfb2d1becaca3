// m1_step_3d.hip -- the fused M1 step for 3-D grids: Cartesian ones (the 192^3 x 12 workload's
// layout), and spherical (ln r, theta, phi) grids with an inflow inner boundary, polar axes and
// periodic phi (the 256 x 64 x 128 x 20 workload).
//
// Same method and arithmetic as k_step_tiled (eq:finite_vol with the reconstruction of
// eq:recon_constraints, the M1 closure, the HLL flux eq:hll with the correction eq:epsilon, the
// backward-Euler interaction update eq:be_update); what differs is how neighbours meet:
//   * a wave is one y row of 16 x columns by 4 consecutive groups, lane = 16 group + column (with
//     one or two groups: of four or two x tiles, each with all its groups; rows past the last
//     group idle):
//     the x neighbours of a lane are the lanes next to it in its 16-lane row, reached by DPP
//     row shifts (no LDS, no barrier).  Columns 0 and 15 are halo: their zones are
//     reconstructed (their face states close the tile) but not updated, and their own outer
//     neighbours are loaded by those two lanes;
//   * a block is NI waves stacked in y and one group quad.  Each row computes the flux at its
//     lower y face from its own reconstruction and that of the row below, both from the
//     plane's states in LDS.  With AR (all rows) the NI rows are updated and the top row also
//     computes the flux at the block's upper face (from the reconstruction of the row above;
//     two rows above the block in LDS); without (the float blocks of 8 and 16 rows, whose
//     register budget at four waves per SIMD has no room for the extra loads) the lower NI - 1
//     rows are updated and the top row only computes the flux at its lower face (its zones are
//     the next tile's first row; one row above the block in LDS).
//     The two rows below the block and those above it are loaded into LDS by all waves
//     together.  The fluxes pass through LDS;
//   * the block marches along z over TM planes with a register window: every z face is
//     computed once, from values each lane loads for its own column one plane ahead;
//   * x faces are computed once (by the lane above the face), y faces once per block (the
//     lower row's upper state is recomputed by the row above instead of exchanged), z faces
//     once; only the halo columns and the faces between tiles repeat work of the neighbouring
//     tiles.
// One block barrier per plane (after the states), which waits for LDS only: the loads of the
// next plane stay in flight.  The update of a plane follows the next plane's barrier.
// What the plane loop waits for is kept out of it by hand: values loaded a plane ahead are moved
// into registers of their own where they are consumed, so that no copy of a load in flight
// (with a wait for it) falls before the barrier, every outer-row item is loaded without a branch,
// and addresses are a uniform base plus a 32-bit lane offset.  With this and the closure's form in
// the squares of f, whole steps with diagnostics: 192^3 x 12 FP64 3681 -> 3546 us, MIXED 2214 ->
// 2142, 256 x 64 x 128 x 20 MIXED (f mostly above 0.9) 2368 -> 2159.
// Stamps taken inside the loop show where the rest goes in double:
// of the two waves on a SIMD the older takes a plane in 6800 cycles and waits 3900 at the barrier
// for the younger one; VALU issue 62 %.
// With VEL (Cartesian grids, in double spherical ones too), Step 1 of the velocity step: the same transport without the
// interaction update, each face flux with the advective flux v^d U of the upwind face state
// added (the face's left state where v^d >= 0), from the normal velocity component on the face;
// the zone-local velocity terms of the flux rows follow in the frequency step.
// Spherical grids (SPH): the same structure with the geometry of the lane's zone from the
// per-axis tables (volume-coordinate slopes, face scale factors for the realizability checks and
// the fluxes, face weights and zone widths for the divergence, proper widths for the optical
// depth; the radial values of the block's columns staged in LDS once, the theta values of the
// wave's row read by scalar loads), the geometric source terms after the divergence, theta faces
// on the polar axis closed; a polar-axis ghost row takes the mirrored row of the plane n_phi/2
// away (with F_theta and F_phi flipped), and an inflow ghost column the prescribed state with its
// own scale factors.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "m1_device.h"
#include "m1_grid.h"
#include "m1_internal.h"
#include "m1_lane.h"
#include "m1_step.h"

namespace fm1 {

// the sign rules: F_c flipped by its sign mask
template <typename R>
__device__ __forceinline__ void c3_fix(const R raw[4], unsigned mx, unsigned my, unsigned mz, R q[4]) {
  q[0] = raw[0];
  q[1] = flip_sign(raw[1], mx);
  q[2] = flip_sign(raw[2], my);
  q[3] = flip_sign(raw[3], mz);
}

// the state at element offset p of a plane (uniform) plus the lane's byte offset
template <typename S, typename R>
__device__ __forceinline__ void c3_load(const StepArgs<S>& a, int64_t p, unsigned off, R q[4]) {
  q[0] = R(ld_off(a.E + p, off));
  q[1] = R(ld_off(a.F[0] + p, off));
  q[2] = R(ld_off(a.F[1] + p, off));
  q[3] = R(ld_off(a.F[2] + p, off));
}

// LDS barrier: waits for the wave's LDS operations only (the global loads of the next plane
// stay in flight); the empty asm statements keep the compiler from moving memory accesses
// across it
__device__ __forceinline__ void c3_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Rows of the plane held in LDS: the block's NI rows in slots 2 .. NI + 1, the two rows below
// in slots 0, 1 and those above in slots NI + 2 (and NI + 3 where every row is updated).  The
// outer rows are loaded by all waves together, one (slot, component) item per wave and load:
// the 4 state components of slot 0, the 4 state components, kappa and sigma of slot 1; above
// the block either those of slot NI + 2 and the 4 state components of NI + 3 (every row
// updated), or the 4 state components of slot NI + 2.
template <bool AR>
constexpr int c3_nitem() { return AR ? 20 : 14; }

// NI waves per block, W waves per SIMD (register budget 512 / W).  RK: whether the launch may be a
// second Runge-Kutta stage (a.Ea read at run time)
template <typename S, int NI, int W, int LIM, bool SPH, bool AR, bool VEL = false, bool RK = true>
__global__ void __launch_bounds__(64 * NI) __attribute__((amdgpu_waves_per_eu(W)))
k_step_3d(StepArgs<S> a, Geo<S> geo, C3Tile tl, VelArgs<S> va) {
  using R = S;
  constexpr int TX = C3_TX;
  constexpr int NS = NI + (AR ? 4 : 3);                   // LDS row slots
  constexpr int NIT = c3_nitem<AR>();
  constexpr int NHI = (NIT + NI - 1) / NI;                // outer-row items per wave
  // double-buffered by plane parity: one barrier per plane (see the plane loop)
  __shared__ R QS[2][6][NS][64];    // E, F_x, F_y, F_z, kappa, sigma of the plane's rows
  __shared__ R FY[2][4][NI + AR][64];  // y flux at the lower face of each row (and the block's upper face)
  __shared__ double red_e[NI], red_m[NI];
  __shared__ int red_u[NI], red_p[NI];

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave = row (uniform)
  const int x = lane & (TX - 1), gq = lane >> 4;
  const int sw = w + 2;                                   // the wave's slot
  const bool top = w == NI - 1;
  const bool idle = !AR && top;          // a row that only computes its lower face flux

  // tile of the block (XCD-aware renumbering; the group quads of a tile adjacent)
  const int b = blockIdx.x;
  const int xcd = b & 7, sl = b >> 3;
  const int L = xcd * tl.xq + min(xcd, tl.xr) + sl;
  const int gb = L % tl.ngb;
  int rest = L / tl.ngb;
  const int tx = rest % tl.ntx;
  rest /= tl.ntx;
  const int ty = rest % tl.nty;
  const int tz = rest / tl.nty;

  const int n0 = a.n[0], n1 = a.n[1], n2 = a.n[2], G = a.G;
  // the row's group and x tile: four groups of one tile, or with one or two groups all groups of
  // RT = 4 or 2 tiles; lanes past the last group repeat it (they never store)
  // (in float the group count is a multiple of 4)
  const int RT = sizeof(R) == 8 ? tl.RT : 1;
  const int g = RT == 1 ? gb * 4 + gq : (G == 2 ? gq & 1 : 0);
  const int gc = sizeof(R) == 8 ? min(g, G - 1) : g;
  const int xt = RT == 1 ? tx : tx * RT + (G == 2 ? gq >> 1 : gq);
  const int xz = xt * (TX - 2) + x - 1;          // zone of the lane's column
  const int y0 = ty * (AR ? NI : NI - 1);        // zone of slot 2
  const int yz = y0 + w;                         // zone of the wave's row
  const int mbeg = tz * tl.TM, mend = min(mbeg + tl.TM, n2);
  const bool upd = !idle && yz < n1 && x >= 1 && x <= TX - 2 && xz < n0 && (sizeof(R) == 4 || g < G);
  const int PL = n0 * n1 * G;                    // elements of a z plane

  const C3Axis ax0 = c3_axis<0>(a), ax1 = c3_axis<1>(a), ax2 = c3_axis<2>(a);
  // sources and sign rules of the lane's column and of its outer x neighbour (columns 0, 15)
  int xs, xf, ys, yf;
  c3_src(ax0, xz, xs, xf);
  c3_src(ax1, yz, ys, yf);
  const bool xedge = x == 0 || x == TX - 1;
  int xef;
  // byte offsets within a plane (below 2^32: a grid has fewer than 2^29 zone-groups)
  unsigned ob = (unsigned)((ys * n0 + xs) * G + gc) * sizeof(S);
  int xeo;
  c3_src(ax0, x == 0 ? xz - 1 : xz + 1, xeo, xef);
  unsigned oe = (unsigned)((ys * n0 + xeo) * G + gc) * sizeof(S);
  // sign masks: F_x flips in reflected columns, F_y in reflected or polar-axis rows, F_z in
  // polar-axis rows (flag bit 2) and in reflected planes
  const unsigned sx = (unsigned)(xf & 1) << 31, sxe = (unsigned)(xef & 1) << 31;
  const unsigned sy = (unsigned)(yf & 1) << 31, sz = (unsigned)((yf >> 2) & 1) << 31;
  // spherical grids: extended indices of the lane's zone for the geometry tables (clamped:
  // lanes outside the grid compute but never store), the phi shift of a polar-axis ghost row,
  // inflow ghosts (flag bit 1) of the lane's column and of its outer neighbour
  const int ex = SPH ? min(max(xz, -2), n0 + 1) + NG : 0;
  const int ey = SPH ? min(max(yz, -2), n1 + 1) + NG : 0;
  const int zsh = (SPH && ((yf >> 2) & 1)) ? n2 / 2 : 0;
  const bool xinf = SPH && ((xf >> 1) & 1), xinfe = SPH && ((xef >> 1) & 1);
  // B of the lane's own zone (clamped into the domain so every lane may load it)
  unsigned oz = (unsigned)((min(max(yz, 0), n1 - 1) * n0 + min(max(xz, 0), n0 - 1)) * G + gc) * sizeof(S);
  // the wave's outer-row items: LDS slot and component (uniform), element offset within a
  // plane and flip of its row and column (per lane), the array (uniform)
  int hslot[NHI], hcomp[NHI], hsh[NHI], hey[NHI];
  unsigned hoff[NHI], hmask[NHI];
  const S* hsrc[NHI];
  for (int k = 0; k < NHI; ++k) {
    // (a wave short of an item repeats one: same value to the same place, and no branch)
    const int it = (w + k * NI) % NIT;
    int slot, comp;
    if (it < 4) { slot = 0; comp = it; }
    else if (it < 10) { slot = 1; comp = it - 4; }
    else if (!AR || it < 16) { slot = NI + 2; comp = it - 10; }
    else { slot = NI + 3; comp = it - 16; }
    int hys, hyf;
    c3_src(ax1, y0 - 2 + slot, hys, hyf);
    hslot[k] = slot;
    hcomp[k] = comp;
    hoff[k] = (unsigned)((hys * n0 + xs) * G + gc) * sizeof(S);
    hmask[k] = comp == 1 ? sx : comp == 2 ? (unsigned)(hyf & 1) << 31 : comp == 3 ? (unsigned)((hyf >> 2) & 1) << 31 : 0u;
    hsh[k] = (SPH && ((hyf >> 2) & 1)) ? n2 / 2 : 0;
    hey[k] = min(max(y0 - 2 + slot, -2), n1 + 1) + NG;
    hsrc[k] = comp == 0 ? a.E : comp <= 3 ? a.F[comp - 1] : comp == 4 ? a.kap : a.sig;
  }
  // plane m (-2 .. n2 + 1, clamped): element offset and F_z's sign mask
  auto plane = [&](int m, unsigned& pm) -> int64_t {
    int zs, zf;
    c3_src(ax2, m, zs, zf);
    pm = (unsigned)(zf & 1) << 31;
    return (int64_t)zs * PL;
  };
  // plane m of a row shifted by sh in phi (a polar-axis ghost row: phi is periodic there)
  auto plane_s = [&](int m, int sh, unsigned& pm) -> int64_t {
    if (sh == 0) return plane(m, pm);
    pm = 0;
    int zz = (m + sh) % n2;
    if (zz < 0) zz += n2;
    return (int64_t)zz * PL;
  };
  // the inflow ghost state of zone (extended ex_, ey_): E and covariant F_k = h_k F^_k with the
  // ghost's own scale factors (spherical grids, inflow on x1 only)
  auto inflow_state = [&](int ex_, int ey_, R q[4]) {
    const double* in = a.inflow + gc * 4;
    R h[3];
    cell_h<R, SPH>(geo, ex_, ey_, h);
    q[0] = R(in[0]);
    for (int c = 0; c < 3; ++c) q[1 + c] = h[c] * R(in[1 + c]);
  };

  const bool want_diag = a.p_energy != nullptr;
  WaveDiag wd;
  const unsigned long long updm = __builtin_amdgcn_ballot_w64(upd);
  const double cdt = a.c * a.dt;
  const R dtR = R(a.dt);
  const R idx0 = geo.idx[0], idx1 = geo.idx[1], idx2 = geo.idx[2];
  const R dx1 = geo.dx[1], dx2 = geo.dx[2];
  const R hdx0 = R(0.5) * geo.dx[0], hdx1 = R(0.5) * dx1, hdx2 = R(0.5) * dx2;
  const R hone[3] = {R(1), R(1), R(1)};
  const double Vz = want_diag ? (SPH ? geo.Wd[0][ex] * geo.Wd[1][ey] * geo.Wd[2][NG]
                                     : geo.Wd[0][NG] * geo.Wd[1][NG] * geo.Wd[2][NG])
                              : 0.0;
  // phi-face scale factors of the lane's column (the same for every plane) and the proper width
  // along phi; cell-centred h for the geometric source
  R hz[3] = {R(1), R(1), R(1)}, ihz[3] = {R(1), R(1), R(1)};
  R dlz = dx2;
  if constexpr (SPH) {
    face_h<R, SPH>(geo, 2, ex, ey, 0, hz);
    face_ih<R, SPH>(geo, 2, ex, ey, 0, ihz);
    dlz = proper_width<R, SPH>(geo, 2, ex, ey);
  }
  // spherical grids: the radial tables at the block's 16 columns, staged in LDS once (the first
  // plane's barrier orders the reads): the plane loop reads them from LDS rather than from the
  // tables (the theta tables, indexed by the wave's row, are scalar loads)
  enum { RG_IRC, RG_RC, RG_HR, RG_IHR, RG_IRF0, RG_IRF1, RG_RF, RG_IDM, RG_IDP, RG_DLO, RG_DHI, RG_IDC, RG_WF0,
         RG_WF1, RG_IW, RG_N };
  __shared__ R RGT[SPH ? RG_N : 1][sizeof(R) == 8 ? 64 : TX];
  const int xl = RT == 1 ? x : lane;          // the column's entry (rows share a tile, or not)
  if constexpr (SPH) {
    if (w == 0 && xl == lane) {
      RGT[RG_IRC][xl] = gld(geo.irc, ex);
      RGT[RG_RC][xl] = gld(geo.rc, ex);
      RGT[RG_HR][xl] = gld(geo.hr, ex);
      RGT[RG_IHR][xl] = gld(geo.ihr, ex);
      RGT[RG_IRF0][xl] = gld(geo.irf, ex);
      RGT[RG_IRF1][xl] = gld(geo.irf, ex + 1);
      RGT[RG_RF][xl] = gld(geo.rf, ex);
      RGT[RG_IDM][xl] = gld(geo.idm[0], ex);
      RGT[RG_IDP][xl] = gld(geo.idp[0], ex);
      RGT[RG_DLO][xl] = gld(geo.dlo[0], ex);
      RGT[RG_DHI][xl] = gld(geo.dhi[0], ex);
      RGT[RG_IDC][xl] = gld(geo.idc[0], ex);
      RGT[RG_WF0][xl] = gld(geo.wf[0], ex);
      RGT[RG_WF1][xl] = gld(geo.wf[0], ex + 1);
      RGT[RG_IW][xl] = gld(geo.iW[0], ex);
    }
  }
  auto rg = [&](int k) -> R { return RGT[SPH ? k : 0][xl]; };
  // eq:epsilon on z faces (zones of equal width along z)
  auto eps_z = [&](R ksL, R ksR) -> R {
    if constexpr (SPH) return epsilon_of(ksL, ksR, dlz, dlz);
    else return epsilon_uniform(ksL, ksR, hdx2);
  };

  // ---- register window along z: q(m), q(m + 1); the upper z face state of zone m and the
  // flux at m - 1/2; kappa and sigma of plane m ----
  R q0[4], q1[4], hiM[4], fPrev[4];
  R k0, s0;
  // values in flight: q(m + 2), the outer x neighbour (columns 0, 15) of plane m and the
  // wave's outer-row items of plane m, kappa, sigma of m + 1 (Pk, Ps) and B of m (PB), all
  // loaded at the top of the plane before
  R Pr[4], Po[4], Ph[NHI], Pk, Ps, PB;
  unsigned y0m, y1m, y2m, y3m;   // F_z sign masks of planes m .. m + 3 (the lane's own row)
  int64_t p1, p2, p3;            // element offsets of planes m + 1, m + 2, m + 3
  FaceAux<R> xM{};               // |F^|^2 and cE of hiM
  // the wave's outer-row items of plane m (element offset off of the unshifted plane m)
  auto load_items = [&](int64_t off, int m) {
    for (int k = 0; k < NHI; ++k) {
        int64_t o = off;
        if (SPH && hsh[k] != 0) {
          unsigned pmx;
          o = plane_s(m, hsh[k], pmx);
        }
        Ph[k] = R(ld_off(hsrc[k] + o, hoff[k]));
        if (SPH && xinf && hcomp[k] <= 3) {
          R qi[4];
          inflow_state(ex, hey[k], qi);
          const int hc = hcomp[k];
          Ph[k] = hc == 0 ? qi[0] : hc == 1 ? qi[1] : hc == 2 ? qi[2] : qi[3];
        }
      }
  };
  // VEL: normal velocity components on the lane's faces (indices clamped into the face arrays:
  // lanes and rows outside the grid compute but never store).  x faces [n2][n1][n0 + 1], y faces
  // [n2][n1 + 1][n0] after the n0 (n1 + 1) n2 x components of v[1], z faces [n2 + 1][n1][n0]
  // after 2 n0 n1 (n2 + 1) components of v[2].
  const int64_t vxc = min(max(xz, 0), n0), vxz = min(max(xz, 0), n0 - 1);
  const int64_t vyr = min(max(yz, 0), n1 - 1), vyf = min(max(yz, 0), n1), vyt = min(max(yz + 1, 0), n1);
  const int64_t nfy = (int64_t)n0 * (n1 + 1) * n2, nfz = (int64_t)n0 * n1 * (n2 + 1);
  auto vel_z = [&](int f) -> R { return R(va.v[2][2 * nfz + ((int64_t)f * n1 + vyr) * n0 + vxz]); };
  R Ux = R(0), Uy = R(0), Uyt = R(0), Uz = R(0);   // face velocities of the plane
  unsigned zm0;   // F_z sign mask of plane m (unshifted): the outer-row items'
  {
    unsigned ya, yb;
    R raw[4], qa[4], qb[4];
    const int64_t p0 = plane_s(mbeg, zsh, y0m);
    c3_load<S, R>(a, p0, ob, raw);
    c3_fix(raw, sx, sy, sz ^ y0m, q0);
    k0 = R(ld_off(a.kap + p0, ob));
    s0 = R(ld_off(a.sig + p0, ob));
    p1 = plane_s(mbeg + 1, zsh, y1m);
    c3_load<S, R>(a, p1, ob, raw);
    c3_fix(raw, sx, sy, sz ^ y1m, q1);
    const int64_t pa = plane_s(mbeg - 2, zsh, ya), pb = plane_s(mbeg - 1, zsh, yb);
    c3_load<S, R>(a, pa, ob, raw);
    c3_fix(raw, sx, sy, sz ^ ya, qa);
    c3_load<S, R>(a, pb, ob, raw);
    c3_fix(raw, sx, sy, sz ^ yb, qb);
    if (SPH && xinf) {
      inflow_state(ex, ey, q0);
      inflow_state(ex, ey, q1);
      inflow_state(ex, ey, qa);
      inflow_state(ex, ey, qb);
    }
    const R ksb = R(ld_off(a.kap + pb, ob)) + R(ld_off(a.sig + pb, ob));
    // face mbeg - 1/2 from zones mbeg - 1 (upper state) and mbeg (lower state)
    for (int c = 0; c < 4; ++c) hiM[c] = fPrev[c] = R(0);
    if (!idle) {
      R lo[4], hiP[4];
      FaceAux<R> xP, xl;
      reconstruct<R, SPH, 3, LIM>(a, geo, 2, NG, qa, qb, q0, ihz, ihz, true, true, lo, hiP, nullptr, nullptr, &xP);
      reconstruct<R, SPH, 3, LIM>(a, geo, 2, NG, qb, q0, q1, ihz, ihz, true, true, lo, hiM, nullptr, &xl, &xM);
      hll<R, SPH, 3, (LIM < 0)>(a, 2, hiP, lo, hz, ihz, eps_z(ksb, k0 + s0), fPrev, &xP, &xl);
      if constexpr (VEL) add_upwind(vel_z(mbeg), hiP, lo, fPrev);
    }
    // in flight into the first plane
    Pk = R(ld_off(a.kap + p1, ob));
    Ps = R(ld_off(a.sig + p1, ob));
    PB = R(ld_off(a.B + (int64_t)mbeg * PL, oz));
    p2 = plane_s(mbeg + 2, zsh, y2m);
    c3_load<S, R>(a, p2, ob, Pr);
    c3_load<S, R>(a, p0, oe, Po);
    if (SPH && xinfe) inflow_state(ex - 1, ey, Po);
    load_items(plane(mbeg, zm0), mbeg);
  }

  // The update of plane m needs the y flux that the row above computes for plane m: it runs
  // after the next plane's barrier, from values the lane keeps (the state, the x and z part of
  // the divergence and the flux at its lower y face, kappa, sigma, B).  With the LDS arrays
  // double-buffered by plane parity, the one barrier per plane orders every LDS access: a
  // buffer written for plane m was last read for plane m - 2, before the barrier of m - 1.
  // (The state, the x and z part and the lower y flux stay apart: folded into one value, which takes
  // a third of the registers, equal y fluxes would no longer cancel exactly.)
  // geometric source terms of the covariant flux components (cell-centred h), from the state qz
  auto add_geometric = [&](const R qz[4], R U[4]) {
    if constexpr (SPH) {
      R h[3], ih[3], P[9], Sg[3];
      h[0] = h[1] = rg(RG_HR);
      h[2] = rg(RG_HR) * gld(geo.hs, ey);
      ih[0] = ih[1] = rg(RG_IHR);
      ih[2] = rg(RG_IHR) * gld(geo.ihs, ey);
      closure_full<R, SPH, 3>(qz, ih, R(a.c), a.closure, P);
      geometric_source<R>(P, h, ih, geo.gam + 4 * min(max(yz, 0), n1 - 1), R(a.c), Sg);
      for (int cc = 0; cc < 3; ++cc) U[1 + cc] += dtR * Sg[cc];
    } else {
      (void)qz;
      (void)U;
    }
  };
  R qU[4], accU[4], fyU[4], kU = R(0), sU = R(0), BU = R(0);
  for (int c = 0; c < 4; ++c) qU[c] = accU[c] = fyU[c] = R(0);
  // the update of plane mu from the kept values and the y flux that the row above computed for it
  // (every lane of the inner rows computes; the lanes that hold a zone of the tile store); bu: the
  // plane's LDS buffer
  auto update = [&](const int mu, const int bu) {
    const int64_t pu = (int64_t)mu * PL;
    R Um[4];
    R acc[4];
    if constexpr (SPH) {
      const R wl = gld(geo.wf[1], ey), wh = gld(geo.wf[1], ey + 1), iW = gld(geo.iW[1], ey);
      for (int c = 0; c < 4; ++c) acc[c] = accU[c] + (wh * FY[bu][c][w + 1][lane] - wl * fyU[c]) * iW;
    } else {
      for (int c = 0; c < 4; ++c) acc[c] = accU[c] + (FY[bu][c][w + 1][lane] - fyU[c]) * idx1;
    }
    for (int c = 0; c < 4; ++c) Um[c] = qU[c] - dtR * acc[c];
    if constexpr (SPH) add_geometric(qU, Um);
    if (RK && a.Ea) {
      // second Runge-Kutta stage: U^- = (U^n + U* + dt L(U*)) / 2
      Um[0] = R(0.5) * (R(ld_off(a.Ea + pu, oz)) + Um[0]);
      for (int c = 0; c < 3; ++c) Um[1 + c] = R(0.5) * (R(ld_off(a.Fa[c] + pu, oz)) + Um[1 + c]);
    }
    S Eo, F1[3];
    double dz = 0.0;
    if (a.src) {
      const double ck = cdt * (double)kU;
      dz = source_update<S, R, 3>(Um, ck, cdt * ((double)kU + (double)sU), ck * (double)BU, Eo, F1);
      if (want_diag) {
        double Fd[3] = {(double)F1[0], (double)F1[1], (double)F1[2]};
        if constexpr (SPH) {
          const double hd = (double)rg(RG_HR), hd2 = hd * (double)gld(geo.hs, ey);
          const double ih = rcp_(hd);
          Fd[0] *= ih;
          Fd[1] *= ih;
          Fd[2] *= rcp_(hd2);
        }
        wave_diag<S, 3>(a.c, (double)Eo, Fd, updm, wd);
      }
    } else {
      Eo = S(Um[0]);
      for (int c = 0; c < 3; ++c) F1[c] = S(Um[1 + c]);
    }
    if (upd) {
      st_off(a.Eo + pu, oz, Eo);
      for (int c = 0; c < 3; ++c) st_off(a.Fo[c] + pu, oz, F1[c]);
    }
    if (a.dEm) {
      // the zone's sum over the rows that hold its groups (lanes 16 apart)
      dz = upd ? dz : 0.0;
      if (RT < 4) dz = lane_pair_sum<16>(dz);
      if (RT < 2) dz = lane_pair_sum<32>(dz);
      if (upd && g == gb * 4) {
        const int64_t zone = ((int64_t)mu * n1 + yz) * n0 + xz;
        if (tl.ngb == 1) a.dEm[zone] = -dz;
        else a.dzp[(int64_t)gb * a.nzones + zone] = dz;
      }
    }
  };
  for (int m = mbeg; m < mend; ++m) {
    const int buf = m & 1;
    R q2[4], qo[4], k1, s1, BM;
    // (the offsets opaque to the compiler in each pass: their extension to 64 bits, hoisted out
    // of the loop, would cost an address addition per access)
    asm("" : "+v"(ob), "+v"(oe), "+v"(oz));
    for (int k = 0; k < NHI; ++k) asm("" : "+v"(hoff[k]));
    // ---- consume the values loaded one plane ago; the plane's rows to LDS ----
    c3_fix(Pr, sx, sy, sz ^ y2m, q2);          // plane m + 2
    c3_fix(Po, sxe, sy, sz ^ y0m, qo);         // outer x neighbour, plane m
    k1 = Pk;
    s1 = Ps;
    BM = PB;
    // (into registers of their own, so that the loads below can target the ones they came from:
    // left to the compiler, the loads go elsewhere and are copied back before the barrier, where
    // the copies wait for them)
    for (int c = 0; c < 4; ++c) asm("" : "+v"(q2[c]), "+v"(qo[c]));
    asm("" : "+v"(k1), "+v"(s1), "+v"(BM));
    if (SPH && xinf) inflow_state(ex, ey, q2);
    if (SPH && xinfe) inflow_state(ex - 1, ey, qo);
    for (int c = 0; c < 4; ++c) QS[buf][c][sw][lane] = q0[c];
    QS[buf][4][sw][lane] = k0;
    QS[buf][5][sw][lane] = s0;
    for (int k = 0; k < NHI; ++k)
      QS[buf][hcomp[k]][hslot[k]][lane] = flip_sign(Ph[k], hmask[k] ^ (hcomp[k] == 3 ? zm0 : 0u));
    // ---- loads for the next plane: q(m + 3), outer neighbours of m + 1, kappa, sigma of
    // m + 2 and B of m + 1 (indices clamped into the ghost range; the last planes' are not
    // used) ----
    p3 = plane_s(min(m + 3, n2 + 1), zsh, y3m);
    c3_load<S, R>(a, p3, ob, Pr);
    if (xedge) c3_load<S, R>(a, p1, oe, Po);
    if constexpr (SPH) {
      load_items(plane(min(m + 1, n2 + 1), zm0), min(m + 1, n2 + 1));
    } else {
      load_items(p1, m + 1);
      zm0 = y1m;
    }
    Pk = R(ld_off(a.kap + p2, ob));
    Ps = R(ld_off(a.sig + p2, ob));
    PB = R(ld_off(a.B + (int64_t)min(m + 1, n2 - 1) * PL, oz));
    if constexpr (VEL) {
      // this plane's face velocities (used after the barrier)
      Ux = R(va.v[0][((int64_t)m * n1 + vyr) * (n0 + 1) + vxc]);
      Uy = R(va.v[1][nfy + ((int64_t)m * (n1 + 1) + vyf) * n0 + vxz]);
      if (AR && top) Uyt = R(va.v[1][nfy + ((int64_t)m * (n1 + 1) + vyt) * n0 + vxz]);
      Uz = vel_z(m + 1);
    }
    c3_barrier();
    if (m > mbeg && !idle) update(m - 1, buf ^ 1);
    const R ks0 = k0 + s0;
    // ---- y: the flux at the lower y face of the row, from the reconstructions of the row
    // below (upper state) and of the row (lower state) ----
    R fy[4];
    {
      R qa[4], qb[4], qc[4], lo[4], hiP[4], hiY[4], loY[4];
      FaceAux<R> xP, xY, xYh;
      for (int c = 0; c < 4; ++c) {
        qa[c] = QS[buf][c][sw - 2][lane];
        qb[c] = QS[buf][c][sw - 1][lane];
      }
      const R ksb = QS[buf][4][sw - 1][lane] + QS[buf][5][sw - 1][lane];
      for (int c = 0; c < 4; ++c) qc[c] = QS[buf][c][sw + 1][lane];
      if constexpr (SPH) {
        // theta faces: scale factors at the face centres of the lane's column; a face on the
        // polar axis is closed (no flux, its face states not checked)
        // (theta faces: 1/h_r = 1/h_theta = 1/r at the column's centre, 1/h_phi with 1/sin theta
        // of the face)
        const R irc = rg(RG_IRC), rc = rg(RG_RC), dly = rg(RG_HR) * geo.dx[1];
        auto ih_th = [&](int ef, R ih[3]) {
          ih[0] = ih[1] = irc;
          ih[2] = irc * gld(geo.isf, ef);
        };
        auto h_th = [&](int ef, R h[3]) {
          h[0] = h[1] = rc;
          h[2] = rc * gld(geo.sf, ef);
        };
        R ihm[3], ih0[3], ih1[3];
        ih_th(ey - 1, ihm);
        ih_th(ey, ih0);
        ih_th(ey + 1, ih1);
        const bool om = gld(geo.wf[1], ey - 1) != R(0), o0f = gld(geo.wf[1], ey) != R(0), o1f = gld(geo.wf[1], ey + 1) != R(0);
        reconstruct<R, SPH, 3, LIM>(a, geo, 1, ey - 1, qa, qb, q0, ihm, ih0, om, o0f, lo, hiP, nullptr, nullptr, &xP);
        reconstruct<R, SPH, 3, LIM>(a, geo, 1, ey, qb, q0, qc, ih0, ih1, o0f, o1f, loY, hiY, nullptr, &xY, &xYh);
        for (int c = 0; c < 4; ++c) fy[c] = R(0);
        if (o0f) {
          R hf[3];
          h_th(ey, hf);
          hll<R, SPH, 3, (LIM < 0)>(a, 1, hiP, loY, hf, ih0, epsilon_of(ksb, ks0, dly, dly), fy, &xP, &xY);
          if constexpr (VEL) add_upwind(Uy, hiP, loY, fy);
        }
        if (AR && top && yz < n1) {
          // the block's upper face (ey + 1 <= n1 - 1 + NG + 1: inside the face tables)
          R qd[4], loA[4], hiA[4], ih2[3], fu[4];
          for (int c = 0; c < 4; ++c) qd[c] = QS[buf][c][sw + 2][lane];
          const R ksa = QS[buf][4][sw + 1][lane] + QS[buf][5][sw + 1][lane];
          ih_th(ey + 2, ih2);
          const bool o2f = gld(geo.wf[1], ey + 2) != R(0);
          FaceAux<R> xA;
          reconstruct<R, SPH, 3, LIM>(a, geo, 1, ey + 1, q0, qc, qd, ih1, ih2, o1f, o2f, loA, hiA, nullptr, &xA);
          for (int c = 0; c < 4; ++c) fu[c] = R(0);
          if (o1f) {
            R hf[3];
            h_th(ey + 1, hf);
            hll<R, SPH, 3, (LIM < 0)>(a, 1, hiY, loA, hf, ih1, epsilon_of(ks0, ksa, dly, dly), fu, &xYh, &xA);
            if constexpr (VEL) add_upwind(Uyt, hiY, loA, fu);
          }
          for (int c = 0; c < 4; ++c) FY[buf][c][NI][lane] = fu[c];
        }
      } else {
        reconstruct<R, false, 3, LIM>(a, geo, 1, 0, qa, qb, q0, hone, hone, true, true, lo, hiP, nullptr, nullptr, &xP);
        reconstruct<R, false, 3, LIM>(a, geo, 1, 0, qb, q0, qc, hone, hone, true, true, loY, hiY, nullptr, &xY, &xYh);
        hll<R, false, 3, (LIM < 0)>(a, 1, hiP, loY, hone, hone, epsilon_uniform(ksb, ks0, hdx1), fy, &xP, &xY);
        if constexpr (VEL) add_upwind(Uy, hiP, loY, fy);
        if (AR && top && yz < n1) {
          // the block's upper face
          R qd[4], loA[4], hiA[4], fu[4];
          for (int c = 0; c < 4; ++c) qd[c] = QS[buf][c][sw + 2][lane];
          const R ksa = QS[buf][4][sw + 1][lane] + QS[buf][5][sw + 1][lane];
          FaceAux<R> xA;
          reconstruct<R, false, 3, LIM>(a, geo, 1, 0, q0, qc, qd, hone, hone, true, true, loA, hiA, nullptr, &xA);
          hll<R, false, 3, (LIM < 0)>(a, 1, hiY, loA, hone, hone, epsilon_uniform(ks0, ksa, hdx1), fu, &xYh, &xA);
          if constexpr (VEL) add_upwind(Uyt, hiY, loA, fu);
          for (int c = 0; c < 4; ++c) FY[buf][c][NI][lane] = fu[c];
        }
      }
      for (int c = 0; c < 4; ++c) FY[buf][c][w][lane] = fy[c];
    }
    R acc[4] = {R(0), R(0), R(0), R(0)};
    if (!idle) {
      // ---- x: reconstruction, the flux at the lower x face of the column (the upper state
      // of the column below by a lane shift), the x part of the divergence ----
      {
        R qm[4], qp[4], loX[4], hiX[4];
        for (int c = 0; c < 4; ++c) {
          qm[c] = col_prev_or(q0[c], qo[c]);
          qp[c] = col_next_or(q0[c], qo[c]);
        }
        R qL[4], fx[4];
        FaceAux<R> xX, xXh, xL;
        if constexpr (SPH) {
          // r faces of the lane's zone; the flux at its lower face
          R ihl[3], ihr[3], hf[3];
          const R isc = gld(geo.isc, ey);
          ihl[0] = ihl[1] = rg(RG_IRF0);
          ihl[2] = rg(RG_IRF0) * isc;
          ihr[0] = ihr[1] = rg(RG_IRF1);
          ihr[2] = rg(RG_IRF1) * isc;
          const R vs[5] = {rg(RG_IDM), rg(RG_IDP), rg(RG_DLO), rg(RG_DHI), rg(RG_IDC)};
          reconstruct<R, SPH, 3, LIM>(a, geo, 0, ex, qm, q0, qp, ihl, ihr, true, true, loX, hiX, vs, &xX, &xXh);
          for (int c = 0; c < 4; ++c) qL[c] = col_prev(hiX[c]);
          const R ksL = col_prev(ks0);
          const R dlx = rg(RG_HR) * geo.dx[0];
          const R dlL = col_prev(dlx);
          hf[0] = hf[1] = rg(RG_RF);
          hf[2] = rg(RG_RF) * gld(geo.sc, ey);
          xL.F2 = col_prev(xXh.F2);
          xL.X = R(a.c) * qL[0];
          hll<R, SPH, 3, (LIM < 0)>(a, 0, qL, loX, hf, ihl, epsilon_of(ksL, ks0, dlL, dlx), fx, &xL, &xX);
          if constexpr (VEL) add_upwind(Ux, qL, loX, fx);
          const R wl = rg(RG_WF0), wh = rg(RG_WF1), iW = rg(RG_IW);
          for (int c = 0; c < 4; ++c) acc[c] = (wh * col_next(fx[c]) - wl * fx[c]) * iW;
        } else {
          reconstruct<R, false, 3, LIM>(a, geo, 0, 0, qm, q0, qp, hone, hone, true, true, loX, hiX, nullptr, &xX, &xXh);
          for (int c = 0; c < 4; ++c) qL[c] = col_prev(hiX[c]);
          const R ksL = col_prev(ks0);
          xL.F2 = col_prev(xXh.F2);
          xL.X = R(a.c) * qL[0];
          hll<R, false, 3, (LIM < 0)>(a, 0, qL, loX, hone, hone, epsilon_uniform(ksL, ks0, hdx0), fx, &xL, &xX);
          if constexpr (VEL) add_upwind(Ux, qL, loX, fx);
          for (int c = 0; c < 4; ++c) acc[c] = (col_next(fx[c]) - fx[c]) * idx0;
        }
      }
      // ---- z: reconstruction of zone m + 1, the flux at m + 1/2; the window's face values
      // move on at once ----
      {
        R nLo[4], nHi[4], fNext[4];
        FaceAux<R> xl, xh;
        reconstruct<R, SPH, 3, LIM>(a, geo, 2, NG, q0, q1, q2, ihz, ihz, true, true, nLo, nHi, nullptr, &xl, &xh);
        hll<R, SPH, 3, (LIM < 0)>(a, 2, hiM, nLo, hz, ihz, eps_z(ks0, k1 + s1), fNext, &xM, &xl);
        xM = xh;
        if constexpr (VEL) add_upwind(Uz, hiM, nLo, fNext);
        for (int c = 0; c < 4; ++c) {
          acc[c] += (fNext[c] - fPrev[c]) * idx2;
          fPrev[c] = fNext[c];
          hiM[c] = nHi[c];
        }
      }
    }
    // ---- keep what the update of plane m needs; advance the window ----
    for (int c = 0; c < 4; ++c) {
      qU[c] = q0[c];
      accU[c] = acc[c];
      fyU[c] = fy[c];
      q0[c] = q1[c];
      q1[c] = q2[c];
    }
    kU = k0;
    sU = s0;
    BU = BM;
    k0 = k1;
    s0 = s1;
    p1 = p2;
    p2 = p3;
    y0m = y1m;
    y1m = y2m;
    y2m = y3m;
  }
  c3_barrier();
  if (!idle) update(mend - 1, (mend - 1) & 1);

  if (want_diag)
    wave_diag_store(wd, upd, Vz, w, lane, NI, red_e, red_m, red_u, red_p, a.p_energy, a.p_maxf2, a.p_nun, a.p_nnp);
}

// ------------------------------------------------------------------------------------------
// every row of a block updated: double blocks, and float blocks of 4 and 12 rows (three waves
// per SIMD)
static bool c3_all_rows(const fornax_m1_desc& D, int NR) { return D.precision == FORNAX_FP64 || NR == 4 || NR == 12; }

C3Tile make_c3_tile(const fornax_m1_desc& D, int NR, int TM) {
  C3Tile tl{};
  tl.nblocks = 0;
  if (D.ndim != 3 || (D.precision != FORNAX_FP64 && D.ngroups % 4 != 0)) return tl;
  const bool sph = D.coord == FORNAX_SPHERICAL_LOGR;
  if (!sph && D.coord != FORNAX_CARTESIAN) return tl;
  // the instantiated block heights: 6, 8 or 12 rows in double, 4, 8, 12 or 16 in float
  // (spherical grids: 8 rows, or 4, 8 or 12 in float)
  const bool dbl = D.precision == FORNAX_FP64;
  if (!(NR == 8 || (!dbl && (NR == 4 || NR == 12)) || (!sph && (NR == (dbl ? 6 : 4) || NR == (dbl ? 12 : 16)))))
    return tl;
  if (TM < 1) return tl;
  // inflow only on the lower x1 boundary of spherical grids; a polar axis (theta, spherical
  // grids) needs a periodic phi axis of even length
  for (int d = 0; d < 3; ++d) {
    if (D.bc_hi[d] == FORNAX_BC_INFLOW || (D.bc_lo[d] == FORNAX_BC_INFLOW && !(sph && d == 0))) return tl;
    if ((D.bc_lo[d] == FORNAX_BC_AXIS || D.bc_hi[d] == FORNAX_BC_AXIS) && !(sph && d == 1)) return tl;
  }
  if (sph && (D.bc_lo[1] == FORNAX_BC_AXIS || D.bc_hi[1] == FORNAX_BC_AXIS) &&
      (D.bc_lo[2] != FORNAX_BC_PERIODIC || D.bc_hi[2] != FORNAX_BC_PERIODIC || D.n[2] % 2 != 0))
    return tl;
  tl.NR = NR;
  tl.TM = TM;
  tl.RT = D.ngroups == 1 ? 4 : (D.ngroups == 2 ? 2 : 1);
  tl.ntx = ((D.n[0] + C3_TX - 3) / (C3_TX - 2) + tl.RT - 1) / tl.RT;
  // tiles of NR rows, or NR - 1 (the top row is the next tile's first)
  tl.nty = c3_all_rows(D, NR) ? (D.n[1] + NR - 1) / NR : (D.n[1] + NR - 2) / (NR - 1);
  tl.ntz = (D.n[2] + TM - 1) / TM;
  tl.ngb = (D.ngroups + 3) / 4;
  const int64_t nb = (int64_t)tl.ntx * tl.nty * tl.ntz * tl.ngb;
  if (nb > (int64_t)1 << 30) return C3Tile{};
  tl.nblocks = (int)nb;
  tl.xq = tl.nblocks / 8;
  tl.xr = tl.nblocks % 8;
  return tl;
}

// Planes per block: a block walks its TM planes (and about three planes' worth of start-up: the
// first planes' loads and the face below its first plane, the last deferred update) one after
// the other, so the kernel takes about the number of rounds of block slots times TM + 3.  The
// tile of NR rows with the least such cost (ties: the longer tile), the slots from the shape's
// W waves per SIMD and the CU count.  Measured on MI355X this picks the fastest of the lengths
// tried in each case: 192 planes at 192^3 x 12 FP64 (one tile along z: 2.6 % faster than 64
// and 1 % than 96), 64 in MIXED (7 % faster than 96, 1 % than 32), 128 on the 256 x 64 x 128 x
// 20 spherical grid in FP64 (1 % faster than 32 and 64) and 32 in MIXED (12 % faster than 64).
static C3Tile c3_tile_by_rounds(const fornax_m1_desc& D, int NR, int W, int cus) {
  const int per_cu = std::max(1, 4 * W / NR);
  const long slots = (long)per_cu * (cus > 0 ? cus : 256);
  C3Tile best{};
  double best_cost = 0.0;
  for (int TM = std::min(8, D.n[2]); TM <= D.n[2]; ++TM) {
    const C3Tile t = make_c3_tile(D, NR, TM);
    if (t.nblocks <= 0) continue;
    const double cost = (double)((t.nblocks + slots - 1) / slots) * (TM + 3);
    if (best.nblocks <= 0 || cost <= best_cost) {
      best = t;
      best_cost = cost;
    }
  }
  return best;
}

C3Tile choose_c3_tile(const fornax_m1_desc& D, int cus) {
  // one y row per wave: 8 rows (spherical grids in float: 12, every row updated at three waves
  // per SIMD).  Measured at 192^3 x 12 (Cartesian) and 256 x 64 x 128 x 20 (spherical): float
  // Cartesian blocks of 12 or 4 rows at three waves per SIMD 3 % and 11 % slower than 8 rows;
  // spherical float 12 rows 9 % faster than 4 rows and 22 % faster than 8 rows at four waves
  // per SIMD, which spill registers.  Waves per SIMD as launch_c3 instantiates the shapes:
  // double 2, float Cartesian 4, float spherical 3.
  const bool dbl = D.precision == FORNAX_FP64;
  const bool sph = D.coord == FORNAX_SPHERICAL_LOGR;
  // Group counts that leave rows idle (5 groups: 3 of 8) run here in double where that is faster
  // than on the tiled kernel (c3_pays).  In float they keep the tiled kernel (make_c3_tile refuses
  // them), and its results bit for bit: it adds the three directions in another order, and the
  // float roundings of a step show in its double diagnostics and steer the limiter of the next.
  return c3_tile_by_rounds(D, (sph && !dbl) ? 12 : 8, dbl ? 2 : (sph ? 3 : 4), cus);
}

bool c3_pays(const fornax_m1_desc& D, const C3Tile& c3, const Tile& tiled, int cus) {
  if (c3.nblocks <= 0 || D.ngroups % 4 == 0 || tiled.nblocks <= 0) return true;
  return plane_kernel_pays(c3.nblocks, c3.TM, tiled.nblocks, tiled.nthreads, tiled.TM, D.n[2],
                           D.coord == FORNAX_SPHERICAL_LOGR, D.limiter == FORNAX_LIMITER_MINMOD,
                           D.limiter == FORNAX_LIMITER_PPM, D.wavespeed == FORNAX_WAVESPEED_M1, cus);
}

// Step 1 of the velocity step: 8 rows at two waves per SIMD in double, 12 rows at three in
// float (launch_c3_vel)
C3Tile choose_c3_vel_tile(const fornax_m1_desc& D, int cus) {
  const bool dbl = D.precision == FORNAX_FP64;
  // in float the grids whose Step 1 runs here, and no others (see choose_c3_tile)
  const bool sph = D.coord == FORNAX_SPHERICAL_LOGR;
  if (!dbl && sph) return C3Tile{};
  // spherical grids, and group counts that leave rows idle, from the size on where the blocks
  // fill the chip; below it one thread per zone-group is faster (measured in double: spherical
  // 32 x 8 x 8 x 12 80 against 49 us, 64 x 16 x 24 x 6 105 against 99, 160 x 48 x 80 x 3 276 against
  // 475; Cartesian 20^3 x 3 55 against 42, 40 x 30 x 30 x 3 72 against 71, 144^3 x 3 791 against 1608).
  // Limiters other than minmod, whose instantiation spills registers, from twice the size on (whole
  // step with MC: 20^3 x 17 86 against 62 us, 26^3 x 10 82 against 72, 200 x 100 x 4 x 3 56 against 74;
  // spherical 64 x 32 x 32 x 4 152 against 124, 128 x 48 x 64 x 1 153 against 140, 64 x 24 x 32 x 12
  // 172 against 216)
  const int64_t nzg = (int64_t)D.n[0] * D.n[1] * D.n[2] * D.ngroups;
  const int other = D.limiter != FORNAX_LIMITER_MINMOD ? 1 : 0;
  if ((sph && nzg < (1 << (18 + other))) || (D.ngroups % 4 != 0 && nzg < (1 << (17 + other)))) return C3Tile{};
  return c3_tile_by_rounds(D, dbl ? 8 : 12, dbl ? 2 : 3, cus);
}

template <typename S>
int launch_c3(fornax_m1_ctx* ctx, const Geo<S>& geo, const StepArgs<S>& a, hipStream_t st) {
  const C3Tile& tl = ctx->c3;
  if (tl.nblocks <= 0) return FORNAX_EUNSUPPORTED;
  if (a.dEm && tl.ngb > 1 && !a.dzp) return FORNAX_EUNSUPPORTED;
  // the minmod instantiation has the -+c bounds built in; the other takes both options at run time
  // and spills in double (24 registers on Cartesian grids, 98 on spherical ones; Step 1 of the
  // velocity step 47 and 126): the rules for odd group counts and for Step 1 (plane_kernel_margin,
  // choose_c3_vel_tile) have lines of their own for it
  const bool mm = a.limiter == FORNAX_LIMITER_MINMOD && a.wavespeed == FORNAX_WAVESPEED_LIGHT;
  const bool sph = ctx->desc.coord == FORNAX_SPHERICAL_LOGR;
  dim3 grid(tl.nblocks), block(64 * tl.NR);
  const VelArgs<S> nova{};
#define FM1_C3(NRV, WV, SP, AR)                                                                                       \
  do {                                                                                                                \
    if (mm && !a.Ea)                                                                                                  \
      hipLaunchKernelGGL((k_step_3d<S, NRV, WV, FORNAX_LIMITER_MINMOD, SP, AR, false, false>), grid, block, 0, st, a,  \
                         geo, tl, nova);                                                                              \
    else if (mm)                                                                                                      \
      hipLaunchKernelGGL((k_step_3d<S, NRV, WV, FORNAX_LIMITER_MINMOD, SP, AR, false, true>), grid, block, 0, st, a,   \
                         geo, tl, nova);                                                                              \
    else                                                                                                              \
      hipLaunchKernelGGL((k_step_3d<S, NRV, WV, -1, SP, AR>), grid, block, 0, st, a, geo, tl, nova);                    \
  } while (0)
  // waves per SIMD: the register budget of each shape (double: 168 or 256 VGPRs; float: 128,
  // or 168 for the 4- and 12-row blocks)
  if constexpr (sizeof(S) == 8) {
    if (sph) FM1_C3(8, 2, true, true);
    else if (tl.NR == 6) FM1_C3(6, 3, false, true);
    else if (tl.NR == 8) FM1_C3(8, 2, false, true);
    else FM1_C3(12, 3, false, true);
  } else {
    if (sph && tl.NR == 4) FM1_C3(4, 3, true, true);
    else if (sph && tl.NR == 12) FM1_C3(12, 3, true, true);
    else if (sph) FM1_C3(8, 4, true, false);
    else if (tl.NR == 4) FM1_C3(4, 3, false, true);
    else if (tl.NR == 8) FM1_C3(8, 4, false, false);
    else if (tl.NR == 12) FM1_C3(12, 3, false, true);
    else FM1_C3(16, 4, false, false);
  }
#undef FM1_C3
  Tile lt{};
  lt.nblocks = tl.nblocks;
  lt.ngb = tl.ngb;
  *ctx->last_tile = lt;
  return hipGetLastError() == hipSuccess ? FORNAX_OK : FORNAX_EDEVICE;
}

template int launch_c3<double>(fornax_m1_ctx*, const Geo<double>&, const StepArgs<double>&, hipStream_t);
template int launch_c3<float>(fornax_m1_ctx*, const Geo<float>&, const StepArgs<float>&, hipStream_t);

// Step 1 of the velocity step (transport with the advective fluxes, no interaction update, no
// diagnostics) on 3-D grids of the kernel's kind, in float Cartesian ones only: 8-row blocks in
// double, 12-row blocks (three waves per SIMD) in float, planes per block chosen at create.
template <typename S>
int launch_c3_vel(fornax_m1_ctx* ctx, const Geo<S>& geo, const StepArgs<S>& a, const VelArgs<S>& va, hipStream_t st) {
  const fornax_m1_desc& D = ctx->desc;
  if (D.ndim != 3) return FORNAX_EUNSUPPORTED;
  if (a.src || a.dEm || a.p_energy || a.Ea) return FORNAX_EUNSUPPORTED;
  constexpr bool dbl = sizeof(S) == 8;
  const C3Tile tl = ctx->c3v;
  constexpr int NRV = dbl ? 8 : 12, WV = dbl ? 2 : 3;
  if (tl.nblocks <= 0 || tl.NR != NRV) return FORNAX_EUNSUPPORTED;
  const bool mm = a.limiter == FORNAX_LIMITER_MINMOD && a.wavespeed == FORNAX_WAVESPEED_LIGHT;
  dim3 grid(tl.nblocks), block(64 * tl.NR);
  if (!dbl && D.coord == FORNAX_SPHERICAL_LOGR) return FORNAX_EUNSUPPORTED;
#define FM1_C3V(LIMV, SP) \
  hipLaunchKernelGGL((k_step_3d<S, NRV, WV, LIMV, SP, true, true, false>), grid, block, 0, st, a, geo, tl, va)
  const bool sph = D.coord == FORNAX_SPHERICAL_LOGR;
  if constexpr (dbl) {
    if (mm && sph) FM1_C3V(FORNAX_LIMITER_MINMOD, true);
    else if (sph) FM1_C3V(-1, true);
  }
  if (!sph && mm) FM1_C3V(FORNAX_LIMITER_MINMOD, false);
  else if (!sph) FM1_C3V(-1, false);
#undef FM1_C3V
  return hipGetLastError() == hipSuccess ? FORNAX_OK : FORNAX_EDEVICE;
}

template int launch_c3_vel<double>(fornax_m1_ctx*, const Geo<double>&, const StepArgs<double>&,
                                   const VelArgs<double>&, hipStream_t);
template int launch_c3_vel<float>(fornax_m1_ctx*, const Geo<float>&, const StepArgs<float>&, const VelArgs<float>&,
                                  hipStream_t);

}  // namespace fm1
