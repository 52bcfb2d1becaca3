// m1_velocity_freq.hip -- Step 2 of the velocity step (frequency advection) and the interaction
// update in double, whole zones per wave.
//
// k_vel_freq_wave: a wave holds 64 / G zones, lanes = groups, and needs no other wave: the
// neighbour groups come by lane shifts, the zone's velocity gradient through the wave's own LDS,
// where 9 lanes per zone (ND^2) each form one component instead of every group forming all of
// them (SHARE; small group counts, with more zones per wave than 64 / ND^2, form them per lane).
// Waves stride over the zones and carry their zone indices along, so no zone index is divided.
//
// Bound by memory: 192^3 zones x 12 groups in 3-D, 14 arrays in and out, 2.08 ms (4.6 TB/s; a plain
// kernel that reads 10 arrays and writes 4 of this size takes 1.8 ms with full aligned waves and
// 1.95 with 60 of 64 lanes), against 2.91 ms for whole zones per block (k_vel_freq: 3 barriers per
// pass, 695 vector instructions against 440).  Loads of the next zones in flight across the pass,
// 2 or 3 waves per SIMD, zones in one run per XCD, or non-temporal access: 2.27 to 2.64 ms, on a
// card where this form took 2.31.
//
// The contractions of a zone are taken through the symmetric matrices S = W + W^T of the two sign
// parts W of the gradient: with f = F^/(cE), P^^ = iso delta + ani f f and the third moment
// Q^ = A (f d + d f + ..) + B f f f, whose A = 3/5 c iso and B = c ani,
//   sum_ij W_ij P^^ji = iso tr W + ani f.(S f)/2,
//   row j of the flux terms = A ((S f)_j + f_j tr W) + B f_j f.(S f)/2.
#include <algorithm>

#include "m1_device.h"
#include "m1_grid.h"
#include "m1_internal.h"
#include "m1_lane.h"
#include "m1_step.h"

namespace fm1 {
namespace {

// the value of the lane one lower / higher in the wave (0 for the lane at the wave's end)
__device__ __forceinline__ double wave_prev(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, 0x138, 0xf, 0xf, true);
}
__device__ __forceinline__ double wave_next(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, 0x130, 0xf, 0xf, true);
}

// the part of x below 0, 0 for the rest (one instruction: fmin would first canonicalise x)
__device__ __forceinline__ double neg_part(double x) {
  double r;
  __asm__("v_min_f64 %0, %1, 0" : "=v"(r) : "v"(x));
  return r;
}

// LDS values of a wave written before are read after (its LDS operations run in order)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a zone's indices, carried along in steps of a fixed number of zones
struct ZoneWalk {
  int i, j, k;
  __device__ __forceinline__ void set(unsigned z, int n0, int n1) {
    const unsigned r = z / (unsigned)n0;
    i = (int)(z - r * (unsigned)n0);
    k = (int)(r / (unsigned)n1);
    j = (int)(r - (unsigned)k * (unsigned)n1);
  }
  __device__ __forceinline__ void advance(const ZoneWalk& s, int n0, int n1) {
    i += s.i;
    j += s.j;
    k += s.k;
    if (i >= n0) {
      i -= n0;
      ++j;
    }
    if (j >= n1) {
      j -= n1;
      ++k;
    }
  }
};

// x where the mask is all ones, exactly 0 where it is 0: both halves are cleared, so that nothing of
// another zone's value (its low bits, a NaN or an infinity) passes a closed edge.
__device__ __forceinline__ double keep_masked(double x, unsigned mask) {
  const unsigned long long m = ((unsigned long long)mask << 32) | mask;
  return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, x) & m);
}

}  // namespace

template <bool SPH, int ND, bool SHARE, bool FN>
__global__ void __launch_bounds__(BLOCK, SPH && ND == 3 ? 3 : 4)
    k_vel_freq_wave(StepArgs<double> a, Geo<double> geo, VelArgs<double> va, int want_diag) {
  constexpr int NC = ND * ND;
  constexpr int NV = NC + 1 + (SPH ? 3 : 0);   // gradient, volume, centroid velocity
  constexpr int NW = BLOCK / 64;
  const int n0 = a.n[0], n1 = a.n[1], n2 = a.n[2];
  const int G = a.G, zpw = 64 / G;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool lane_ok = lane < zpw * G;
  const int grp = lane % G, lz = min(lane / G, zpw - 1);
  __shared__ double sG[NW][SHARE ? 64 / NC * NV : 1];
  __shared__ double sdz[NW][64];
  // the group's frequency geometry
  double idm = 0.0, rnlo = 0.0, idnu = 0.0, dnu = 0.0;
  if (lane_ok) {
    const double nlo = va.nu[grp], nhi = va.nu[grp + 1];
    const double nc = 0.5 * (nlo + nhi);
    if (grp > 0) idm = 1.0 / (nc - 0.5 * (va.nu[grp - 1] + nlo));
    dnu = nhi - nlo;
    idnu = 1.0 / dnu;
    rnlo = nlo;
  }
  const double half = 0.5 * dnu;
  const unsigned interior = lane_ok && grp > 0 && grp < G - 1 ? ~0u : 0u;
  const unsigned lower = lane_ok && grp > 0 ? ~0u : 0u;
  const double c = a.c, dt = a.dt, cdt = c * dt;

  // the wave's zones: zb, zb + stride, ...; the lane's own zone and, with SHARE, the zone and
  // component whose slope it forms
  const unsigned nzones = (unsigned)a.nzones;
  const unsigned stride = gridDim.x * NW * (unsigned)zpw;
  unsigned zb = (blockIdx.x * NW + (unsigned)w) * (unsigned)zpw;
  ZoneWalk step, own, prod;
  step.set(stride, n0, n1);
  own.set(zb + lz, n0, n1);
  const int pz = lane / NC, pc = lane - pz * NC;
  const int pi = pc / ND, pd = pc - pi * ND;
  const bool prod_ok = SHARE && pz < zpw;
  int64_t pup = 1, pm0 = 0, pm1 = 0;
  const double* pv = nullptr;
  double pidx = 0.0;
  if constexpr (SHARE) {
    prod.set(zb + pz, n0, n1);
    pm0 = n0 + (pd == 0), pm1 = n1 + (pd == 1);
    pup = pd == 0 ? 1 : pd == 1 ? n0 : (int64_t)n0 * n1;
    const int64_t nf = pm0 * pm1 * (n2 + (pd == 2));
    pv = (pd == 0 ? va.v[0] : pd == 1 ? va.v[1] : va.v[2]) + pi * nf;
    pidx = pd == 0 ? geo.idx[0] : pd == 1 ? geo.idx[1] : geo.idx[2];
  }
  WaveDiag wd;
  for (; zb < nzones; zb += stride, own.advance(step, n0, n1)) {
    const size_t eb = (size_t)zb * G;
    const bool act = lane_ok && zb + lz < nzones;
    // the velocities and volume factors of the lane's slope first: they are waited for first.
    // Zones past the grid's end (last waves): any zone of the last plane, never used
    double lo = 0.0, hi = 0.0, w0 = 0.0, w1 = 0.0, w2 = 0.0, dl = 0.0;
    if constexpr (SHARE) {
      const int pk = min(prod.k, n2 - 1);
      const double* vp = pv + ((pk * pm1 + prod.j) * pm0 + prod.i);
      lo = vp[0];
      hi = vp[pup];
      w0 = gld(geo.Wd[0], prod.i + NG);
      w1 = gld(geo.Wd[1], prod.j + NG);
      w2 = gld(geo.Wd[2], pk + NG);
      if constexpr (SPH)
        dl = gld(pd == 0 ? geo.dlo[0] : pd == 1 ? geo.dlo[1] : geo.dlo[2],
                 (pd == 0 ? prod.i : pd == 1 ? prod.j : pk) + NG);
      prod.advance(step, n0, n1);
    }
    // the zones' state and coefficients; lanes past the last zone-group read that one
    unsigned off = 8u * min((unsigned)lane, (unsigned)min((size_t)(zpw * G), (size_t)nzones * G - eb) - 1);
    __asm__("" : "+v"(off));
    double q[4] = {0.0, 0.0, 0.0, 0.0}, fn[3] = {0.0, 0.0, 0.0};
    q[0] = ld_off(a.E + eb, off);
    for (int cc = 0; cc < ND; ++cc) q[1 + cc] = ld_off(a.F[cc] + eb, off);
    if constexpr (FN)
      for (int cc = 0; cc < ND; ++cc) fn[cc] = ld_off(va.Fn[cc] + eb, off);
    const double kd = ld_off(a.kap + eb, off), sd = ld_off(a.sig + eb, off), Bd = ld_off(a.B + eb, off);
    // dv[3 ic + jd] = d v^ic / d x^jd of the zone, its volume, its centroid velocity
    double dv[9], vb[3] = {0.0, 0.0, 0.0}, V;
    for (int t = 0; t < 9; ++t) dv[t] = 0.0;
    const int oi = own.i, oj = own.j;
    if constexpr (SHARE) {
      double* o = &sG[w][pz * NV];
      if (prod_ok) {
        o[pc] = (hi - lo) * pidx;
        o[NC] = w0 * w1 * w2;
        // the component's value at the zone's volume centroid
        if (SPH && pi == pd) o[NC + 1 + (SPH ? pd : 0)] = lo - (hi - lo) * (dl * pidx);
      }
      wave_sync();
      const double* s = &sG[w][lz * NV];
      for (int ic = 0; ic < ND; ++ic)
        for (int jd = 0; jd < ND; ++jd) dv[3 * ic + jd] = s[ic * ND + jd];
      V = s[NC];
      if constexpr (SPH)
        for (int kk = 0; kk < ND; ++kk) vb[kk] = s[NC + 1 + kk];
    } else {
      const int ok = min(own.k, n2 - 1);
      for (int jd = 0; jd < ND; ++jd) {
        const int64_t m0 = n0 + (jd == 0), m1 = n1 + (jd == 1), nf = m0 * m1 * (n2 + (jd == 2));
        const int64_t up = jd == 0 ? 1 : jd == 1 ? n0 : (int64_t)n0 * n1;
        const double* vp = va.v[jd] + (ok * m1 + oj) * m0 + oi;
        for (int ic = 0; ic < ND; ++ic) {
          const double lo = vp[ic * nf], hi = vp[ic * nf + up];
          dv[3 * ic + jd] = (hi - lo) * geo.idx[jd];
          if (SPH && ic == jd)
            vb[jd] = lo - (hi - lo) * (gld(geo.dlo[jd], (jd == 0 ? oi : jd == 1 ? oj : ok) + NG) * geo.idx[jd]);
        }
      }
      V = geo.Wd[0][oi + NG] * geo.Wd[1][oj + NG] * geo.Wd[2][ok + NG];
    }
    // Step 1 on the transport kernel left the zone-local velocity terms of the flux rows to this
    // one: <Gamma^l_ik> <v^i> F_l - <v^i_;k> F_i = - v^i_,k F_i of U^n (the connection is
    // symmetric in its lower indices)
    if constexpr (FN)
      for (int kk = 0; kk < ND; ++kk)
        for (int ic = 0; ic < ND; ++ic) q[1 + kk] = fma(-dv[3 * ic + kk], dt * fn[ic], q[1 + kk]);
    // <v^i_;k> in the frame of the physical components (times h_i / h_k)
    double h[3] = {1.0, 1.0, 1.0}, ih[3] = {1.0, 1.0, 1.0};
    double Vt[9];
    for (int t = 0; t < 9; ++t) Vt[t] = dv[t];
    if constexpr (SPH) {
      cell_h<double, SPH>(geo, oi + NG, oj + NG, h);
      cell_ih<double, SPH>(geo, oi + NG, oj + NG, ih);
      const double* g = geo.gam + 4 * oj;
      const double G323 = g[0], G133 = g[1], G233 = g[2], G222 = g[3];
      Vt[0] += vb[0];
      Vt[1] -= vb[1];
      Vt[3] += vb[1];
      Vt[4] += fma(G222, vb[1], vb[0]);
      Vt[8] += fma(G323, vb[1], vb[0]);
      if constexpr (ND == 3) {
        Vt[2] = fma(G133, vb[2], Vt[2]);
        Vt[5] = fma(G233, vb[2], Vt[5]);
        Vt[6] += vb[2];
        Vt[7] = fma(G323, vb[2], Vt[7]);
        const double r02 = h[0] * ih[2], r20 = h[2] * ih[0];
        Vt[2] *= r02;
        Vt[5] *= r02;
        Vt[6] *= r20;
        Vt[7] *= r20;
      }
    }
    // f = F^/(cE), |f| <= 1, and the closure's coefficients over E; E <= 0, |f| > 1 and a subnormal
    // cE, whose reciprocal is infinite (f^2 is then no number), in a branch that only waves holding
    // one take
    const double E = q[0];
    double cE = c * E;
    const double icE = rcp_(cE);
    double f[3] = {0.0, 0.0, 0.0}, f2 = 0.0;
    for (int k = 0; k < ND; ++k) {
      f[k] = (SPH ? q[1 + k] * ih[k] : q[1 + k]) * icE;
      f2 = fma(f[k], f[k], f2);
    }
    if (__builtin_amdgcn_ballot_w64(!(E > 0.0) || !(f2 <= 1.0))) {
      __asm__ volatile("");
      // (the same f for a cE of ordinary size; a tiny one from the state scaled by 2^600, exactly)
      const double up = cE < 0x1p-400 ? 0x1p600 : 1.0;
      const double iu = rcp_(c * (E * up));
      f2 = 0.0;
      for (int k = 0; k < ND; ++k) {
        f[k] = (SPH ? q[1 + k] * ih[k] : q[1 + k]) * up * iu;
        f2 = fma(f[k], f[k], f2);
      }
      const double sc = rcp_(sqrt_(f2));
      const bool pos = E > 0.0, big = f2 > 1.0;
      for (int k = 0; k < ND; ++k) f[k] = pos ? (big ? f[k] * sc : f[k]) : 0.0;
      f2 = pos ? (big ? 1.0 : f2) : 0.0;
      cE = pos ? cE : 0.0;
    }
    double iso = 1.0 / 3.0, ani = 0.0;
    if (!a.closure) {
      const double s = sqrt_(fma(-3.0, f2, 4.0));
      const double r = rcp_((1.0 + s) * (2.0 + s));
      iso = (1.0 - f2) * (2.0 + s) * r;
      ani = fma(3.0, s, 3.0) * r;
    }
    iso *= idnu;
    ani *= idnu;
    const double eiso = E * iso, eani = 0.5 * (E * ani), yt = 0.6 * (cE * iso), ya = 0.5 * (cE * ani);
    // the parts of the contractions, sd = 0 where the gradient is below 0 (taken at a group's
    // upper edge) and 1 (at its lower edge): energy row, flux rows
    double W[2][9];
    for (int t = 0; t < 9; ++t) {
      // (the rounded component, not its last product contracted into the difference, whose
      // rounding would remain in the part that has to be exactly 0)
      if ((t / 3 < ND && t % 3 < ND) || (SPH && t % 4 == 0)) __asm__("" : "+v"(Vt[t]));
      W[0][t] = neg_part(Vt[t]);
      W[1][t] = Vt[t] - W[0][t];
    }
    double val[2][4];
    for (int sd2 = 0; sd2 < 2; ++sd2) {
      const double* M = W[sd2];
      const double s01 = M[1] + M[3], s02 = M[2] + M[6], s12 = M[5] + M[7];
      const double tr = M[0] + M[4] + M[8];
      double sf[3];
      sf[0] = 2.0 * M[0] * f[0] + s01 * f[1] + s02 * f[2];
      sf[1] = s01 * f[0] + 2.0 * M[4] * f[1] + s12 * f[2];
      sf[2] = s02 * f[0] + s12 * f[1] + 2.0 * M[8] * f[2];
      const double fsf = f[0] * sf[0] + f[1] * sf[1] + f[2] * sf[2];
      val[sd2][0] = fma(eani, fsf, eiso * tr);
      const double u = fma(ya, fsf, yt * tr);
      for (int k = 0; k < ND; ++k) {
        const double y = fma(yt, sf[k], u * f[k]);
        val[sd2][1 + k] = SPH ? h[k] * y : y;
      }
    }
    const double vP = (val[0][0] + val[1][0]) * dnu;
    // edge values by limited slopes over the group-centre distances, then the fluxes through the
    // group's lower edge; the upper edge's is the next lane's
    for (int r = 0; r <= ND; ++r) {
      double ed[2];
      for (int sd2 = 0; sd2 < 2; ++sd2) {
        const double v = val[sd2][r];
        const double am = (v - wave_prev(v)) * idm;
        const double ap = wave_next(am);
        ed[sd2] = fma(minmod(keep_masked(am, interior), ap), sd2 == 0 ? half : -half, v);
      }
      const double em = wave_prev(ed[0]);
      const double fl = keep_masked(rnlo * (em + ed[1]), lower);
      q[r] = fma(dt, (wave_next(fl) - fl) - (r == 0 ? vP : 0.0), q[r]);
    }
    // Steps 3 and 4
    const double ck = cdt * kd, cks = cdt * (kd + sd), jB = ck * Bd;
    double E1, F1[3] = {0.0, 0.0, 0.0};
    const double dz = source_update<double, double, ND>(q, ck, cks, jB, E1, F1);
    if (act) {
      st_off(a.Eo + eb, off, E1);
      for (int cc = 0; cc < ND; ++cc) st_off(a.Fo[cc] + eb, off, F1[cc]);
    }
    if (want_diag) {
      const double Ed = act ? E1 : 0.0;
      double Fd[3] = {0.0, 0.0, 0.0};
      for (int k = 0; k < ND; ++k) Fd[k] = SPH ? F1[k] * ih[k] : F1[k];
      wd.esum = fma(V, Ed, wd.esum);
      wave_diag_count<double, ND>(c, Ed, Fd, __builtin_amdgcn_ballot_w64(act), wd);
    }
    if (a.dEm) {
      sdz[w][lane] = dz;
      wave_sync();
      if (act && grp == 0) {
        double s = 0.0;
        for (int g2 = 0; g2 < G; ++g2) s += sdz[w][lane + g2];
        a.dEm[zb + lz] = -s;
      }
      wave_sync();
    } else if constexpr (SHARE) {
      wave_sync();
    }
  }
  if (!want_diag) return;
  __shared__ double we[NW], wm[NW];
  __shared__ int wu[NW], wp[NW];
  wave_diag_store(wd, lane_ok, 1.0, w, lane, NW, we, wm, wu, wp, a.p_energy, a.p_maxf2, a.p_nun, a.p_nnp);
}

namespace {
template <bool SPH, int ND, bool FN>
int launch_freq(const StepArgs<double>& b, const Geo<double>& geo, const VelArgs<double>& va, int nb, int want,
                hipStream_t st) {
  // one lane per (zone, component) of the velocity gradient
  if ((64 / b.G) * ND * ND <= 64)
    hipLaunchKernelGGL((k_vel_freq_wave<SPH, ND, true, FN>), dim3(nb), dim3(BLOCK), 0, st, b, geo, va, want);
  else if constexpr (ND > 1)
    hipLaunchKernelGGL((k_vel_freq_wave<SPH, ND, false, FN>), dim3(nb), dim3(BLOCK), 0, st, b, geo, va, want);
  return hipGetLastError() == hipSuccess ? FORNAX_OK : FORNAX_EDEVICE;
}
}  // namespace

int launch_vel_freq_wave(const fornax_m1_ctx* ctx, const StepArgs<double>& b, const VelArgs<double>& va, int* nblocks,
                         int want, hipStream_t st) {
  const int64_t zpb = (int64_t)(64 / b.G) * (BLOCK / 64);
  const int64_t slots = 64 * (int64_t)(ctx->cus > 0 ? ctx->cus : 256);
  const bool sph = ctx->desc.coord == FORNAX_SPHERICAL_LOGR;
  // as many blocks per CU at least as the registers hold: 4, on spherical 3-D grids 3 (384 x 384 x 24
  // 315 -> 305 us against the step tiling's blocks, 256 x 256 x 24 142 -> 135; 4 on the spherical
  // 96 x 32 x 48 x 12 leave a round of blocks a third full: this kernel 51 -> 62 us)
  const int64_t need = std::min<int64_t>((b.nzones + zpb - 1) / zpb, slots);
  const int nb = (int)stride_blocks(need, ctx->nb_partials, ctx->nb_entries, sph && ctx->desc.ndim == 3 ? 3 : 4,
                                    ctx->cus);
  *nblocks = nb;
  const int shape = ctx->desc.ndim * 2 + (sph ? 1 : 0);
  if (va.Fn[0])   // 3-D grids only
    return sph ? launch_freq<true, 3, true>(b, ctx->geo_d, va, nb, want, st)
               : launch_freq<false, 3, true>(b, ctx->geo_d, va, nb, want, st);
  switch (shape) {
    case 2: return launch_freq<false, 1, false>(b, ctx->geo_d, va, nb, want, st);
    case 3: return launch_freq<true, 1, false>(b, ctx->geo_d, va, nb, want, st);
    case 4: return launch_freq<false, 2, false>(b, ctx->geo_d, va, nb, want, st);
    case 5: return launch_freq<true, 2, false>(b, ctx->geo_d, va, nb, want, st);
    case 6: return launch_freq<false, 3, false>(b, ctx->geo_d, va, nb, want, st);
    default: return launch_freq<true, 3, false>(b, ctx->geo_d, va, nb, want, st);
  }
}

}  // namespace fm1
