// m1_matter.hip -- the radiation-matter energy exchange (Interaction Terms: the inner
// backward-Euler update of every group, eq:be_update, inside the outer solve for the matter
// temperature; photons: one equation) and the matter model's opacities and emission.
//
// Layout: a zone's groups on consecutive lanes (lanes per zone = the power of two >= G, at
// most 64, so a zone never spans two waves); the outer iteration is uniform over a zone's
// lanes and the group sums are butterfly reductions among them.  Everything in double.

#include <hip/hip_runtime.h>

#include <cmath>

#include "m1_device.h"
#include "m1_internal.h"
#include "m1_lane.h"

namespace fm1 {

namespace {

constexpr int MBLOCK = 256;

struct MatterTab {
  const double* nu_edge;   // [G + 1]
  const double* nu_c;      // [G]
  const double* kg;        // [G]
  double a_rad, tol;
  int maxn;
};

template <typename S>
struct MatterArgs {
  S* E;
  S* F[3];
  const S* sig;
  const double* cv;
  const double* kappa0;
  double* T;
  double* dEm;
  int* iters;
  MatterTab tab;
  int G, ndim, lg;      // lanes per zone = 1 << lg
  int64_t nzones;
  double c, dt;
};

// 1/x and sqrt(x) of normal positive arguments to about an ulp: the hardware estimates refined
// by two Newton-Raphson steps (the library division and square root spend twice the
// instructions on scaling and on the last half ulp).
__device__ __forceinline__ double rcp2(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// a b + c with the constant c held in scalar registers: a Horner step is then one instruction (the
// compiler copies a constant addend into vector registers first, one move per step).  a and b
// never come straight from a transcendental instruction.
__device__ __forceinline__ double fma_c(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

// e^(-x) and e^(-x) - 1 for 0 <= x <= EXP_MAX: x = -n ln 2 - r with |r| <= ln(2)/2 (ln 2 in two
// parts, the first of 42 bits so that n times it is exact), e^r - 1 by its Taylor series through
// r^13 (the next term is below 5e-18 there), scaled by 2^n.  e^(-EXP_MAX) underflows to 0.
constexpr double EXP_MAX = 800.0;
__device__ __forceinline__ void exp_neg(double x, double& q, double& em) {
  const double n = rint(x * -1.4426950408889634);
  const double r = fma(n, -0x1.ef35793c7673p-45, fma(n, -0x1.62e42fefa38p-1, -x));
  double p = 1.0 / 6227020800.0;
  p = fma_c(p, r, 1.0 / 479001600.0);
  p = fma_c(p, r, 1.0 / 39916800.0);
  p = fma_c(p, r, 1.0 / 3628800.0);
  p = fma_c(p, r, 1.0 / 362880.0);
  p = fma_c(p, r, 1.0 / 40320.0);
  p = fma_c(p, r, 1.0 / 5040.0);
  p = fma_c(p, r, 1.0 / 720.0);
  p = fma_c(p, r, 1.0 / 120.0);
  p = fma_c(p, r, 1.0 / 24.0);
  p = fma_c(p, r, 1.0 / 6.0);
  p = fma_c(p, r, 0.5);
  const double e = fma(r * r, p, r);
  const int k = (int)n;
  const double s = ldexp(1.0, k);
  q = ldexp(1.0 + e, k);
  em = fma(s, e, s - 1.0);
}

// The Planck integrals int x^3 / (e^x - 1) dx of one group edge: from 0 below the split, to
// infinity from the split on.  The split lies where the two are about equal, which makes the
// worst cancellation between a group's two edge values smallest, and both series are short and
// of fixed length: 14 coefficients below it, four sums of PLANCK_N terms above it (a split at 1.5,
// where 12 Bernoulli terms suffice, needs 26 terms above it).
constexpr double PLANCK_SPLIT = 3.5;
constexpr int PLANCK_N = 10;   // e^(-3.5 n) terms left out: 3e-17 of the integral at the split
// int_0^split and int_split^inf (their sum is pi^4/15)
constexpr double PLANCK_HS = 3.242940546215698, PLANCK_HH = 3.250998856051131;
// sum_{j >= 1} B_2j / ((2j)! (2j + 3)) y^(j-1), the even part of the expansion
// int_0^x = x^3 (1/3 - x/8 + sum_j B_2j/((2j)! (2j+3)) x^(2j)), as the polynomial in y = x^2 that
// interpolates it at the 14 Chebyshev points of [0, split^2] (4e-18 of the integral), highest
// power first
constexpr double c_low[14] = {
    -4.579610424450894e-25,  5.874799171410437e-23,  -4.006866021371855e-21, 2.0518102281657752e-19,
    -9.313783042183928e-18,  4.0790272619149505e-16, -1.7835812091183352e-14, 7.871924029860963e-13,
    -3.522789804744265e-11,  1.605904329043872e-09,  -7.51563251067359e-08,   3.674309229841219e-06,
    -0.000198412698412694,   0.016666666666666666};

__device__ __forceinline__ double planck_low(double x) {
  const double y = x * x;
  double p = c_low[0];
#pragma unroll
  for (int k = 1; k < 14; ++k) p = fma_c(p, y, c_low[k]);
  return x * y * fma(y, p, fma(x, -0.125, 1.0 / 3.0));
}

// sum over n of int_x^inf x^3 e^(-n x) = x^3 q^n/n + 3 x^2 q^n/n^2 + 6 x q^n/n^3 + 6 q^n/n^4,
// q = e^(-x): four polynomials in q, each by Horner's rule (independent chains)
__device__ __forceinline__ double planck_high(double x, double q) {
  constexpr double N = PLANCK_N;
  double a = 1.0 / N, b = 1.0 / (N * N), c = 1.0 / (N * N * N), d = 1.0 / (N * N * N * N);
#pragma unroll
  for (int n = PLANCK_N - 1; n >= 1; --n) {
    const double m = n;
    a = fma_c(a, q, 1.0 / m);
    b = fma_c(b, q, 1.0 / (m * m));
    c = fma_c(c, q, 1.0 / (m * m * m));
    d = fma_c(d, q, 1.0 / (m * m * m * m));
  }
  return q * fma(x, fma(x, fma(x, a, 3.0 * b), 6.0 * c), 6.0 * d);
}

// one edge's value, below the split (low) or above it, at x[0] and, with P = 2, at a nearby x[1]
// (relatively 1e-7 apart) in the same form: the integral over [x[1], x[0]] by the midpoint rule
// (its error, the cube of the width, is far below rounding)
template <int P>
__device__ __forceinline__ void planck_edge(const double* x, bool low, double* v) {
  const double xc = fmin(x[0], EXP_MAX);
  double q, em;
  exp_neg(xc, q, em);
  if (low) v[0] = planck_low(xc);
  else v[0] = planck_high(xc, q);
  if constexpr (P == 2) {
    // x^3 / (e^x - 1) at the midpoint, from e^(-x) there (x = 0: 0)
    const double w = xc - fmin(x[1], EXP_MAX), u = 0.5 * w;
    const double m = xc - u;
    const double e = fma(q, u * fma(u, 0.5, 1.0), em);   // e^(-m) - 1
    const double f = w * (m * m * m) * (1.0 + e) * rcp2(xc > 0.0 ? -e : 1.0);
    v[1] = low ? v[0] - f : v[0] + f;
  }
}

// integral over a group from the values va, vb of its edges, each from 0 (its flag set) or to
// infinity, without subtracting two nearly equal integrals
__device__ __forceinline__ double planck_part(bool a_low, bool b_low, double va, double vb) {
  return b_low ? vb - va : (a_low ? (PLANCK_HS - va) + (PLANCK_HH - vb) : va - vb);
}

// the value v of the lane whose byte address (4 x lane) is addr
__device__ __forceinline__ double lane_value(int addr, double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute(addr, (int)(unsigned)b);
  const unsigned hi = (unsigned)__builtin_amdgcn_ds_bpermute(addr, (int)(unsigned)(b >> 32));
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// v of the next lane (a zone's last lane does not use it): a row shift where zones lie inside
// 16-lane rows, through LDS otherwise
__device__ __forceinline__ double next_lane(double v, int lg) {
  if (lg <= 4) return row_dpp<0x101>(v);
  return lane_value((((int)threadIdx.x + 1) & 63) << 2, v);
}

// A lane's group: opacity and emission at P nearby temperatures (T[1] = T[0] (1 + 1e-7)).  A
// lane evaluates the Planck integral at its group's lower edge and takes the upper edge's value
// from the next lane; a zone's last lane, when it holds a group, evaluates the top edge itself
// (lanes past the last group evaluate the top edge).  All lanes of a zone call together.
struct GroupLane {
  double nuc, nlo, nhi, pnorm;
  double ntop;       // the top edge where the zone's last lane holds a group, else infinite
  bool last;         // the zone's last lane
  int lg;
  __device__ __forceinline__ GroupLane(const MatterTab& tab, int G, int g, int lg_) : lg(lg_) {
    const int gg = g < G ? g : 0;
    nuc = tab.nu_c[gg];
    nlo = tab.nu_edge[g < G ? g : G];
    nhi = tab.nu_edge[gg + 1];
    last = g == (1 << lg) - 1;
    ntop = G == (1 << lg) ? tab.nu_edge[G] : INFINITY;
    pnorm = tab.a_rad * 15.0 / (M_PI * M_PI * M_PI * M_PI);
  }
  // EX: quotients and root correctly rounded (an error of x = nu/T shows x times as large in e^(-x)):
  // for the coefficients that are kept as they are
  template <int P, bool EX = false>
  __device__ __forceinline__ void at(const double* T, double kq, double* kap, double* B) const {
    static_assert(P == 1 || !EX, "one temperature");
    double iT[P], xa[P], va[P], vb[P];
    double qa, em;
    if constexpr (EX) {
      exp_neg(fmin(nuc / T[0], EXP_MAX), qa, em);
      kap[0] = kq / sqrt(T[0]) * -em;
      xa[0] = nlo / T[0];
    } else {
      double is[P];
      iT[0] = rcp2(T[0]);
      is[0] = sqrt_(iT[0]);
      const double a = fmin(nuc * iT[0], EXP_MAX);
      exp_neg(a, qa, em);
      kap[0] = kq * is[0] * -em;
      if constexpr (P == 2) {
        // 1/T' and 1/sqrt(T') from those of T by the binomial series in (T' - T)/T
        const double e = (T[1] - T[0]) * iT[0];
        iT[1] = fma(iT[0], e * (e - 1.0), iT[0]);
        is[1] = fma(is[0], e * fma(e, 0.375, -0.5), is[0]);
        // e^(-a') - 1 = (e^(-a) - 1) + e^(-a) (e^u - 1), u = a - a' small
        const double u = a - fmin(nuc * iT[1], EXP_MAX);
        const double e1 = fma(qa, u * fma(u, fma(u, 1.0 / 6.0, 0.5), 1.0), em);
        kap[1] = kq * is[1] * -e1;
      }
      for (int p = 0; p < P; ++p) xa[p] = nlo * iT[p];
    }
    const double Ts = PLANCK_SPLIT * T[0];
    const bool al = nlo < Ts, bl = nhi < Ts;   // (the edge between two lanes: the same for both)
    planck_edge<P>(xa, al, va);
    for (int p = 0; p < P; ++p) vb[p] = next_lane(va[p], lg);
    if (ntop < INFINITY) {
      if (last) {
        double xt[P];
        for (int p = 0; p < P; ++p) xt[p] = EX ? ntop / T[0] : ntop * iT[p];
        planck_edge<P>(xt, bl, vb);
      }
    } else if (last) {
      for (int p = 0; p < P; ++p) vb[p] = 0.0;
    }
    for (int p = 0; p < P; ++p) {
      const double T2 = T[p] * T[p];
      B[p] = pnorm * (T2 * T2) * planck_part(al, bl, va[p], vb[p]);
    }
  }
};

// One lane per zone-group, a zone's groups on consecutive lanes (as k_matter_source): each lane
// evaluates one edge instead of its group's two.  512^2 x 16 in double: 39 us (145 us with both
// edges per lane, library exponentials and data-dependent series lengths; 34 us with reciprocal
// estimates, whose emission far in the Wien tail is off twice as far).
template <typename S>
__global__ void __launch_bounds__(MBLOCK) k_matter_coeffs(MatterArgs<S> a, S* kap_out, S* B_out) {
  const int64_t gt = (int64_t)blockIdx.x * MBLOCK + threadIdx.x;
  const int64_t z = gt >> a.lg;
  const int g = (int)(gt & ((1 << a.lg) - 1));
  if (z >= a.nzones) return;   // whole zones leave together
  const GroupLane gr(a.tab, a.G, g, a.lg);
  const bool on = g < a.G;
  const double T = a.T[z];
  double kap, B;
  gr.at<1, true>(&T, a.kappa0[z] * a.tab.kg[on ? g : 0], &kap, &B);
  if (on) {
    const int64_t i = z * a.G + g;
    kap_out[i] = (S)kap;
    B_out[i] = (S)B;
  }
}

// The interaction update with the outer solve.  Bound by double-precision VALU work (the bytes
// take a tenth of its time), so the work per residual is what counts: the residual and its
// forward-difference neighbour are evaluated together (every accepted temperature needs both),
// sharing the exponentials, and the group sums are lane permutations instead of LDS round
// trips.  512^2 x 16 in double, 3.1 iterations in the slowest zone of a wave: 211 us (767 us with
// separate residuals, library exponentials and series of data-dependent length); VALU issue about
// 60 % of the cycles at five waves per SIMD.
template <typename S>
__global__ void __launch_bounds__(MBLOCK) __attribute__((amdgpu_waves_per_eu(5))) k_matter_source(MatterArgs<S> a) {
  const int64_t gt = (int64_t)blockIdx.x * MBLOCK + threadIdx.x;
  const int64_t z = gt >> a.lg;
  const int g = (int)(gt & ((1 << a.lg) - 1));
  if (z >= a.nzones) return;   // whole zones leave together
  const bool on = g < a.G;
  const int gg = on ? g : 0;
  const int64_t zg = z * a.G + gg;
  const double Em = on ? (double)a.E[zg] : 0.0;
  const double cv = a.cv[z], k0 = a.kappa0[z], Tm = a.T[z];
  const double kq = on ? k0 * a.tab.kg[gg] : 0.0;
  const double cdt = a.c * a.dt;
  const GroupLane gr(a.tab, a.G, g, a.lg);

  // r(T) = cv (T - T^-) + sum_g (E_g(T) - E_g^-), E_g(T) - E_g^- = c dt kappa (B - E^-) / (1 + c dt kappa)
  auto residual = [&](double T) {
    double kap, B;
    gr.at<1>(&T, kq, &kap, &B);
    const double ck = cdt * kap;
    return cv * (T - Tm) + zone_sum(on ? ck * (B - Em) * rcp2(1.0 + ck) : 0.0, a.lg);
  };
  // r(T) and r(T + h), h = 1e-7 T
  auto residual2 = [&](double T, double& r, double& rh) {
    const double Tp[2] = {T, T + 1e-7 * T};
    double kap[2], B[2], s[2];
    gr.at<2>(Tp, kq, kap, B);
    for (int p = 0; p < 2; ++p) {
      const double ck = cdt * kap[p];
      s[p] = zone_sum(on ? ck * (B[p] - Em) * rcp2(1.0 + ck) : 0.0, a.lg);
    }
    r = cv * (Tp[0] - Tm) + s[0];
    rh = cv * (Tp[1] - Tm) + s[1];
  };

  // outer solve: Newton with a forward-difference derivative and backtracking, then bisection.
  // One loop over trial temperatures Tn (one copy of the residual's code): the first is T^-,
  // taken as it is; a later one replaces T where it lowers |r|, else the step is halved
  double T = Tm, Tn = Tm, r = 0.0, T1 = Tm, d = 0.0, lam = 1.0;
  int it = -1, ls = 0, it_out = 0;
  bool done = false;
  while (true) {
    double rn, rhn;
    residual2(Tn, rn, rhn);
    if (it < 0 || fabs(rn) < fabs(r)) {
      const bool conv = it >= 0 && fabs(Tn - T) <= a.tab.tol * Tn;
      T = Tn;
      r = rn;
      ++it;
      if (conv) {
        T1 = T;
        it_out = it;
        done = true;
        break;
      }
      if (it >= a.tab.maxn) break;
      const double h = 1e-7 * T;
      const double dr = rhn - rn;   // J h
      if (!(dr > 0.0)) break;
      d = -r * h * rcp2(dr);
      if (fabs(d) <= a.tab.tol * T) {
        T1 = T + d;
        it_out = it + 1;
        done = true;
        break;
      }
      lam = 1.0;
      ls = 0;
    } else {
      lam *= 0.5;
      ++ls;
    }
    while (ls <= 10 && !((Tn = T + lam * d) > 0.0)) {
      lam *= 0.5;
      ++ls;
    }
    if (ls > 10) break;
  }
  if (!done) {
    const double esum = zone_sum(on ? fmax(Em, 0.0) : 0.0, a.lg);
    double lo = 0.0, hi = Tm + esum / cv;
    int steps = 0;
    while (hi - lo > 1e-13 * hi && steps < 400) {
      const double mid = 0.5 * (lo + hi);
      if (residual(mid) > 0.0)
        hi = mid;
      else
        lo = mid;
      ++steps;
    }
    T1 = 0.5 * (lo + hi);
    it_out = -steps;
  }

  // the groups at T^{n+1}, the fluxes with the new opacity (every lane of the zone calls)
  double kap, B;
  gr.at<1>(&T1, kq, &kap, &B);
  if (on) {
    a.E[zg] = (S)((Em + cdt * kap * B) / (1.0 + cdt * kap));
    const double den = 1.0 + cdt * (kap + (double)a.sig[zg]);
    for (int k = 0; k < a.ndim; ++k) a.F[k][zg] = (S)((double)a.F[k][zg] / den);
  }
  if (g == 0) {
    a.T[z] = T1;
    if (a.dEm) a.dEm[z] = cv * (T1 - Tm);
    if (a.iters) a.iters[z] = it_out;
  }
}

template <typename S>
void fill_matter(const fornax_m1_ctx* ctx, MatterArgs<S>& a, const fornax_m1_matter* m) {
  const int G = ctx->desc.ngroups;
  a.G = G;
  a.ndim = ctx->desc.ndim;
  int lg = 0;
  while ((1 << lg) < G) ++lg;
  a.lg = lg;
  a.nzones = (int64_t)ctx->desc.n[0] * ctx->desc.n[1] * ctx->desc.n[2];
  a.c = ctx->desc.c;
  a.cv = m->cv;
  a.kappa0 = m->kappa0;
  a.T = m->T;
  a.tab.nu_edge = ctx->mat_tab;
  a.tab.nu_c = ctx->mat_tab + (G + 1);
  a.tab.kg = ctx->mat_tab + (2 * G + 1);
  a.tab.a_rad = ctx->mat_a;
  a.tab.tol = ctx->mat_tol;
  a.tab.maxn = ctx->mat_maxn;
  a.dEm = nullptr;
  a.iters = nullptr;
  a.sig = nullptr;
  a.E = nullptr;
  for (int k = 0; k < 3; ++k) a.F[k] = nullptr;
}

template <typename S>
int launch_matter_coeffs_t(fornax_m1_ctx* ctx, const fornax_m1_matter* m, void* kap, void* B, hipStream_t st) {
  MatterArgs<S> a;
  fill_matter<S>(ctx, a, m);
  const int64_t n = a.nzones << a.lg;
  if (n == 0) return FORNAX_OK;
  hipLaunchKernelGGL(k_matter_coeffs<S>, dim3((unsigned)((n + MBLOCK - 1) / MBLOCK)), dim3(MBLOCK), 0, st, a, (S*)kap,
                     (S*)B);
  return hipGetLastError() == hipSuccess ? FORNAX_OK : FORNAX_EDEVICE;
}

template <typename S>
int launch_matter_source_t(fornax_m1_ctx* ctx, fornax_m1_state* io, const void* sigma, const fornax_m1_matter* m,
                           double dt, double* dEm, int* iters, hipStream_t st) {
  MatterArgs<S> a;
  fill_matter<S>(ctx, a, m);
  a.E = (S*)io->E;
  for (int k = 0; k < ctx->desc.ndim; ++k) a.F[k] = (S*)io->F[k];
  a.sig = (const S*)sigma;
  a.dt = dt;
  a.dEm = dEm;
  a.iters = iters;
  const int64_t n = a.nzones << a.lg;
  if (n == 0) return FORNAX_OK;
  hipLaunchKernelGGL(k_matter_source<S>, dim3((unsigned)((n + MBLOCK - 1) / MBLOCK)), dim3(MBLOCK), 0, st, a);
  return hipGetLastError() == hipSuccess ? FORNAX_OK : FORNAX_EDEVICE;
}

}  // namespace

}  // namespace fm1

int fm1_launch_matter_coeffs(fornax_m1_ctx* ctx, const fornax_m1_matter* m, void* kap, void* B, hipStream_t stream) {
  if (ctx->desc.precision == FORNAX_FP64) return fm1::launch_matter_coeffs_t<double>(ctx, m, kap, B, stream);
  return fm1::launch_matter_coeffs_t<float>(ctx, m, kap, B, stream);
}

int fm1_launch_matter_source(fornax_m1_ctx* ctx, fornax_m1_state* io, const void* sigma, const fornax_m1_matter* m,
                             double dt, double* dEm, int* iters, hipStream_t stream) {
  if (ctx->desc.precision == FORNAX_FP64)
    return fm1::launch_matter_source_t<double>(ctx, io, sigma, m, dt, dEm, iters, stream);
  return fm1::launch_matter_source_t<float>(ctx, io, sigma, m, dt, dEm, iters, stream);
}
