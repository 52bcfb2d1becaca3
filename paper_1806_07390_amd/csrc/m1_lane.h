// m1_lane.h -- device helpers of the step kernels whose waves are rows of 16 x columns by 4
// groups (or units): x neighbours by lane shifts, sums over a zone's groups by row swaps, the
// ghost rules of an axis, loads at a uniform base plus a 32-bit lane offset.
#pragma once

#include "m1_device.h"
#include "m1_internal.h"

namespace fm1 {

constexpr int C3_TX = 16;   // x columns of a wave row (14 updated)

// the value of the lane one column lower (row_shr:1) / higher (row_shl:1) in the same 16-lane
// row; the lanes at the row's ends receive 0 (bound_ctrl: they never use it, and no register
// has to be cleared first)
template <typename R>
__device__ __forceinline__ R col_prev(R v) {
  return __builtin_amdgcn_update_dpp(R(0), v, 0x111, 0xf, 0xf, true);
}
template <typename R>
__device__ __forceinline__ R col_next(R v) {
  return __builtin_amdgcn_update_dpp(R(0), v, 0x101, 0xf, 0xf, true);
}

// the same with the lane at the row's end (no lane below / above it) keeping `old`
template <typename R>
__device__ __forceinline__ R col_prev_or(R v, R old) {
  return __builtin_amdgcn_update_dpp(old, v, 0x111, 0xf, 0xf, false);
}
template <typename R>
__device__ __forceinline__ R col_next_or(R v, R old) {
  return __builtin_amdgcn_update_dpp(old, v, 0x101, 0xf, 0xf, false);
}

// v of this lane plus v of the lane 16 (S = 16) or 32 (S = 32) apart, by the row swaps of
// gfx950 (VALU; the lane sums are formed in the same order as a shuffle sum would)
template <int S>
__device__ __forceinline__ double lane_pair_sum(double v) {
  struct W {
    unsigned lo, hi;
  };
  const W w = __builtin_bit_cast(W, v);
  W a, b;
  if constexpr (S == 16) {
    const auto l = __builtin_amdgcn_permlane16_swap(w.lo, w.lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(w.hi, w.hi, false, false);
    a = W{l[0], h[0]};
    b = W{l[1], h[1]};
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap(w.lo, w.lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(w.hi, w.hi, false, false);
    a = W{l[0], h[0]};
    b = W{l[1], h[1]};
  }
  return __builtin_bit_cast(double, a) + __builtin_bit_cast(double, b);
}

template <int CTRL>
__device__ __forceinline__ double row_dpp(double v) {
  return __builtin_amdgcn_update_dpp(0.0, v, CTRL, 0xf, 0xf, true);
}

// sum of v over the 2^lg lanes of a zone, in every lane: butterfly order; inside a 16-lane row
// by lane permutations of the VALU (neighbour pairs, pairs of pairs, mirrored halves and rows:
// the lanes of a pair or a half hold equal sums by then)
__device__ __forceinline__ double zone_sum(double v, int lg) {
  if (lg >= 1) v += row_dpp<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  if (lg >= 2) v += row_dpp<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  if (lg >= 3) v += row_dpp<0x141>(v);   // row_half_mirror
  if (lg >= 4) v += row_dpp<0x140>(v);   // row_mirror
  if (lg >= 5) v += __shfl_xor(v, 16);
  if (lg >= 6) v += __shfl_xor(v, 32);
  return v;
}

// the advective flux v U of the upwind face state added to a face flux (the left state where
// v >= 0)
template <typename R>
__device__ __forceinline__ void add_upwind(R v, const R qL[4], const R qR[4], R flux[4]) {
  const bool left = v >= R(0);
  for (int c = 0; c < 4; ++c) flux[c] += v * (left ? qL[c] : qR[c]);
}

// The ghost rules of one axis, taken from the launch's table at each use (measured: faster
// than copies of the table held in scalar registers for the whole kernel, which crowd out the
// other uniform values).
struct C3Axis {
  const StepArgsBase* a;
  int d;
};
template <int D>
__device__ __forceinline__ C3Axis c3_axis(const StepArgsBase& a) { return C3Axis{&a, D}; }
// Ghost rule of index e (clamped into -2 .. n + 1 first): source zone and flags (bit 0 flips
// the flux component along the axis), selected without indexing the table by a per-lane value.
__device__ __forceinline__ void c3_src(const C3Axis& ax, int e, int& src, int& fl) {
  const StepArgsBase& a = *ax.a;
  const int D = ax.d;
  const int n = a.n[D];
  e = e < -2 ? -2 : (e > n + 1 ? n + 1 : e);
  src = e;
  fl = 0;
  if (e < 0 || e >= n) {
    const int k = e < 0 ? e + 2 : e - n + 2;
    src = k == 0 ? a.gsrc[D][0] : k == 1 ? a.gsrc[D][1] : k == 2 ? a.gsrc[D][2] : a.gsrc[D][3];
    fl = k == 0 ? a.gfl[D][0] : k == 1 ? a.gfl[D][1] : k == 2 ? a.gfl[D][2] : a.gfl[D][3];
  }
}

// the element at a uniform pointer plus a 32-bit byte offset of the lane (one scalar base and
// one vector register of address, no 64-bit address arithmetic per lane)
template <typename S>
__device__ __forceinline__ S ld_off(const S* base, unsigned off) {
  return *reinterpret_cast<const S*>(reinterpret_cast<const char*>(base) + off);
}
template <typename S>
__device__ __forceinline__ void st_off(S* base, unsigned off, S v) {
  *reinterpret_cast<S*>(reinterpret_cast<char*>(base) + off) = v;
}

// v with its sign flipped where the sign mask (0 or the top bit) says so
__device__ __forceinline__ double flip_sign(double v, unsigned mask) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v) ^ ((unsigned long long)mask << 32);
  return __builtin_bit_cast(double, b);
}
__device__ __forceinline__ float flip_sign(float v, unsigned mask) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, v) ^ mask);
}

// Diagnostics of a wave whose lanes keep their role (a zone column, updated or not) over the
// whole kernel: each lane's sum of E^{n+1} and largest f^2 (as the ratio fnum / fden), and the
// wave's counts, taken from the compare masks by the scalar unit.  Called by all lanes of the
// wave together; the lanes outside `upd` hold values that the reduction at the end ignores.
// The largest f^2 is compared by cross-multiplication, its selects run only in waves where some
// lane finds a larger one.
struct WaveDiag {
  double esum = 0.0, fnum = 0.0, fden = 1.0;
  int nun = 0, nnp = 0;
};
// SEL: by selects in every wave instead (the 2-D tiles, whose planes are short chains of
// latencies: 512 x 512 x 16 0.7 % faster than with the branch; the 3-D kernel the other way round).
template <typename S, int ND, bool SEL = false>
__device__ __forceinline__ void wave_diag_count(double c, double E1, const double F1[3], unsigned long long upd,
                                                WaveDiag& wd) {
  double Es = E1, F2 = 0.0;
  for (int k = 0; k < ND; ++k) F2 += F1[k] * F1[k];
  // tiny states: f and the counts are those of the state scaled by a power of two, in waves that
  // hold such a zone only
  if (sizeof(S) == 8 && (__builtin_amdgcn_ballot_w64(fabs(E1) < DIAG_SMALL) & upd)) {
    __asm__ volatile("");
    const int k2 = fabs(E1) < DIAG_SMALL ? diag_scale(E1) : 0;
    Es = ldexp(E1, k2);
    F2 = 0.0;
    for (int k = 0; k < ND; ++k) {
      const double fk = ldexp(F1[k], k2);
      F2 += fk * fk;
    }
  }
  const double cE = c * Es, cE2 = cE * cE;
  const bool up = Es > 0.0 && F2 * wd.fden > wd.fnum * cE2;
  if (SEL || __builtin_amdgcn_ballot_w64(up)) {
    wd.fnum = up ? F2 : wd.fnum;
    wd.fden = up ? cE2 : wd.fden;
  }
  constexpr double u = (sizeof(S) == 8) ? 0x1p-53 : 0x1p-24;
  const double lim = cE * (1.0 + 8.0 * u);
  // |F^| > lim: every state with E < 0 counts, else compare the squares
  wd.nun += __builtin_popcountll(__builtin_amdgcn_ballot_w64(lim < 0.0 || F2 > lim * lim) & upd);
  wd.nnp += __builtin_popcountll(__builtin_amdgcn_ballot_w64(!(E1 > 0.0)) & upd);
}
template <typename S, int ND>
__device__ __forceinline__ void wave_diag(double c, double E1, const double F1[3], unsigned long long upd,
                                          WaveDiag& wd) {
  wd.esum += E1;
  wave_diag_count<S, ND>(c, E1, F1, upd, wd);
}

// The block's partials of the diagnostics from its waves' (nw <= 16), each zone's volume V the
// same for the lane's zones; s*: LDS of nw entries.  Every wave of the block calls.
__device__ __forceinline__ void wave_diag_store(const WaveDiag& wd, bool upd, double V,
                                                int w, int lane, int nw, double* se, double* sm, int* su, int* sp,
                                                double* p_energy, double* p_maxf2, int* p_nun, int* p_nnp) {
  double e = upd ? V * wd.esum : 0.0, mf = upd ? wd.fnum / wd.fden : 0.0;
  for (int off = 32; off > 0; off >>= 1) {
    e += __shfl_xor(e, off);
    mf = fmax(mf, __shfl_xor(mf, off));
  }
  if (lane == 0) {
    se[w] = e;
    sm[w] = mf;
    su[w] = wd.nun;
    sp[w] = wd.nnp;
  }
  __syncthreads();
  if (w == 0 && lane == 0) {
    double te = 0.0, tm = 0.0;
    int tu = 0, tp = 0;
    for (int k = 0; k < nw; ++k) {
      te += se[k];
      tm = fmax(tm, sm[k]);
      tu += su[k];
      tp += sp[k];
    }
    p_energy[blockIdx.x] = te;
    p_maxf2[blockIdx.x] = tm;
    p_nun[blockIdx.x] = tu;
    p_nnp[blockIdx.x] = tp;
  }
}

}  // namespace fm1
