// gm_adjoint_dev.hpp -- device pieces shared by the adjoint kernels
// (gm_adjoint.hip, node arguments as chains; gm_factor_adjoint.hip, factored): the
// split of a node's contribution into a function of its argument and one of each
// coordinate, and the per-component factors applied at the end.
#pragma once

#include "gm_adjoint.hpp"
#include "gm_math.hpp"

namespace gm {

// b^E for a compile-time E >= 1 by binary powering (E <= 18 here: at most
// five multiplications, a few ulp).
template <int E>
__device__ __forceinline__ double ipow(double b) {
  double y = 1.0, p = b;
  bool first = true;
#pragma unroll
  for (int e = E; e > 0; e >>= 1) {
    if (e & 1) {
      y = first ? p : y * p;
      first = false;
    }
    if (e > 1) p = p * p;
  }
  return y;
}

// The factor that turns the factored sums (times the region volume, summed
// over the regions) into dI/da_j (component j < D) and dI/du_j (D + j).  It
// depends on the parameters only, so it is applied once per block.
template <int D, int FAM>
__device__ __forceinline__ double adj_scale(const DevParams& P, int k) {
  const int j = k < D ? k : k - D;
  if constexpr (FAM == kOsc) {
    return k < D ? -1.0 : (k == D ? -6.283185307179586476925286766559 : 0.0);
  } else if constexpr (FAM == kProductPeak) {
    return k < D ? 2.0 / (P.a[j] * P.a[j] * P.a[j]) : 2.0;
  } else if constexpr (FAM == kCornerPeak) {
    return k < D ? -(double)(D + 1) : 0.0;
  } else if constexpr (FAM == kGaussian) {
    return k < D ? -2.0 * P.a[j] : 2.0 * P.a[j] * P.a[j];
  } else if constexpr (FAM == kC0) {
    return k < D ? -1.0 : P.a[j];
  } else {
    return k < D ? 1.0 : 0.0;
  }
}

// Per-family split of a node's contribution into phi(s) and psi_j(x_j)
// (the same quantities adj_node accumulates, without the class weight).
template <int FAM>
struct AdjSplit {
  // the empty chain: comb(kEmpty, t) == t exactly
  static constexpr double kEmpty = (FAM == kProductPeak) ? 1.0 : 0.0;
  // per-coordinate term of the argument and its combination
  __device__ static __forceinline__ double term(const DevParams& P, int j, double x) {
    if constexpr (FAM == kOsc || FAM == kCornerPeak) {
      return P.a[j] * x;
    } else if constexpr (FAM == kProductPeak) {
      const double t = x - P.u[j];
      return fm::rcp(P.inv_a2[j] + t * t);
    } else if constexpr (FAM == kGaussian) {
      const double t = P.a[j] * (x - P.u[j]);
      return t * t;
    } else if constexpr (FAM == kC0) {
      return P.a[j] * fabs(x - P.u[j]);
    } else {
      return (x > P.u[j]) ? -__builtin_inf() : P.a[j] * x;
    }
  }
  __device__ static __forceinline__ double comb(double s, double t) {
    if constexpr (FAM == kProductPeak) return s * t;
    else return s + t;
  }
  // phi on N independent arguments at once (the N-wide outer functions
  // interleave their dependent FMA chains)
  template <int D, int N>
  __device__ static __forceinline__ void phi_n(const DevParams& P, const double (&s)[N],
                                               double (&f)[N]) {
    double a[N];
    if constexpr (FAM == kOsc) {
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] = P.c0 + s[i];
      fm::sin_n<N>(a, f);
    } else if constexpr (FAM == kProductPeak) {
#pragma unroll
      for (int i = 0; i < N; ++i) f[i] = s[i];
    } else if constexpr (FAM == kCornerPeak) {
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] = ipow<D + 2>(1.0 + s[i]);
      fm::rcp_n<N>(a, f);
    } else if constexpr (FAM == kGaussian || FAM == kC0) {
#pragma unroll
      for (int i = 0; i < N; ++i) a[i] = -s[i];
      fm::exp_n<N>(a, f);
    } else {
      fm::exp_n<N>(s, f);  // the discontinuous family: exp(-inf) = 0 outside its box
    }
  }
  template <int D>
  __device__ static __forceinline__ double phi(const DevParams& P, double s) {
    const double a[1] = {s};
    double f[1];
    phi_n<D, 1>(P, a, f);
    return f[0];
  }
  // add w psi(x) for axis j into the factored sums
  template <int D>
  __device__ static __forceinline__ void add_point(const DevParams& P, int j, double x, double w,
                                                   double (&acc)[2 * D]) {
    if constexpr (FAM == kOsc || FAM == kCornerPeak || FAM == kDiscontinuous) {
      acc[j] = fma(w, x, acc[j]);
    } else if constexpr (FAM == kProductPeak) {
      const double t = x - P.u[j];
      const double r = w * fm::rcp(P.inv_a2[j] + t * t);
      acc[j] += r;
      acc[D + j] = fma(r, t, acc[D + j]);
    } else if constexpr (FAM == kGaussian) {
      const double t = x - P.u[j];
      acc[j] = fma(w * t, t, acc[j]);
      acc[D + j] = fma(w, t, acc[D + j]);
    } else {
      const double t = x - P.u[j];
      acc[j] = fma(w, fabs(t), acc[j]);
      acc[D + j] += (t > 0.0) ? w : ((t < 0.0) ? -w : 0.0);
    }
  }
  // add w (psi(+) Phi^+ + psi(-) Phi^-) for axis j into the factored sums
  template <int D>
  __device__ static __forceinline__ void add_axis(const DevParams& P, int j, double xp, double xm,
                                                  double wp, double wm, double (&acc)[2 * D]) {
    if constexpr (FAM == kOsc || FAM == kCornerPeak || FAM == kDiscontinuous) {
      acc[j] = fma(wp, xp, fma(wm, xm, acc[j]));
    } else if constexpr (FAM == kProductPeak) {
      const double tp = xp - P.u[j], tm = xm - P.u[j];
      const double rp = wp * fm::rcp(P.inv_a2[j] + tp * tp);
      const double rm = wm * fm::rcp(P.inv_a2[j] + tm * tm);
      acc[j] += rp + rm;
      acc[D + j] = fma(rp, tp, fma(rm, tm, acc[D + j]));
    } else if constexpr (FAM == kGaussian) {
      const double tp = xp - P.u[j], tm = xm - P.u[j];
      acc[j] = fma(wp * tp, tp, fma(wm * tm, tm, acc[j]));
      acc[D + j] = fma(wp, tp, fma(wm, tm, acc[D + j]));
    } else {
      const double tp = xp - P.u[j], tm = xm - P.u[j];
      acc[j] = fma(wp, fabs(tp), fma(wm, fabs(tm), acc[j]));
      const double sp = (tp > 0.0) ? wp : ((tp < 0.0) ? -wp : 0.0);
      const double sm = (tm > 0.0) ? wm : ((tm < 0.0) ? -wm : 0.0);
      acc[D + j] += sp + sm;
    }
  }
};

// A copy of x the optimiser cannot relate to x (no instruction is emitted).
__device__ __forceinline__ double opaque(double x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Sum over the wavefront (a fixed butterfly; lane 0's result is used).
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

}  // namespace gm
