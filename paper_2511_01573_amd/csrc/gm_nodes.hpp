// gm_nodes.hpp -- factored node values of the fully symmetric rules (Sec. 2) for
// the integrand families of Sec. 4 that are products over the axes (Gaussian,
// product peak, C0, discontinuous) or the real part of one (oscillatory).
//
// A node of the rules moves at most three coordinates off the centre, or all
// of them (the corners).  With f(x) = prod_j T_j(x_j) the factors T_j are formed
// once per region (seven positions per axis) and a node is the product of a
// few combinations that many nodes share:
//   - the centre factors of every axis the node does not move, from prefix,
//     suffix and in-between products, and the factors of the moved axes;
//   - at a corner, an entry of a table over the leading axes' sign patterns
//     and one of a table over the last axes'.
// A node then costs one multiply-add into its class sum, instead of an
// exponential (16 operations) behind a chain of additions: the kernels are
// bound by FP64 issue, so operations per node are what counts.  The
// oscillatory family is Re(e^{i theta} prod_j e^{i a_j (x_j - c_j)}) with theta
// the angle at the centre, summed in double-double: the centre's own factors
// are 1, +-l h are conjugates (three sine-cosine pairs per axis), and a node is
// two multiply-adds.
// Every node is evaluated; only the order in which its factors meet differs
// from the definition's, so a node's relative rounding is that of d factors and
// d - 1 products instead of that of one outer function of a rounded sum (which
// grows with the size of the exponent or angle).
#pragma once

#include <type_traits>

#include "gm_corner.hpp"

namespace gm {

struct Cplx {
  double r, i;
};


template <int FAM>
struct Alg {
  static_assert(base_family(FAM) != FAM, "a factored kernel family");
  // oscillatory: factors are rotations, and the centre's are 1
  static constexpr bool kUnitCentre = FAM == kOscF;
  using T = std::conditional_t<kUnitCentre, Cplx, double>;

  __device__ static __forceinline__ double comb(double a, double b) {
    return a * b;
  }
  __device__ static __forceinline__ Cplx comb(Cplx a, Cplx b) {
    return Cplx{fma(a.r, b.r, -(a.i * b.i)), fma(a.r, b.i, a.i * b.r)};
  }
  // the empty product
  __device__ static __forceinline__ T none() {
    if constexpr (kUnitCentre) return Cplx{1.0, 0.0};
    else return 1.0;
  }
  // Terms of axis j at the coordinates x[0..N).
  template <int N>
  __device__ static __forceinline__ void terms(const DevParams& P, int j, const double (&x)[N],
                                               T (&t)[N]) {
    if constexpr (FAM == kGaussianF) {
      double a[N];
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const double s = P.a[j] * (x[q] - P.u[j]);
        a[q] = -(s * s);
      }
      fm::exp_n<N>(a, t);
    } else if constexpr (FAM == kC0F) {
      double a[N];
#pragma unroll
      for (int q = 0; q < N; ++q) a[q] = -(P.a[j] * fabs(x[q] - P.u[j]));
      fm::exp_n<N>(a, t);
    } else if constexpr (FAM == kDiscontinuousF) {
      double a[N];
#pragma unroll
      for (int q = 0; q < N; ++q) a[q] = P.a[j] * x[q];
      fm::exp_n<N>(a, t);
#pragma unroll
      for (int q = 0; q < N; ++q) t[q] = x[q] > P.u[j] ? 0.0 : t[q];
    } else if constexpr (FAM == kProductPeakF) {
      double a[N];
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const double s = x[q] - P.u[j];
        a[q] = P.inv_a2[j] + s * s;
      }
      fm::rcp_n<N>(a, t);
    }
  }

  // Terms of axis j at c + lam h and c - lam h.
  __device__ static __forceinline__ void pair(const DevParams& P, int j, double c, double h,
                                              double lam, T& tp, T& tm) {
    if constexpr (kUnitCentre) {
      const double x[1] = {P.a[j] * (lam * h)}, xl[1] = {0.0};
      double s[1], k[1];
      fm::sincos_n<1, false>(x, xl, s, k);
      tp = Cplx{k[0], s[0]};
      tm = Cplx{k[0], -s[0]};
    } else {
      const double x[2] = {fma(lam, h, c), fma(-lam, h, c)};
      T t[2];
      terms<2>(P, j, x, t);
      tp = t[0];
      tm = t[1];
    }
  }
  // The centre factor of axis j into tc[j] (a rotation's is 1 and has no place there).
  __device__ static __forceinline__ void centre(const DevParams& P, int j, double c, T* tc) {
    if constexpr (!kUnitCentre) {
      const double x[1] = {c};
      T t[1];
      terms<1>(P, j, x, t);
      tc[j] = t[0];
    }
  }
  // The rotation family's base e^{i (c0 + sum a_j c_j)}: the angle is summed in
  // double-double, so it carries no rounding of its own.
  template <int D>
  __device__ static __forceinline__ T base(const DevParams& P, const double (&c)[D]) {
    if constexpr (kUnitCentre) {
      double hi = P.c0, lo = 0.0;
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const double p = P.a[j] * c[j];
        const double pe = fma(P.a[j], c[j], -p);
        double s, e;
        two_sum(hi, p, s, e);
        hi = s;
        lo += e + pe;
      }
      const double x[1] = {hi}, xl[1] = {lo};
      double s[1], k[1];
      fm::sincos_n<1, true>(x, xl, s, k);
      return Cplx{k[0], s[0]};
    } else {
      return none();
    }
  }

  // The value of a whole node, of a node in two parts, and the same added to
  // running sums (FIRST: starting them).
  __device__ static __forceinline__ double value(T a) {
    if constexpr (kUnitCentre) return a.r;
    else return a;
  }
  template <int N>
  __device__ static __forceinline__ void nodes(const T (&a)[N], const T (&b)[N], double (&f)[N]) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      if constexpr (kUnitCentre) f[q] = fma(a[q].r, b[q].r, -(a[q].i * b[q].i));
      else f[q] = a[q] * b[q];
    }
  }
  template <int N, bool FIRST>
  __device__ static __forceinline__ void accumulate(const T (&a)[N], const T (&b)[N],
                                                    double (&acc)[N]) {
    if constexpr (kUnitCentre) {
#pragma unroll
      for (int q = 0; q < N; ++q) acc[q] = FIRST ? a[q].r * b[q].r : fma(a[q].r, b[q].r, acc[q]);
#pragma unroll
      for (int q = 0; q < N; ++q) acc[q] = fma(-a[q].i, b[q].i, acc[q]);
    } else {
#pragma unroll
      for (int q = 0; q < N; ++q) acc[q] = FIRST ? a[q] * b[q] : fma(a[q], b[q], acc[q]);
    }
  }
};

// ---------------------------------------------------------------------------
// Corner sweep.
// ---------------------------------------------------------------------------
// Products of the 2^M sign patterns of axes J .. J+M-1 (sign + before sign -),
// each behind s (PREFIX), else starting with the pattern's first factor.
template <int D, int FAM, int J, int M, bool PREFIX>
__device__ __forceinline__ void sign_table(typename Alg<FAM>::T s,
                                           const typename Alg<FAM>::T (&tp)[D],
                                           const typename Alg<FAM>::T (&tm)[D],
                                           typename Alg<FAM>::T* out) {
  using F = Alg<FAM>;
  if constexpr (M == 0) {
    out[0] = s;
  } else {
    typename F::T a = tp[J], b = tm[J];
    if constexpr (PREFIX) {
      a = F::comb(s, a);
      b = F::comb(s, b);
    }
    sign_table<D, FAM, J + 1, M - 1, true>(a, tp, tm, out);
    sign_table<D, FAM, J + 1, M - 1, true>(b, tp, tm, out + (1 << (M - 1)));
  }
}

// Sum of the corners whose first LB coordinates have the signs of `lane_bits`
// (bit j set -> -l5), 2^(D - LB) of them, added to S5 in groups.  A corner is
// an entry of the leading axes' table (G) times one of the last axes' (R, up to
// 16 entries, kept in registers).  A group's NA running sums of at most eight
// corners each hide the latency of the accumulation; they are added pairwise,
// so a corner passes through at most 8 + log2 NA roundings before the
// compensated sum, a rotation (two multiply-adds a corner) through 16 + log2 NA (the
// chain form's plain sum of 16 corners: 15).
template <int D, int FAM, int LB>
__device__ __forceinline__ void corner_sum(typename Alg<FAM>::T base,
                                           const typename Alg<FAM>::T (&tp)[D],
                                           const typename Alg<FAM>::T (&tm)[D],
                                           uint32_t lane_bits, KSum& S5) {
  using F = Alg<FAM>;
  using T = typename F::T;
  constexpr int NC = D - LB;
  static_assert(NC >= 3, "several lanes only from d = 9 on, 64 at most");
  constexpr int RB = NC >= 8 ? 4 : (NC + 1) / 2;  // last axes, table R
  constexpr int GMAX = F::kUnitCentre ? 3 : 4;    // unrolled axes before them, table G
  constexpr int GB = NC - RB < GMAX ? NC - RB : GMAX;
  constexpr int NO = NC - RB - GB;                // looped axes
  T pl = base;
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    T t = tp[j];
    if ((lane_bits >> j) & 1u) t = tm[j];
    pl = (j == 0 && !F::kUnitCentre) ? t : F::comb(pl, t);
  }
  constexpr int NR = 1 << RB;
  constexpr int NA = NR < 8 ? NR : 8;            // running sums
  constexpr int NG = 1 << GB, GS = NG < 4 ? NG : 4;  // entries of G, and of a group
  T R[NR];
  sign_table<D, FAM, D - RB, RB, false>(F::none(), tp, tm, R);
#pragma unroll 1
  for (uint32_t m = 0; m < (1u << NO); ++m) {
    T pre = pl;
#pragma unroll
    for (int q = 0; q < NO; ++q) {
      T t = tp[LB + q];
      if ((m >> q) & 1u) t = tm[LB + q];
      pre = (LB + q == 0 && !F::kUnitCentre) ? t : F::comb(pre, t);
    }
    T G[NG];
    sign_table<D, FAM, LB + NO, GB, F::kUnitCentre || LB + NO != 0>(pre, tp, tm, G);
#pragma unroll
    for (int g0 = 0; g0 < NG; g0 += GS) {
      double acc[NA];
#pragma unroll
      for (int g = 0; g < GS; ++g) {
        T a[NA];
#pragma unroll
        for (int q = 0; q < NA; ++q) a[q] = G[g0 + g];
#pragma unroll
        for (int k = 0; k < NR; k += NA) {
          T b[NA];
#pragma unroll
          for (int q = 0; q < NA; ++q) b[q] = R[k + q];
          if (g == 0 && k == 0) F::template accumulate<NA, true>(a, b, acc);
          else F::template accumulate<NA, false>(a, b, acc);
        }
      }
#pragma unroll
      for (int w = NA / 2; w >= 1; w >>= 1) {
#pragma unroll
        for (int q = 0; q < w; ++q) acc[q] = acc[q] + acc[q + w];
      }
      ks_add(S5, acc[0]);
    }
  }
}

}  // namespace gm
