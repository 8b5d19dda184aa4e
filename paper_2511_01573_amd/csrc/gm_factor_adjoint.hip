// gm_factor_adjoint.hip -- adjoint kernel of the gradient mode for the factored
// families (gm_nodes.hpp), d = 7..10, degree 7 or 9: the sums of gm_adjoint.hip
// with node values that are products of tabulated factors.
//
// A node's contribution to axis j is phi psi_j(x_j), phi its value (for the
// oscillatory family, cosine's derivative: the imaginary part of the rotation
// product), so per axis only the phi sums of the nodes at each of its offsets
// are needed.  A node's product is formed inside the multiply-add that adds it
// to such a sum, once for the sum of its last moved axis and once for the
// running sums of its row, which go to the other moved axes at the row's end:
// two multiply-adds per node (rotations: four) and no exponential; at a corner
// the last axes' sums are kept per entry of their table and the leading axes'
// per entry of theirs.  About 4500 FP64 operations a region at d = 8, degree 9
// (the chain form, 1089 exponentials, about 20000).  One lane per region, every
// class in one launch: the offsets' sums stay in registers.
// d = 8 Gaussian, degree 9, 1.35e6 leaves and active regions: 433 us (3.1e9
// regions/s, 14 TFLOP/s; the chain form's two launches: 1620 us).
#include "gm_adjoint_dev.hpp"
#include "gm_nodes.hpp"

namespace gm {

// acc += phi(a b)
__device__ __forceinline__ void add_phi(double a, double b, double& acc) { acc = fma(a, b, acc); }
__device__ __forceinline__ void add_phi(Cplx a, Cplx b, double& acc) {
  acc = fma(a.r, b.i, acc);
  acc = fma(a.i, b.r, acc);
}
__device__ __forceinline__ double phi_of(double a) { return a; }
__device__ __forceinline__ double phi_of(Cplx a) { return a.i; }
__device__ __forceinline__ double scaled(double a, double w) { return a * w; }
__device__ __forceinline__ Cplx scaled(Cplx a, double w) { return Cplx{a.r * w, a.i * w}; }

// The corner class, weight w: phi sums of either side of every axis into acc.
template <int D, int FAM>
__device__ __forceinline__ void factor_adj_corners(const DevParams& P, const RuleConsts& K, double w,
                                                   typename Alg<FAM>::T base,
                                                   const double (&c)[D], const double (&h)[D],
                                                   double (&acc)[2 * D]) {
  using F = Alg<FAM>;
  using T = typename F::T;
  using S = AdjSplit<base_family(FAM)>;
  constexpr int RB = 4, NR = 1 << RB;     // last axes, table R
  constexpr int GB = 3, NG = 1 << GB;     // unrolled axes before them, table G
  constexpr int NO = D - RB - GB;         // looped axes
  T tp[D], tm[D];
#pragma unroll
  for (int j = 0; j < D; ++j) F::pair(P, j, c[j], h[j], K.lam5, tp[j], tm[j]);
  T R[NR];
  sign_table<D, FAM, D - RB, RB, false>(F::none(), tp, tm, R);
  double rs[NR];           // per entry of R
  double fp[D], fm_[D];    // either side of the leading axes
#pragma unroll
  for (int q = 0; q < NR; ++q) rs[q] = 0.0;
#pragma unroll
  for (int j = 0; j < D; ++j) fp[j] = fm_[j] = 0.0;
  double total = 0.0;
#pragma unroll 1
  for (uint32_t m = 0; m < (1u << NO); ++m) {
    T pre = scaled(base, w);
#pragma unroll
    for (int q = 0; q < NO; ++q) {
      T t = tp[q];
      if ((m >> q) & 1u) t = tm[q];
      pre = F::comb(pre, t);
    }
    T G[NG];
    sign_table<D, FAM, NO, GB, true>(pre, tp, tm, G);
    double gs[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      double s[2] = {0.0, 0.0};
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        add_phi(G[g], R[q], rs[q]);
        add_phi(G[g], R[q], s[q & 1]);
      }
      gs[g] = s[0] + s[1];
    }
    // G's entries: the first of its axes is the highest bit, + before -
#pragma unroll
    for (int j = 0; j < GB; ++j) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if ((g >> (GB - 1 - j)) & 1) fm_[NO + j] += gs[g];
        else fp[NO + j] += gs[g];
      }
    }
    const double sum = ((gs[0] + gs[1]) + (gs[2] + gs[3])) + ((gs[4] + gs[5]) + (gs[6] + gs[7]));
#pragma unroll
    for (int q = 0; q < NO; ++q) {
      if ((m >> q) & 1u) fm_[q] += sum;
      else fp[q] += sum;
    }
    total += sum;
  }
#pragma unroll
  for (int j = 0; j < RB; ++j) {
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      if ((q >> (RB - 1 - j)) & 1) fm_[D - RB + j] += rs[q];
      else fp[D - RB + j] += rs[q];
    }
  }
  if constexpr (F::kUnitCentre) acc[D] += total;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const double cj = opaque(c[j]), hj = opaque(h[j]);
    S::template add_axis<D>(P, j, fma(K.lam5, hj, cj), fma(-K.lam5, hj, cj), fp[j], fm_[j], acc);
  }
}

// Centre factors and their suffix products (tc[k] ... tc[D-1]).
template <int D, int FAM>
__device__ __forceinline__ void centre_factors(const DevParams& P, const double (&c)[D],
                                               typename Alg<FAM>::T (&tc)[D],
                                               typename Alg<FAM>::T (&suf)[D + 1]) {
  using F = Alg<FAM>;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const double x[1] = {c[j]};
    typename F::T t[1];
    F::template terms<1>(P, j, x, t);
    tc[j] = t[0];
  }
  suf[D - 1] = tc[D - 1];
#pragma unroll
  for (int k = D - 2; k >= 0; --k) suf[k] = F::comb(tc[k], suf[k + 1]);
}

// Class 6 (+-l6 e_i), weight w, into acc.
template <int D, int FAM>
__device__ __forceinline__ void factor_adj_class6(const DevParams& P, const RuleConsts& K, double w,
                                                  typename Alg<FAM>::T base, const double (&c)[D],
                                                  const double (&h)[D], double (&acc)[2 * D]) {
  using F = Alg<FAM>;
  using T = typename F::T;
  using S = AdjSplit<base_family(FAM)>;
  constexpr bool U = F::kUnitCentre;
  T tc[D], suf[D + 1];
  if constexpr (!U) centre_factors<D, FAM>(P, c, tc, suf);
  double W = 0.0, sp[D], sm[D];
  T pre = scaled(base, w);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    T t6p, t6m;
    F::pair(P, i, c[i], h[i], K.lam6, t6p, t6m);
    const T o = U || i == D - 1 ? pre : F::comb(pre, suf[i + 1]);
    sp[i] = sm[i] = 0.0;
    add_phi(o, t6p, sp[i]);
    add_phi(o, t6m, sm[i]);
    W += sp[i] + sm[i];
    if constexpr (!U) pre = F::comb(pre, tc[i]);
  }
  if constexpr (U) acc[D] += W;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    S::template add_point<D>(P, j, c[j], W - (sp[j] + sm[j]), acc);
    S::template add_axis<D>(P, j, fma(K.lam6, h[j], c[j]), fma(-K.lam6, h[j], c[j]), sp[j], sm[j], acc);
  }
}

// Classes 1-4 (R9: 7 and 8 too), weights w[]: their phi sum W and those of the
// nodes with x_j at +l2, -l2, +l3, -l3 from the centre (g[0..4)).
template <int D, int FAM, bool R9>
__device__ __forceinline__ void factor_adj_others(const DevParams& P, const RuleConsts& K,
                                                  const double* w, typename Alg<FAM>::T base,
                                                  const double (&c)[D], const double (&h)[D],
                                                  double& Wout, double (&g)[4][D]) {
  using F = Alg<FAM>;
  using T = typename F::T;
  constexpr bool U = F::kUnitCentre;
  T tc[D], t2p[D], t2m[D], t3p[D], t3m[D], suf[D + 1];
#pragma unroll
  for (int j = 0; j < D; ++j) {
    F::pair(P, j, c[j], h[j], K.lam2, t2p[j], t2m[j]);
    F::pair(P, j, c[j], h[j], K.lam3, t3p[j], t3m[j]);
  }
  if constexpr (!U) centre_factors<D, FAM>(P, c, tc, suf);
  double(&g2p)[D] = g[0], (&g2m)[D] = g[1], (&g3p)[D] = g[2], (&g3m)[D] = g[3];
  double W = w[0] * phi_of(U ? base : T(suf[0]));
#pragma unroll
  for (int j = 0; j < D; ++j) g2p[j] = g2m[j] = g3p[j] = g3m[j] = 0.0;
  T pre = base;
#pragma unroll
  for (int i = 0; i < D; ++i) {
    {  // one moved axis
      const T o = U ? base : i == 0 ? suf[1] : i == D - 1 ? pre : F::comb(pre, suf[i + 1]);
      const T o1 = scaled(o, w[1]), o2 = scaled(o, w[2]);
      double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
      add_phi(o1, t2p[i], s0);
      add_phi(o1, t2m[i], s1);
      add_phi(o2, t3p[i], s2);
      add_phi(o2, t3m[i], s3);
      W += (s0 + s1) + (s2 + s3);
      g2p[i] += s0;
      g2m[i] += s1;
      g3p[i] += s2;
      g3m[i] += s3;
    }
    if (i < D - 1) {
      T m = pre;  // product of the centre factors below j except i's
      double r2p = 0.0, r2m = 0.0, r3p = 0.0, r3m = 0.0;  // row i
#pragma unroll
      for (int j = i + 1; j < D; ++j) {
        const bool none = !U && i == 0 && j == 1;
        const T o = U ? base : j == D - 1 ? m : none ? suf[j + 1] : F::comb(m, suf[j + 1]);
        {
          const T o4 = scaled(o, w[3]);
          const T ip = F::comb(o4, t3p[i]), im = F::comb(o4, t3m[i]);
          add_phi(ip, t3p[j], g3p[j]);
          add_phi(ip, t3m[j], g3m[j]);
          add_phi(ip, t3p[j], r3p);
          add_phi(im, t3p[j], r3m);
          add_phi(im, t3p[j], g3p[j]);
          add_phi(im, t3m[j], g3m[j]);
          add_phi(ip, t3m[j], r3p);
          add_phi(im, t3m[j], r3m);
        }
        if constexpr (R9) {
          const T o7 = scaled(o, w[6]);
          const T i3p = F::comb(o7, t3p[i]), i3m = F::comb(o7, t3m[i]);
          const T i2p = F::comb(o7, t2p[i]), i2m = F::comb(o7, t2m[i]);
          add_phi(i3p, t2p[j], g2p[j]);
          add_phi(i3p, t2m[j], g2m[j]);
          add_phi(i2p, t3p[j], g3p[j]);
          add_phi(i2p, t3m[j], g3m[j]);
          add_phi(i3p, t2p[j], r3p);
          add_phi(i3m, t2p[j], r3m);
          add_phi(i2p, t3p[j], r2p);
          add_phi(i2m, t3p[j], r2m);
          add_phi(i3m, t2p[j], g2p[j]);
          add_phi(i3m, t2m[j], g2m[j]);
          add_phi(i2m, t3p[j], g3p[j]);
          add_phi(i2m, t3m[j], g3m[j]);
          add_phi(i3p, t2m[j], r3p);
          add_phi(i3m, t2m[j], r3m);
          add_phi(i2p, t3m[j], r2p);
          add_phi(i2m, t3m[j], r2m);
          if (j < D - 1) {
            // row (i, j) of the triples: sums per sign pattern of (i, j)
            const T a0 = scaled(t3p[i], w[7]), a1 = scaled(t3m[i], w[7]);
            T ij[4] = {F::comb(a0, t3p[j]), F::comb(a0, t3m[j]), F::comb(a1, t3p[j]),
                       F::comb(a1, t3m[j])};
            if constexpr (U) {
#pragma unroll
              for (int q = 0; q < 4; ++q) ij[q] = F::comb(base, ij[q]);
            }
            T m3 = m;
            double u[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = j + 1; k < D; ++k) {
              const bool none3 = none && k == 2;
              T kp = t3p[k], km = t3m[k];
              if constexpr (!U) {
                const T o3 = k == D - 1 ? m3 : none3 ? suf[k + 1] : F::comb(m3, suf[k + 1]);
                kp = F::comb(o3, kp);
                km = F::comb(o3, km);
                m3 = none3 ? tc[k] : F::comb(m3, tc[k]);
              }
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                add_phi(ij[q], kp, u[q]);
                add_phi(ij[q], kp, g3p[k]);
                add_phi(ij[q], km, g3m[k]);
                add_phi(ij[q], km, u[q]);
              }
            }
            const double ip = u[0] + u[1], im = u[2] + u[3];
            r3p += ip;
            r3m += im;
            g3p[j] += u[0] + u[2];
            g3m[j] += u[1] + u[3];
          }
        }
        if constexpr (!U) m = none ? tc[j] : F::comb(m, tc[j]);
        // (rows kept apart: mixed, their partial products would not fit the registers)
        __builtin_amdgcn_sched_barrier(0);
      }
      // the row's nodes all move axis i
      W += (r2p + r2m) + (r3p + r3m);
      g2p[i] += r2p;
      g2m[i] += r2m;
      g3p[i] += r3p;
      g3m[i] += r3m;
    }
    if constexpr (!U) pre = i == 0 ? tc[0] : F::comb(pre, tc[i]);
  }
  Wout = W;
}

// A wavefront takes 64 consecutive regions per step; the lanes' contributions
// (times the region volume) join the wavefront's double-double totals as in
// adjoint_kernel (a fixed order).
template <int D, int FAM, bool R9>
__global__ __launch_bounds__(kAdjBlock) __attribute__((amdgpu_waves_per_eu(2)))
void factor_adjoint_kernel(AdjArgs A) {
  __shared__ dd wtot[kAdjBlock / 64][2 * D];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < 2 * D; ++j) wtot[wv][j] = dd{0.0, 0.0};
  for (int64_t rb = (int64_t)blockIdx.x * kAdjBlock + 64 * wv; rb < A.n;
       rb += (int64_t)gridDim.x * kAdjBlock) {
    const int64_t r = rb + lane;
    double acc[2 * D];
#pragma unroll
    for (int j = 0; j < 2 * D; ++j) acc[j] = 0.0;
    double vol = 0.0;
    if (r < A.n) {
      using F = Alg<FAM>;
      using S = AdjSplit<base_family(FAM)>;
      const double* w = R9 ? A.K.w9 : A.K.w;
      double W, g[4][D];
      // The region is read again for each group of classes (from the L2): held
      // through the sweep of classes 4, 7 and 8, whose sums and factors take 200
      // registers at d = 8, it would spill.
      {
        double c[D], h[D];
        vol = ldexp(A.vol_omega, -load_region<D>(A.R, r, c, h));
        const typename F::T base = F::template base<D>(A.P, c);
        factor_adj_corners<D, FAM>(A.P, A.K, w[4], base, c, h, acc);
        if constexpr (R9) factor_adj_class6<D, FAM>(A.P, A.K, w[5], base, c, h, acc);
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      {
        double c[D], h[D];
        load_region<D>(A.R, r, c, h);
        factor_adj_others<D, FAM, R9>(A.P, A.K, w, F::template base<D>(A.P, c), c, h, W, g);
      }
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      {
        double c[D], h[D];
        load_region<D>(A.R, r, c, h);
        if constexpr (F::kUnitCentre) acc[D] += W;
#pragma unroll
        for (int j = 0; j < D; ++j) {
          const double moved = (g[0][j] + g[1][j]) + (g[2][j] + g[3][j]);
          S::template add_point<D>(A.P, j, c[j], W - moved, acc);
          S::template add_axis<D>(A.P, j, fma(A.K.lam2, h[j], c[j]), fma(-A.K.lam2, h[j], c[j]),
                                  g[0][j], g[1][j], acc);
          S::template add_axis<D>(A.P, j, fma(A.K.lam3, h[j], c[j]), fma(-A.K.lam3, h[j], c[j]),
                                  g[2][j], g[3][j], acc);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 2 * D; ++j) {
      const double v = wave_sum_f64(vol * acc[j]);
      if (lane == 0) dd_add(wtot[wv][j], v);
    }
  }
  __syncthreads();
  if (tid < 2 * D) {
    dd v = wtot[0][tid];
    for (int k = 1; k < kAdjBlock / 64; ++k) v = dd_sum(v, wtot[k][tid]);
    const double sc = adj_scale<D, base_family(FAM)>(A.P, tid);
    double* p = A.partials + ((int64_t)blockIdx.x * 2 * kMaxDim + threadIdx.x) * 2;
    p[0] = v.hi * sc;
    p[1] = v.lo * sc;
  }
}

#ifndef GM_FAMILY
#error "compile with -DGM_FAMILY=<8..12>"
#endif

template <int D>
static AdjFn fadj_d(bool r9) {
  return r9 ? factor_adjoint_kernel<D, GM_FAMILY, true> : factor_adjoint_kernel<D, GM_FAMILY, false>;
}

#define GM_CAT2(a, b) a##b
#define GM_CAT(a, b) GM_CAT2(a, b)

AdjFn GM_CAT(factor_adjoint_f, GM_FAMILY)(int d, bool r9) {
  static_assert(kFactorMinDim == 7 && kAdjFactoredMaxDim == 10, "the cases below");
  switch (d) {
    case 7: return fadj_d<7>(r9);
    case 8: return fadj_d<8>(r9);
    case 9: return fadj_d<9>(r9);
    case 10: return fadj_d<10>(r9);
    default: return nullptr;
  }
}

GM_CHECK_UNIT_F(factor_adjoint, GM_FAMILY)

}  // namespace gm
