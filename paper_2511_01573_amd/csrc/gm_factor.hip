// gm_factor.hip -- the degree-7 rule kernel for the factored families: the
// Genz-Malik rule, embedded-rule error estimate and fourth-difference split
// axis of gm_rule.hip (arXiv 2511.01573, Sec. 2) with the node values of
// gm_nodes.hpp.
//
// Mappings.  One lane per region (TPR), everything unrolled but the corners'
// outer loop: at d = 8 about 1800 FP64 operations a region, 950 of them the 56
// exponentials of the Gaussian's factors (the chain form: 7600).  Above d = 10
// also L = 2^l lanes of one wavefront per region (WPR), for sets too small to
// fill the GPU: the lanes form the region's factors and partial products together
// in LDS, deal out the class 2-4 nodes as work items (an axis: 4 nodes and its
// fourth difference; an axis pair: 4 nodes), sweep the corners behind their own
// signs of the first l axes, and combine the class sums with shuffles.  The
// line between them: target_lanes in gm_api.hip.
#include "gm_nodes.hpp"

namespace gm {

// ---------------------------------------------------------------------------
// TPR: one lane per region.
// ---------------------------------------------------------------------------
template <int D, int FAM>
__device__ __forceinline__ RegionResult factor_region(const DevParams& P, const RuleConsts& K,
                                                      const double (&c)[D], const double (&h)[D],
                                                      double vol) {
  using F = Alg<FAM>;
  using T = typename F::T;
  constexpr bool U = F::kUnitCentre;
  // Factors at the centre and at +-l3 (= +-l4); suf[k] = tc[k] ... tc[D-1].
  T tc[D], t3p[D], t3m[D], suf[D + 1];
  const T base = F::template base<D>(P, c);
#pragma unroll
  for (int j = 0; j < D; ++j) F::pair(P, j, c[j], h[j], K.lam3, t3p[j], t3m[j]);
  if constexpr (!U) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const double x[1] = {c[j]};
      T t[1];
      F::template terms<1>(P, j, x, t);
      tc[j] = t[0];
    }
    suf[D - 1] = tc[D - 1];
#pragma unroll
    for (int k = D - 2; k >= 0; --k) suf[k] = F::comb(tc[k], suf[k + 1]);
  }
  const double f0 = F::value(U ? base : suf[0]);
  KSum S2 = {0.0, 0.0}, S3 = {0.0, 0.0}, S4 = {0.0, 0.0}, S5 = {0.0, 0.0};
  double Dv[D];
  double scale = 0.0;
  T pre = base;  // tc[0] ... tc[i-1]
#pragma unroll
  for (int i = 0; i < D; ++i) {
    // classes 2 and 3 on axis i
    {
      T t2p, t2m;
      F::pair(P, i, c[i], h[i], K.lam2, t2p, t2m);
      const T o = U ? base : i == 0 ? suf[1] : i == D - 1 ? pre : F::comb(pre, suf[i + 1]);
      const T a[4] = {o, o, o, o}, b[4] = {t2p, t2m, t3p[i], t3m[i]};
      double f[4];
      F::template nodes<4>(a, b, f);
      ks_add(S2, f[0] + f[1]);
      ks_add(S3, f[2] + f[3]);
      double sc;
      fourth_diff(K, f0, f[0], f[1], f[2], f[3], Dv[i], sc);
      scale = sc > scale ? sc : scale;
    }
    // class 4, row i: the four sign patterns of (i, j), j > i, in a running
    // sum each; m is the product of the centre factors below j except i's
    if (i < D - 1) {
      T m = pre, rp, rm;
      if constexpr (U) {
        rp = F::comb(base, t3p[i]);
        rm = F::comb(base, t3m[i]);
      }
      double acc[4];
#pragma unroll
      for (int j = i + 1; j < D; ++j) {
        if constexpr (!U) {
          const T o = j == D - 1 ? m : (i == 0 && j == 1) ? suf[j + 1] : F::comb(m, suf[j + 1]);
          rp = F::comb(o, t3p[i]);
          rm = F::comb(o, t3m[i]);
          m = (i == 0 && j == 1) ? tc[j] : F::comb(m, tc[j]);
        }
        const T a[4] = {rp, rp, rm, rm}, b[4] = {t3p[j], t3m[j], t3p[j], t3m[j]};
        if (j == i + 1) F::template accumulate<4, true>(a, b, acc);
        else F::template accumulate<4, false>(a, b, acc);
      }
      ks_add(S4, (acc[0] + acc[1]) + (acc[2] + acc[3]));
    }
    if constexpr (!U) pre = i == 0 ? tc[0] : F::comb(pre, tc[i]);
  }
  {
    T t5p[D], t5m[D];
#pragma unroll
    for (int j = 0; j < D; ++j) F::pair(P, j, c[j], h[j], K.lam5, t5p[j], t5m[j]);
    corner_sum<D, FAM, 0>(base, t5p, t5m, 0u, S5);
  }
  RegionResult r;
  rule_combine(K, f0, ks_val(S2), ks_val(S3), ks_val(S4), ks_val(S5), vol, r);
  split_axis<D>(K, Dv, scale, c, h, r);
  r.nonfinite |= !Fam<base_family(FAM)>::in_range(P, c, h);
  return r;
}

template <int D, int FAM, bool BATCH>
__global__ __launch_bounds__(kRuleBlock) __attribute__((amdgpu_waves_per_eu(2)))
void factor_tpr_kernel(RuleArgs A) {
  int64_t start, end;
  int buf;
  if (!active_range<BATCH>(A, start, end, buf)) return;
  const RegionSrc R = region_src<BATCH>(A, buf);
  const int64_t stride = (int64_t)gridDim.x * kRuleBlock;
  dd qs = {0.0, 0.0}, es = {0.0, 0.0};
  int nonfin = 0;
  // (siblings in neighbouring lanes, as in rule_tpr_kernel)
  const bool pairs = R.pending;
  int64_t v = start + (int64_t)blockIdx.x * kRuleBlock + threadIdx.x;
  const auto region_of = [&](int64_t k) {
    return pairs ? ((k & 1) ? R.nkeep + (k >> 1) : (k >> 1)) : k;
  };
  // The next region's record is read while this one is evaluated, and the list's
  // entry it depends on while the one before is (kAhead: where the registers hold
  // a second record; 203 -> 240 at d = 8).  Loads and arithmetic took turns: 0.080
  // ns a region, the sum of 0.046 of FP64 issue and 0.033 of HBM time; now 0.068.
  constexpr bool kAhead = !BATCH && D <= 9;
  Record<D> next;
  int64_t e = 0;
  if (v < end) {
    e = list_entry(R, region_of(v));
    if constexpr (kAhead) {
      load_record<D>(R, region_of(v), e, next);
      if (v + stride < end) e = list_entry(R, region_of(v + stride));
    }
  }
  for (; v < end; v += stride) {
    const int64_t r = region_of(v);
    double c[D], h[D];
    Record<D> cur;
    if constexpr (kAhead) {
      cur = next;
      if (v + stride < end) load_record<D>(R, region_of(v + stride), e, next);
      if (v + 2 * stride < end) e = list_entry(R, region_of(v + 2 * stride));
    } else {
      load_record<D>(R, r, e, cur);
      if (v + stride < end) e = list_entry(R, region_of(v + stride));
    }
    const int lvl = form_region<D>(R, r, cur, c, h);
    double volo;
    const DevParams& P = region_params<BATCH>(A, buf, r, volo);
    const double vol = ldexp(volo, -lvl);
    const RegionResult o = factor_region<D, FAM>(P, A.K, c, h, vol);
    store_result(A, r, o);
    dd_add(qs, o.q);
    dd_add(es, o.err);
    nonfin |= o.nonfinite;
  }
  if constexpr (!BATCH) block_partials(A, qs, es, nonfin);
}

// ---------------------------------------------------------------------------
// WPR: L = 2^LOG2L lanes per region (d > 10).
// ---------------------------------------------------------------------------
// LDS per region: the factors of every axis at +-l2, +-l3, +-l5 and the centre,
// the products of the centre factors before and after each axis, and the region
// itself.  An axis' fourth difference and its scale take the place of its +-l2
// factors, which its axis nodes alone read (with four lanes a region the slots
// decide how many workgroups a CU holds).
template <int D, int FAM>
struct FactorSlot {
  using T = typename Alg<FAM>::T;
  static constexpr bool U = Alg<FAM>::kUnitCentre;
  T t2[2][D], t3[2][D], t5[2][D];
  T tc[U ? 1 : D], pre[U ? 1 : D], suf[U ? 1 : D];
  double c[D], h[D];

  __device__ __forceinline__ void put_diff(int i, double dv, double sc) {
    if constexpr (U) {
      t2[0][i] = T{dv, sc};
    } else {
      t2[0][i] = dv;
      t2[1][i] = sc;
    }
  }
  __device__ __forceinline__ double dv(int i) const {
    if constexpr (U) return t2[0][i].r;
    else return t2[0][i];
  }
  __device__ __forceinline__ double sc(int i) const {
    if constexpr (U) return t2[0][i].i;
    else return t2[1][i];
  }
};

template <int D, int FAM, int LOG2L>
__global__ __launch_bounds__(kRuleBlock) void factor_wpr_kernel(RuleArgs A) {
  using F = Alg<FAM>;
  using T = typename F::T;
  constexpr bool U = F::kUnitCentre;
  constexpr int L = 1 << LOG2L;
  constexpr int RPB = kRuleBlock / L;  // regions per block step
  constexpr int NPAIR = D * (D - 1) / 2;
  __shared__ FactorSlot<D, FAM> slots[RPB];
  int64_t start, n;
  int buf;
  if (!active_range<false>(A, start, n, buf)) return;
  const RegionSrc R = region_src<false>(A, buf);
  const RuleConsts& K = A.K;
  const int g = threadIdx.x >> LOG2L;  // region slot in the block
  const int s = threadIdx.x & (L - 1);
  FactorSlot<D, FAM>& sl = slots[g];
  dd qs = {0.0, 0.0}, es = {0.0, 0.0};
  int nonfin = 0;
  for (int64_t rb = start + (int64_t)blockIdx.x * RPB; rb < n; rb += (int64_t)gridDim.x * RPB) {
    const int64_t r = rb + g;
    const bool valid = r < n;
    double volo;
    const DevParams& P = region_params<false>(A, buf, valid ? r : start, volo);
    // The region's factors, the axes dealt out to the lanes.
    const int lvl = load_axes<D, L>(R, valid, r, valid ? list_entry(R, r) : 0, s,
                                    [&](int j, double c, double h) {
                                      sl.c[j] = c;
                                      sl.h[j] = h;
                                      F::pair(P, j, c, h, K.lam2, sl.t2[0][j], sl.t2[1][j]);
                                      F::pair(P, j, c, h, K.lam3, sl.t3[0][j], sl.t3[1][j]);
                                      F::pair(P, j, c, h, K.lam5, sl.t5[0][j], sl.t5[1][j]);
                                      F::centre(P, j, c, sl.tc);
                                    });
    wave_lds_sync();
    const T base = F::template base<D>(P, sl.c);
    __syncthreads();
    T tc[U ? 1 : D];
    T full = base;
    if constexpr (!U) {
#pragma unroll
      for (int j = 0; j < D; ++j) tc[j] = sl.tc[j];
      // prefixes by lane 0, suffixes by lane 1 of the region
      if (s == 0) {
        T p = F::none();
#pragma unroll
        for (int k = 0; k < D; ++k) {
          sl.pre[k] = p;
          p = k == 0 ? tc[0] : F::comb(p, tc[k]);
        }
      } else if (s == 1) {
        T p = F::none();
#pragma unroll
        for (int k = D - 1; k >= 0; --k) {
          sl.suf[k] = p;
          p = k == D - 1 ? tc[k] : F::comb(p, tc[k]);
        }
      }
      full = tc[0];
#pragma unroll
      for (int k = 1; k < D; ++k) full = F::comb(full, tc[k]);
      __syncthreads();
    }
    const double f0 = F::value(full);
    KSum S2 = {0.0, 0.0}, S3 = {0.0, 0.0}, S4 = {0.0, 0.0}, S5 = {0.0, 0.0};
    for (int i = s; i < D; i += L) {
      T o = base;
      if constexpr (!U) o = F::comb(sl.pre[i], sl.suf[i]);
      const T a[4] = {o, o, o, o}, b[4] = {sl.t2[0][i], sl.t2[1][i], sl.t3[0][i], sl.t3[1][i]};
      double f[4];
      F::template nodes<4>(a, b, f);
      ks_add(S2, f[0] + f[1]);
      ks_add(S3, f[2] + f[3]);
      double dv, scv;
      fourth_diff(K, f0, f[0], f[1], f[2], f[3], dv, scv);
      sl.put_diff(i, dv, scv);
    }
    // Class 4, one axis pair per item: the centre factors between the two axes
    // are multiplied from the lane's registers with the item's bounds as
    // predicates.
    for (int it = s; it < NPAIR; it += L) {
      int i, j;
      pair_of<D>(it, i, j);
      T o = base;
      if constexpr (!U) {
        o = F::comb(sl.pre[i], sl.suf[j]);
#pragma unroll
        for (int k = 1; k < D - 1; ++k) {
          const T t = F::comb(o, tc[k]);
          if (k > i && k < j) o = t;
        }
      }
      const T ip = F::comb(o, sl.t3[0][i]), im = F::comb(o, sl.t3[1][i]);
      const T jp = sl.t3[0][j], jm = sl.t3[1][j];
      const T a[4] = {ip, ip, im, im}, b[4] = {jp, jm, jp, jm};
      double f[4];
      F::template nodes<4>(a, b, f);
      ks_add(S4, (f[0] + f[1]) + (f[2] + f[3]));
    }
    // Class 5: this lane's 2^(D - LOG2L) corners.
    {
      T t5p[D], t5m[D];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        t5p[j] = sl.t5[0][j];
        t5m[j] = sl.t5[1][j];
      }
      corner_sum<D, FAM, LOG2L>(base, t5p, t5m, (uint32_t)s, S5);
    }
    // Combine the L lanes of the group.
#pragma unroll
    for (int m = L / 2; m >= 1; m >>= 1) {
      S2 = ks_merge(S2, shfl_xor_ks(S2, m));
      S3 = ks_merge(S3, shfl_xor_ks(S3, m));
      S4 = ks_merge(S4, shfl_xor_ks(S4, m));
      S5 = ks_merge(S5, shfl_xor_ks(S5, m));
    }
    __syncthreads();
    if (s == 0 && valid) {
      RegionResult o;
      const double vol = ldexp(volo, -lvl);
      rule_combine(K, f0, ks_val(S2), ks_val(S3), ks_val(S4), ks_val(S5), vol, o);
      double dv[D], scale = 0.0;
#pragma unroll
      for (int i = 0; i < D; ++i) {
        dv[i] = sl.dv(i);
        scale = sl.sc(i) > scale ? sl.sc(i) : scale;
      }
      split_axis<D>(K, dv, scale, sl.c, sl.h, o);
      o.nonfinite |= !Fam<base_family(FAM)>::in_range(P, sl.c, sl.h);
      store_result(A, r, o);
      dd_add(qs, o.q);
      dd_add(es, o.err);
      nonfin |= o.nonfinite;
    }
    __syncthreads();
  }
  block_partials(A, qs, es, nonfin);
}

// ---------------------------------------------------------------------------
// Dispatch over (d, mapping) for the kernel family this translation unit is
// built for (-DGM_RULE_FAMILY=k, k = kOscF .. kDiscontinuousF).
// ---------------------------------------------------------------------------
#ifndef GM_RULE_FAMILY
#error "compile with -DGM_RULE_FAMILY=<8..12>"
#endif

template <int D, bool B>
static RuleKernelFn pick(int log2l) {
  constexpr int F = GM_RULE_FAMILY;
  if constexpr (B && (D < kBatchFactorMinDim || D > kBatchMaxDim)) {
    return nullptr;
  } else {
    if (log2l < 0) return factor_tpr_kernel<D, F, B>;
    if constexpr (D > kTprMaxDim) {
      if (log2l == 2) return factor_wpr_kernel<D, F, 2>;
      if (log2l == 4) return factor_wpr_kernel<D, F, 4>;
      if (log2l == 6) return factor_wpr_kernel<D, F, 6>;
    }
    return nullptr;
  }
}

template <bool B>
static RuleKernelFn factor_fn(int d, int log2l) {
  switch (d) {
    case 7: return pick<7, B>(log2l);
    case 8: return pick<8, B>(log2l);
    case 9: return pick<9, B>(log2l);
    case 10: return pick<10, B>(log2l);
    case 11: return pick<11, B>(log2l);
    case 12: return pick<12, B>(log2l);
    case 13: return pick<13, B>(log2l);
    case 14: return pick<14, B>(log2l);
    case 15: return pick<15, B>(log2l);
    case 16: return pick<16, B>(log2l);
    default: return nullptr;
  }
}

#define GM_CAT2(a, b) a##b
#define GM_CAT(a, b) GM_CAT2(a, b)

RuleKernelFn GM_CAT(factor_kernel_f, GM_RULE_FAMILY)(int d, int log2l, bool batch) {
  return batch ? factor_fn<true>(d, log2l) : factor_fn<false>(d, log2l);
}

GM_CHECK_UNIT_F(factor, GM_RULE_FAMILY)

}  // namespace gm
