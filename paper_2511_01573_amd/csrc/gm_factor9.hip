// gm_factor9.hip -- the degree-9 rule kernel for the factored families: the
// rule, embedded rules, error models and split axis of gm_rule9.hip (the
// "9-order" reading of arXiv 2511.01573, Sec. 2) with the node values of
// gm_nodes.hpp.
//
// Mappings.  One lane per region (TPR, d <= 10), everything unrolled: no lane
// waits for another, and a triple's eight nodes are one multiply-add each between
// the product of its first two moved factors and that of the third with the
// unmoved ones.  About 3150 FP64 operations a region at d = 8, 1200 of them the
// factors: d = 8 C0, 1.0e6 regions: 130 us (7.5e9 regions/s, 24 TFLOP/s; the
// chain kernel's eight lanes per region: 1100 us).  Above d = 10, and in small
// sets at d = 9 and 10, the 64 lanes of a wavefront per region as in gm_rule9.hip:
// the region's factors, and the products of its centre factors before an axis, after
// it and strictly between two, are formed by its lanes together in LDS, so a node of an axis pair or triple (77% of the 1089 nodes at d = 8) is two
// to four multiplications of shared products instead of an exponential behind a
// chain over the axes that it does not move.
#include "gm_nodes.hpp"
#include "gm_rule9.hpp"

namespace gm {

template <int D, int FAM>
struct Factor9Slot {
  using T = typename Alg<FAM>::T;
  static constexpr bool U = Alg<FAM>::kUnitCentre;
  // per-coordinate terms at the perturbed positions: [0] +l2, [1] -l2,
  // [2] +l3 (= +l4), [3] -l3, [4] +l6, [5] -l6; after the axis nodes, which
  // alone use l6, [4] and [5] hold +l5 and -l5
  T tp[6][D];
  T tc[U ? 1 : D], pre[U ? 1 : D], suf[U ? 1 : D];
  T mid[U ? 1 : D * (D - 1) / 2];  // strictly between axes i < j: [j (j - 1) / 2 + i]
  double c[D], h[D], dv[D], sc[D];
};

// Three wavefronts per SIMD up to d = 10 (the rotation family spills 16 registers
// there); two above, where the compiler uses 128 to 200 registers (rotations: 200 to
// 256, with up to 18 spilled from d = 14 on).
template <int D, int FAM, int LOG2L>
__global__ __launch_bounds__(kRuleBlock) __attribute__((amdgpu_waves_per_eu(D <= 10 ? 3 : 2)))
void factor9_kernel(RuleArgs A) {
  using F = Alg<FAM>;
  using T = typename F::T;
  constexpr bool U = F::kUnitCentre;
  constexpr int L = 1 << LOG2L;
  constexpr int RPB = kRuleBlock / L;  // regions per block step
  constexpr int NPAIR = D * (D - 1) / 2;
  constexpr int NTRI = D * (D - 1) * (D - 2) / 6;
  static_assert(LOG2L <= D && LOG2L <= 6, "at least one corner and one wavefront per region");
  __shared__ Factor9Slot<D, FAM> slots[RPB];
  int64_t start, n;
  int buf;
  if (!active_range<false>(A, start, n, buf)) return;
  const RegionSrc R = region_src<false>(A, buf);
  const RuleConsts& K = A.K;
  const int g = threadIdx.x >> LOG2L;  // region slot in the block
  const int s = threadIdx.x & (L - 1);
  Factor9Slot<D, FAM>& sl = slots[g];
  dd qs = {0.0, 0.0}, es = {0.0, 0.0};
  int nonfin = 0;
  for (int64_t rb = start + (int64_t)blockIdx.x * RPB; rb < n; rb += (int64_t)gridDim.x * RPB) {
    const int64_t r = rb + g;
    const bool valid = r < n;
    double volo;
    const DevParams& P = region_params<false>(A, buf, valid ? r : start, volo);
    const int lvl = load_axes<D, L>(R, valid, r, valid ? list_entry(R, r) : 0, s,
                                    [&](int j, double c, double h) {
                                      sl.c[j] = c;
                                      sl.h[j] = h;
                                      F::pair(P, j, c, h, K.lam2, sl.tp[0][j], sl.tp[1][j]);
                                      F::pair(P, j, c, h, K.lam3, sl.tp[2][j], sl.tp[3][j]);
                                      F::pair(P, j, c, h, K.lam6, sl.tp[4][j], sl.tp[5][j]);
                                      F::centre(P, j, c, sl.tc);
                                    });
    wave_lds_sync();
    const T base = F::template base<D>(P, sl.c);
    __syncthreads();
    T full = base;
    if constexpr (!U) {
      // by rows (first axis i)
      for (int i = s; i < D; i += L) {
        T m = F::none();
        for (int j = i + 1; j < D; ++j) {
          sl.mid[j * (j - 1) / 2 + i] = m;
          m = F::comb(m, sl.tc[j]);
        }
        sl.suf[i] = m;
        m = F::none();
        for (int j = 0; j < i; ++j) m = F::comb(m, sl.tc[j]);
        sl.pre[i] = m;
      }
      __syncthreads();
      full = F::comb(sl.pre[D - 1], sl.tc[D - 1]);
    }
    const double f0 = F::value(full);
    KSum S2 = {0.0, 0.0}, S3 = {0.0, 0.0}, S4 = {0.0, 0.0}, S5 = {0.0, 0.0};
    KSum S6 = {0.0, 0.0}, S7 = {0.0, 0.0}, S8 = {0.0, 0.0};
    // The three node groups run one after the other, so the lanes of a
    // wavefront stay on the same code path.
    // Axes: +-l2, +-l3, +-l6 along axis i and its fourth difference.
    for (int i = s; i < D; i += L) {
      const T b[6] = {sl.tp[0][i], sl.tp[1][i], sl.tp[2][i], sl.tp[3][i], sl.tp[4][i], sl.tp[5][i]};
      double f[6];
      T o = base;
      if constexpr (!U) o = F::comb(sl.pre[i], sl.suf[i]);
      const T a[6] = {o, o, o, o, o, o};
      F::template nodes<6>(a, b, f);
      ks_add(S2, f[0] + f[1]);
      ks_add(S3, f[2] + f[3]);
      ks_add(S6, f[4] + f[5]);
      double dv, scv;
      fourth_diff(K, f0, f[0], f[1], f[2], f[3], dv, scv);
      sl.dv[i] = dv;
      sl.sc[i] = scv;
    }
    // the corner terms take the l6 terms' place (each lane the axes it alone
    // read there)
    for (int j = s; j < D; j += L) F::pair(P, j, sl.c[j], sl.h[j], K.lam5, sl.tp[4][j], sl.tp[5][j]);
    // Axis pairs i < j: class 4 (+-l4, +-l4) and class 7 in both orders.
    for (int it = s; it < NPAIR; it += L) {
      const int pk = kItems<D>.pair[it];
      const int i = pk & 15, j = pk >> 4;
      T o = base;
      if constexpr (!U) o = F::comb(F::comb(sl.pre[i], sl.mid[it]), sl.suf[j]);
      const T i3p = F::comb(o, sl.tp[2][i]), i3m = F::comb(o, sl.tp[3][i]);
      const T i2p = F::comb(o, sl.tp[0][i]), i2m = F::comb(o, sl.tp[1][i]);
      const T j3p = sl.tp[2][j], j3m = sl.tp[3][j], j2p = sl.tp[0][j], j2m = sl.tp[1][j];
      // class 4, then class 7: (+-l3 on i, +-l2 on j) and (+-l2 on i, +-l3 on j)
      const T a[12] = {i3p, i3p, i3m, i3m, i3p, i3p, i3m, i3m, i2p, i2p, i2m, i2m};
      const T b[12] = {j3p, j3m, j3p, j3m, j2p, j2m, j2p, j2m, j3p, j3m, j3p, j3m};
      double f[12];
      F::template nodes<12>(a, b, f);
      ks_add(S4, (f[0] + f[1]) + (f[2] + f[3]));
      ks_add(S7, ((f[4] + f[5]) + (f[6] + f[7])) + ((f[8] + f[9]) + (f[10] + f[11])));
    }
    // Axis triples i < j < k: class 8.
    for (int it = s; it < NTRI; it += L) {
      const int tk3 = kItems<D>.tri[it];
      const int i = tk3 & 15, j = (tk3 >> 4) & 15, k = tk3 >> 8;
      T o = base;
      if constexpr (!U)
        o = F::comb(F::comb(sl.pre[i], sl.mid[j * (j - 1) / 2 + i]),
                    F::comb(sl.mid[k * (k - 1) / 2 + j], sl.suf[k]));
      const T ip = F::comb(o, sl.tp[2][i]), im = F::comb(o, sl.tp[3][i]);
      const T jp = sl.tp[2][j], jm = sl.tp[3][j], kp = sl.tp[2][k], km = sl.tp[3][k];
      const T pp = F::comb(ip, jp), pm = F::comb(ip, jm), mp = F::comb(im, jp), mm = F::comb(im, jm);
      const T a[8] = {pp, pp, pm, pm, mp, mp, mm, mm}, b[8] = {kp, km, kp, km, kp, km, kp, km};
      double f[8];
      F::template nodes<8>(a, b, f);
      ks_add(S8, ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])));
    }
    __syncthreads();
    // Class 5: this lane's 2^(D - LOG2L) corners.
    {
      T t5p[D], t5m[D];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        t5p[j] = sl.tp[4][j];
        t5m[j] = sl.tp[5][j];
      }
      corner_sum<D, FAM, LOG2L>(base, t5p, t5m, (uint32_t)s, S5);
    }
    // Combine the L lanes of the region: each lane's compensated class sums
    // are rounded once and added across the lanes in a butterfly (a + b and
    // b + a round alike, so every lane ends with the same totals).
    double Ts[7] = {ks_val(S2), ks_val(S3), ks_val(S4), ks_val(S5),
                   ks_val(S6), ks_val(S7), ks_val(S8)};
#pragma unroll
    for (int m = L / 2; m >= 1; m >>= 1) {
#pragma unroll
      for (int q = 0; q < 7; ++q) Ts[q] = Ts[q] + __shfl_xor(Ts[q], m, 64);
    }
    __syncthreads();
    if (s == 0 && valid) {
      const double vol = ldexp(volo, -lvl);
      RegionResult o;
      rule9_combine(K, f0, Ts, vol, o);
      double dv[D], scale = 0.0;
#pragma unroll
      for (int i = 0; i < D; ++i) {
        dv[i] = sl.dv[i];
        scale = sl.sc[i] > scale ? sl.sc[i] : scale;
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
// TPR: one lane per region.
// ---------------------------------------------------------------------------
// Class sums: a row of pairs or triples (all of one first axis, or of one first two)
// is added plainly, a running sum per sign pattern, and enters the compensated total
// as one: a node passes through at most d + 2 roundings on the way (a rotation, two
// multiply-adds a node, 2 d + 2), where the several-lane kernels have 2 or 3.  Against
// 80-bit sums over regions of runs at d = 7 to 10, rms error of the value and of err,
// relative to the magnitudes summed: 4.1e-17 to 6.3e-17, 0.68 to 1.07 times the chain
// form's; rotations 0.12 to 0.32 times.
template <int D, int FAM>
__device__ __forceinline__ RegionResult factor9_region(const DevParams& P, const RuleConsts& K,
                                                       const double (&c)[D], const double (&h)[D],
                                                       double vol) {
  using F = Alg<FAM>;
  using T = typename F::T;
  constexpr bool U = F::kUnitCentre;
  T tc[D], t2p[D], t2m[D], t3p[D], t3m[D], suf[D + 1];
  const T base = F::template base<D>(P, c);
#pragma unroll
  for (int j = 0; j < D; ++j) {
    F::pair(P, j, c[j], h[j], K.lam2, t2p[j], t2m[j]);
    F::pair(P, j, c[j], h[j], K.lam3, t3p[j], t3m[j]);
  }
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
  KSum S6 = {0.0, 0.0}, S7 = {0.0, 0.0}, S8 = {0.0, 0.0};
  double Dv[D];
  double scale = 0.0;
  T pre = base;  // tc[0] ... tc[i-1]
#pragma unroll
  for (int i = 0; i < D; ++i) {
    // classes 2, 3 and 6 on axis i
    {
      T t6p, t6m;
      F::pair(P, i, c[i], h[i], K.lam6, t6p, t6m);
      const T o = U ? base : i == 0 ? suf[1] : i == D - 1 ? pre : F::comb(pre, suf[i + 1]);
      const T a[6] = {o, o, o, o, o, o}, b[6] = {t2p[i], t2m[i], t3p[i], t3m[i], t6p, t6m};
      double f[6];
      F::template nodes<6>(a, b, f);
      ks_add(S2, f[0] + f[1]);
      ks_add(S3, f[2] + f[3]);
      ks_add(S6, f[4] + f[5]);
      double sc;
      fourth_diff(K, f0, f[0], f[1], f[2], f[3], Dv[i], sc);
      scale = sc > scale ? sc : scale;
    }
    if (i < D - 1) {
      // row i of the pairs: a running sum per sign pattern (class 4: 4, class
      // 7: 8); m is the product of the centre factors below j except i's
      T m = pre;
      double acc4[4], acc7[8];
#pragma unroll
      for (int j = i + 1; j < D; ++j) {
        const bool none = !U && i == 0 && j == 1;  // no factor below j but i's
        const T o = U ? base : j == D - 1 ? m : none ? suf[j + 1] : F::comb(m, suf[j + 1]);
        const T i3p = F::comb(o, t3p[i]), i3m = F::comb(o, t3m[i]);
        const T i2p = F::comb(o, t2p[i]), i2m = F::comb(o, t2m[i]);
        const T a4[4] = {i3p, i3p, i3m, i3m}, b4[4] = {t3p[j], t3m[j], t3p[j], t3m[j]};
        const T a7[8] = {i3p, i3p, i3m, i3m, i2p, i2p, i2m, i2m};
        const T b7[8] = {t2p[j], t2m[j], t2p[j], t2m[j], t3p[j], t3m[j], t3p[j], t3m[j]};
        if (j == i + 1) {
          F::template accumulate<4, true>(a4, b4, acc4);
          F::template accumulate<8, true>(a7, b7, acc7);
        } else {
          F::template accumulate<4, false>(a4, b4, acc4);
          F::template accumulate<8, false>(a7, b7, acc7);
        }
        if (j < D - 1) {
          // row (i, j) of the triples
          T ij[4] = {F::comb(t3p[i], t3p[j]), F::comb(t3p[i], t3m[j]), F::comb(t3m[i], t3p[j]),
                     F::comb(t3m[i], t3m[j])};
          if constexpr (U) {
#pragma unroll
            for (int q = 0; q < 4; ++q) ij[q] = F::comb(base, ij[q]);
          }
          T m3 = m;
          double acc8[8];
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
            const T a8[8] = {ij[0], ij[0], ij[1], ij[1], ij[2], ij[2], ij[3], ij[3]};
            const T b8[8] = {kp, km, kp, km, kp, km, kp, km};
            if (k == j + 1) F::template accumulate<8, true>(a8, b8, acc8);
            else F::template accumulate<8, false>(a8, b8, acc8);
          }
          ks_add(S8, ((acc8[0] + acc8[1]) + (acc8[2] + acc8[3])) +
                         ((acc8[4] + acc8[5]) + (acc8[6] + acc8[7])));
        }
        if constexpr (!U) m = none ? tc[j] : F::comb(m, tc[j]);
      }
      ks_add(S4, (acc4[0] + acc4[1]) + (acc4[2] + acc4[3]));
      ks_add(S7, ((acc7[0] + acc7[1]) + (acc7[2] + acc7[3])) +
                     ((acc7[4] + acc7[5]) + (acc7[6] + acc7[7])));
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
  const double T7[7] = {ks_val(S2), ks_val(S3), ks_val(S4), ks_val(S5),
                        ks_val(S6), ks_val(S7), ks_val(S8)};
  rule9_combine(K, f0, T7, vol, r);
  split_axis<D>(K, Dv, scale, c, h, r);
  r.nonfinite |= !Fam<base_family(FAM)>::in_range(P, c, h);
  return r;
}

template <int D, int FAM>
__global__ __launch_bounds__(kRuleBlock) __attribute__((amdgpu_waves_per_eu(2)))
void factor9_tpr_kernel(RuleArgs A) {
  int64_t start, end;
  int buf;
  if (!active_range<false>(A, start, end, buf)) return;
  const RegionSrc R = region_src<false>(A, buf);
  const int64_t stride = (int64_t)gridDim.x * kRuleBlock;
  dd qs = {0.0, 0.0}, es = {0.0, 0.0};
  int nonfin = 0;
  // (siblings in neighbouring lanes, as in rule_tpr_kernel)
  const bool pairs = R.pending;
  int64_t v = start + (int64_t)blockIdx.x * kRuleBlock + threadIdx.x;
  for (; v < end; v += stride) {
    const int64_t r = pairs ? ((v & 1) ? R.nkeep + (v >> 1) : (v >> 1)) : v;
    double c[D], h[D];
    const int lvl = load_active<D>(R, r, c, h);
    const RegionResult o = factor9_region<D, FAM>(A.P, A.K, c, h, ldexp(A.vol_omega, -lvl));
    store_result(A, r, o);
    dd_add(qs, o.q);
    dd_add(es, o.err);
    nonfin |= o.nonfinite;
  }
  block_partials(A, qs, es, nonfin);
}

#ifndef GM_RULE_FAMILY
#error "compile with -DGM_RULE_FAMILY=<8..12>"
#endif

#define GM_F9_CAT2(a, b) a##b
#define GM_F9_CAT(a, b) GM_F9_CAT2(a, b)

template <int D>
static RuleKernelFn f9_pick(int log2l) {
  constexpr int F = GM_RULE_FAMILY;
  if constexpr (D <= kTprMaxDim) {
    if (log2l < 0) return factor9_tpr_kernel<D, F>;
  }
  if constexpr (D >= kFactor9WideMinDim) {
    if (log2l == rule9_log2l_wide(D)) return factor9_kernel<D, F, rule9_log2l_wide(D)>;
  }
  return nullptr;
}

RuleKernelFn GM_F9_CAT(factor9_kernel_f, GM_RULE_FAMILY)(int d, int log2l) {
  switch (d) {
    case 7: return f9_pick<7>(log2l);
    case 8: return f9_pick<8>(log2l);
    case 9: return f9_pick<9>(log2l);
    case 10: return f9_pick<10>(log2l);
    case 11: return f9_pick<11>(log2l);
    case 12: return f9_pick<12>(log2l);
    case 13: return f9_pick<13>(log2l);
    case 14: return f9_pick<14>(log2l);
    case 15: return f9_pick<15>(log2l);
    case 16: return f9_pick<16>(log2l);
    default: return nullptr;
  }
}

GM_CHECK_UNIT_F(factor9, GM_RULE_FAMILY)

}  // namespace gm
