// gm_rule9.hpp -- pieces shared by the degree-9 rule kernels (gm_rule9.hip, node
// arguments as chains; gm_factor9.hip, factored): the work-item tables and the
// combination of the class sums into the rule value and error estimate.
#pragma once

#include "gm_corner.hpp"

namespace gm {

// Work-item tables: the axis pairs (i, j) and triples (i, j, k), packed 4
// bits per index, ordered by their last index so that the lanes of a round
// run tail chains of about the same length.
template <int D>
struct ItemTable {
  uint16_t pair[D * (D - 1) / 2 + 1];
  uint16_t tri[D * (D - 1) * (D - 2) / 6 + 1];
};

template <int D>
constexpr ItemTable<D> make_items() {
  ItemTable<D> t{};
  int n = 0;
  for (int j = 1; j < D; ++j)
    for (int i = 0; i < j; ++i) t.pair[n++] = (uint16_t)(i | (j << 4));
  n = 0;
  for (int k = 2; k < D; ++k)
    for (int j = 1; j < k; ++j)
      for (int i = 0; i < j; ++i) t.tri[n++] = (uint16_t)(i | (j << 4) | (k << 8));
  return t;
}

template <int D>
__device__ constexpr ItemTable<D> kItems = make_items<D>();

// Class sums (f0 the centre, T the classes 2 to 8) into the degree-9 rule value,
// the embedded rules and the error estimate (the head of gm_rule9.hip).
__device__ __forceinline__ void rule9_combine(const RuleConsts& K, double f0, const double (&T)[7],
                                              double vol, RegionResult& r) {
  const double S[8] = {f0, T[0], T[1], T[2], T[3], T[4], T[5], T[6]};
  r.nonfinite = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) r.nonfinite |= !isfinite(S[q]);
  double q9 = K.w9[0] * S[0];
  double n1 = K.e9[0] * S[0];
#pragma unroll
  for (int q = 1; q < 8; ++q) {
    q9 = q9 + K.w9[q] * S[q];
    n1 = n1 + K.e9[q] * S[q];
  }
  n1 = fabs(n1);
  double q7 = K.w[0] * S[0];
  double d75 = K.e[0] * S[0];
#pragma unroll
  for (int q = 1; q < 5; ++q) {
    q7 = q7 + K.w[q] * S[q];
    d75 = d75 + K.e[q] * S[q];
  }
  const double n2 = fabs(d75);
  const double q5 = q7 - d75;
  const double q3 = K.q3[0] * S[0] + K.q3[1] * S[2];
  const double n3 = fabs(q5 - q3);
  r.q = vol * q9;
  r.err = K.err_model ? vol * (n1 * fmin(1.0, 2.0 * fmax(n1 / n2, n2 / n3))) : vol * n1;
}

}  // namespace gm
