// Host build of the kernels' sine-cosine pairs and of their quick reciprocal
// (paper_2511_01573_amd/csrc/gm_math.hpp) for tests/test_device_math_pairs.py.
#include "gm_math.hpp"
extern "C" {
void gm_test_sincos(const double* x, const double* xl, double* s, double* c, long n, int tail) {
  for (long i = 0; i < n; ++i) {
    const double a[1] = {x[i]}, l[1] = {xl[i]};
    double sn[1], cs[1];
    if (tail) gm::fm::sincos_n<1, true>(a, l, sn, cs);
    else gm::fm::sincos_n<1, false>(a, l, sn, cs);
    s[i] = sn[0];
    c[i] = cs[0];
  }
}
void gm_test_rcp3(const double* x, double* y, long n) {
  for (long i = 0; i < n; ++i) {
    const double a[1] = {x[i]};
    double r[1];
    gm::fm::rcp3_n<1>(a, r);
    y[i] = r[0];
  }
}
}
