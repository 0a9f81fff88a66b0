// Host-side check of the double Box-Muller pair (normals64_with) against an
// 80-bit evaluation, with a reciprocal square root good to 2^-24 as the
// device's is.  Prints the largest relative error in units of 2^-53 and exits
// nonzero when it exceeds the bound given as the first argument.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../../paper_2110_15425_amd/csrc/normal64.hpp"

namespace {

double worst = 0.0;
unsigned long long n_tests = 0;

void check(uint64_t ma, uint64_t mb, double noise) {  // u = (m + 1) 2^-53, m < 2^53
  cm::Words w{(uint32_t)(ma << 11) | 0x155u, (uint32_t)(ma >> 21), (uint32_t)(mb << 11) | 0x2AAu,
              (uint32_t)(mb >> 21)};
  double z[2];
  cm::normals64_with(w, cm::kNormTabValues,
                     [&](double x) { return (double)(1.0L / sqrtl((long double)x)) * (1.0 + noise); }, z[0], z[1]);
  const uint64_t na = ma + 1, nb = mb + 1, one = 1ull << 53;
  const long double lu = na > one / 2 ? log1pl(-(long double)(one - na) * 0x1p-53L) : logl((long double)na * 0x1p-53L);
  const long double rho = sqrtl(-2.0L * lu);
  const uint64_t quad = (nb + (one >> 3)) >> 51;  // the nearest quarter turn, and the rest exactly
  const long double a = 6.283185307179586476925286766559L * ((long double)(int64_t)(nb - (quad << 51)) * 0x1p-53L);
  const long double c = cosl(a), s = sinl(a);
  const long double C[4] = {c, -s, -c, s}, S[4] = {s, c, -s, -c};
  const long double want[2] = {rho * C[quad & 3], rho * S[quad & 3]};
  for (int k = 0; k < 2; ++k) {
    ++n_tests;
    const long double d = fabsl((long double)z[k] - want[k]), m = fabsl(want[k]);
    // a zero of the exact pair (u_a = 1, or a quarter turn): within 10^-150
    const double e = m == 0.0L ? (d < 1e-149L ? 0.0 : 1e300) : (double)(d / m * 0x1p53L);
    if (!(e <= worst)) worst = e == e ? e : 1e300;
  }
}

}  // namespace

int main(int, char** argv) {
  std::mt19937_64 g(5);
  const uint64_t one = 1ull << 53;
  auto any = [&] { return g() >> 11; };
  const double noise[3] = {0.0, 6e-8, -6e-8};
  for (int k = 0; k < 3; ++k) {
    for (int d = -2; d <= 2; ++d) {
      for (int e = 0; e <= 53; ++e)         // either side of each interval's edge, at every exponent
        for (int i = 0; i < 256; ++i) {
          const uint64_t edge = (uint64_t)ldexp(1.0 + i / 256.0, e);
          const uint64_t m = edge - 1 + (uint64_t)d;
          if (m < one) check(m, any(), noise[k]);
        }
      for (uint64_t j = 0; j <= 256; ++j) {  // and of each part of the circle
        const uint64_t m = j * (one >> 8) - 1 + (uint64_t)d;
        if (m < one) check(any(), m, noise[k]);
      }
    }
    for (uint64_t m = 0; m < 4096; ++m) {    // smallest and largest uniforms
      check(m, any(), noise[k]);
      check(one - 1 - m, any(), noise[k]);
      check(any(), m, noise[k]);
      check(any(), one - 1 - m, noise[k]);
      check(one - 1 - m, one - 1 - m, noise[k]);
    }
    for (int i = 0; i < 300000; ++i) check(any() >> (g() % 53), any(), noise[k]);
    for (int i = 0; i < 300000; ++i) check(one - 1 - (any() >> (g() % 53)), any(), noise[k]);
  }
  printf("tests %llu worst %.3f\n", n_tests, worst);
  return !(worst <= atof(argv[1]));
}
