// CPU check of the LDS line transforms of the momentum-space kernels (line_dft,
// dft_places): every even length up to 64, both signs, both precisions and two strides,
// against a direct DFT in long double.  Built by hipcc for the host only.
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <vector>

#include "ov_kernels.hpp"

using namespace ov;
using cld = std::complex<long double>;

template <class R>
double worst(int N, int st, int sgn) {
  const long double pi2 = 2 * 3.141592653589793238462643383279503L;
  std::vector<c2<R>> a((size_t)N * st), tw(N), out((size_t)N * st, c2<R>{R(99), R(99)});
  unsigned s = 12345u + 7u * (unsigned)N;
  auto rnd = [&]() {
    s = s * 1664525u + 1013904223u;
    return (R)((double)(s >> 8) / 16777216.0 - 0.5);
  };
  for (auto& v : a) {
    v.x = rnd();
    v.y = rnd();
  }
  for (int m = 0; m < N; ++m)
    tw[m] = c2<R>{(R)std::cos(pi2 * m / N), (R)std::sin(pi2 * m / N)};
  for (int g = 0; g < dft_groups(N); ++g) {
    c2<R> o[4];
    int at[4];
    line_dft<R>(a.data(), st, N, tw.data(), g, (R)sgn, o);
    dft_places(N, g, st, at);
    for (int q = 0; q < 4; ++q) out[at[q]] = o[q];
  }
  long double err = 0, nrm = 0;
  for (int k = 0; k < N; ++k) {
    cld acc = 0;
    for (int j = 0; j < N; ++j)
      acc += cld(a[(size_t)j * st].x, a[(size_t)j * st].y) *
             std::polar(1.0L, sgn * pi2 * (long double)(j * k % N) / N);
    const c2<R> v = out[(size_t)k * st];
    err = std::max(err, std::abs(acc - cld(v.x, v.y)));
    nrm = std::max(nrm, std::abs(acc));
  }
  return (double)(err / nrm);
}

int main() {
  double w64 = 0, w32 = 0;
  for (int N = 2; N <= 64; N += 2)
    for (int st : {1, 5})
      for (int sgn : {-1, 1}) {
        w64 = std::max(w64, worst<double>(N, st, sgn));
        w32 = std::max(w32, worst<float>(N, st, sgn));
      }
  std::printf("worst fp64 %.2e fp32 %.2e\n", w64, w32);
  // 64 terms of up to sqrt(2)/2, each rounded three times at most: 64 x 3 x 2^-53 of sums
  // that are at least as large as one term
  const bool ok = w64 < 192 * 1.2e-16 && w32 < 192 * 6e-8;
  if (ok) std::printf("line_dft ok\n");
  return ok ? 0 : 1;
}
