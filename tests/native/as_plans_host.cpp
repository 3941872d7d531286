// Host-side check of the angular-spectrum plans and the half-aperture codelets:
// HalfDft against a direct double-precision DFT whose input (or kept output)
// is the middle half, every AsPlanFor plan (natural positions and
// frequencies, Cooley-Tukey twiddles) against a direct DFT, and the mean gain of
// the 10- and 20-point codelets.  Exits non-zero on any failure.
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2306_11268_amd/csrc/plan.hpp"

using cd = std::complex<double>;

static std::vector<cd> dft(const std::vector<cd>& x, int sign) {
  const int n = (int)x.size();
  std::vector<cd> y(n);
  for (int k = 0; k < n; ++k)
    for (int j = 0; j < n; ++j) y[k] += x[j] * std::polar(1.0, sign * 2.0 * M_PI * (double)((1LL * j * k) % n) / n);
  return y;
}

static bool close(const char* what, int n, const std::vector<cd>& a, const std::vector<cd>& b) {
  double num = 0, den = 0;
  for (size_t i = 0; i < a.size(); ++i) { num += std::norm(a[i] - b[i]); den += std::norm(b[i]); }
  const double e = std::sqrt(num / den);
  std::printf("%s %d rel=%.2e %s\n", what, n, e, e < 1e-6 ? "ok" : "FAIL");
  return e < 1e-6;  // float32 transforms of up to 1024 points: about 2e-7
}

template <int R>
static bool half(std::mt19937& g) {
  std::normal_distribution<double> nd;
  std::vector<cd> x(R), full(R);
  float2 xs[R / 2], X[R], back[R / 2];
  for (int i = 0; i < R / 2; ++i) {
    xs[i] = lr::c2((float)nd(g), (float)nd(g));
    x[R / 4 + i] = cd(xs[i].x, xs[i].y);
  }
  lr::HalfDft<R>::forward(xs, X);
  std::vector<cd> got(R);
  for (int i = 0; i < R; ++i) got[i] = cd(X[i].x, X[i].y);
  bool ok = close("half forward", R, got, dft(x, -1));
  for (int i = 0; i < R; ++i) { X[i] = lr::c2((float)nd(g), (float)nd(g)); full[i] = cd(X[i].x, X[i].y); }
  lr::HalfDft<R>::inverse(X, back);
  const std::vector<cd> ref = dft(full, +1);
  std::vector<cd> a(R / 2), b(R / 2);
  for (int i = 0; i < R / 2; ++i) { a[i] = cd(back[i].x, back[i].y); b[i] = ref[R / 4 + i]; }
  return ok & close("half inverse", R, a, b);
}

template <int N>
static bool plan(std::mt19937& g) {
  using PL = typename lr::AsPlanFor<N>::type;
  std::normal_distribution<double> nd;
  std::vector<cd> x(N), got(N);
  std::vector<float2> v(N), w(N);
  for (int i = 0; i < N; ++i) { v[i] = lr::c2((float)nd(g), (float)nd(g)); x[i] = cd(v[i].x, v[i].y); }
  // (natural order at every length but the Good-Thomas 350)
  bool ok = PL::N == N && PL::PFA == (N == 350);
  for (int j = 0; j < PL::N2; ++j) {
    float2 a[PL::N1];
    for (int k = 0; k < PL::N1; ++k) a[k] = v[PL::PFA ? PL::pos(k, j) : j + PL::N2 * k];
    lr::Dft<PL::N1, -1>::run(a);
    for (int k = 0; k < PL::N1; ++k) w[j + PL::N2 * k] = a[k];
  }
  for (int k1 = 0; k1 < PL::N1; ++k1) {
    float2 b[PL::N2];
    for (int j = 0; j < PL::N2; ++j) b[j] = PL::PFA ? w[PL::N2 * k1 + j] : lr::cmul(w[PL::N2 * k1 + j], PL::twiddle(k1, j));
    lr::Dft<PL::N2, -1>::run(b);
    for (int k2 = 0; k2 < PL::N2; ++k2) got[PL::PFA ? PL::freq(k1, k2) : k1 + PL::N1 * k2] = cd(b[k2].x, b[k2].y);
  }
  return ok & close("plan", N, got, dft(x, -1));
}

// Mean gain Re<X, got>/<X, X> - 1 over random vectors.  4000 vectors of R values
// leave a standard error of about 1e-7 / sqrt(8000 R) < 4e-10; the constants
// rounded to nearest give 8e-9, the chosen ones 3e-9.
template <int R, int SIGN>
static bool gain(std::mt19937& g) {
  std::normal_distribution<double> nd;
  double num = 0, den = 0;
  for (int t = 0; t < 4000; ++t) {
    std::vector<cd> x(R);
    float2 v[R];
    for (int i = 0; i < R; ++i) { v[i] = lr::c2((float)nd(g), (float)nd(g)); x[i] = cd(v[i].x, v[i].y); }
    lr::Dft<R, SIGN>::run(v);
    const std::vector<cd> ref = dft(x, SIGN);
    for (int i = 0; i < R; ++i) {
      num += std::real((cd(v[i].x, v[i].y) - ref[i]) * std::conj(ref[i]));
      den += std::norm(ref[i]);
    }
  }
  const bool ok = std::abs(num / den) < 5e-9;
  std::printf("gain %d %d 1%+.2e %s\n", R, SIGN, num / den, ok ? "ok" : "FAIL");
  return ok;
}

int main() {
  std::mt19937 g(77);
  bool ok = half<8>(g) & half<16>(g) & half<20>(g) & half<32>(g);
  ok &= plan<64>(g) & plan<100>(g) & plan<128>(g) & plan<200>(g) & plan<256>(g) & plan<350>(g) & plan<400>(g);
  ok &= plan<500>(g) & plan<512>(g) & plan<1000>(g) & plan<1024>(g);
  ok &= gain<10, -1>(g) & gain<10, 1>(g) & gain<20, -1>(g) & gain<20, 1>(g);
  std::printf(ok ? "ALL OK\n" : "FAILURES\n");
  return ok ? 0 : 1;
}
