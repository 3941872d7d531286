// Precision of the angular-spectrum transforms, on the host: the device functions
// of the passes (A-step, item twiddles, B-step, half apertures), compiled as
// plain C++, against 64 bits, next to the length's general plan (PlanFor, whole
// transforms, roots rounded to nearest) on the same inputs.  A length whose
// passes round worse than that plan fails.
//
// 1-D transforms of normal random values; forward from, and inverse to, the
// whole grid or its middle half.  Prints the relative r.m.s. error of both and
// the mean gain, which adds up over the transforms of a network.
#include <hip/hip_runtime.h>

#include <complex>
#include <random>
#include <vector>

#include "../../paper_2306_11268_amd/csrc/as_impl.hpp"

using cd = std::complex<double>;
using namespace lr;
constexpr int N = LR_FFT_N;

static std::vector<float2> nearest_roots() {
  std::vector<float2> w(N + 1);
  for (int k = 0; k <= N; ++k) {
    const cdbl z = unit_root(k, N, -1);
    w[k] = c2((float)z.re, (float)z.im);
  }
  return w;
}

// The general plan: the steps of tile.hpp.
template <int SIGN>
static void reference(const std::vector<float2>& in, std::vector<float2>& out) {
  using PL = typename PlanFor<N>::type;
  static const std::vector<float2> w = nearest_roots();
  auto times = [](float2 v, int k1, int j) {
    if (PL::PFA) return v;
    auto by = [&](float2 u, float2 w) { return SIGN < 0 ? cmul(u, w) : cmulc(u, w); };
    if (PL::N2 < 32 || j < 8 || j % 8 == 0) return by(v, w[k1 * j]);
    return by(v, cmul(w[k1 * (j % 8)], w[k1 * (j / 8 * 8)]));
  };
  std::vector<float2> v(N);
  float2 a[PL::N1], b[PL::N2];
  if (SIGN < 0) {
    for (int j = 0; j < PL::N2; ++j) {
      for (int k = 0; k < PL::N1; ++k) a[k] = in[PL::pos(k, j)];
      Dft<PL::N1, -1>::run(a);
      for (int k = 0; k < PL::N1; ++k) v[PL::N2 * k + j] = a[k];
    }
    for (int k1 = 0; k1 < PL::N1; ++k1) {
      for (int j = 0; j < PL::N2; ++j) b[j] = j ? times(v[PL::N2 * k1 + j], k1, j) : v[PL::N2 * k1];
      Dft<PL::N2, -1>::run(b);
      for (int k = 0; k < PL::N2; ++k) out[PL::freq(k1, k)] = b[k];
    }
  } else {
    for (int k1 = 0; k1 < PL::N1; ++k1) {
      for (int k = 0; k < PL::N2; ++k) b[k] = in[PL::freq(k1, k)];
      Dft<PL::N2, 1>::run(b);
      for (int j = 0; j < PL::N2; ++j) v[PL::N2 * k1 + j] = j ? times(b[j], k1, j) : b[j];
    }
    for (int j = 0; j < PL::N2; ++j) {
      for (int k = 0; k < PL::N1; ++k) a[k] = v[PL::N2 * k + j];
      Dft<PL::N1, 1>::run(a);
      for (int k = 0; k < PL::N1; ++k) out[PL::pos(k, j)] = a[k];
    }
  }
}

// The passes' own functions.
template <class PL, int SIGN, bool HALF>
static void passes(const std::vector<float2>& in, std::vector<float2>& out) {
  using IT = AsItems<PL>;
  constexpr int KN = IT::KN(HALF), K0 = IT::K0(HALF);
  std::vector<float2> v(N);
  float2 u[KN], x[PL::N1], y[PL::N2];
  if (SIGN < 0) {
    for (int j = 0; j < PL::N2; ++j) {
      for (int k = 0; k < KN; ++k) u[k] = in[PL::pos(k + K0, j)];
      as_a_forward<IT, HALF>(u, x);
      for (int k = 0; k < PL::N1; ++k) v[PL::N2 * k + j] = x[k];
    }
    for (int k1 = 0; k1 < PL::N1; ++k1) {
      for (int j = 0; j < PL::N2; ++j) y[j] = v[PL::N2 * k1 + j];
      item_forward<IT>(k1, y);
      for (int k = 0; k < PL::N2; ++k) out[PL::freq(k1, k)] = y[k];
    }
  } else {
    for (int k1 = 0; k1 < PL::N1; ++k1) {
      for (int k = 0; k < PL::N2; ++k) y[k] = in[PL::freq(k1, k)];
      item_inverse<IT>(k1, y);
      for (int j = 0; j < PL::N2; ++j) v[PL::N2 * k1 + j] = y[j];
    }
    for (int j = 0; j < PL::N2; ++j) {
      for (int k = 0; k < PL::N1; ++k) x[k] = v[PL::N2 * k + j];
      as_a_inverse<IT, HALF>(x, u);
      for (int k = 0; k < KN; ++k) out[PL::pos(k + K0, j)] = u[k];
    }
  }
}

struct Error {
  double num = 0, gain = 0, den = 0;
  void add(float2 got, cd ref) {
    const cd d = cd(got.x, got.y) - ref;
    num += std::norm(d);
    gain += std::real(d * std::conj(ref));
    den += std::norm(ref);
  }
  double rms() const { return std::sqrt(num / den); }
};

// More than 2.5 % above the general plan fails: 12 outputs each of 20000 / sqrt(N)
// vectors on the same inputs leave under 0.5 %, and the half transforms of 400
// points round 2 % worse, which a hop makes up for (its 1/N^2 is not rounded by
// itself, its mean gain is taken out).  The far field has no such product; a
// whole transform of it may not round worse at all.
template <int SIGN, bool HALF, bool FAR = false>
static bool compare() {
  std::mt19937 g(11);
  std::normal_distribution<double> nd;
  std::vector<cd> root(N);
  for (int i = 0; i < N; ++i) root[i] = std::polar(1.0, SIGN * 2.0 * M_PI * i / N);
  Error own, ref;
  for (int t = 0; t < 20000 / std::sqrt(N); ++t) {
    std::vector<float2> x(N), a(N), b(N);
    for (int i = 0; i < N; ++i) {
      x[i] = c2((float)nd(g), (float)nd(g));
      if (HALF && SIGN < 0 && (i < N / 4 || i >= 3 * N / 4)) x[i] = c2(0.f, 0.f);
    }
    passes<AsPlan<N, FAR>, SIGN, HALF>(x, a);
    reference<SIGN>(x, b);
    for (int q = 0; q < 12; ++q) {
      const int k = HALF && SIGN > 0 ? N / 4 + (int)(g() % (N / 2)) : (int)(g() % N);
      cd s = 0;
      for (int i = 0; i < N; ++i) s += cd(x[i].x, x[i].y) * root[(long)i * k % N];
      own.add(a[k], s);
      ref.add(b[k], s);
    }
  }
  const bool ok = own.rms() < (FAR ? 1.0005 : 1.025) * ref.rms();
  std::printf("N=%d %s %s: %.3e (gain %+.1e), general plan %.3e (%+.1e), ratio %.4f %s\n", N,
              FAR ? "far" : SIGN < 0 ? "forward" : "inverse", HALF ? "half" : "whole", own.rms(), own.gain / own.den, ref.rms(),
              ref.gain / ref.den, own.rms() / ref.rms(), ok ? "ok" : "FAIL");
  return ok;
}

int main() {
  bool ok = compare<-1, false>() & compare<1, false>();
  if constexpr (as_half_plan<N>()) ok &= compare<-1, true>() & compare<1, true>();
  ok &= compare<-1, false, true>();
  std::printf(ok ? "ALL OK\n" : "FAILURES\n");
  return ok ? 0 : 1;
}
