// Host-side check of the difference-form interpolation and of its reverse
// (hweno_point_diff, hweno_point_diff_vjp) against the direct forms (hweno_point,
// hweno_point_vjp) for linear weights over the whole accepted range (0, 1), also
// next to its ends. Prints one line per check and "ALL OK".
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <random>

#include "hweno_adjoint_diff.h"

using namespace hweno;

static std::mt19937_64 rng(815);
static double unif(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }
static int failures = 0;
// The largest relative difference; a value that is not finite stays.
struct Worst {
  double v = 0.0;
  void add(double got, double want, double scale) {
    const double e = std::fabs(got - want) / scale;
    if (!(e <= v)) v = e;
    if (!std::isfinite(got) || !std::isfinite(want)) v = NAN;
  }
};
// Both forms in double: differences of the data and of the smoothness
// indicators cost a few digits of 16 each, which leaves 1e-9 (float: of the
// single-precision result, 4 roundings of 6e-8).
template <typename T>
constexpr double kTol = sizeof(T) == 8 ? 1e-9 : 2.5e-7;

template <typename T>
static void check(double gamma0, double d0, double scale) {
  Scheme s{};
  const double h = 0.05;
  s.dx = s.dy = h;
  s.idx = s.idy = 1.0 / h;
  s.gamma0 = gamma0;
  s.g1 = 0.5 * (1.0 - gamma0);
  s.d0 = d0;
  s.d1 = 0.5 * (1.0 - d0);
  s.eps = 1e-10;
  const double lam = Carried<T>::lam, vts = point_vt_scale<T>(s);
  const PointK k = point_k(s, lam, vts);
  Worst forward, reverse;
  for (int trial = 0; trial < 200; ++trial) {
    // differences of a few scales, equal data among them (float data, so that
    // both types see the same stencil)
    const double e1 = trial == 0 ? 0.0 : (float)(scale * unif(-1, 1)), e2 = trial == 0 ? 0.0 : (float)(scale * unif(-1, 1));
    const double vm = trial == 0 ? 0.0 : (float)(scale * unif(-20, 20)), vp = trial == 0 ? 0.0 : (float)(scale * unif(-20, 20));
    double uR, uL, vt;
    hweno_point<double>(-e1, 0.0, e2, vm, vp, s, h, 1.0 / h, uR, uL, vt);
    T dR, dL, at;
    const T S = T(lam * h * (vm + vp)), D = T(lam * h * (vm - vp));
    hweno_point_diff<T>(T(e1), T(e2), S, D, k, dR, dL, at);
    const double m = std::fabs(e1) + std::fabs(e2) + h * (std::fabs(vm) + std::fabs(vp)) + 1e-300;
    forward.add((double)dR, uR, m);
    forward.add(-(double)dL, uL, m);
    forward.add((double)at * vts / h, vt, m / h);
    if (sizeof(T) != 8) continue;
    const double gR = unif(-1, 1), gL = unif(-1, 1), gT = unif(-1, 1);
    double b[5] = {};
    hweno_point_vjp(-e1, 0.0, e2, vm, vp, s, h, 1.0 / h, gR, gL, gT, b[0], b[1], b[2], b[3], b[4]);
    T r_, l_, t_, g1, g2, gS, gD;
    hweno_point_diff_vjp<kOutAll, T>(T(e1), T(e2), S, D, k, T(gR), T(-gL), T(gT * vts / h), r_, l_, t_, g1, g2, gS, gD);
    double mag = 1.0;
    for (double x : b) mag = std::fmax(mag, std::fabs(x));
    reverse.add(-(double)g1, b[0], mag);
    reverse.add((double)g2, b[2], mag);
    reverse.add(lam * h * ((double)gS + (double)gD), b[3], mag);
    reverse.add(lam * h * ((double)gS - (double)gD), b[4], mag);
    forward.add((double)r_, (double)dR, m);
    forward.add((double)l_, (double)dL, m);
    forward.add((double)t_, (double)at, m);
  }
  const bool ok = forward.v <= kTol<T> && reverse.v <= kTol<T>;
  if (!ok) ++failures;
  std::printf("%s gamma0 %-8.1e d0 %-8.1e differences %-6.0e forward %.1e reverse %.1e %s\n",
              sizeof(T) == 8 ? "f64" : "f32", gamma0, d0, scale, forward.v, reverse.v, ok ? "ok" : "FAIL");
}

int main() {
  const double ends[] = {4.9e-324, 1e-300, 1e-160, 1e-100, 1e-30, 1e-3, 0.5, 0.95, 1.0 - 1.2e-16};
  for (double gamma0 : ends)
    for (double d0 : ends)
      for (double scale : {1e-4, 1.0, 1e3}) {
        check<double>(gamma0, d0, scale);
        check<float>(gamma0, d0, scale);
      }
  if (failures) { std::printf("%d FAILED\n", failures); return 1; }
  std::printf("ALL OK\n");
  return 0;
}
