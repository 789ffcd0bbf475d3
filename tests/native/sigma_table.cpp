// The sigma_8 quadrature of plan creation against the same sum on one thread.  Prints the largest
// relative difference and the best times of both in milliseconds.
#include <chrono>
#include <cmath>
#include <cstdio>

#include "host_math.hpp"

using namespace pin;

static double now_ms() {
  return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

// composite Simpson in ln k with as many evaluations of the integrand (64000)
static double serial(double radius, double gamma, double ns) {
  const double a = std::log(1e-7), b = std::log(1e3);
  const int n = 64000;
  const double h = (b - a) / n;
  double total = 0.0;
  for (int i = 0; i <= n; ++i) {
    const double k = std::exp(a + i * h), t = bbks_transfer(k, gamma), w = tophat_window(k * radius);
    total += (i == 0 || i == n ? 1 : i % 2 ? 4 : 2) * k * k * k * std::pow(k, ns) * t * t * w * w;
  }
  return total * h / 3 / (2 * 3.14159265358979323846 * 3.14159265358979323846);
}

int main() {
  double parts = 1e30, one = 1e30, worst = 0.0;
  for (int r = 0; r < 15; ++r) {
    double t = now_ms();
    const double s = sigma2_tophat_unit(8.0, 0.21, 1.0);
    parts = std::fmin(parts, now_ms() - t);
    t = now_ms();
    const double q = serial(8.0, 0.21, 1.0);
    one = std::fmin(one, now_ms() - t);
    worst = std::fmax(worst, std::fabs(s / q - 1.0));
  }
  std::printf("%.3g %.3f %.3f\n", worst, parts, one);
  return 0;
}
