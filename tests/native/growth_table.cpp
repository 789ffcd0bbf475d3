// growth_table against its own quadrature done panel by panel on one thread.  Prints whether repeated
// tables are the same bits, the largest relative difference of D from the serial sum, and the best
// times of both in milliseconds.
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "host_math.hpp"

using namespace pin;

namespace {

double now_ms() {
  return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

// 16-point Gauss-Legendre nodes and weights by Newton steps on the Legendre recurrence
void nodes(double (&x)[16], double (&w)[16]) {
  for (int i = 0; i < 16; ++i) {
    double t = std::cos(3.14159265358979323846 * (i + 0.75) / 16.5), dp = 1.0;
    for (int it = 0; it < 50; ++it) {
      double p0 = 1.0, p1 = t;
      for (int k = 2; k <= 16; ++k) {
        const double p2 = ((2 * k - 1) * t * p1 - (k - 1) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      dp = 16 * (t * p1 - p0) / (t * t - 1.0);
      t -= p1 / dp;
    }
    x[i] = t;
    w[i] = 2.0 / ((1.0 - t * t) * dp * dp);
  }
}

// D at the table's nodes, one panel after another
std::vector<double> serial(double om, const GrowthTable& g) {
  double x[16], w[16];
  nodes(x, w);
  const double ol = 1.0 - om;
  auto panel = [&](double a, double b) {
    double s = 0.0;
    for (int i = 0; i < 16; ++i) {
      const double e = std::exp(0.5 * (a + b) + 0.5 * (b - a) * x[i]);
      s += w[i] * std::pow(e, 2.5) * std::pow(om + ol * e * e * e, -1.5);
    }
    return 0.5 * (b - a) * s;
  };
  const double ys = std::log(1e-8);
  double I = 0.4 * std::pow(1e-8, 2.5) * std::pow(om, -1.5);
  for (int p = 0; p < 4000; ++p) I += panel(ys + (g.y0 - ys) * p / 4000, ys + (g.y0 - ys) * (p + 1) / 4000);
  std::vector<double> d(kGrowthNodes);
  double I1 = I;
  for (int i = 0; i < kGrowthNodes; ++i) {
    if (i > 0)
      for (int q = 0; q < 4; ++q) I += panel(g.y0 + (i - 1 + q / 4.0) * g.h, g.y0 + (i - 1 + (q + 1) / 4.0) * g.h);
    d[i] = I;
  }
  for (int p = 0; p < 4000; ++p) I1 += panel(g.y0 * (1.0 - p / 4000.0), g.y0 * (1.0 - (p + 1) / 4000.0));
  const double norm = 2.5 * om * std::sqrt(om + ol) * I1;
  for (int i = 0; i < kGrowthNodes; ++i) {
    const double a = std::exp(g.y0 + i * g.h);
    d[i] *= 2.5 * om * std::sqrt(om / (a * a * a) + ol) / norm;
  }
  return d;
}

}  // namespace

int main() {
  const double om = 0.25;
  GrowthTable g = growth_table(om);
  double table = 1e30, quadrature = 1e30, worst = 0.0;
  bool same = true;
  for (int k = 0; k < 9; ++k) {
    double t = now_ms();
    const GrowthTable again = growth_table(om);
    table = std::fmin(table, now_ms() - t);
    same = same && again.d == g.d && std::memcmp(again.poly.data(), g.poly.data(), g.poly.size() * 8) == 0;
    t = now_ms();
    const std::vector<double> d = serial(om, g);
    quadrature = std::fmin(quadrature, now_ms() - t);
    for (int i = 0; i < kGrowthNodes; ++i) worst = std::fmax(worst, std::fabs(g.d[i] / d[i] - 1.0));
  }
  std::printf("%d %.3g %.3f %.3f\n", same ? 1 : 0, worst, table, quadrature);
  return 0;
}
