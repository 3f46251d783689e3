// Error of the staged interpolation's window sum on fp32 grids (gp_window.h)
// against fp64, beside the order whose place it took: four lanes' quarters of the
// window's rows, each added in fp32 and joined in fp64; and beside rows joined one by
// one in fp64 where ROWS asks for that.  Random and smooth grids, every width.
#include <array>
#include <cmath>
#include <cstdio>
#include <random>
#include <utility>
#include <vector>

#include "../../paper_2407_03608_amd/csrc/gp_window.h"

namespace {
struct F2 {
  float x, y;
};
std::mt19937_64 gen(7);
double uniform(double a, double b) { return std::uniform_real_distribution<double>(a, b)(gen); }
double normal() { return std::normal_distribution<double>()(gen); }

int failures = 0;

template <int D, int W, bool ROWS>
void width(bool smooth) {
  constexpr int RG = D == 2 ? 2 : 1, HP = (W + RG - 1) / RG;
  constexpr int S1 = W | 1, S2 = D > 2 ? S1 * W : S1, N = S1 * W * (D > 2 ? W : 1);
  const int samples = 6000;
  double e_now = 0, e_quarters = 0, e_rows = 0, e_plain = 0, size = 0;
  std::vector<F2> g(N + S1);
  for (int t = 0; t < samples; ++t) {
    float p[3][W];
    for (int r = 0; r < 3; ++r) {
      const double del = uniform(-0.5 * W, -0.5 * W + 1);
      for (int q = 0; q < W; ++q) {
        const double z = (del + q) * 2.0 / W, u = 1 - z * z;
        p[r][q] = (float)(u >= 0 ? std::exp(2.3 * W * (std::sqrt(u) - 1)) : 0.0);
      }
    }
    double k[6][4];
    for (auto& wave : k) {
      for (int r = 0; r < 3; ++r) wave[r] = uniform(-M_PI / 2, M_PI / 2);
      wave[3] = uniform(0, 2 * M_PI);
    }
    for (int c = 0; c < N; ++c) {
      const int q0 = c % S1, q1 = c / S1 % W, q2 = D > 2 ? c / (S1 * W) : 0;
      double a = 0, b = 0;
      if (smooth)
        for (auto& wave : k) {
          const double ph = wave[0] * q0 + wave[1] * q1 + wave[2] * q2 + wave[3];
          a += std::cos(ph);
          b += std::sin(ph);
        }
      else {
        a = normal();
        b = normal();
      }
      g[c] = F2{(float)a, (float)b};
    }
    // fp64, and the row sums of the former order (fp32 along a row)
    constexpr int NR = D > 2 ? W * W : W;
    double ex = 0, rows = 0;
    float quarter[4] = {0, 0, 0, 0}, plain = 0;
    for (int row = 0; row < NR; ++row) {
      const int q1 = row % W, q2 = D > 2 ? row / W : 0;
      const F2* tr = g.data() + q2 * S2 * (D > 2) + q1 * S1;
      double d = 0;
      float s = 0;
      for (int q0 = 0; q0 < W; ++q0) {
        d += (double)p[0][q0] * tr[q0].x;
        s = std::fmaf(p[0][q0], tr[q0].x, s);
      }
      const double wd = (double)p[1][q1] * (D > 2 ? (double)p[2][q2] : 1.0);
      const float wf = D > 2 ? p[1][q1] * p[2][q2] : p[1][q1];
      ex += wd * d;
      rows += (double)wf * (double)s;
      quarter[row % 4] = std::fmaf(wf, s, quarter[row % 4]);
      plain = std::fmaf(wf, s, plain);
    }
    const double quarters = (double)quarter[0] + quarter[1] + quarter[2] + quarter[3];
    // the kernel's sum: RG lanes, joined in fp64
    double now = 0;
    float p0[W], pm[W];
    for (int q = 0; q < W; ++q) {
      p0[q] = p[0][q];
      pm[q] = p[1][q];
    }
    for (int rg = 0; rg < RG; ++rg) {
      double bx, by;
      float ph[HP];
      for (int j = 0; j < HP; ++j) ph[j] = rg + RG * j < W ? p[D - 1][rg + RG * j] : 0.f;
      const int last = rg + RG * (HP - 1) < W ? RG * (HP - 1) * S2 : 0;
      if constexpr (D > 2) {
        gp::window_sum<float, F2, D, W, HP, RG, S1, S2, ROWS>(g.data() + rg * S2, last, p0, pm, ph, &bx, &by);
      } else {
        float none[1] = {0};
        gp::window_sum<float, F2, D, W, HP, RG, S1, S2, ROWS>(g.data() + rg * S2, last, p0, ph, none, &bx, &by);
      }
      now += bx;
    }
    auto sq = [](double v) { return v * v; };
    e_now += sq(now - ex);
    e_quarters += sq(quarters - ex);
    e_rows += sq(rows - ex);
    e_plain += sq(plain - ex);
    size += sq(ex);
  }
  const double u = std::sqrt(size) * std::ldexp(1.0, -24);
  const double now = std::sqrt(e_now) / u, old = std::sqrt(ROWS ? e_rows : e_quarters) / u;
  // 6000 samples: 2 % of statistical error on the ratio
  const bool ok = now <= 1.02 * old;
  failures += !ok;
  std::printf("%d-D w=%d %s %s: %.3f, former %.3f, all in fp32 %.3f%s\n", D, W, smooth ? "smooth" : "random",
              ROWS ? "rows" : "", now, old, std::sqrt(e_plain) / u, ok ? "" : "  FAIL");
}

template <int D, bool ROWS, int... W>
void widths(std::integer_sequence<int, W...>) {
  (width<D, W + 2, ROWS>(false), ...);
  (width<D, W + 2, ROWS>(true), ...);
}
}  // namespace

int main() {
  widths<2, false>(std::make_integer_sequence<int, 15>());  // 2 .. 16
  widths<3, false>(std::make_integer_sequence<int, 6>());   // 2 .. 7
  width<3, 7, true>(false);
  width<3, 7, true>(true);
  width<3, 8, true>(false);
  width<3, 8, true>(true);
  width<3, 9, true>(false);
  width<3, 9, true>(true);
  width<3, 12, true>(false);
  width<3, 12, true>(true);
  std::printf("%d failures\n", failures);
  return failures != 0;
}
