// SCDM's block bound against the value the update computes: random columns and
// unit directions, the direction turned towards the column so that what is
// left after the downdate runs from all of the norm to far below the rounding
// of the projection.  The projection is summed as the pick does (64 lanes, the
// normalisation applied to each value, a butterfly) and as the update does (in order,
// fused).  Prints the number of cases whose bound exceeds the updated norm,
// for the library's bound and for a margin relative to what is left.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2309_00651_amd/csrc/scdm_bound.hpp"

int main() {
  std::mt19937_64 rng(17);
  std::normal_distribution<double> nd;
  int over = 0, over_relative = 0, loose = 0, cases = 0;
  for (int n : {1, 2, 8, 63, 64, 65, 128, 300, 1000})
    for (int e = 0; e <= 18; ++e)
      for (int rep = 0; rep < 40; ++rep, ++cases) {
        std::vector<double> a(n), r(n), q(n);
        double na = 0.0, nr = 0.0;
        for (int i = 0; i < n; ++i) a[i] = nd(rng), na += a[i] * a[i];
        for (int i = 0; i < n; ++i) {
          r[i] = a[i] + std::pow(10.0, -0.5 * e) * std::sqrt(na / n) * nd(rng);
          nr += r[i] * r[i];
        }
        const double inv = 1.0 / std::sqrt(nr);
        for (int i = 0; i < n; ++i) q[i] = r[i] * inv;
        double lane[64] = {}, sq[64] = {};
        for (int i = 0; i < n; ++i) {
          lane[i % 64] = std::fma(r[i] * inv, a[i], lane[i % 64]);
          sq[i % 64] = std::fma(a[i], a[i], sq[i % 64]);
        }
        for (int s = 32; s > 0; s >>= 1)
          for (int l = 0; l < s; ++l) lane[l] += lane[l + s], sq[l] += sq[l + s];
        double t = 0.0, w = 0.0;
        for (int i = 0; i < n; ++i) t = std::fma(q[i], a[i], t), w = std::fma(a[i], a[i], w);
        const double now = std::fmax(std::fma(-t, t, w), 0.0);
        const double bound = hfx::scdm_lower_bound(w, lane[0], sq[0], n);
        over += bound > now;
        over_relative += (w - lane[0] * lane[0]) * (1.0 - 1e-12) > now;
        // not below the norm by more than the margin where that norm is large
        loose += e == 0 && n > 1 && bound < now - 1e-9 * w;
      }
  std::printf("cases %d over %d over_relative %d loose %d\n", cases, over, over_relative, loose);
  return 0;
}
