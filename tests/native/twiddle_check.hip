// The balanced float32 twiddle tables of the reduced pair grids: every factor is
// a float32 neighbour of the exact one, and the norm errors of a leg (one r of a
// stage, over k) cancel as far as its neighbours allow.  Prints the largest
// distance in units of the last place below 1, the largest excess of a leg's mean
// norm error over the smallest that any choice of neighbours gives (legs of up to
// 6 factors: every choice tried), the largest mean of the longer legs, and the
// largest means of these tables and of unit_f32's.
#include <cmath>
#include <cstdio>
#include <vector>

#include "../../paper_2309_00651_amd/csrc/twiddle.hpp"

using namespace hfx;

static std::vector<float> near(double x) {
  const float f = (float)x;
  if ((double)f == x) return {f};
  return {f, std::nextafter(f, (double)f < x ? 2.0f : -2.0f)};
}

int main() {
  const std::vector<std::vector<int>> schedules = {
      {4, 8}, {4, 9}, {4, 10}, {4, 12}, {6, 9}, {12, 5}, {8, 8}, {6, 8}, {8, 6},
      {6, 10}, {9, 8}, {10, 8}, {12, 8}, {8, 12}};
  double ulp[2] = {0, 0}, mean[2] = {0, 0}, excess = 0, longer = 0;
  for (const auto& r : schedules) {
    const std::vector<double> t = twiddle_table(r.data(), (int)r.size());
    const std::vector<float> b = balanced_twiddles_f32(r.data(), (int)r.size());
    if (b.size() != t.size()) return 1;
    const int ns = r[0], legs = r[1] - 1;  // two stages: only the second has factors
    for (int mode = 0; mode < 2; ++mode)
      for (int leg = 0; leg < legs; ++leg) {
        double sum = 0.0;
        std::vector<double> sums = {0.0};  // of every choice
        for (int k = 0; k < ns; ++k) {
          const size_t at = 2 * (size_t)(k * legs + leg);
          float c = b[at], s = b[at + 1];
          if (mode) unit_f32(t[at], t[at + 1], &c, &s);
          const double dc = c - t[at], ds = s - t[at + 1];
          ulp[mode] = std::fmax(ulp[mode], std::fmax(std::fabs(dc), std::fabs(ds)) * 16777216.0);
          sum += dc * t[at] + ds * t[at + 1];
          if (mode == 0 && ns <= 6) {
            std::vector<double> next;
            for (double x : sums)
              for (float c2 : near(t[at]))
                for (float s2 : near(t[at + 1]))
                  next.push_back(x + (c2 - t[at]) * t[at] + (s2 - t[at + 1]) * t[at + 1]);
            sums = next;
          }
        }
        if (mode == 0 && ns <= 6) {
          double best = 1.0;
          for (double x : sums) best = std::fmin(best, std::fabs(x));
          excess = std::fmax(excess, (std::fabs(sum) - best) / ns);
        } else if (mode == 0) {
          longer = std::fmax(longer, std::fabs(sum) / ns);
        }
        mean[mode] = std::fmax(mean[mode], std::fabs(sum) / ns);
      }
  }
  std::printf("%.3f %.3e %.3e %.3e %.3e\n", ulp[0], excess, longer, mean[0], mean[1]);
  return 0;
}
