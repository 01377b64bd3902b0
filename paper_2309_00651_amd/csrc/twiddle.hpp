// Host-side construction of Stockham stage twiddle tables.
//
// For a radix schedule (R_0, ..., R_{S-1}) the table lists, for every stage
// with span Ns > 1 (Ns = R_0 ... R_{s-1}), the factors W_{Ns R}^{r k}
// = exp(-2 pi i r k / (Ns R)) for k = 0..Ns-1, r = 1..R-1, at index
// k*(R-1) + r-1 after the entries of the earlier stages.  Values are
// evaluated in float64 and rounded once to the working precision.
#pragma once

#include <cmath>
#include <vector>

#include "trig.hpp"

namespace hfx {

// float32 representation of a unit complex number: among the float32
// neighbours (within two units in the last place) of cos and sin, the pair
// whose norm c^2 + s^2 is closest to 1 (ties: smaller angle error).  A norm
// error scales every value passing through the twiddle and, being one-sided
// for plain rounding, biases transform energies; an angle error keeps the
// transform unitary.
inline void unit_f32(double c, double s, float* cf, float* sf) {
  const float c0 = (float)c, s0 = (float)s;
  float bc = c0, bs = s0;
  double best_norm = 1e300, best_ang = 1e300;
  const double ang = std::atan2(s, c);
  auto step = [](float x, int d) {
    for (; d > 0; --d) x = std::nextafter(x, 2.0f);
    for (; d < 0; ++d) x = std::nextafter(x, -2.0f);
    return x;
  };
  for (int dc = -2; dc <= 2; ++dc)
    for (int ds = -2; ds <= 2; ++ds) {
      const float ct = step(c0, dc), st = step(s0, ds);
      const double nrm = std::fabs((double)ct * ct + (double)st * st - 1.0);
      double da = std::fabs(std::atan2((double)st, (double)ct) - ang);
      if (da > 3.14159265358979323846) da = 2 * 3.14159265358979323846 - da;
      if (nrm < best_norm || (nrm == best_norm && da < best_ang)) {
        best_norm = nrm;
        best_ang = da;
        bc = ct;
        bs = st;
      }
    }
  *cf = bc;
  *sf = bs;
}

inline std::vector<double> twiddle_table(const int* radices, int count) {
  std::vector<double> out;  // interleaved (re, im)
  long long ns = 1;
  for (int s = 0; s < count; ++s) {
    const int r_s = radices[s];
    if (ns > 1) {
      for (long long k = 0; k < ns; ++k) {
        for (int r = 1; r < r_s; ++r) {
          const SinCos w = sincos_2pi(-(long long)r * k, ns * r_s);
          out.push_back(w.c);
          out.push_back(w.s);
        }
      }
    }
    ns *= r_s;
  }
  return out;
}

// float32 table of the same layout for the reduced pair grids.  A transform of
// one frequency passes its value through one leg r of a stage and meets that
// leg's factors for every k, so its gain, and with it the energy's bias, is the
// mean of the factors' norm errors over k; single norms need not be exact.
// Each factor is one of the four float32 neighbours of (cos, sin), chosen so that
// the norm errors of every leg cancel (to below 1e-9 of their mean where six
// factors can be chosen; legs with two or three inexact ones keep up to 2e-9),
// where unit_f32 moves factors by up to two units to make each norm exact.
// (Transform alone, rms error / gain, unit_f32 and this table: 48 points (6, 8)
// 1.20e-7 / -1.5e-9 and 0.86e-7 / -0.7e-9, 60 (6, 10) 1.05e-7 / 2.4e-9 and 0.93e-7
// / -0.4e-9, 72 (9, 8) 1.31e-7 / -2.4e-9 and 0.93e-7 / -1.0e-9.)
inline std::vector<float> balanced_twiddles_f32(const int* radices, int count) {
  struct Choice {
    float c, s;
    double norm, cost;  // norm error; squared distance
  };
  const std::vector<double> t = twiddle_table(radices, count);
  std::vector<float> out(t.size());
  auto neighbours = [](double x, float* lo, float* hi) {
    *lo = *hi = (float)x;
    if ((double)*lo < x)
      *hi = std::nextafter(*lo, 2.0f);
    else if ((double)*lo > x)
      *lo = std::nextafter(*hi, -2.0f);
  };
  long long ns = 1, off = 0;
  for (int s = 0; s < count; ++s) {
    const int legs = radices[s] - 1;
    for (int r = 0; ns > 1 && r < legs; ++r) {
      std::vector<std::vector<Choice>> of(ns);
      std::vector<int> pick(ns, 0);
      double norm = 0.0, cost = 0.0;  // sums over k
      for (long long k = 0; k < ns; ++k) {
        const double c = t[2 * (off + k * legs + r)], sn = t[2 * (off + k * legs + r) + 1];
        float cl, ch, sl, sh;
        neighbours(c, &cl, &ch);
        neighbours(sn, &sl, &sh);
        for (float x : {cl, ch})
          for (float y : {sl, sh}) {
            const double dx = x - c, dy = y - sn;
            of[k].push_back({x, y, dx * c + dy * sn, dx * dx + dy * dy});
          }
        for (int q = 1; q < 4; ++q)
          if (of[k][q].cost < of[k][pick[k]].cost) pick[k] = q;
        norm += of[k][pick[k]].norm;
        cost += of[k][pick[k]].cost;
      }
      // from the rounded factors, every choice of up to six of those that are
      // not exact: the least cost plus the sum's square, weighted.
      std::vector<long long> free;
      for (long long k = 0; k < ns && free.size() < 6; ++k)
        if (of[k][0].c != of[k][3].c || of[k][0].s != of[k][3].s) free.push_back(k);
      auto total = [](double n, double c) { return c + 1e6 * n * n; };
      for (long long k : free) {
        norm -= of[k][pick[k]].norm;
        cost -= of[k][pick[k]].cost;
      }
      int best = 0;
      double least = 1e300;
      for (int code = 0; code < 1 << 2 * free.size(); ++code) {
        double n = norm, c = cost;
        for (size_t f = 0; f < free.size(); ++f) {
          n += of[free[f]][code >> 2 * f & 3].norm;
          c += of[free[f]][code >> 2 * f & 3].cost;
        }
        if (total(n, c) < least) {
          least = total(n, c);
          best = code;
        }
      }
      for (size_t f = 0; f < free.size(); ++f) pick[free[f]] = best >> 2 * f & 3;
      for (long long k = 0; k < ns; ++k) {
        out[2 * (off + k * legs + r)] = of[k][pick[k]].c;
        out[2 * (off + k * legs + r) + 1] = of[k][pick[k]].s;
      }
    }
    if (ns > 1) off += ns * legs;
    ns *= radices[s];
  }
  return out;
}

}  // namespace hfx
