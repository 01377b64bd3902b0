// The resampling matrices that the library builds for its reduced pair grids,
// against the direct cosine sum in extended precision: both forms unpacked from
// their fragment order, every compiled pipeline of both precisions, each axis, both
// directions.  Linked with libhfx.so (host functions only).  Prints one line
// per matrix: a b kmax, the largest error of the plain form, of the split form
// (high and low parts of E and O summed), 1 where the split form's high parts are
// multiples of 2^-24, and the sum over a row of |high parts| that bounds the
// exact product; and the bounds the dispatch rule checks.
#include <cmath>
#include <cstdio>
#include <tuple>
#include <vector>

#include "../../paper_2309_00651_amd/csrc/hfx_internal.hpp"

static long double direct(int a, int b, int kmax, int i, int j) {
  const long double pi = 3.14159265358979323846264338327950288L;
  long double s = 1.0L;
  for (int k = 1; k <= kmax; ++k) {
    const long long m = (long long)k * (i * a - j * b) % (a * b);
    s += 2.0L * std::cos(2.0L * pi * m / (a * b));
  }
  return s / a;
}

static void check(int a, int b, int kmax) {
  std::vector<double> m(hfx::resample_entries(a, b)), q(hfx::resample_split_entries(a, b));
  hfx::resample_matrix(a, b, kmax, m.data());
  hfx::resample_split_matrix(a, b, kmax, q.data());
  const int rb = (b + 15) / 16, hb = (b / 2 + 15) / 16, step = hb * 256 + 8;
  double plain = 0.0, split = 0.0, most = 0.0;
  int whole = 1;
  for (int i = 0; i < b; ++i)
    for (int j = 0; j < a; ++j) {
      const double got = m[((size_t)(j / 4) * rb + i / 16) * 64 + i % 16 + 16 * (j % 4)];
      plain = std::fmax(plain, std::fabs((double)(got - direct(a, b, kmax, i, j))));
    }
  // rows and padding beyond b are zeros
  for (int s = 0; s < a / 4; ++s)
    for (int i = b; i < 16 * rb; ++i)
      for (int l = 0; l < 4; ++l)
        if (m[((size_t)s * rb + i / 16) * 64 + i % 16 + 16 * l] != 0.0) plain = 1.0;
  auto part = [&](int i, int j, int which) -> double {  // 0 Eh, 1 El, 2 Oh, 3 Ol
    const double* f = &q[(size_t)(j / 4) * step];
    if (i == b / 2) return which < 2 ? f[hb * 256 + 4 * which + j % 4] : 0.0;
    return f[(i / 16) * 256 + 64 * which + i % 16 + 16 * (j % 4)];
  };
  for (int i = 0; i <= b / 2; ++i) {
    double row = 0.0;
    for (int j = 0; j <= a / 2; ++j) {
      const long double e = (long double)part(i, j, 0) + part(i, j, 1);
      const long double o = (long double)part(i, j, 2) + part(i, j, 3);
      const int mir = (a - j) % a;
      const bool self = mir == j;
      // x_j's coefficient: e u + o w with u = 2 x_j where j pairs with itself
      const long double rj = self ? 2.0L * e : e + o, rm = self ? rj : e - o;
      split = std::fmax(split, (double)std::fabs(rj - direct(a, b, kmax, i, j)));
      split = std::fmax(split, (double)std::fabs(rm - direct(a, b, kmax, i, mir)));
      for (int w = 0; w < 4; w += 2) {
        const double h = part(i, j, w) * 16777216.0;
        if (h != std::rint(h)) whole = 0;
        row += 2.0 * std::fabs(part(i, j, w));
      }
    }
    most = std::fmax(most, row);
  }
  // padded rows and columns of the blocks are zeros
  for (int s = 0; s < (a / 2 + 4) / 4; ++s)
    for (int i = 0; i < 16 * hb; ++i)
      for (int l = 0; l < 4; ++l)
        if (i >= b / 2 || 4 * s + l > a / 2)
          for (int w = 0; w < 4; ++w)
            if (q[(size_t)s * step + (i / 16) * 256 + 64 * w + i % 16 + 16 * l] != 0.0) split = 1.0;
  std::printf("matrix %d %d %d %.3e %.3e %d %.3f\n", a, b, kmax, plain, split, whole, most);
}

int main() {
  for (int prec = 0; prec < 2; ++prec) {
    int count = 0;
    const hfx::Variant* v = prec ? hfx::reduced_f64(&count) : hfx::reduced_f32(&count);
    for (int i = 0; i < count; ++i) {
      const int bx = (v[i].nf - 1) / 4, bz = (v[i].nfz - 1) / 4;
      std::printf("variant %d %d %d %d %d\n", 2 * v[i].nf, 2 * v[i].nfz, v[i].n, v[i].nz, v[i].min_orb);
      // the widest band of the matrices is the widest that the dispatch accepts
      for (auto [nf, n, band] : {std::tuple<int, int, int>{v[i].nf, v[i].n, bx}, {v[i].nfz, v[i].nz, bz}}) {
        std::printf("band %d %d %d\n", nf, n, band);
        check(2 * nf, n, band);
        check(n, 2 * nf, 3 * band);
      }
    }
  }
  return 0;
}
