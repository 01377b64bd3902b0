// Band-limited resampling of orbitals and K psi between the caller's grid and
// the reduced pair grids of a plan (see ReducedPipeline); part of
// exchange_common.hip.
//
// A periodic function with frequencies |k| <= kmax, 2 kmax + 1 <= a, is known
// exactly from its a samples; its values at b points are R f with
//   R[i][j] = (1/a) (1 + 2 sum_{k=1..kmax} cos 2 pi k (i/b - j/a)),
// one matrix per axis.  The three axes are applied one after the other as
// float64 products on the matrix cores (float32 data is widened on the way in
// and rounded once on the way out).  A dense product per axis costs 2 a b
// flops per line where an FFT pair would cost less, but it is n_orb lines
// against n_orb^2 / 4 pair transforms: 96^3 -> 72^3 takes 0.33 GFLOP per
// orbital each way.
//
// float64 plans take a split product (below): a plain sum of 48 to 128 terms
// is 2e-16 to 4e-16 off in float64, and six of them in a row added more to K
// psi than the pair transforms do (against 80-bit arithmetic, 8 orbitals of 5
// Ha: 6.4e-16 on 64^3 and 8.2e-16 on 120^3, where the caller's grid has 2.5e-16 and
// 4.9e-16; with it 3.8e-16 and 6.0e-16, of which psi on the pair grid is 0.5e-16,
// the way back 0.7e-16 and the pair transforms 2.3e-16 at 64^3; the rest is what
// those float64 orbitals hold outside the declared band, which the caller's
// grid keeps).  It costs a tenth of K psi at 64 orbitals (120^3 12.9 -> 14.4 ms).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "hfx_internal.hpp"

namespace hfx {

namespace {
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kRsThreads = 256;
constexpr int kRsTiles = 2;  // 16-line tiles per wavefront
constexpr int kMaxLen = 128;
}  // namespace

// Fragment order: entry ((4-point step s, 16-row block p), lane l) holds
// R[16 p + l % 16][4 s + l / 16] (rows beyond b are zeros), the A operand of
// v_mfma_f64_16x16x4 for lane l: one contiguous 512-byte load per wavefront.
// R in extended precision: value(i, j).
struct ResampleKernel {
  int a, b, kmax;
  std::vector<long double> val;
  std::vector<char> known;
  ResampleKernel(int a_, int b_, int k) : a(a_), b(b_), kmax(k), val(a_ * b_, 0.0L), known(a_ * b_, 0) {}
  // R depends on d = (i/b - j/a) ab mod ab alone; the sum over k in closed form,
  // sin((2 kmax + 1) pi d / ab) / sin(pi d / ab), its angles reduced exactly and, as
  // it is even in d, to the smaller of d and ab - d (no cancellation at the poles)
  long double value(int i, int j) {
    const int ab = a * b, e = ((i * a - j * b) % ab + ab) % ab, d = e < ab - e ? e : ab - e;
    if (!known[d]) {
      const long double pi = 3.14159265358979323846264338327950288L;
      const long long m = (2LL * kmax + 1) * d % (2LL * ab);
      val[d] = d == 0 ? (2 * kmax + 1) / (long double)a
                      : std::sin(pi * m / ab) / (std::sin(pi * d / ab) * a);
      known[d] = 1;
    }
    return val[d];
  }
};

size_t resample_entries(int a, int b) { return (size_t)(a / 4) * ((b + 15) / 16) * 64; }

void resample_matrix(int a, int b, int kmax, double* out) {
  ResampleKernel r(a, b, kmax);
  const int rb = (b + 15) / 16;
  for (int s = 0; s < a / 4; ++s)
    for (int p = 0; p < rb; ++p)
      for (int l = 0; l < 64; ++l) {
        const int i = 16 * p + l % 16, j = 4 * s + l / 16;
        out[((size_t)s * rb + p) * 64 + l] = i < b ? (double)r.value(i, j) : 0.0;
      }
}

// Split products.  R[b-i][a-j] = R[i][j], so with u_j, w_j = x_j +- x_(a-j) and
// E, O = (R[i][j] +- R[i][a-j]) / 2 over j <= a/2 (half of that where j pairs
// with itself), e = E u and o = O w over i <= b/2, the results are e_i + o_i
// and, at b - i, e_i - o_i: half the products of the plain form.  Each factor
// is split in a high part of few bits and the rest,
//   E = Eh + El,  Eh a multiple of 2^-kMatBits,
//   u = uh + ul,  uh a multiple of 2^-kDataBits times a power of two above |x|,
// so that the terms of Eh uh and their sums are whole multiples of one unit
// and below 2^53 of it: that product is exact, and Eh ul + El u, a 2^-20th of it,
// carries the roundings.  A result is rounded once.  Where a value exceeds the
// scale that the orbital's largest sample sets, sums round as in the plain
// form; nothing else changes.
constexpr int kMatBits = 24, kDataBits = 26;

//
// Step s (columns 4 s ..) of the fragments: Eh, El, Oh, Ol of every 16-row block
// p of the rows below b / 2, 64 lanes each (lane l: row 16 p + l % 16, column 4 s
// + l / 16), then Eh and El of row b / 2 (O is zero there), 4 columns each: a block
// of its own would be most of the products' padding at 64, 96 and 128 points.
constexpr int split_blocks(int b) { return (b / 2 + 15) / 16; }
constexpr int split_step(int blocks) { return blocks * 256 + 8; }
static int split_steps(int a) { return (a / 2 + 1 + 3) / 4; }
size_t resample_split_entries(int a, int b) {
  return (size_t)split_steps(a) * split_step(split_blocks(b));
}

void resample_split_matrix(int a, int b, int kmax, double* out) {
  ResampleKernel r(a, b, kmax);
  const int rb = split_blocks(b);
  const long double unit = (long double)(1 << kMatBits);
  auto put = [&](int i, int j, double* e, double* o, int stride) {
    long double x = 0.0L, y = 0.0L;
    if (i <= b / 2 && j <= a / 2) x = r.value(i, j), y = r.value(i, (a - j) % a);
    const bool self = j == 0 || 2 * j == a;
    const long double ev = (x + y) / (self ? 4 : 2), ov = self ? 0.0L : (x - y) / 2;
    e[0] = (double)(std::rint(ev * unit) / unit);
    e[stride] = (double)(ev - e[0]);
    if (!o) return;
    o[0] = (double)(std::rint(ov * unit) / unit);
    o[stride] = (double)(ov - o[0]);
  };
  for (int s = 0; s < split_steps(a); ++s) {
    double* f = out + (size_t)s * split_step(rb);
    for (int p = 0; p < rb; ++p)
      for (int l = 0; l < 64; ++l) {
        const int i = 16 * p + l % 16;
        put(i < b / 2 ? i : b, 4 * s + l / 16, f + p * 256 + l, f + p * 256 + 128 + l, 64);
      }
    for (int q = 0; q < 4; ++q) put(b / 2, 4 * s + q, f + rb * 256 + q, nullptr, 4);
  }
}

// psi at its even points: a thread per output point.
__global__ void __launch_bounds__(kRsThreads) k_decimate(const double* __restrict__ psi, int n, int nz,
                                                 long long total, double* __restrict__ out64,
                                                 float* __restrict__ out32) {
  const int h = n / 2, hz = nz / 2;
  const long long stride = (long long)gridDim.x * kRsThreads;
  for (long long i = (long long)blockIdx.x * kRsThreads + threadIdx.x; i < total; i += stride) {
    const int x = (int)(i % h);
    long long r = i / h;
    const int y = (int)(r % h);
    r /= h;
    const int z = (int)(r % hz);
    const long long o = r / hz;
    const double v = psi[((o * nz + 2 * z) * n + 2 * y) * n + 2 * x];
    out64[i] = v;
    if (out32) out32[i] = (float)v;
  }
}

void launch_decimate(const double* psi, int n_orb, int n, int nz, double* out64, float* out32,
                     hipStream_t s) {
  const long long total = (long long)n_orb * (n / 2) * (n / 2) * (nz / 2);
  const long long blocks = std::min<long long>((total + kRsThreads - 1) / kRsThreads, 16384);
  hipLaunchKernelGGL(k_decimate, dim3((unsigned)blocks), dim3(kRsThreads), 0, s, psi, n, nz, total, out64,
                     out32);
}

// acc[q][p] = sum over the a points of 16 lines per q: point j of lane lr's
// line at line[q][(lk + j) * stride], fragments as above.  The operands of
// the next D steps are in flight (a ring of registers): one step's products,
// RB x NC x 64 cycles, are shorter than an L2 access, and an HBM access
// takes several.  OWN: the line plus own[q] times that at more[q].
template <int RB, int NC, int D, bool OWN = false, typename S>
__device__ __forceinline__ void line_products(const S* (&line)[NC], long long stride,
                                              const double* f, int steps, f64x4 (&acc)[NC][RB],
                                              const S* const* more = nullptr,
                                              const double* own = nullptr) {
  S x[D][NC], y[OWN ? D : 1][OWN ? NC : 1];
  double r[D][RB];
  auto load = [&](int k, int s) {
    const int at = s < steps ? s : steps - 1;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      x[k][q] = line[q][at * 4 * stride];
      if constexpr (OWN) y[k][q] = more[q][at * 4 * stride];
    }
#pragma unroll
    for (int p = 0; p < RB; ++p) r[k][p] = f[(at * RB + p) * 64];
    asm volatile("" ::: "memory");  // or the loads sink to their use in a later step
  };
#pragma unroll
  for (int q = 0; q < NC; ++q)
#pragma unroll
    for (int p = 0; p < RB; ++p) acc[q][p] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < D; ++k) load(k, k);
  for (int s = 0; s < steps; s += D) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      if (s + k < steps) {
        double v[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          v[q] = (double)x[k][q];
          if constexpr (OWN) v[q] += own[q] * (double)y[k][q];
        }
#pragma unroll
        for (int p = 0; p < RB; ++p)
#pragma unroll
          for (int q = 0; q < NC; ++q)
            acc[q][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(r[k][p], v[q], acc[q][p], 0, 0, 0);
      }
      load(k, s + k + D);
    }
  }
}

// out[g][i][c] = sum_j R[i][j] in[g][j][c] (g < ng, i < b, j < a, c < width):
// an axis that is not the fastest.  A wavefront owns 16 kRsTiles neighbouring columns
// (of the ng width columns in all), loads their points straight into the B
// operand (128-byte segments) and keeps all b rows of results: the data moves
// once, R comes from L2.  a: a multiple of 4.  OWN (K psi back to the caller's
// grid, group g orbital g): in_g - v0 mu_gg psi_g in place of in_g.
template <typename S, typename O, int RB, bool OWN>
__global__ void __launch_bounds__(kRsThreads) k_axis(const S* __restrict__ in, O* __restrict__ out,
                                             const double* __restrict__ frag, int a, int b,
                                             int width, long long columns,
                                             const S* __restrict__ psi,
                                             const double* __restrict__ mu, int n_orb, double v0) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const S *src[kRsTiles], *more[kRsTiles];
  double own[kRsTiles];
  O* dst[kRsTiles];
  bool ok[kRsTiles];
#pragma unroll
  for (int q = 0; q < kRsTiles; ++q) {
    const long long col = (((long long)blockIdx.x * (kRsThreads / 64) + wave) * kRsTiles + q) * 16 + lr;
    ok[q] = col < columns;
    const long long g = ok[q] ? col / width : 0;
    const long long c = ok[q] ? col - g * width : 0;
    src[q] = in + (g * a + lk) * width + c;
    more[q] = OWN ? psi + (g * a + lk) * width + c : nullptr;
    own[q] = OWN ? -v0 * mu[g * (n_orb + 1)] : 0.0;
    dst[q] = out + (g * b + lk) * width + c;
  }
  f64x4 acc[kRsTiles][RB];
  line_products<RB, kRsTiles, 2, OWN>(src, width, frag + lane, a / 4, acc, more, own);
  // result i of lane l: row 16 p + l / 16 + 4 i, column l % 16
#pragma unroll
  for (int q = 0; q < kRsTiles; ++q)
#pragma unroll
    for (int p = 0; p < RB; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (ok[q] && 16 * p + lk + 4 * i < b)
          dst[q][(long long)(16 * p + 4 * i) * width] = (O)acc[q][p][i];
}

// The x and y axes of one plane per workgroup: a x a points to b x b.  The
// rows are loaded straight into the B operand (16 rows x 32 bytes per load; the
// other parts of each line are the next steps'), their b results stay in LDS
// [a][b + 1], and the columns go from there to HBM: the intermediate never
// leaves the compute unit.  A wavefront takes kRsTiles x 16 rows or columns, so each
// fragment of R feeds kRsTiles products (with one, the L1 access rate was the bound,
// 85 % of its cycles, and the matrix cores ran at 49 %).
template <typename O, int RB>
__global__ void __launch_bounds__(256) k_plane_axes(const double* __restrict__ in,
                                                    O* __restrict__ out,
                                                    const double* __restrict__ frag, int a, int b) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* u = reinterpret_cast<double*>(smem_raw);
  const int pitch = b + 1;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const int first = (threadIdx.x >> 6) * 16 * kRsTiles;  // of the wavefront's lines
  const double* src = in + (long long)blockIdx.x * a * a;
  O* dst = out + (long long)blockIdx.x * b * b;
  f64x4 acc[kRsTiles][RB];
  const double* line[kRsTiles];
  if (first < a) {
#pragma unroll
    for (int q = 0; q < kRsTiles; ++q) {
      const int y = first + 16 * q + lr;
      line[q] = src + (y < a ? y : 0) * a + lk;
    }
    line_products<RB, kRsTiles, 4>(line, 1, frag + lane, a / 4, acc);
#pragma unroll
    for (int q = 0; q < kRsTiles; ++q) {
      const int y = first + 16 * q + lr;
      if (y < a)
#pragma unroll
        for (int p = 0; p < RB; ++p)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (16 * p + lk + 4 * i < b) u[y * pitch + 16 * p + lk + 4 * i] = acc[q][p][i];
    }
  }
  __syncthreads();
  if (first < b) {
#pragma unroll
    for (int q = 0; q < kRsTiles; ++q) {
      const int x = first + 16 * q + lr;
      line[q] = u + lk * pitch + (x < b ? x : 0);
    }
    line_products<RB, kRsTiles, 3>(line, pitch, frag + lane, a / 4, acc);
#pragma unroll
    for (int q = 0; q < kRsTiles; ++q) {
      const int x = first + 16 * q + lr;
      if (x < b)
#pragma unroll
        for (int p = 0; p < RB; ++p)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (16 * p + lk + 4 * i < b) dst[(long long)(16 * p + lk + 4 * i) * b + x] = (O)acc[q][p][i];
    }
  }
}

// Largest |value| of an orbital's nr points, kMaxParts partial maxima each
// (grid: kMaxParts x orbitals).  Every 16th run of 64 points is read, a few rows
// of a plane apart and at other rows in the next plane: the functions are
// band-limited, and the scale need not hold every value (see above).
constexpr int kMaxParts = 16;
constexpr long long kMaxStep = 64 * 16;
__global__ void __launch_bounds__(kRsThreads) k_absmax(const double* __restrict__ in, long long nr,
                                               double* __restrict__ part) {
  __shared__ double red[kRsThreads / 64];
  const double* x = in + (long long)blockIdx.y * nr;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double m = 0.0;
  for (long long r = ((long long)blockIdx.x * (kRsThreads / 64) + wave) * kMaxStep + lane; r < nr;
       r += kMaxParts * (kRsThreads / 64) * kMaxStep)
    m = fmax(m, fabs(x[r]));
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) m = fmax(m, __shfl_xor(m, s));
  if (lane == 0) red[wave] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kRsThreads / 64; ++w) m = fmax(m, red[w]);
    part[(long long)blockIdx.y * kMaxParts + blockIdx.x] = m;
  }
}

// c with (x + c) - c = x rounded to kDataBits bits below 2^margin times the
// orbital's largest sample; 0 (no split) where there is none or no room.
__device__ __forceinline__ double split_constant(const double* __restrict__ part, int margin) {
  double m = 0.0;
#pragma unroll
  for (int k = 0; k < kMaxParts; ++k) m = fmax(m, part[k]);
  return m > 1e-280 && m < 1e280 ? ldexp(1.5, ilogb(m) + 1 + margin + 52 - kDataBits) : 0.0;
}

// e, o of 16 lines (lane l: line l % 16): eh + el, oh + ol [p] of rows 16 p + ...
// (result i of lane l: row 16 p + l / 16 + 4 i), and th + tl of row b / 2.  Point j
// of the lane's line at line[j * stride]; f: fragments; fs: 2 split_step(RB)
// doubles of LDS.  Called by every wavefront of the workgroup: each step's
// fragments come from L2 once for all of them (a wavefront fetching its own, 8
// KB for 24 products, kept the L2 busy: k_axis_split 836 us, 540 with this, 64
// orbitals between 120 and 96 points).  The points of the next four steps are
// in flight.
template <int RB>
struct SplitSums {
  f64x4 eh[RB], el[RB], oh[RB], ol[RB];
  double th, tl;
};
template <int RB>
__device__ __forceinline__ void split_products(const double* line, long long stride, int a,
                                               const double* __restrict__ f, double* fs, double c,
                                               SplitSums<RB>& y) {
  constexpr int FR = split_step(RB), D = 4;
  const int tid = threadIdx.x, nt = blockDim.x;  // nt >= 256
  const int lane = tid & 63, lk = lane >> 4;
  const int steps = (a / 2 + 1 + 3) / 4;
  double x[D][2], r[RB + 1];
  auto load_points = [&](int k, int s) {
    const int at = s < steps ? s : steps - 1;
    const int j = 4 * at + lk;  // at most a / 2 + 3
    x[k][0] = line[j * stride];
    x[k][1] = line[(j == 0 ? 0 : a - j) * stride];
    asm volatile("" ::: "memory");  // or the loads sink to their use in a later step
  };
  auto load_fragments = [&](int s) {
    const int at = s < steps ? s : steps - 1;
#pragma unroll
    for (int q = 0; q <= RB; ++q)
      if (tid + q * nt < FR) r[q] = f[at * FR + tid + q * nt];
  };
  auto stage_fragments = [&](int buf) {
#pragma unroll
    for (int q = 0; q <= RB; ++q)
      if (tid + q * nt < FR) fs[buf * FR + tid + q * nt] = r[q];
  };
#pragma unroll
  for (int p = 0; p < RB; ++p) y.eh[p] = y.el[p] = y.oh[p] = y.ol[p] = f64x4{0.0, 0.0, 0.0, 0.0};
  y.th = y.tl = 0.0;
  load_fragments(0);
#pragma unroll
  for (int k = 0; k < D; ++k) load_points(k, k);
  stage_fragments(0);
  __syncthreads();
  for (int s = 0; s < steps; s += D) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      if (s + k >= steps) break;
      const double h0 = (x[k][0] + c) - c, h1 = (x[k][1] + c) - c;
      const double l0 = x[k][0] - h0, l1 = x[k][1] - h1;
      const double uh = h0 + h1, ul = l0 + l1, wh = h0 - h1, wl = l0 - l1;
      const double u = uh + ul, w = wh + wl;
      load_fragments(s + k + 1);
      load_points(k, s + k + D);
      const double* g = fs + (k & 1) * FR;
      const double rh = g[RB * 256 + lk], rl = g[RB * 256 + 4 + lk];
      g += lane;
#pragma unroll
      for (int p = 0; p < RB; ++p) {
        const double m = g[p * 256], q = g[p * 256 + 128];
        y.eh[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(m, uh, y.eh[p], 0, 0, 0);
        y.oh[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(q, wh, y.oh[p], 0, 0, 0);
        y.el[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(m, ul, y.el[p], 0, 0, 0);
        y.ol[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(q, wl, y.ol[p], 0, 0, 0);
      }
#pragma unroll
      for (int p = 0; p < RB; ++p) {
        y.el[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[p * 256 + 64], u, y.el[p], 0, 0, 0);
        y.ol[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[p * 256 + 192], w, y.ol[p], 0, 0, 0);
      }
      y.th += rh * uh;
      y.tl += rh * ul + rl * u;
      stage_fragments((k & 1) ^ 1);  // last read before the previous barrier
      __syncthreads();
    }
  }
#pragma unroll
  for (int m = 16; m < 64; m *= 2) {
    y.th += __shfl_xor(y.th, m);
    y.tl += __shfl_xor(y.tl, m);
  }
}

// store(row, value) for the b results of the lane's line.
template <int RB, class F>
__device__ __forceinline__ void split_results(int b, const SplitSums<RB>& y, F&& store) {
  const int lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int p = 0; p < RB; ++p)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 16 * p + lk + 4 * i;
      const double eh = y.eh[p][i], el = y.el[p][i], oh = y.oh[p][i], ol = y.ol[p][i];
      if (row < b / 2) store(row, (eh + oh) + (el + ol));
      if (row > 0 && row < b / 2) store(b - row, (eh - oh) + (el - ol));
    }
  if (lk == 0) store(b / 2, y.th + y.tl);
}

// k_axis with split products; the scale of column c of group g is group g's
// (one group per orbital).
template <int RB>
__global__ void __launch_bounds__(kRsThreads) __attribute__((amdgpu_waves_per_eu(2)))
k_axis_split(const double* __restrict__ in, double* __restrict__ out,
             const double* __restrict__ frag, const double* __restrict__ part, int margin, int a,
             int b, int width, long long columns) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long col = ((long long)blockIdx.x * (kRsThreads / 64) + wave) * 16 + (lane & 15);
  const bool ok = col < columns;
  const long long g = ok ? col / width : 0;
  const long long c = ok ? col - g * width : 0;
  __shared__ double fs[2 * split_step(RB)];
  SplitSums<RB> y;
  split_products<RB>(in + g * a * width + c, width, a, frag, fs,
                     split_constant(part + g * kMaxParts, margin), y);
  if (!ok) return;
  double* dst = out + g * b * width + c;
  split_results<RB>(b, y, [&](int row, double v) { dst[(long long)row * width] = v; });
}

// k_plane_axes with split products, 16 rows or columns per wavefront (up to
// eight of them); planes: of one orbital.
template <int RB>
__global__ void __launch_bounds__(512)
k_plane_split(const double* __restrict__ in, double* __restrict__ out,
              const double* __restrict__ frag, const double* __restrict__ part, int margin, int a,
              int b, int planes) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* u = reinterpret_cast<double*>(smem_raw);  // [a][b + 1]
  __shared__ double fs[2 * split_step(RB)];
  const int pitch = b + 1;
  const int at = (threadIdx.x >> 6) * 16 + (threadIdx.x & 15);  // the lane's row, then column
  const double* src = in + (long long)blockIdx.x * a * a;
  double* dst = out + (long long)blockIdx.x * b * b;
  const double* pt = part + (long long)(blockIdx.x / planes) * kMaxParts;
  SplitSums<RB> y;
  // (lines beyond the plane repeat the first)
  split_products<RB>(src + (at < a ? at : 0) * a, 1, a, frag, fs, split_constant(pt, margin), y);
  if (at < a)
    split_results<RB>(b, y, [&](int row, double v) { u[at * pitch + row] = v; });
  __syncthreads();
  split_products<RB>(u + (at < b ? at : 0), pitch, a, frag, fs, split_constant(pt, margin + 2), y);
  if (at < b)
    split_results<RB>(b, y, [&](int row, double v) { dst[(long long)row * b + at] = v; });
}

// f(std::integral_constant<int, RB>) with RB = ceil(b / 16), 3..8.
template <class F>
static void with_rows(int b, F&& f) {
  switch ((b + 15) / 16) {
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    default: f(std::integral_constant<int, 8>{});
  }
}

// The same with RB = split_blocks(b), 2..4.
template <class F>
static void with_half_rows(int b, F&& f) {
  switch (split_blocks(b)) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    default: f(std::integral_constant<int, 4>{});
  }
}

template <bool OWN = false, typename S, typename O>
static void axis(const S* in, O* out, const double* frag, int a, int b, int width, long long groups,
                 hipStream_t s, const S* psi = nullptr, const double* mu = nullptr, int n_orb = 0,
                 double v0 = 0.0) {
  const long long columns = groups * width, per = (long long)(kRsThreads / 64) * kRsTiles * 16;
  with_rows(b, [&](auto rb) {
    hipLaunchKernelGGL((k_axis<S, O, decltype(rb)::value, OWN>),
                       dim3((unsigned)((columns + per - 1) / per)), dim3(kRsThreads), 0, s, in, out, frag,
                       a, b, width, columns, psi, mu, n_orb, v0);
  });
}

template <typename O>
static void plane_axes(const double* in, O* out, const double* frag, int a, int b,
                       long long planes, hipStream_t s) {
  with_rows(b, [&](auto rb) {
    const int waves = (std::max(a, b) + 16 * kRsTiles - 1) / (16 * kRsTiles);
    hipLaunchKernelGGL((k_plane_axes<O, decltype(rb)::value>), dim3((unsigned)planes),
                       dim3(64 * waves), (size_t)a * (b + 1) * 8, s, in, out, frag, a, b);
  });
}

// Raise the dynamic-LDS limit of the plane kernels (once per process).
hipError_t prepare_resample() {
  hipError_t e = hipSuccess;
  for (int b = 48; b <= kMaxLen; b += 16)
    with_rows(b, [&](auto rb) {
      const void* k[2] = {reinterpret_cast<const void*>(&k_plane_axes<double, decltype(rb)::value>),
                          reinterpret_cast<const void*>(&k_plane_axes<float, decltype(rb)::value>)};
      for (const void* f : k)
        if (e == hipSuccess)
          e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  kMaxLen * (kMaxLen + 1) * 8);
    });
  for (int b = 48; b <= kMaxLen; b += 16)
    with_half_rows(b, [&](auto rb) {
      if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_plane_split<decltype(rb)::value>),
                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                kMaxLen * (kMaxLen + 1) * 8);
    });
  return e;
}

// The intermediate grid of one orbital: planes first to a smaller grid, z
// first to a larger one.
size_t resample_tmp_bytes(int a, int az, int b, int bz) {
  return (b < a ? (size_t)az * b * b : (size_t)bz * a * a) * 8;
}

static void axis_split(const double* in, double* out, const double* frag, const double* part,
                       int margin, int a, int b, int width, int orbs, hipStream_t s) {
  const long long columns = (long long)orbs * width, per = kRsThreads / 4;
  with_half_rows(b, [&](auto rb) {
    hipLaunchKernelGGL((k_axis_split<decltype(rb)::value>),
                       dim3((unsigned)((columns + per - 1) / per)), dim3(kRsThreads), 0, s, in, out,
                       frag, part, margin, a, b, width, columns);
  });
}

static void planes_split(const double* in, double* out, const double* frag, const double* part,
                         int margin, int a, int b, int planes, int orbs, hipStream_t s) {
  with_half_rows(b, [&](auto rb) {
    hipLaunchKernelGGL((k_plane_split<decltype(rb)::value>), dim3((unsigned)(planes * orbs)),
                       dim3(64 * ((std::max(a, b) + 15) / 16)), (size_t)a * (b + 1) * 8, s, in, out,
                       frag, part, margin, a, b, planes);
  });
}

// Margins: interpolation raises a band-limited function's largest value little,
// 2^2 per axis is allowed for, and 2^3 for what the samples missed.
void launch_resample_split(const double* in, double* out, int n_orb, int a, int az, int b, int bz,
                           const double* rx, const double* rz, double* part, void* tmp,
                           size_t tmp_bytes, hipStream_t s) {
  const size_t one = resample_tmp_bytes(a, az, b, bz);
  const int per = (int)std::max<size_t>(1, std::min<size_t>(n_orb, tmp_bytes / one));
  const long long na = (long long)az * a * a, nb = (long long)bz * b * b;
  double* t = static_cast<double*>(tmp);
  hipLaunchKernelGGL(k_absmax, dim3(kMaxParts, n_orb), dim3(kRsThreads), 0, s, in, na, part);
  for (int o = 0; o < n_orb; o += per) {
    const int k = std::min(per, n_orb - o);
    const double* pt = part + (size_t)o * kMaxParts;
    if (b < a) {
      planes_split(in + o * na, t, rx, pt, 3, a, b, az, k, s);
      axis_split(t, out + o * nb, rz, pt, 7, az, bz, b * b, k, s);
    } else {
      axis_split(in + o * na, t, rz, pt, 3, az, bz, a * a, k, s);
      planes_split(t, out + o * nb, rx, pt, 5, a, b, bz, k, s);
    }
  }
}

size_t resample_scale_bytes(int n_orb) { return (size_t)n_orb * kMaxParts * 8; }

// psi, mu, v0 (float32 K psi back): K psi without v0 mu_aa psi_a came in, psi the
// orbitals on the pair grid.  That term is the largest of a float32 sum whose
// other terms would each be rounded at its size; added here, in float64, it is
// not rounded before the result is.
template <typename S, typename O>
void launch_resample(const S* in, O* out, int n_orb, int a, int az, int b, int bz,
                     const double* rx, const double* rz, void* tmp, size_t tmp_bytes,
                     hipStream_t s, const S* psi, const double* mu, double v0) {
  const size_t one = resample_tmp_bytes(a, az, b, bz);
  const int per = (int)std::max<size_t>(1, std::min<size_t>(n_orb, tmp_bytes / one));
  const long long na = (long long)az * a * a, nb = (long long)bz * b * b;
  double* t = static_cast<double*>(tmp);
  for (int o = 0; o < n_orb; o += per) {
    const int k = std::min(per, n_orb - o);
    if constexpr (std::is_same_v<S, double>) {
      plane_axes(in + o * na, t, rx, a, b, (long long)k * az, s);
      axis(t, out + o * nb, rz, az, bz, b * b, k, s);
    } else {
      if (psi)
        axis<true>(in + o * na, t, rz, az, bz, a * a, k, s, psi + o * na,
                   mu + (size_t)o * (n_orb + 1), n_orb, v0);
      else
        axis(in + o * na, t, rz, az, bz, a * a, k, s);
      plane_axes(t, out + o * nb, rx, a, b, (long long)k * bz, s);
    }
  }
}

template void launch_resample<double, float>(const double*, float*, int, int, int, int, int,
                                             const double*, const double*, void*, size_t,
                                             hipStream_t, const double*, const double*, double);
template void launch_resample<float, float>(const float*, float*, int, int, int, int, int,
                                            const double*, const double*, void*, size_t,
                                            hipStream_t, const float*, const double*, double);

}  // namespace hfx
