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
size_t resample_entries(int a, int b) { return (size_t)(a / 4) * ((b + 15) / 16) * 64; }

void resample_matrix(int a, int b, int kmax, double* out) {
  // R depends on d = (i/b - j/a) ab mod ab alone; the sum over k in closed form,
  // sin((2 kmax + 1) pi d / ab) / sin(pi d / ab), its angles reduced exactly
  const int ab = a * b, rb = (b + 15) / 16;
  const long double pi = 3.14159265358979323846264338327950288L;
  std::vector<double> val(ab, 0.0);
  std::vector<char> known(ab, 0);
  for (int s = 0; s < a / 4; ++s)
    for (int p = 0; p < rb; ++p)
      for (int l = 0; l < 64; ++l) {
        const int i = 16 * p + l % 16, j = 4 * s + l / 16;
        double v = 0.0;
        if (i < b) {
          const int d = ((i * a - j * b) % ab + ab) % ab;
          if (!known[d]) {
            const long long m = (2LL * kmax + 1) * d % (2LL * ab);
            val[d] = d == 0 ? (double)((2 * kmax + 1) / (long double)a)
                            : (double)(std::sin(pi * m / ab) / (std::sin(pi * d / ab) * a));
            known[d] = 1;
          }
          v = val[d];
        }
        out[((size_t)s * rb + p) * 64 + l] = v;
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
// takes several.
template <int RB, int NC, int D, typename S>
__device__ __forceinline__ void line_products(const S* (&line)[NC], long long stride,
                                              const double* f, int steps, f64x4 (&acc)[NC][RB]) {
  S x[D][NC];
  double r[D][RB];
  auto load = [&](int k, int s) {
    const int at = s < steps ? s : steps - 1;
#pragma unroll
    for (int q = 0; q < NC; ++q) x[k][q] = line[q][at * 4 * stride];
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
#pragma unroll
        for (int p = 0; p < RB; ++p)
#pragma unroll
          for (int q = 0; q < NC; ++q)
            acc[q][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(r[k][p], (double)x[k][q], acc[q][p],
                                                             0, 0, 0);
      }
      load(k, s + k + D);
    }
  }
}

// out[g][i][c] = sum_j R[i][j] in[g][j][c] (g < ng, i < b, j < a, c < width):
// an axis that is not the fastest.  A wavefront owns 16 kRsTiles neighbouring columns
// (of the ng width columns in all), loads their points straight into the B
// operand (128-byte segments) and keeps all b rows of results: the data moves
// once, R comes from L2.  a: a multiple of 4.
template <typename S, typename O, int RB>
__global__ void __launch_bounds__(kRsThreads) k_axis(const S* __restrict__ in, O* __restrict__ out,
                                             const double* __restrict__ frag, int a, int b,
                                             int width, long long columns) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const S* src[kRsTiles];
  O* dst[kRsTiles];
  bool ok[kRsTiles];
#pragma unroll
  for (int q = 0; q < kRsTiles; ++q) {
    const long long col = (((long long)blockIdx.x * (kRsThreads / 64) + wave) * kRsTiles + q) * 16 + lr;
    ok[q] = col < columns;
    const long long g = ok[q] ? col / width : 0;
    const long long c = ok[q] ? col - g * width : 0;
    src[q] = in + (g * a + lk) * width + c;
    dst[q] = out + (g * b + lk) * width + c;
  }
  f64x4 acc[kRsTiles][RB];
  line_products<RB, kRsTiles, 2>(src, width, frag + lane, a / 4, acc);
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

template <typename S, typename O>
static void axis(const S* in, O* out, const double* frag, int a, int b, int width, long long groups,
                 hipStream_t s) {
  const long long columns = groups * width, per = (long long)(kRsThreads / 64) * kRsTiles * 16;
  with_rows(b, [&](auto rb) {
    hipLaunchKernelGGL((k_axis<S, O, decltype(rb)::value>),
                       dim3((unsigned)((columns + per - 1) / per)), dim3(kRsThreads), 0, s, in, out, frag,
                       a, b, width, columns);
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
  return e;
}

// The intermediate grid of one orbital: planes first to a smaller grid, z
// first to a larger one.
size_t resample_tmp_bytes(int a, int az, int b, int bz) {
  return (b < a ? (size_t)az * b * b : (size_t)bz * a * a) * 8;
}

template <typename S, typename O>
void launch_resample(const S* in, O* out, int n_orb, int a, int az, int b, int bz,
                     const double* rx, const double* rz, void* tmp, size_t tmp_bytes,
                     hipStream_t s) {
  const size_t one = resample_tmp_bytes(a, az, b, bz);
  const int per = (int)std::max<size_t>(1, std::min<size_t>(n_orb, tmp_bytes / one));
  const long long na = (long long)az * a * a, nb = (long long)bz * b * b;
  double* t = static_cast<double*>(tmp);
  for (int o = 0; o < n_orb; o += per) {
    const int k = std::min(per, n_orb - o);
    if constexpr (std::is_same_v<S, double>)
      if (b < a) {
        plane_axes(in + o * na, t, rx, a, b, (long long)k * az, s);
        axis(t, out + o * nb, rz, az, bz, b * b, k, s);
        continue;
      }
    axis(in + o * na, t, rz, az, bz, a * a, k, s);
    plane_axes(t, out + o * nb, rx, a, b, (long long)k * bz, s);
  }
}

template void launch_resample<double, double>(const double*, double*, int, int, int, int, int,
                                              const double*, const double*, void*, size_t,
                                              hipStream_t);
template void launch_resample<double, float>(const double*, float*, int, int, int, int, int,
                                             const double*, const double*, void*, size_t,
                                             hipStream_t);
template void launch_resample<float, float>(const float*, float*, int, int, int, int, int,
                                            const double*, const double*, void*, size_t,
                                            hipStream_t);

}  // namespace hfx
