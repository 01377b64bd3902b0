// Loewdin orthonormalisation in float64: Psi <- S^(-1/2) Psi (orbital-major
// storage), S = dV Psi Psi^T.
//
// S^(-1/2) comes from the coupled Newton-Schulz iteration
//   Y_0 = S / c, Z_0 = I, c = max row sum of |S| (so the spectrum lies in
//   (0, 1]; c = 1 for orthonormal input, which then converges in two steps),
//   T_k = (3 I - Z_k Y_k) / 2,  Y_{k+1} = Y_k T_k,  Z_{k+1} = T_k Z_k,
// whose Z_k converges quadratically to (S/c)^(-1/2); then S^(-1/2) = Z / sqrt(c).
// Every step is three dense float64 products on the matrix cores.
// Convergence is decided on the device: the step in which max|Z Y - I| <
// 1e-10 is the last one applied, and a flag in device memory turns the
// remaining launches into no-ops, so the host never waits; up to 64 orbitals
// run in one workgroup and one launch.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "hfx_internal.hpp"

namespace hfx {

namespace {
constexpr int TM = 64;
constexpr int KB = 16;
typedef double f64x4 __attribute__((ext_vector_type(4)));
}  // namespace

// C[M][N] = alpha * A[M][K] B[K][N] (row-major, leading dims lda, ldb, ldc),
// skipped entirely when *flag != 0.  4 wavefronts x (2 x 2) MFMA f64 16x16x4
// (lane l: A[l%16][l/16], B[l/16][l%16], result i = D[l/16 + 4i][l%16]).
__global__ void __launch_bounds__(256) k_gemm_nn_f64(const double* __restrict__ a, int lda,
                                                     const double* __restrict__ b, long long ldb,
                                                     double* __restrict__ c, long long ldc, int M,
                                                     long long N, int K, double alpha,
                                                     const int* __restrict__ flag) {
  if (flag && flag[0]) return;
  __shared__ double as[TM][KB + 1];
  __shared__ double bs[KB][TM + 1];
  const long long tiles_n = (N + TM - 1) / TM;
  const int ti = (int)(blockIdx.x / tiles_n);
  const long long tj = blockIdx.x % tiles_n;
  const int row0 = ti * TM;
  const long long col0 = tj * TM;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  const int lr = lane & 15, lk = lane >> 4;
  f64x4 acc[2][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[p][q] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < K; k0 += KB) {
    // A tile 64 x 16: 4 values per thread; B tile 16 x 64: 4 values per thread
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = tid + u * 256;
      const int ar = e / KB, ak = e % KB;
      const int gr = row0 + ar, gk = k0 + ak;
      as[ar][ak] = (gr < M && gk < K) ? a[(long long)gr * lda + gk] : 0.0;
      const int bk = e / TM, bc = e % TM;
      const int gbk = k0 + bk;
      const long long gbc = col0 + bc;
      bs[bk][bc] = (gbk < K && gbc < N) ? b[(long long)gbk * ldb + gbc] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < KB; kk += 4)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          acc[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(as[wr + p * 16 + lr][kk + lk],
                                                           bs[kk + lk][wc + q * 16 + lr],
                                                           acc[p][q], 0, 0, 0);
    __syncthreads();
  }
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = row0 + wr + p * 16 + lk + 4 * i;
        const long long cc = col0 + wc + q * 16 + lr;
        if (r < M && cc < N) c[(long long)r * ldc + cc] = alpha * acc[p][q][i];
      }
}

// Newton-Schulz state in device memory: done flag, completed steps; err[k % 2]:
// max |Z Y - I| of step k as the bits of a non-negative double (ordered like
// the value, so an integer atomic max applies); c.
struct NsState {
  int done, steps, pad[2];
  unsigned long long err[2];
  double c;
};
constexpr double kNsConverged = 1e-10;  // a step that starts closer than this is the last

// c = max row sum of |S| (a bound on the spectral radius of the symmetric S,
// tight when S is close to diagonal); Y0 = S / c, Z0 = I.
__global__ void __launch_bounds__(256) k_ns_init(const double* __restrict__ s, int n,
                                                 double* __restrict__ y, double* __restrict__ z,
                                                 NsState* __restrict__ st) {
  __shared__ double red[256];
  double m = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) {
    double r = 0.0;
    for (int j = 0; j < n; ++j) r += fabs(s[(long long)i * n + j]);
    m = fmax(m, r);
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  const double c = red[0];
  const long long nn = (long long)n * n;
  for (long long i = threadIdx.x; i < nn; i += 256) {
    y[i] = s[i] / c;
    z[i] = (i / n == i % n) ? 1.0 : 0.0;
  }
  if (threadIdx.x == 0) {
    st->c = c;
    st->done = 0;
    st->steps = 0;
    st->err[0] = st->err[1] = 0ull;
  }
}

// One n x n x n float64 product C = A B on 32 x 32 tiles (4 wavefronts, one
// 16 x 16 MFMA block each): acc[i] is C[row][col] at rows row + 4 i.
__device__ __forceinline__ void ns_product(const double* __restrict__ a,
                                           const double* __restrict__ b, int n, int tile,
                                           double __attribute__((ext_vector_type(4))) & acc,
                                           int& row, int& col) {
  constexpr int T = 32, KB = 16;
  __shared__ double as[T][KB + 1];
  __shared__ double bs[KB][T + 1];
  const int tiles = (n + T - 1) / T;
  const int row0 = (tile / tiles) * T, col0 = (tile % tiles) * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = (wave >> 1) * 16, wc = (wave & 1) * 16;
  const int lr = lane & 15, lk = lane >> 4;
  acc = {0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < n; k0 += KB) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int e = tid + 256 * u;
      const int ar = e / KB, ak = e % KB;
      as[ar][ak] = (row0 + ar < n && k0 + ak < n) ? a[(long long)(row0 + ar) * n + k0 + ak] : 0.0;
      const int bk = e / T, bc = e % T;
      bs[bk][bc] = (k0 + bk < n && col0 + bc < n) ? b[(long long)(k0 + bk) * n + col0 + bc] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < KB; kk += 4)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(as[wr + lr][kk + lk], bs[kk + lk][wc + lr], acc,
                                                 0, 0, 0);
    __syncthreads();
  }
  row = row0 + wr + lk;
  col = col0 + wc + lr;
}

// First product of step k, P = Z Y: T = (3 I - P) / 2, max |P - I| to err[k % 2].
// A step after one that started within kNsConverged ends the iteration.
__global__ void __launch_bounds__(256) k_ns_first(const double* __restrict__ z,
                                                  const double* __restrict__ y,
                                                  double* __restrict__ t, int n, int k,
                                                  NsState* __restrict__ st) {
  if (st->done) return;
  if (k > 0 && __longlong_as_double((long long)st->err[(k - 1) & 1]) < kNsConverged) {
    if (blockIdx.x == 0 && threadIdx.x == 0) st->done = 1;
    return;
  }
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  f64x4 acc;
  int row, col;
  ns_product(z, y, n, blockIdx.x, acc, row, col);
  double m = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = row + 4 * i;
    if (r < n && col < n) {
      const double d = acc[i] - (r == col ? 1.0 : 0.0);
      m = fmax(m, fabs(d));
      t[(long long)r * n + col] = (r == col ? 1.0 : 0.0) - 0.5 * d;
    }
  }
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) m = fmax(m, __shfl_xor(m, s));
  if (threadIdx.x % 64 == 0)
    atomicMax(&st->err[k & 1], (unsigned long long)__double_as_longlong(m));
}

// The other two products of step k side by side, Y T and T Z.
__global__ void __launch_bounds__(256) k_ns_step(const double* __restrict__ y,
                                                 const double* __restrict__ t,
                                                 const double* __restrict__ z,
                                                 double* __restrict__ yn, double* __restrict__ zn,
                                                 int n, int k, NsState* __restrict__ st) {
  if (st->done) return;
  const int half = gridDim.x / 2;
  const bool second = (int)blockIdx.x >= half;
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  f64x4 acc;
  int row, col;
  ns_product(second ? t : y, second ? z : t, n, second ? blockIdx.x - half : blockIdx.x, acc, row,
             col);
  double* c = second ? zn : yn;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (row + 4 * i < n && col < n) c[(long long)(row + 4 * i) * n + col] = acc[i];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->steps = k + 1;
    st->err[(k + 1) & 1] = 0ull;  // of the next step
  }
}

// The whole iteration for n <= 64 in one workgroup, Y, Z and T in LDS: 16
// wavefronts, one 16 x 16 block each; 64 is what the LDS holds three times
// (96 would need 223 KB).  Launches bound it before, 160 of them and those
// after convergence empty: orthonormalising 16 / 64 orbitals on 24^3 took 490 /
// 499 us, now 25 / 79.  From 65 on two launches per step (were four, one of
// them a single thread): 128 orbitals 599 -> 337 us, 256 936 -> 604.
constexpr int kNsSmall = 64;
__global__ void __launch_bounds__(1024) k_ns_small(double* __restrict__ s, int n, int max_iter) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int L = kNsSmall, LD = L + 1;
  double* y = reinterpret_cast<double*>(smem_raw);
  double* z = y + L * LD;
  double* t = z + L * LD;
  __shared__ double red[L], red2[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  for (int e = tid; e < L * L; e += 1024) {
    const int r = e / L, c = e % L;
    y[r * LD + c] = r < n && c < n ? s[(long long)r * n + c] : 0.0;
    z[r * LD + c] = r == c && r < n ? 1.0 : 0.0;
    t[r * LD + c] = 0.0;
  }
  __syncthreads();
  if (tid < L) {
    double a = 0.0;
    for (int c = 0; c < n; ++c) a += fabs(y[tid * LD + c]);
    red[tid] = a;
  }
  __syncthreads();
  double cmax = 0.0;
  for (int r = 0; r < n; ++r) cmax = fmax(cmax, red[r]);
  for (int e = tid; e < L * L; e += 1024) y[(e / L) * LD + e % L] /= cmax;
  __syncthreads();
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  const int nb = (n + 15) / 16;
  const int br = (wave / 4) * 16, bc = (wave % 4) * 16;  // the wavefront's block
  const bool mine = wave / 4 < nb && wave % 4 < nb;
  auto product = [&](const double* a, const double* b) {
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < 16 * nb; k += 4)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[(br + lr) * LD + k + lk],
                                                 b[(k + lk) * LD + bc + lr], acc, 0, 0, 0);
    return acc;
  };
  for (int it = 0; it < max_iter; ++it) {
    double m = 0.0;
    if (mine) {
      const f64x4 p = product(z, y);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = br + lk + 4 * i, c = bc + lr;
        if (r < n && c < n) {
          const double d = p[i] - (r == c ? 1.0 : 0.0);
          m = fmax(m, fabs(d));
          t[r * LD + c] = (r == c ? 1.0 : 0.0) - 0.5 * d;
        }
      }
    }
#pragma unroll
    for (int sh = 32; sh > 0; sh >>= 1) m = fmax(m, __shfl_xor(m, sh));
    if (lane == 0) red2[wave] = m;
    __syncthreads();
    f64x4 yn = {0.0, 0.0, 0.0, 0.0}, zn = yn;
    if (mine) {
      yn = product(y, t);
      zn = product(t, z);
    }
    double err = 0.0;
    for (int w = 0; w < 16; ++w) err = fmax(err, red2[w]);
    __syncthreads();
    if (mine)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int at = (br + lk + 4 * i) * LD + bc + lr;
        y[at] = yn[i];
        z[at] = zn[i];
      }
    __syncthreads();
    if (err < kNsConverged) break;
  }
  const double rc = sqrt(cmax);
  for (int e = tid; e < n * n; e += 1024) s[e] = z[(e / n) * LD + e % n] / rc;
}

__global__ void __launch_bounds__(256) k_ns_final(const double* __restrict__ z0,
                                                  const double* __restrict__ z1, long long nn,
                                                  const NsState* __restrict__ st,
                                                  double* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const double* z = (st->steps & 1) ? z1 : z0;
  if (i < nn) out[i] = z[i] / sqrt(st->c);
}

__global__ void __launch_bounds__(256) k_copy_cols(const double* __restrict__ tmp, int n,
                                                   long long cc, double* __restrict__ psi,
                                                   long long nr, long long c0) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)n * cc) return;
  const long long r = i / cc, k = i % cc;
  psi[r * nr + c0 + k] = tmp[i];
}

static void gemm_nn(const double* a, int lda, const double* b, long long ldb, double* c,
                    long long ldc, int M, long long N, int K, double alpha, const int* flag,
                    hipStream_t st) {
  const long long tiles = (long long)((M + TM - 1) / TM) * ((N + TM - 1) / TM);
  hipLaunchKernelGGL(k_gemm_nn_f64, dim3((unsigned)tiles), dim3(256), 0, st, a, lda, b, ldb, c,
                     ldc, M, N, K, alpha, flag);
}

constexpr int kNsSmallLds = 3 * kNsSmall * (kNsSmall + 1) * 8;

// Raise the dynamic-LDS limit of the one-workgroup iteration.
hipError_t prepare_inverse_sqrt() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ns_small),
                             hipFuncAttributeMaxDynamicSharedMemorySize, kNsSmallLds);
}

// s: n x n overlap in, S^(-1/2) out.  work: >= 5 n^2 doubles + 64 bytes.
// Step k reads (Y, Z)[k % 2] and writes (Y, Z)[(k + 1) % 2]; the final
// result is Z[steps % 2], read on the device.
hipError_t launch_inverse_sqrt(double* s, int n, double* work, int max_iter, hipStream_t st) {
  const long long nn = (long long)n * n;
  if (n <= kNsSmall) {
    hipLaunchKernelGGL(k_ns_small, dim3(1), dim3(1024), kNsSmallLds, st, s, n, max_iter);
    return hipGetLastError();
  }
  double* y[2] = {work, work + nn};
  double* z[2] = {work + 2 * nn, work + 3 * nn};
  double* t = work + 4 * nn;
  NsState* state = reinterpret_cast<NsState*>(work + 5 * nn);
  hipLaunchKernelGGL(k_ns_init, dim3(1), dim3(256), 0, st, s, n, y[0], z[0], state);
  const int tiles = (n + 31) / 32;
  const unsigned g = (unsigned)(tiles * tiles);
  for (int it = 0; it < max_iter; ++it) {
    const int cur = it & 1, nxt = cur ^ 1;
    hipLaunchKernelGGL(k_ns_first, dim3(g), dim3(256), 0, st, z[cur], y[cur], t, n, it, state);
    hipLaunchKernelGGL(k_ns_step, dim3(2 * g), dim3(256), 0, st, y[cur], t, z[cur], y[nxt], z[nxt],
                       n, it, state);
  }
  const unsigned eb = (unsigned)((nn + 255) / 256);
  hipLaunchKernelGGL(k_ns_final, dim3(eb), dim3(256), 0, st, z[0], z[1], nn, state, s);
  return hipGetLastError();
}

// dst = m src for n <= 512 rows, dst == src allowed.
//
// A wavefront owns RB 16-row blocks of the result and two 16-column tiles; the
// RW wavefronts that share the columns cover the rows, so a workgroup reads all
// it needs of its columns before its barrier and may then overwrite them.
// Nothing is staged in LDS: src rows are the B operand as they lie (128-byte
// segments), and m comes in fragment order from L2 (k_fragments), one
// contiguous 512-byte load per 16 x 4 block that feeds both column tiles.  The
// operands of two steps are in flight.  Bound by the float64 matrix rate: 116
// GFLOP at 256 orbitals on 96^3.  (Columns staged in LDS, 64 KB per workgroup,
// and m read from its rows with branches around the edges took 3.25 ms there:
// a staging phase that nothing hides, and waits at every branch.)
//
// Fragment ((4-column step s, 16-row block p), lane l) of m: m[16 p + l % 16]
// [4 s + l / 16], zero beyond n.
__global__ void __launch_bounds__(256) k_fragments(const double* __restrict__ m, int n, int blocks,
                                                   int total, double* __restrict__ frag) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int l = e & 63, p = (e >> 6) % blocks, s = (e >> 6) / blocks;
  const int row = 16 * p + (l & 15), col = 4 * s + (l >> 4);
  frag[e] = row < n && col < n ? m[(long long)row * n + col] : 0.0;
}

template <int RB, typename S>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_apply_left(const double* __restrict__ frag, int n, int blocks, int rw, const S* src, double* dst,
             long long nr) {
  constexpr int NC = 2, D = 2;
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int cw = (int)(blockDim.x >> 6) / rw;  // column groups of the workgroup
  const int p0 = (wave % rw) * RB;             // first row block (blocks is a multiple of RB)
  const long long c0 = ((long long)blockIdx.x * cw + wave / rw) * 16 * NC + lr;
  const S* col[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) col[q] = src + (c0 + 16 * q < nr ? c0 + 16 * q : 0);
  const double* f = frag + (long long)p0 * 64 + lane;
  const int steps = (n + 3) / 4;
  double r[D][RB];
  S x[D][NC];
  auto load = [&](int k, int s) {
    const int at = s < steps ? s : steps - 1;
    const int row = 4 * at + lk < n ? 4 * at + lk : n - 1;
#pragma unroll
    for (int q = 0; q < NC; ++q) x[k][q] = col[q][(long long)row * nr];
#pragma unroll
    for (int p = 0; p < RB; ++p) r[k][p] = f[((long long)at * blocks + p) * 64];
    asm volatile("" ::: "memory");  // or the loads sink to their use in a later step
  };
  f64x4 acc[RB][NC];
#pragma unroll
  for (int p = 0; p < RB; ++p)
#pragma unroll
    for (int q = 0; q < NC; ++q) acc[p][q] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < D; ++k) load(k, k);
  for (int s = 0; s < steps; s += D)
#pragma unroll
    for (int k = 0; k < D; ++k) {
      if (s + k < steps) {
        // rows beyond n (last step): zeros, not the clamped row times zero
        const bool in = 4 * (s + k) + lk < n;
#pragma unroll
        for (int p = 0; p < RB; ++p)
#pragma unroll
          for (int q = 0; q < NC; ++q)
            acc[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(r[k][p], in ? (double)x[k][q] : 0.0,
                                                             acc[p][q], 0, 0, 0);
      }
      load(k, s + k + D);
    }
  __syncthreads();  // every wavefront has read the workgroup's columns
  // result i of lane l: row (l / 16) + 4 i of the block, column l % 16
#pragma unroll
  for (int p = 0; p < RB; ++p)
#pragma unroll
    for (int q = 0; q < NC; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 16 * (p0 + p) + lk + 4 * i;
        if (row < n && c0 + 16 * q < nr) dst[(long long)row * nr + c0 + 16 * q] = acc[p][q][i];
      }
}

// Launches k_apply_left for n <= 512; tmp holds the fragments of m
// (2 n + 80 values per row at most: n x min(nr, 32768) doubles are there).
template <typename S>
static void apply_left(const double* m, const S* src, double* dst, int n, long long nr, double* tmp,
                       hipStream_t st) {
  const int nb = (n + 15) / 16;
  const int rw = (nb + 7) / 8;          // row wavefronts, up to 8 blocks each
  const int rb = (nb + rw - 1) / rw;    // blocks per wavefront
  const int blocks = rw * rb, total = (n + 3) / 4 * blocks * 64;
  hipLaunchKernelGGL(k_fragments, dim3((total + 255) / 256), dim3(256), 0, st, m, n, blocks, total,
                     tmp);
  const int cw = 4 / rw;
  const long long per = (long long)cw * 32;
  const dim3 grid((unsigned)((nr + per - 1) / per)), block(64 * rw * cw);
  auto go = [&](auto rbc) {
    hipLaunchKernelGGL((k_apply_left<decltype(rbc)::value, S>), grid, block, 0, st, tmp, n, blocks,
                       rw, src, dst, nr);
  };
  switch (rb) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 5: go(std::integral_constant<int, 5>{}); break;
    case 6: go(std::integral_constant<int, 6>{}); break;
    case 7: go(std::integral_constant<int, 7>{}); break;
    default: go(std::integral_constant<int, 8>{});
  }
}

// dst <- m src (n x n times n x nr; dst == src allowed).  n <= 512: one pass
// (k_apply_left); larger n: column chunks through tmp (n x 32768 doubles)
// and a copy to dst.
void launch_apply_left(const double* m, const double* src, double* dst, int n, long long nr,
                       double* tmp, hipStream_t st) {
  if (n <= 512) {
    apply_left(m, src, dst, n, nr, tmp, st);
    return;
  }
  const long long cc = 32768;
  for (long long c0 = 0; c0 < nr; c0 += cc) {
    const long long w = c0 + cc <= nr ? cc : nr - c0;
    gemm_nn(m, n, src + c0, nr, tmp, w, n, w, n, 1.0, nullptr, st);
    const long long tot = (long long)n * w;
    hipLaunchKernelGGL(k_copy_cols, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, tmp,
                       n, w, dst, nr, c0);
  }
}

// dst <- m widen(src) for a float32 source (n <= 512, dst distinct from
// src); returns false for larger n, where the caller widens first.
bool launch_apply_left_f32(const double* m, const float* src, double* dst, int n, long long nr,
                           double* tmp, hipStream_t st) {
  if (n > 512) return false;
  apply_left(m, src, dst, n, nr, tmp, st);
  return true;
}

}  // namespace hfx
