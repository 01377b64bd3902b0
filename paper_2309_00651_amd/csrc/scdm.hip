// SCDM localisation (selected columns of the density matrix; the Methods'
// MTACE subsection uses SCDM-localised orbitals for s-MTACE).  Grid points
// c_1..c_N are chosen by column-pivoted QR of the N_orb x N_r matrix Psi^T:
// step k takes the point whose residual, after the directions of the points
// chosen so far are projected out, has the largest norm (ties: the smallest
// index).  The localised functions xi_k(r) = sum_i psi_i(r) psi_i(c_k) are the
// density-matrix columns at those points; the caller orthonormalises them.
//
// Only the pivots are needed, so no Q or R of the N_r columns is formed: the
// squared residual norms w_r are kept and downdated, w_r -= (q_k . a_r)^2,
// where q_k (N_orb values) is the normalised residual of the chosen column,
// obtained by classical Gram-Schmidt applied twice against q_1..q_(k-1) in one
// workgroup.  Downdating every point in every step reads Psi N_orb times
// (73 us a step at 128 orbitals on 72^3, 9 of the call's 14 ms).  Norms only
// fall, though, so a norm that is some steps behind is an upper bound: the
// points are kept in blocks of 256 with their largest norm, and a step brings
// up to date only the blocks whose bound reaches the value that a candidate
// point is known to have now (a handful of 1458 in the median step there, 31 us
// on average with the steps that find no good bound).  Every norm still
// receives its downdates one by one and in order, so pivots and norms are
// those of the plain method.  Tried and slower: the directions staged in LDS
// instead of scalar loads (62 us), and sweeps over all blocks every 16 steps
// with bounds from blocks that lag (18 us a step and 184 per sweep, but a
// longer pick).
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <type_traits>

#include "hfx_internal.hpp"
#include "scdm_bound.hpp"

namespace hfx {

namespace {
constexpr int NTS = 256;   // threads per workgroup and points per block
constexpr int NTP = 1024;  // threads of the pick

// State of the blocks: w, and per block its largest w, where, and the number
// of directions already applied; bound[0]: what a block must reach to matter.
struct ScdmState {
  double* w;
  double* bmax;
  double* bound;
  int* barg;
  int* stamp;
  int blocks;
};
}  // namespace

// (v, i) wins over (u, j): larger value, then smaller index
__device__ __forceinline__ bool beats(double v, int i, double u, int j) {
  return v > u || (v == u && i < j);
}

template <int THREADS>
__device__ void block_argmax(double& v, int& i, double* sv, int* si) {
  const int tid = threadIdx.x;
  sv[tid] = v;
  si[tid] = i;
  __syncthreads();
  for (int s = THREADS / 2; s > 0; s >>= 1) {
    if (tid < s && beats(sv[tid + s], si[tid + s], sv[tid], si[tid])) {
      sv[tid] = sv[tid + s];
      si[tid] = si[tid + s];
    }
    __syncthreads();
  }
  v = sv[0];
  i = si[0];
  __syncthreads();
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s);
  return v;
}

// w_r = sum_i psi_i(r)^2 and the blocks' maxima (one workgroup per block).
// Norms are never NaN (here, and by fmax in the updates), and ties go to the
// smaller index, so every block maximum names a point of the grid, whatever
// the orbitals hold.
__global__ void __launch_bounds__(NTS) k_scdm_norms(const double* __restrict__ psi, int n,
                                                     long long nr, ScdmState st) {
  __shared__ double sv[NTS];
  __shared__ int si[NTS];
  const long long r = (long long)blockIdx.x * NTS + threadIdx.x;
  double s = -1.0;
  if (r < nr) {
    s = 0.0;
#pragma unroll 16
    for (int i = 0; i < n; ++i) {
      const double x = psi[(long long)i * nr + r];
      s += x * x;
    }
    // a point with a NaN is never chosen: its norm would neither win nor lose
    // a comparison and would hide the other points of its block
    if (!(s >= 0.0)) s = -1.0;
    st.w[r] = s;
  }
  int at = r < nr ? (int)r : INT_MAX;
  block_argmax<NTS>(s, at, sv, si);
  if (threadIdx.x == 0) {
    st.bmax[blockIdx.x] = s;
    st.barg[blockIdx.x] = at;
    st.stamp[blockIdx.x] = 0;
    if (blockIdx.x == 0) st.bound[0] = 0.0;
  }
}

// Brings the blocks whose bound reaches bound[0] up to date with the
// directions q_stamp .. q_(k-1): w_r -= (q . a_r)^2 for the points not chosen
// yet (chosen points hold -1), up to eight directions per read of Psi.
__global__ void __launch_bounds__(NTS) k_scdm_update(const double* __restrict__ psi, int n,
                                                      long long nr, int k,
                                                      const double* __restrict__ qm, ScdmState st) {
  __shared__ double sv[NTS];
  __shared__ int si[NTS];
  const double need = st.bound[0];
  for (int b = blockIdx.x; b < st.blocks; b += gridDim.x) {
    if (st.bmax[b] < need) continue;
    const long long r = (long long)b * NTS + threadIdx.x;
    const bool in = r < nr;
    const double* __restrict__ col = psi + (in ? r : 0);
    double v = in ? st.w[r] : -1.0;
    auto apply = [&](auto gc, int s0) {
      constexpr int G = decltype(gc)::value;
      double t[G];
#pragma unroll
      for (int g = 0; g < G; ++g) t[g] = 0.0;
      const double* __restrict__ q = qm + (long long)s0 * n;
#pragma unroll 16
      for (int i = 0; i < n; ++i) {
        const double x = col[(long long)i * nr];
#pragma unroll
        for (int g = 0; g < G; ++g) t[g] += q[(long long)g * n + i] * x;
      }
      if (v >= 0.0) {
#pragma unroll
        for (int g = 0; g < G; ++g) v = fmax(v - t[g] * t[g], 0.0);
      }
    };
    int s = st.stamp[b];
    for (; s + 8 <= k; s += 8) apply(std::integral_constant<int, 8>{}, s);
    if (s + 4 <= k) {
      apply(std::integral_constant<int, 4>{}, s);
      s += 4;
    }
    if (s + 2 <= k) {
      apply(std::integral_constant<int, 2>{}, s);
      s += 2;
    }
    if (s < k) apply(std::integral_constant<int, 1>{}, s);
    if (in) st.w[r] = v;
    int at = in ? (int)r : INT_MAX;
    block_argmax<NTS>(v, at, sv, si);
    if (threadIdx.x == 0) {
      st.bmax[b] = v;
      st.barg[b] = at;
      st.stamp[b] = k;
    }
  }
}

// Step k: the point of the largest block maximum is the pivot (blocks that
// were not brought up to date have bounds below it); its column a =
// (psi_i(c_k))_i is orthogonalised against q_0..q_(k-1) (rows of qm) twice and
// normalised into q_k.  A vanishing residual (linearly dependent orbitals)
// or a non-finite column gives a NaN direction; the norms it is applied to
// become zero, and the later pivots are arbitrary points.  Then the bound of the next
// step: every wavefront takes the best point among its share of the blocks
// that are up to date and downdates it with q_k; some point has at least the
// largest of these norms (less what the two sums of a projection may differ
// by), so blocks below it cannot hold the next pivot.
__global__ void __launch_bounds__(NTP) k_scdm_pick(const double* __restrict__ psi, int n,
                                                    long long nr, int k, double* __restrict__ qm,
                                                    int* __restrict__ piv, ScdmState st) {
  extern __shared__ double sh[];  // sv[NTP], a[n], c[n]
  double* sv = sh;                // argmax and partial sums
  double* a = sh + NTP;
  double* c = a + n;
  int* si = reinterpret_cast<int*>(a);  // argmax, before a is loaded
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int WV = NTP / 64;
  double best = -1.0, cand = -1.0;
  int bi = INT_MAX, ci = INT_MAX;
  for (int b = tid; b < st.blocks; b += NTP) {
    const double v = st.bmax[b];
    const int at = st.barg[b];
    if (beats(v, at, best, bi)) {
      best = v;
      bi = at;
    }
  }
  block_argmax<NTP>(best, bi, sv, si);
  const int p = bi;
  if (tid == 0) {
    piv[k] = p;
    st.w[p] = -1.0;  // never chosen again
  }
  // the wavefronts' candidates, outside the pivot's block
  for (int b = tid; b < st.blocks; b += NTP)
    if (st.stamp[b] == k && b != p / NTS && beats(st.bmax[b], st.barg[b], cand, ci)) {
      cand = st.bmax[b];
      ci = st.barg[b];
    }
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) {
    const double v = __shfl_xor(cand, s);
    const int i = __shfl_xor(ci, s);
    if (beats(v, i, cand, ci)) {
      cand = v;
      ci = i;
    }
  }
  for (int i = tid; i < n; i += NTP) a[i] = psi[(long long)i * nr + p];
  __syncthreads();
  for (int pass = 0; pass < 2 && k > 0; ++pass) {
    // c_j = q_j . a, one wavefront per j
    for (int j = wave; j < k; j += WV) {
      double s = 0.0;
      for (int i = lane; i < n; i += 64) s += qm[(long long)j * n + i] * a[i];
      s = wave_sum(s);
      if (lane == 0) c[j] = s;
    }
    __syncthreads();
    // a -= sum_j c_j q_j: 64 elements per step, the j shared by the wavefronts
    for (int i0 = 0; i0 < n; i0 += 64) {
      const int i = i0 + lane;
      double s = 0.0;
      if (i < n) {
#pragma unroll 8
        for (int j = wave; j < k; j += WV) s += c[j] * qm[(long long)j * n + i];
      }
      sv[tid] = s;
      __syncthreads();
      if (wave == 0 && i < n) {
        double t = 0.0;
        for (int u = 0; u < WV; ++u) t += sv[u * 64 + lane];
        a[i] -= t;
      }
      __syncthreads();
    }
  }
  double s2 = 0.0;
  for (int i = tid; i < n; i += NTP) s2 += a[i] * a[i];
  s2 = wave_sum(s2);
  if (lane == 0) sv[wave] = s2;
  __syncthreads();
  double nrm = 0.0;
  for (int u = 0; u < WV; ++u) nrm += sv[u];
  const double inv = nrm > 0.0 ? 1.0 / sqrt(nrm) : NAN;
  for (int i = tid; i < n; i += NTP) qm[(long long)k * n + i] = a[i] * inv;
  // the next step's bound
  double t = 0.0, x2 = 0.0;
  if (ci != INT_MAX)
    for (int i = lane; i < n; i += 64) {
      const double x = psi[(long long)i * nr + ci];
      t += a[i] * inv * x;
      x2 += x * x;
    }
  t = wave_sum(t);
  x2 = wave_sum(x2);
  __syncthreads();
  if (lane == 0) sv[wave] = ci == INT_MAX ? 0.0 : scdm_lower_bound(cand, t, x2, n);
  __syncthreads();
  if (tid == 0) {
    double m = 0.0;
    for (int u = 0; u < WV; ++u) m = sv[u] > m ? sv[u] : m;
    st.bound[0] = m;
  }
}

// b[k][i] = psi_i(c_k)
__global__ void __launch_bounds__(NTS) k_scdm_gather(const double* __restrict__ psi, int n,
                                                      long long nr, const int* __restrict__ piv,
                                                      double* __restrict__ b) {
  const long long e = (long long)blockIdx.x * NTS + threadIdx.x;
  if (e >= (long long)n * n) return;
  const int k = (int)(e / n), i = (int)(e - (long long)k * n);
  b[e] = psi[(long long)i * nr + piv[k]];
}

static size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t scdm_scratch_bytes(long long nr) {
  const size_t blocks = (size_t)(nr + NTS - 1) / NTS;
  return up256((size_t)nr * 8) + up256(blocks * 8) + up256(8) + 2 * up256(blocks * 4);
}

void launch_scdm_pivots(const double* psi, int n, long long nr, char* scratch, double* qm,
                        int* piv, hipStream_t st) {
  ScdmState s;
  s.blocks = (int)((nr + NTS - 1) / NTS);
  auto take = [&](size_t bytes) {
    char* p = scratch;
    scratch += up256(bytes);
    return p;
  };
  s.w = reinterpret_cast<double*>(take((size_t)nr * 8));
  s.bmax = reinterpret_cast<double*>(take((size_t)s.blocks * 8));
  s.bound = reinterpret_cast<double*>(take(8));
  s.barg = reinterpret_cast<int*>(take((size_t)s.blocks * 4));
  s.stamp = reinterpret_cast<int*>(take((size_t)s.blocks * 4));
  hipLaunchKernelGGL(k_scdm_norms, dim3((unsigned)s.blocks), dim3(NTS), 0, st, psi, n, nr, s);
  const size_t pick_lds = ((size_t)NTP + (2 * n > NTP / 2 ? 2 * n : NTP / 2)) * 8;
  const unsigned grid = (unsigned)(s.blocks < kScdmParts ? s.blocks : kScdmParts);
  for (int k = 0; k < n; ++k) {
    if (k > 0)
      hipLaunchKernelGGL(k_scdm_update, dim3(grid), dim3(NTS), 0, st, psi, n, nr, k, qm, s);
    hipLaunchKernelGGL(k_scdm_pick, dim3(1), dim3(NTP), pick_lds, st, psi, n, nr, k, qm, piv, s);
  }
}

void launch_scdm_gather(const double* psi, int n, long long nr, const int* piv, double* b,
                        hipStream_t st) {
  const long long tot = (long long)n * n;
  hipLaunchKernelGGL(k_scdm_gather, dim3((unsigned)((tot + NTS - 1) / NTS)), dim3(NTS), 0, st,
                     psi, n, nr, piv, b);
}

}  // namespace hfx
