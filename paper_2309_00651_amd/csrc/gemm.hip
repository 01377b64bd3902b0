// Dense contractions over the grid: C = alpha * A B^T with A, B [n][nr]
// (orbital-major, grid points contiguous).  Used for the exchange matrix
// M = dV Psi^T (K Psi), the overlap S = dV Psi^T Psi and the float32 plans'
// pair-density means (1/N_r) Psi^T Psi.
//
// The long grid dimension is cut into chunks; one workgroup computes one
// TM x TN tile of C over one chunk on the matrix cores and stores a float64
// partial, and a second kernel sums the partials over the chunks in a fixed
// order (results are bitwise reproducible).  Inside a workgroup, K-blocks of
// KB grid points are staged through double-buffered LDS: the vector loads of
// block k+1 are in flight while block k feeds the MFMAs.  Workgroups of one
// chunk are consecutive in the XCD-aware order, so the chunk's rows of A and B
// come from HBM once and are shared through the XCD's L2.  When A and B are
// the same matrix only the tiles on and above the diagonal are computed.
//
// Split precision (float32 plans, exchange matrix): A is float64 and is split
// as a = hi + lo with hi = fl32(a), lo = fl32(a - hi); hi*b and lo*b go to two
// float32 MFMA accumulators that are folded into float64 registers every
// KFOLD grid points, so A's float64 information reaches the result and the
// float32 accumulation length stays bounded.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "hfx_internal.hpp"

namespace hfx {

namespace {
constexpr int KFOLD = 32;       // float32 accumulation length before folding

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// MODE 0: float64 A and B, float64 MFMA.  MODE 1: split A, float32 B.
// MODE 2: as 0 on |A| and |B| (the screening overlaps int |phi_i phi_j|).
// TILE: the output tile, the smallest of 16, 32, 64 and 128 that holds the
// orbitals (128 above).  A small set on the 128 tile was bound by work done
// for padding: 13 orbitals on 64^3 took 152 us in the product and 146 us in
// summing 512 padded 128 KB partials, for 27 MB of input; on the 16 tile the
// two take 24 us (K psi and E_x 511 -> 237 us; two channels of 21 and 18
// orbitals on 64^2 x 128 2247 -> 1524 us).  The small tiles
// only stream A, so they take longer K-blocks (KB grid points per LDS stage,
// whole 128-byte segments per row at least) and twice the workgroups; a 16 x
// 16 tile is one MFMA block, and its four wavefronts split the K-block (KS).
template <int MODE, int TILE>
struct Cfg {
  static constexpr int TM = TILE;                                // C tile rows (A rows)
  static constexpr int TN = MODE == 1 && TILE == 128 ? 64 : TILE;  // C tile columns (B rows)
  static constexpr int KB = TILE >= 64 ? 16 : TILE == 32 ? 32 : 64;
  static constexpr int KS = TILE == 16 ? 4 : 1;    // wavefronts along the K-block
  static constexpr int WM = KS > 1 ? TM : TM / 2;  // rows per wavefront (2 x 2 wavefronts)
  static constexpr int WN = KS > 1 ? TN : TN / 2;
  static constexpr int BM = WM / 16, BN = WN / 16;  // 16 x 16 MFMA blocks per wavefront
  static constexpr int APT = TM * KB / 256;         // A values per thread and K-block
  static constexpr int BPT = TN * KB / 256;         // B values per thread
  // workgroups per product: one round of resident workgroups (two per
  // compute unit; small tiles, bound by loads in flight, four)
  static constexpr int TARGET_WG = TILE == 128 ? 512 : 1024;
};

// Tile of a product of n orbitals.  The split product keeps 32 as its
// smallest: its float32 accumulators fold every KFOLD points of one wavefront.
int tile_of(int n, int mode) {
  if (n > 64) return 128;
  if (n > 32) return 64;
  return n > 16 || mode == 1 ? 32 : 16;
}

__device__ __forceinline__ int xcd_order(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int xcd = b & 7, idx = b >> 3;
  return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

// The tiles of a product, their chunks and workgroups.  "off" tiles: all of
// them, or, in a symmetric product, those above the diagonal; a symmetric
// product's diagonal tiles ("diag") load A once and skip the 16 x 16 blocks
// below the diagonal (10 block products per wavefront for 16 at a 128 tile),
// so they take longer chunks of the grid, in proportion.
struct GemmShape {
  int tiles_m, tiles_n, n_off, n_diag, chunks_o, chunks_d;
  long long len_o, len_d;
};

template <int MODE, int TILE>
GemmShape gemm_shape(int n, long long nr, bool sym) {
  using C = Cfg<MODE, TILE>;
  GemmShape g;
  g.tiles_m = (n + C::TM - 1) / C::TM;
  g.tiles_n = (n + C::TN - 1) / C::TN;
  g.n_diag = sym ? g.tiles_m : 0;
  g.n_off = sym ? g.tiles_m * (g.tiles_m - 1) / 2 : g.tiles_m * g.tiles_n;
  // whole rounds: TARGET_WG workgroups run at once, one more would double
  // the time of the product.  A diagonal tile costs 10/16 of another one.
  auto fit = [&](long long chunks, int* count, long long* len) {
    const long long max_chunks = (nr + 4 * C::KB - 1) / (4 * C::KB);  // at least 4 K-blocks each
    if (chunks > max_chunks) chunks = max_chunks;
    if (chunks < 1) chunks = 1;
    *len = (nr + chunks - 1) / chunks;
    *len = (*len + C::KB - 1) / C::KB * C::KB;
    *count = (int)((nr + *len - 1) / *len);
  };
  fit((long long)C::TARGET_WG * 16 / (16 * g.n_off + 10 * g.n_diag), &g.chunks_o, &g.len_o);
  const long long left = (long long)C::TARGET_WG - (long long)g.n_off * g.chunks_o;
  fit(g.n_diag ? left / g.n_diag : 1, &g.chunks_d, &g.len_d);
  return g;
}
}  // namespace

// MFMA 16x16x4 operand layout (one 64-wide wavefront, lane l):
//   A operand: A[l % 16][l / 16]   (16 x 4)
//   B operand: B[l / 16][l % 16]   (4 x 16)
//   result, 4 values i = 0..3:  f32: D[4 (l / 16) + i][l % 16]
//                               f64: D[(l / 16) + 4 i][l % 16]
// (both checked on gfx950 against a host product).
// One product of a launch: C = alpha A B^T over nr points, its chunking and
// tiles (gemm_shape), partials and output.  A launch carries up to
// kMaxGroup of them with one tile size (a GramGroup, by value as the kernel
// argument); product s owns the logical workgroups [start[s], start[s + 1])
// of the product kernel and [rstart[s], rstart[s + 1]) of the reduction.
// Each product keeps its own chunking, so its result is the same whether
// launched alone or with others.
struct GramJob {
  const double* a;
  const void* b;
  double* part;
  double* c;
  double alpha;
  long long nr;
  GemmShape g;
  int n, sym;
};
struct GramGroup {
  GramJob j[kMaxGroup];
  int start[kMaxGroup + 1];
  int rstart[kMaxGroup + 1];
  int count;
};
__device__ __forceinline__ int gram_locate(const int* start, int count, int L, int& s) {
  int k = 0;
#pragma unroll
  for (int i = 1; i < kMaxGroup; ++i)
    if (i < count && L >= start[i]) k = i;
  s = k;
  return L - start[k];
}

template <int MODE, int TILE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
k_gram(GramGroup grp) {
  int js = 0;
  const int L = gram_locate(grp.start, grp.count, xcd_order(blockIdx.x, gridDim.x), js);
  const GramJob& J = grp.j[js];
  const double* __restrict__ a = J.a;
  const void* __restrict__ bv = J.b;
  const int n = J.n;
  const long long nr = J.nr;
  using C = Cfg<MODE, TILE>;
  constexpr int TM = C::TM, TN = C::TN, BM = C::BM, BN = C::BN, KB = C::KB, KS = C::KS;
  constexpr bool SPLIT = MODE == 1;
  static_assert(!SPLIT || KS == 1, "the split product folds one wavefront's accumulators");
  using BT = typename std::conditional<SPLIT, float, double>::type;
  using AT = typename std::conditional<SPLIT, float, double>::type;  // LDS type of A
  const BT* __restrict__ b = static_cast<const BT*>(bv);
  __shared__ AT as_hi[2][TM][KB + 1];
  __shared__ float as_lo[SPLIT ? 2 : 1][SPLIT ? TM : 1][KB + 1];
  __shared__ BT bs[2][TN][KB + 1];

  // workgroup -> tile and chunk (chunk-major inside each class of tiles)
  const int first_d = J.g.n_off * J.g.chunks_o;
  const bool diag = !SPLIT && L >= first_d;
  int ti, tj, c;
  double* out;
  if (diag) {
    const int l = L - first_d;
    ti = tj = l % J.g.n_diag;
    c = l / J.g.n_diag;
    out = J.part + ((long long)first_d + (long long)ti * J.g.chunks_d + c) * TM * TN;
  } else {
    const int t = L % J.g.n_off;
    c = L / J.g.n_off;
    if (J.sym) {
      int rem = t;
      ti = 0;
      while (rem >= J.g.tiles_n - 1 - ti) {
        rem -= J.g.tiles_n - 1 - ti;
        ++ti;
      }
      tj = ti + 1 + rem;
    } else {
      ti = t / J.g.tiles_n;
      tj = t - ti * J.g.tiles_n;
    }
    out = J.part + ((long long)t * J.g.chunks_o + c) * TM * TN;
  }
  const int row0 = ti * TM, col0 = tj * TN;
  const long long len = diag ? J.g.len_d : J.g.len_o;
  const long long r_begin = (long long)c * len;
  const long long r_end = r_begin + len < nr ? r_begin + len : nr;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  // Diagonal tiles: wavefronts 0 and 3 hold the diagonal quarters of the tile
  // (BM (BM + 1) / 2 blocks each); 1 and 2 share the quarter above the
  // diagonal (PH = BM / 2 of its block rows each, wavefront 2 the lower
  // ones); the quarter below it is not computed.
  constexpr int PH = BM / 2;
  const bool half = KS == 1 && (wave == 1 || wave == 2);
  const bool idle = KS == 1 && PH == 0 && wave == 2;  // one block: wavefront 1 has it
  const bool lower = KS == 1 && wave == 2;
  const int wr = KS > 1 ? 0 : (diag && lower) ? 16 * PH : (wave >> 1) * C::WM;
  const int wc = KS > 1 ? 0 : (diag && lower) ? C::WN : (wave & 1) * C::WN;
  const int lr = lane & 15, lk = lane >> 4;

  // loader maps: APT consecutive points of one A row per thread, BPT of one
  // B row (BPT <= APT)
  constexpr int APT = C::APT, BPT = C::BPT;
  const int a_row = tid / (KB / APT), a_k = (tid % (KB / APT)) * APT;
  const int b_row = tid / (KB / BPT), b_k = (tid % (KB / BPT)) * BPT;
  const bool a_ok = row0 + a_row < n;
  const bool b_ok = col0 + b_row < n;
  const double* __restrict__ a_ptr = a + (long long)(a_ok ? row0 + a_row : 0) * nr;
  const BT* __restrict__ b_ptr = b + (long long)(b_ok ? col0 + b_row : 0) * nr;

  double ra[APT];
  BT rb[BPT];
  auto load = [&](long long r0) {
    const long long ra0 = r0 + a_k, rb0 = r0 + b_k;
    if (a_ok && ra0 + APT <= r_end) {
      const double2* p = reinterpret_cast<const double2*>(a_ptr + ra0);
#pragma unroll
      for (int u = 0; u < APT / 2; ++u) {
        const double2 v = p[u];
        ra[2 * u] = v.x;
        ra[2 * u + 1] = v.y;
      }
    } else {
#pragma unroll
      for (int u = 0; u < APT; ++u) ra[u] = (a_ok && ra0 + u < r_end) ? a_ptr[ra0 + u] : 0.0;
    }
    if (diag) return;  // B is A
    if (b_ok && rb0 + BPT <= r_end) {
      if constexpr (SPLIT) {
        const float4 v = *reinterpret_cast<const float4*>(b_ptr + rb0);
        rb[0] = v.x;
        rb[1] = v.y;
        rb[2] = v.z;
        rb[3] = v.w;
      } else {
        const double2* p = reinterpret_cast<const double2*>(b_ptr + rb0);
#pragma unroll
        for (int u = 0; u < BPT / 2; ++u) {
          const double2 v = p[u];
          rb[2 * u] = v.x;
          rb[2 * u + 1] = v.y;
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < BPT; ++u) rb[u] = (b_ok && rb0 + u < r_end) ? b_ptr[rb0 + u] : BT(0);
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int u = 0; u < APT; ++u) {
      if constexpr (SPLIT) {
        const float hi = (float)ra[u];
        as_hi[buf][a_row][a_k + u] = hi;
        as_lo[buf][a_row][a_k + u] = (float)(ra[u] - (double)hi);
      } else {
        as_hi[buf][a_row][a_k + u] = MODE == 2 ? fabs(ra[u]) : ra[u];
      }
    }
    if (diag) return;
#pragma unroll
    for (int u = 0; u < BPT; ++u) {
      if constexpr (MODE == 2)
        bs[buf][b_row][b_k + u] = fabs(rb[u]);
      else
        bs[buf][b_row][b_k + u] = rb[u];
    }
  };

  int buf = 0;
  if (r_begin < r_end) {
    load(r_begin);
    stage(0);
  }
  __syncthreads();
  // for every K-block: the next block's loads in flight during mul(kk), the
  // MFMA step at K offset kk, then fold(last)
  auto blocks = [&](auto&& mul, auto&& fold) {
    for (long long r0 = r_begin; r0 < r_end; r0 += KB) {
      const bool more = r0 + KB < r_end;
      if (more) load(r0 + KB);
#pragma unroll
      for (int s = 0; s < KB / 4 / KS; ++s) mul(4 * (KS > 1 ? wave * (KB / 4 / KS) + s : s) + lk);
      fold(!more);
      if (more) stage(buf ^ 1);  // the other buffer: last read before the previous barrier
      __syncthreads();
      buf ^= 1;
    }
  };
  auto store = [&](int p, int q, const f64x4& v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int rr = wr + 16 * p + (SPLIT ? 4 * lk + i : lk + 4 * i);
      const int cc = wc + 16 * q + lr;
      out[rr * TN + cc] = v[i];
    }
  };
  if constexpr (KS > 1) {
    // one 16 x 16 block: the wavefronts' K shares summed in order
    f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
    blocks(
        [&](int kk) {
          const double ad = as_hi[buf][lr][kk], bd = diag ? ad : bs[buf][lr][kk];
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ad, bd, acc, 0, 0, 0);
        },
        [](bool) {});
    __shared__ double sum[KS][256];
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[wave][(lk + 4 * i) * 16 + lr] = acc[i];
    __syncthreads();
    double v = sum[0][tid];
#pragma unroll
    for (int w = 1; w < KS; ++w) v += sum[w][tid];
    out[tid] = v;
  } else if (!SPLIT && diag) {
    // the blocks p <= q; of the two block rows of a sharing wavefront (BM =
    // 4), block (1, 0) takes the place of (2, 2) and the last two are unused
    f64x4 acc[BM][BN];
#pragma unroll
    for (int p = 0; p < BM; ++p)
#pragma unroll
      for (int q = p; q < BN; ++q) acc[p][q] = f64x4{0.0, 0.0, 0.0, 0.0};
    blocks(
        [&](int kk) {
          double ad[BM], bd[BN];
#pragma unroll
          for (int p = 0; p < BM; ++p) {
            // rows beyond a sharing wavefront's own repeat its first
            const int pr = half && p >= (PH > 0 ? PH : 1) ? 0 : p;
            ad[p] = as_hi[buf][wr + 16 * pr + lr][kk];
            bd[p] = as_hi[buf][wc + 16 * p + lr][kk];
          }
#pragma unroll
          for (int p = 0; p < BM; ++p)
#pragma unroll
            for (int q = p; q < BN; ++q) {
              double x = ad[p], y = bd[q];
              if (BM == 4 && p == 2 && q == 2) {
                x = half ? ad[1 % BM] : x;
                y = half ? bd[0] : y;
              }
              acc[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc[p][q], 0, 0, 0);
            }
        },
        [](bool) {});
#pragma unroll
    for (int p = 0; p < BM; ++p)
#pragma unroll
      for (int q = p; q < BN; ++q) {
        if (idle) continue;
        if (!half || p < (PH > 0 ? PH : 1))
          store(p, q, acc[p][q]);
        else if (BM == 4 && p == 2 && q == 2)
          store(1, 0, acc[p][q]);
      }
  } else {
    f64x4 acc64[BM][BN];
    f32x4 acch[SPLIT ? BM : 1][SPLIT ? BN : 1], accl[SPLIT ? BM : 1][SPLIT ? BN : 1];
#pragma unroll
    for (int p = 0; p < BM; ++p)
#pragma unroll
      for (int q = 0; q < BN; ++q) {
        acc64[p][q] = f64x4{0.0, 0.0, 0.0, 0.0};
        if constexpr (SPLIT) {
          acch[p][q] = f32x4{0.f, 0.f, 0.f, 0.f};
          accl[p][q] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    int since_fold = 0;
    blocks(
        [&](int kk) {
          if constexpr (SPLIT) {
            float ah[BM], al[BM], bx[BN];
#pragma unroll
            for (int p = 0; p < BM; ++p) {
              ah[p] = as_hi[buf][wr + 16 * p + lr][kk];
              al[p] = as_lo[buf][wr + 16 * p + lr][kk];
            }
#pragma unroll
            for (int q = 0; q < BN; ++q) bx[q] = bs[buf][wc + 16 * q + lr][kk];
#pragma unroll
            for (int p = 0; p < BM; ++p)
#pragma unroll
              for (int q = 0; q < BN; ++q) {
                acch[p][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(ah[p], bx[q], acch[p][q], 0, 0, 0);
                accl[p][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(al[p], bx[q], accl[p][q], 0, 0, 0);
              }
          } else {
            double ad[BM], bd[BN];
#pragma unroll
            for (int p = 0; p < BM; ++p) ad[p] = as_hi[buf][wr + 16 * p + lr][kk];
#pragma unroll
            for (int q = 0; q < BN; ++q) bd[q] = bs[buf][wc + 16 * q + lr][kk];
#pragma unroll
            for (int p = 0; p < BM; ++p)
#pragma unroll
              for (int q = 0; q < BN; ++q)
                acc64[p][q] =
                    __builtin_amdgcn_mfma_f64_16x16x4f64(ad[p], bd[q], acc64[p][q], 0, 0, 0);
          }
        },
        [&](bool last) {
          if constexpr (SPLIT) {
            since_fold += KB;
            if (since_fold >= KFOLD || last) {
#pragma unroll
              for (int p = 0; p < BM; ++p)
#pragma unroll
                for (int q = 0; q < BN; ++q) {
#pragma unroll
                  for (int i = 0; i < 4; ++i)
                    acc64[p][q][i] += (double)acch[p][q][i] + (double)accl[p][q][i];
                  acch[p][q] = f32x4{0.f, 0.f, 0.f, 0.f};
                  accl[p][q] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
              since_fold = 0;
            }
          }
        });
#pragma unroll
    for (int p = 0; p < BM; ++p)
#pragma unroll
      for (int q = 0; q < BN; ++q) store(p, q, acc64[p][q]);
  }
}

// C[i][j] = alpha * sum_c part[tile(i, j)][c][i % TM][j % TN] in a fixed
// order over c; symmetric products sum i <= j and write both halves.  A
// workgroup sums 16 neighbouring columns of one row: 16 threads per column
// take every 16th chunk each (one thread per element, walking 512 chunks
// 128 KB apart, was bound by its chain of loads: 167 us at 64 orbitals), and
// their sums are added in order.
constexpr int RC = 16;  // columns per reduction workgroup
template <int MODE, int TILE>
__global__ void __launch_bounds__(256) k_gram_reduce(GramGroup grp) {
  int js = 0;
  const int blk = gram_locate(grp.rstart, grp.count, (int)blockIdx.x, js);
  const GramJob& J = grp.j[js];
  using C = Cfg<MODE, TILE>;
  const int n = J.n;
  const int per_row = (n + RC - 1) / RC;
  const int i = blk / per_row, j0 = (blk - i * per_row) * RC;
  if (J.sym && j0 + RC <= i) return;  // written from the other half
  __shared__ double red[RC][256 / RC + 1];
  const int e = threadIdx.x % RC, sl = threadIdx.x / RC;
  const int j = j0 + e;
  const bool ok = j < n && (!J.sym || j >= i);
  double s = 0.0;
  if (ok) {
    const int ti = i / C::TM, tj = j / C::TN;
    long long first;
    int count;
    if (J.sym && ti == tj) {
      first = (long long)J.g.n_off * J.g.chunks_o + (long long)ti * J.g.chunks_d;
      count = J.g.chunks_d;
    } else {
      int tile = J.sym ? tj - ti - 1 : ti * J.g.tiles_n + tj;
      if (J.sym)
        for (int r = 0; r < ti; ++r) tile += J.g.tiles_n - 1 - r;
      first = (long long)tile * J.g.chunks_o;
      count = J.g.chunks_o;
    }
    const double* p = J.part + first * C::TM * C::TN + (long long)(i % C::TM) * C::TN + (j % C::TN);
#pragma unroll 4
    for (int c = sl; c < count; c += 256 / RC) s += p[(long long)c * C::TM * C::TN];
  }
  red[e][sl] = s;
  __syncthreads();
  if (sl == 0 && ok) {
    double v = red[e][0];
    for (int k = 1; k < 256 / RC; ++k) v += red[e][k];
    v *= J.alpha;
    J.c[(long long)i * n + j] = v;
    if (J.sym) J.c[(long long)j * n + i] = v;
  }
}

template <int MODE, int TILE>
static GramJob gram_job(const double* a, const void* b, int n, long long nr, double alpha,
                        bool sym, double* part, double* c) {
  GramJob j{};
  j.a = a;
  j.b = b;
  j.part = part;
  j.c = c;
  j.alpha = alpha;
  j.nr = nr;
  j.g = gemm_shape<MODE, TILE>(n, nr, sym);
  j.n = n;
  j.sym = sym ? 1 : 0;
  return j;
}

// The products of jobs[0..count) in one launch of the product kernel and
// one of the reduction.
template <int MODE, int TILE>
static void launch_gram_group(const GramJob* jobs, int count, hipStream_t s) {
  GramGroup g{};
  g.count = count;
  int blocks = 0, rblocks = 0;
  for (int i = 0; i < count; ++i) {
    const GemmShape& sh = jobs[i].g;
    g.j[i] = jobs[i];
    g.start[i] = blocks;
    g.rstart[i] = rblocks;
    blocks += sh.n_off * sh.chunks_o + sh.n_diag * sh.chunks_d;
    rblocks += jobs[i].n * ((jobs[i].n + RC - 1) / RC);
  }
  g.start[count] = blocks;
  g.rstart[count] = rblocks;
  hipLaunchKernelGGL((k_gram<MODE, TILE>), dim3((unsigned)blocks), dim3(256), 0, s, g);
  hipLaunchKernelGGL((k_gram_reduce<MODE, TILE>), dim3((unsigned)rblocks), dim3(256), 0, s, g);
}

// Calls f(std::integral_constant<int, TILE>) for the tile of n orbitals.
template <int MODE, class F>
static void with_tile(int n, F&& f) {
  switch (tile_of(n, MODE)) {
    case 16:
      if constexpr (MODE != 1) f(std::integral_constant<int, 16>{});
      break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    case 64: f(std::integral_constant<int, 64>{}); break;
    default: f(std::integral_constant<int, 128>{});
  }
}

template <int MODE>
static void launch_gram(const double* a, const void* b, int n, long long nr, double alpha,
                        bool sym, double* part, double* c, hipStream_t s) {
  with_tile<MODE>(n, [&](auto tile) {
    constexpr int TILE = decltype(tile)::value;
    const GramJob j = gram_job<MODE, TILE>(a, b, n, nr, alpha, sym, part, c);
    launch_gram_group<MODE, TILE>(&j, 1, s);
  });
}

size_t gemm_partial_bytes(int n_orb, long long nr) {
  size_t best = 0;
  auto take = [&](const GemmShape& g, size_t tile) {
    best = std::max(best, ((size_t)g.n_off * g.chunks_o + (size_t)g.n_diag * g.chunks_d) * tile * 8);
  };
  with_tile<0>(n_orb, [&](auto tile) {
    constexpr int TILE = decltype(tile)::value;
    for (int sym = 0; sym < 2; ++sym) take(gemm_shape<0, TILE>(n_orb, nr, sym != 0), TILE * TILE);
  });
  with_tile<1>(n_orb, [&](auto tile) {
    using C = Cfg<1, decltype(tile)::value>;
    take(gemm_shape<1, decltype(tile)::value>(n_orb, nr, false), C::TM * C::TN);
  });
  return best;
}

void launch_xtx_split(const double* a, const float* b, int n, long long nr, double alpha,
                      double* part, double* c, hipStream_t s) {
  launch_gram<1>(a, b, n, nr, alpha, false, part, c, s);
}

void launch_xtx_f64(const double* a, const double* b, int n, long long nr, double alpha,
                    double* part, double* c, hipStream_t s) {
  launch_gram<0>(a, b, n, nr, alpha, a == b, part, c, s);
}

void launch_xtx_abs(const double* a, int n, long long nr, double alpha, double* part, double* c,
                    hipStream_t s) {
  launch_gram<2>(a, a, n, nr, alpha, true, part, c, s);
}

// One launch per tile size among the products.
void launch_gram_self_group(const double* const* a, const int* n, const long long* nr,
                            const double* alpha, double* const* part, double* const* c,
                            int count, hipStream_t s) {
  for (int t : {16, 32, 64, 128})
    for (int first = 0; first < count; ++first) {
      if (tile_of(n[first], 0) != t) continue;
      with_tile<0>(n[first], [&](auto tile) {
        constexpr int TILE = decltype(tile)::value;
        GramJob jobs[kMaxGroup];
        int k = 0;
        for (int i = first; i < count; ++i)
          if (tile_of(n[i], 0) == t)
            jobs[k++] = gram_job<0, TILE>(a[i], a[i], n[i], nr[i], alpha[i], true, part[i], c[i]);
        launch_gram_group<0, TILE>(jobs, k, s);
      });
      break;
    }
}

}  // namespace hfx
