// Dense FP64 linear algebra on CDNA4 matrix cores and the HBM-streaming solve.
//
// The paper obtains the capacitance matrix by inverting the elastance A
// (Sec. II.A, Eq. 3) and projects it onto the charge-neutral subspace (Eq. 4).
// Here A = L L^T by a blocked right-looking Cholesky (64-wide panels: a
// one-workgroup diagonal factorisation, a panel solve and a trailing
// symmetric update as MFMA GEMMs), X = L^-1 by blocked forward substitution,
// and A^-1 = X^T X as a triangular-aware MFMA GEMM.
//
// v_mfma_f64_16x16x4f64 operand layout (lane l of a wave64):
//   A operand: element (row l%16, k l/16); B operand: (k l/16, col l%16);
//   result register r: element (row l/16 + 4 r, col l%16).
#include <algorithm>
#include <cstdlib>

#include "cpm_internal.h"

namespace cpm {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// GEMM: C = beta C + alpha op(A) op(B), T x T tile per workgroup of 4 T threads, K
// in slabs of 16 through two alternating LDS buffers, one barrier per slab, the
// next slab's global loads (of the next tile at a tile's end) in flight.  M and N
// are multiples of 64, K of 16.  The FP64 matrix rate bounds large products: a
// register-only loop reaches 50-57 TFLOP/s with one wave per SIMD and 66-67 with
// two or more.
//
// T = 64, a workgroup (four waves of 32 x 32) per tile: 80 registers and 36 KiB of
// LDS, so that four workgroups share a CU.  Tiles in row-major order, only those
// on and below the diagonal for tri.  K runs in one chain in ascending order, as it
// always has: the same bits, which the split-BF16 copies and refinement residuals
// need.  One LDS buffer and two barriers per slab reached less (before -> now, in
// TFLOP/s, random operands): K = 512, N = 8192 NN 49 -> 60, its lower triangle NT
// 40 -> 53, N = 2432 31 -> 43; X^T X of a lower-triangular X, n = 8192 41 -> 58,
// n = 2944 30 -> 37; N = K = 2944, M = 1024 45 -> 56.  Rank-64 updates are bound by
// the traffic of C and stay: 12224 x 448 x 64 24 us.  128 x 128 tiles, two
// workgroups per CU, gave the same or less for want of tiles (K = 512 lower
// triangle n = 4096 39 against 49), 5 % more only in the largest X^T X.
//
// SPLIT, T = 128 (eight waves of 64 x 32): too few tiles for the chip, so all tiles'
// slabs, in tile order, are cut into GT_RUNS equal runs, one workgroup per CU.  A
// run writes the tiles that it begins; the head of a run that continues a tile goes
// to the work array (128 KiB per run) and k_gemm_f64_join adds it, so that every
// sum has one fixed order.  The kernel has to stay within 128 registers (212
// when 32 store addresses were hoisted: 343 us instead of 291 for M = 1024 below).
// C must not overlap A or B.  Before -> T = 64 -> split, N = K = 2944: M = 64 169 ->
// 140 -> 64 us, M = 256 171 -> 142 -> 102, M = 512 280 -> 220 -> 177.
// ---------------------------------------------------------------------------
// LDS pitch (16 rows of a read on distinct banks); doubles of a split tile; runs
constexpr int GT_P = 18, GT_PART = 128 * 128, GT_LRUNS = 8, GT_RUNS = 1 << GT_LRUNS;

// The tiles in row-major order (tri: those on and below the diagonal); kmode: a
// tile's K begins at its own first row.
struct GtGeom {
  int M, N, K, tri, kmode, tm, tn;
  int total;                                         // slabs of all tiles (split)
  __device__ int kbeg(int bm) const { return kmode ? bm * 64 : 0; }
  int tiles() const { return tri ? tm * tn - tn * (tn - 1) / 2 : tm * tn; }   // (tri: tm >= tn)
  __device__ void tile(int w, int& bm, int& bn) const {
    const int head = tn * (tn - 1) / 2;              // tiles of the rows 0 .. tn - 2
    if (tri && w < head) {                           // row bm holds bm + 1 tiles
      bm = (int)((sqrtf(8.f * w + 1.f) - 1.f) * 0.5f);
      while (bm * (bm + 1) / 2 > w) --bm;
      while ((bm + 1) * (bm + 2) / 2 <= w) ++bm;
      bn = w - bm * (bm + 1) / 2;
    } else {
      const int t = tri ? w - head : w;
      bm = t / tn;
      bn = t - bm * tn;
      if (tri) bm += tn - 1;
    }
  }
  // split: the first slab of run w, and the tile and slab of a position in all slabs
  __device__ int begin(int w) const { return (int)((long)total * w >> GT_LRUNS); }
  __device__ void locate(int it, int& bm, int& bn, int& s) const {
    const int t = it / (K / 16);
    bm = t / tn;
    bn = t - bm * tn;
    s = it - t * (K / 16);
  }
};

template <int T>
struct GtWave {                                      // this thread's part of a tile
  static constexpr int BI = T / 32, BJ = 2;          // MFMA block rows and columns of a wave
  static constexpr int WC = T / 32;                  // waves side by side
  static __device__ int wm() { return (int)(threadIdx.x >> 6) / WC * (16 * BI); }
  static __device__ int wn() { return (int)(threadIdx.x >> 6) % WC * 32; }
  // tile row of register r of block row i and tile column of block column j
  static __device__ int row(int i, int r) { return wm() + 16 * i + (int)((threadIdx.x & 63) >> 4) + 4 * r; }
  static __device__ int col(int j) { return wn() + 16 * j + (int)(threadIdx.x & 15); }
};

// one operand's slabs: a thread moves a row and 4 k (row-major operand) or a k and 4
// rows (k-major one); rows past the operand's last are its last
template <bool KMAJOR>
struct GtLoader {
  const double* p;
  d2v x, y;
  __device__ void start(const double* M, int ld, int row0, int rows, int k) {
    const int tid = threadIdx.x;
    p = KMAJOR ? M + (size_t)(k + (tid & 15)) * ld + min(row0 + (tid >> 4) * 4, rows - 4)
               : M + (size_t)min(row0 + (tid >> 2), rows - 1) * ld + k + (tid & 3) * 4;
  }
  __device__ void next(int ld) { p += KMAJOR ? (size_t)16 * ld : 16; }
  __device__ void load() {
    const d2v* q = reinterpret_cast<const d2v*>(p);
    x = q[0];
    y = q[1];
  }
  __device__ void store(double (*s)[GT_P]) const {
    const int tid = threadIdx.x;
    if (KMAJOR) {
      const int kk = tid & 15, r = (tid >> 4) * 4;
      s[r][kk] = x.x; s[r + 1][kk] = x.y;
      s[r + 2][kk] = y.x; s[r + 3][kk] = y.y;
    } else {
      double* d = &s[tid >> 2][(tid & 3) * 4];
      *reinterpret_cast<d2v*>(d) = x;
      *reinterpret_cast<d2v*>(d + 2) = y;
    }
  }
};

// acc += one slab's product
template <int T>
__device__ inline void gt_slab(const double (*sA)[GT_P], const double (*sB)[GT_P],
                               v4d (&acc)[GtWave<T>::BI][GtWave<T>::BJ]) {
  using W = GtWave<T>;
  const int l15 = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4, wm = W::wm(), wn = W::wn();
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    double a[W::BI], b[W::BJ];
#pragma unroll
    for (int i = 0; i < W::BI; ++i) a[i] = sA[wm + 16 * i + l15][4 * h + lg];
#pragma unroll
    for (int j = 0; j < W::BJ; ++j) b[j] = sB[wn + 16 * j + l15][4 * h + lg];
#pragma unroll
    for (int i = 0; i < W::BI; ++i)
#pragma unroll
      for (int j = 0; j < W::BJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
  }
}

constexpr int GT_LDS64 = 2 * 2 * 64 * GT_P;          // doubles of LDS of a 64-tile

// one 64 x 64 tile by 256 threads: C = beta C + alpha A B over slabs of 16 k; A, B
// and C at the tile's first row, column and k; rowmap: C's rows (-1: none)
template <bool TA, bool TB>
__device__ __forceinline__ void gemm_tile64(double* lds, const double* A, int lda, const double* B, int ldb,
                                   int K, double alpha, double beta, double* C, int ldc,
                                   const int* rowmap) {
  using W = GtWave<64>;
  auto sA = reinterpret_cast<double (*)[64][GT_P]>(lds);
  auto sB = sA + 2;
  GtLoader<TA> la;
  GtLoader<!TB> lb;
  la.start(A, lda, 0, 64, 0);
  lb.start(B, ldb, 0, 64, 0);
  la.load();
  lb.load();
  la.store(sA[0]);
  lb.store(sB[0]);
  __syncthreads();
  v4d acc[W::BI][W::BJ];
#pragma unroll
  for (int i = 0; i < W::BI; ++i)
#pragma unroll
    for (int j = 0; j < W::BJ; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};
  int buf = 0;
  for (int k = 0; k < K; k += 16) {
    if (k + 16 < K) {                                // (the last slab loads itself again)
      la.next(lda);
      lb.next(ldb);
    }
    la.load();
    lb.load();
    gt_slab<64>(sA[buf], sB[buf], acc);
    la.store(sA[buf ^ 1]);
    lb.store(sB[buf ^ 1]);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int i = 0; i < W::BI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int row = W::row(i, r);
      if (rowmap) {                                  // scattered output rows (-1: skip)
        row = rowmap[row];
        if (row < 0) continue;
      }
#pragma unroll
      for (int j = 0; j < W::BJ; ++j) {
        double* cp = C + (size_t)row * ldc + W::col(j);
        const double v = alpha * acc[i][j][r];
        *cp = (beta != 0.0) ? v + beta * (*cp) : v;
      }
    }
}

template <bool TA, bool TB>
__global__ void __launch_bounds__(256, 4) k_gemm_f64(GtGeom g, double alpha,
                                                     const double* __restrict__ A, int lda,
                                                     const double* __restrict__ B, int ldb,
                                                     double beta, double* C, int ldc) {
  __shared__ __align__(16) double lds[GT_LDS64];
  int bm, bn;
  g.tile(blockIdx.x, bm, bn);
  const size_t m0 = 64 * bm, n0 = 64 * bn, k0 = g.kbeg(bm);
  gemm_tile64<TA, TB>(lds, TA ? A + k0 * lda + m0 : A + m0 * lda + k0, lda,
                      TB ? B + n0 * ldb + k0 : B + k0 * ldb + n0, ldb, g.K - (int)k0, alpha, beta,
                      C + m0 * ldc + n0, ldc, nullptr);
}

__global__ void __launch_bounds__(512, 4) k_gemm_f64_split(GtGeom g, double alpha,
                                                           const double* __restrict__ A, int lda,
                                                           const double* __restrict__ B, int ldb,
                                                           double beta, double* C, int ldc,
                                                           double* __restrict__ part) {
  using W = GtWave<128>;
  __shared__ __align__(16) double sA[2][128][GT_P];
  __shared__ __align__(16) double sB[2][128][GT_P];
  // workgroups of one XCD (every eighth) take neighbouring runs
  const int w = (int)(blockIdx.x & 7) * (GT_RUNS / 8) + (int)(blockIdx.x >> 3), end = g.begin(w + 1);
  int it = g.begin(w), bm, bn, s0, buf = 0;
  if (it >= end) return;
  g.locate(it, bm, bn, s0);
  GtLoader<false> la;
  GtLoader<true> lb;
  la.start(A, lda, bm * 128, g.M, 16 * s0);
  lb.start(B, ldb, bn * 128, g.N, 16 * s0);
  la.load();
  lb.load();
  la.store(sA[0]);
  lb.store(sB[0]);
  __syncthreads();
  while (it < end) {
    const int ns = min(g.K / 16 - s0, end - it);
    const int nn = bn + 1 < g.tn ? bn + 1 : 0, nm = nn ? bm : bm + 1;   // the next tile
    it += ns;
    v4d acc[W::BI][W::BJ];
#pragma unroll
    for (int i = 0; i < W::BI; ++i)
#pragma unroll
      for (int j = 0; j < W::BJ; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < ns; ++s) {
      if (s + 1 < ns) {
        la.next(lda);
        lb.next(ldb);
      } else if (it < end) {
        la.start(A, lda, nm * 128, g.M, 0);
        lb.start(B, ldb, nn * 128, g.N, 0);
      }
      la.load();                                     // (a run's last slab loads itself again)
      lb.load();
      gt_slab<128>(sA[buf], sB[buf], acc);
      la.store(sA[buf ^ 1]);
      lb.store(sB[buf ^ 1]);
      __syncthreads();
      buf ^= 1;
    }
    if (s0 == 0) {
#pragma unroll
      for (int i = 0; i < W::BI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = bm * 128 + W::row(i, r);
          if (row >= g.M) continue;
#pragma unroll
          for (int j = 0; j < W::BJ; ++j) {
            const int col = bn * 128 + W::col(j);
            if (col >= g.N) continue;
            double* cp = C + (size_t)row * ldc + col;
            const double v = alpha * acc[i][j][r];
            *cp = (beta != 0.0) ? v + beta * (*cp) : v;
          }
        }
    } else {                                         // at most the run's first tile
      unsigned o = w * GT_PART + threadIdx.x;
      asm("" : "+v"(o));                             // (keeps 32 addresses out of the slab loop)
#pragma unroll
      for (int i = 0; i < W::BI; ++i)
#pragma unroll
        for (int j = 0; j < W::BJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) part[o + ((i * 2 + j) * 4 + r) * 512] = acc[i][j][r];
    }
    s0 = 0;
    bm = nm;
    bn = nn;
  }
}

// C += alpha (the later K parts of a tile, in order of k); blockIdx.x = the run
// that holds the tile's second part, blockIdx.y = MFMA block row
__global__ void __launch_bounds__(512) k_gemm_f64_join(GtGeom g, double alpha, double* C, int ldc,
                                                       const double* __restrict__ part) {
  using W = GtWave<128>;
  const int w = blockIdx.x + 1, i = blockIdx.y;
  const int it = g.begin(w);
  if (it >= g.total) return;
  int bm, bn, s;
  g.locate(it, bm, bn, s);
  if (s == 0 || g.begin(w - 1) > it - s) return;     // a tile's start, or a third part
  const int tend = it - s + g.K / 16;
  v4d acc[2] = {(v4d){0.0, 0.0, 0.0, 0.0}, (v4d){0.0, 0.0, 0.0, 0.0}};
  for (int v = w; v < GT_RUNS && g.begin(v) < tend; ++v) {
    if (g.begin(v) == g.begin(v + 1)) continue;
    const double* pv = part + (size_t)v * GT_PART + threadIdx.x;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[j][r] += pv[((i * 2 + j) * 4 + r) * 512];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = bm * 128 + W::row(i, r);
    if (row >= g.M) continue;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = bn * 128 + W::col(j);
      if (col < g.N) C[(size_t)row * ldc + col] += alpha * acc[j][r];
    }
  }
}

// The planes' products of the assembly of A in one launch (their rows follow one
// another in the atom map): a plane alone fills the chip only in large cells.  2880
// atoms, six planes of 480 to 512 rows, K = 672: six launches 308 us,
// one 154.
__global__ void __launch_bounds__(256, 4) k_gemm_planes(AsmPlanes pl, int tn, double alpha, double beta,
                                                        const double* __restrict__ G, int ldG,
                                                        const double* __restrict__ F, double* A,
                                                        int npad, const int* __restrict__ amap) {
  __shared__ __align__(16) double lds[GT_LDS64];
  const int bm = blockIdx.x / tn, bn = blockIdx.x % tn;
  int p = 0;
  while (bm >= pl.tile_end[p]) ++p;
  if (64 * bn >= pl.ncols[p]) return;
  // (beta an argument: a constant 1 would contract alpha acc + A into one rounding)
  gemm_tile64<false, false>(lds, G + (size_t)64 * bm * ldG, ldG, F + (size_t)p * ldG * npad + 64 * bn,
                            npad, ldG, alpha, beta, A + 64 * bn, npad, amap + 64 * bm);
}

void launch_gemm_planes(hipStream_t st, const AsmPlanes& pl, int n, double alpha, const double* G,
                        int ldG, const double* F, double* A, int npad, const int* amap) {
  int tn = 0;
  for (int p = 0; p < n; ++p) tn = std::max(tn, pl.ncols[p] / 64);
  if (n > 0 && pl.tile_end[n - 1] > 0 && tn > 0)
    hipLaunchKernelGGL(k_gemm_planes, dim3(pl.tile_end[n - 1] * tn), dim3(256), 0, st, pl, tn, alpha,
                       1.0, G, ldG, F, A, npad, amap);
}

// Split up to two 64-tiles per CU, where unsplit workgroups have a CU to themselves
// or share it unevenly: N = K = 2944 with M = 512 (368 tiles) 220 -> 177 us, M = 1024
// (736 tiles) 316 -> 305, not worth twice the work array.  Short products do not
// repay the partial tiles and the second launch: 256 x 1024 x 1024 (1024 slabs of
// 128-tiles) 48 -> 38 us, 2048 x 576 x 576 50 -> 52, 256 x 576 x 576 29 -> 40.
size_t gemm_f64_work(int M, int N, int K) {
  const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
  const bool split = K >= 1024 && (long)(M / 64) * (N / 64) <= 512 && tiles * (K / 16) >= 1024;
  return split ? (size_t)GT_PART * GT_RUNS : 0;
}

size_t gemm_f64_most_work(int N, int K) {
  size_t most = 0;
  for (int M = 64; (long)(M / 64) * (N / 64) <= 512; M += 64) most = std::max(most, gemm_f64_work(M, N, K));
  return most;
}

void launch_gemm_f64(hipStream_t st, bool transA, bool transB, int M, int N, int K, double alpha,
                     const double* A, int lda, const double* B, int ldb, double beta, double* C,
                     int ldc, int tri, int kmode, GemmWork work) {
  if (M <= 0 || N <= 0) return;
  const size_t need = gemm_f64_work(M, N, K);
  if (need > 0 && work.len >= need && !transA && !transB && !tri && !kmode) {
    const GtGeom g{M, N, K, 0, 0, (M + 127) / 128, (N + 127) / 128,
                   ((M + 127) / 128) * ((N + 127) / 128) * (K / 16)};
    hipLaunchKernelGGL(k_gemm_f64_split, dim3(GT_RUNS), dim3(512), 0, st, g, alpha, A, lda, B, ldb,
                       beta, C, ldc, work.p);
    hipLaunchKernelGGL(k_gemm_f64_join, dim3(GT_RUNS - 1, 4), dim3(512), 0, st, g, alpha, C, ldc,
                       work.p);
    return;
  }
  const GtGeom g{M, N, K, tri, kmode, M / 64, N / 64, 0};
#define CPM_GT(TA, TB)                                                                              \
  hipLaunchKernelGGL((k_gemm_f64<TA, TB>), dim3(g.tiles()), dim3(256), 0, st, g, alpha, A, lda, B,  \
                     ldb, beta, C, ldc)
  if (transA) {
    if (transB) CPM_GT(true, true); else CPM_GT(true, false);
  } else {
    if (transB) CPM_GT(false, true); else CPM_GT(false, false);
  }
#undef CPM_GT
}

// ---------------------------------------------------------------------------
// Diagonal 64x64 block of the Cholesky factorisation and the inverse of its
// factor, in one workgroup, in four panels of 16 columns.  The chain of 64 roots and
// reciprocals bounds it, so wave 0 factors a panel alone in registers, a lane per
// row of the block and every row at once: a step reads the pivot and the column's
// entries in the panel from their lanes, and its updates fill the latency of the
// next step's root.  The columns right of the panel follow by MFMA, 16 x 16 blocks
// over the waves.  The other waves meanwhile form the inverse, as far as panels are
// complete: the diagonal 16 x 16 blocks by forward substitution, then block column
// k by one wave, X_ik = -X_ii sum_{j=k}^{i-1} L_ij X_jk by MFMA.  Every element is
// one chain of FMAs in ascending order of the summed index, which FP64 MFMA keeps.
// A pivot <= 0 (or NaN) records 1 + its global index in *flag (first one wins) and
// continues with 1.
// 34.5 us in one workgroup of 16 waves with the root and a division in the chain and
// the inverse afterwards; alone now 12.4: 1.0 us loads, 2.0 per panel (330 clocks per column
// before the LDS reads of its entries were moved behind the next root, 290 after),
// 0.3-0.6 for the columns right of it, 1.8 for what of the inverse needs the last
// panel.
// ---------------------------------------------------------------------------
// lane l's value of v, in every lane (l uniform)
__device__ inline double readlane_f64(double v, int l) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(x >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// d = sqrt(x) and 1 / d, both correctly rounded, for x well inside the FP64 range
// unless d is all ones: Goldschmidt's iteration for the root and half its reciprocal
// together, then each one's residual by FMA (Markstein).  Eight operations in a
// chain instead of about 30 of sqrt(x) and a division, with equal results.
__device__ inline void root_and_reciprocal(double x, double& d, double& rd) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  r = fma(-h, g, 0.5);
  d = fma(fma(-g, g, x), h, g);
  h = fma(h, r, h);
  h += h;
  rd = fma(fma(-d, h, 1.0), h, h);
}

// panel p0 of the block in LDS, by one wave; FAST: by root_and_reciprocal; false if
// that is not exact for a pivot (the block is as before then, bc and rd are not)
template <bool FAST>
__device__ __forceinline__ bool potrf_panel(double (*a)[65], double* bc, double* rd, int p0, int lane, int* flag,
                                   int k0) {
  double v[16], lc[16], dl = 1.0;          // lc: column j's entries in the panel
#pragma unroll
  for (int t = 0; t < 16; ++t) v[t] = a[lane][p0 + t];
  double piv = readlane_f64(v[0], p0), d, rdj;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if (FAST) {
      root_and_reciprocal(piv, d, rdj);
    } else {
      if (!(piv > 0.0)) {
        if (lane == 0) atomicCAS(flag, 0, k0 + p0 + j + 1);
        piv = 1.0;
      }
      d = sqrt(piv);
      rdj = 1.0 / d;
    }
    // the previous column's updates past the next one: its entries come by LDS,
    // whose latency the root covers
#pragma unroll
    for (int c = j + 1; c < 16; ++c)
      if (j > 0) v[c] -= v[j - 1] * lc[c];
    __builtin_amdgcn_sched_barrier(0);
    v[j] *= rdj;                           // column j of L below the diagonal
    if (j < 15) {
      // (the next pivot's lane multiplies its own entry, ahead of the others)
      piv = readlane_f64(v[j + 1] - v[j] * v[j], p0 + j + 1);
      bc[lane] = v[j];
#pragma unroll
      for (int c = j + 2; c < 16; ++c) lc[c] = bc[p0 + c];
      v[j + 1] -= v[j] * readlane_f64(v[j], p0 + j + 1);
    }
    if (lane == p0 + j) dl = d;
    rd[p0 + j] = rdj;                      // (every lane the same)
    __builtin_amdgcn_sched_barrier(0);
  }
  if (FAST && __any(!(dl > 0x1p-200 && dl < 0x1p200) || (__double_as_longlong(dl) << 12 | 0xfff) == -1))
    return false;
  if (lane >= p0) {
#pragma unroll
    for (int t = 0; t < 16; ++t) a[lane][p0 + t] = v[t];
    if (lane < p0 + 16) a[lane][lane] = dl;
  }
  return true;
}

// X = the inverse of L's diagonal block at p0 by forward substitution, a lane per
// column (one wave); entries above the diagonal come out as zero
__device__ __forceinline__ void invert16(const double (*a)[65], const double* rd, int p0, int lane,
                                double* X) {
  if (lane < 16) {
    double s[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = r == lane ? 1.0 : 0.0;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      s[t] *= rd[p0 + t];
#pragma unroll
      for (int r = t + 1; r < 16; ++r) s[r] -= a[p0 + r][p0 + t] * s[t];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) X[r * 65 + lane] = s[r];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// acc + L x: L 16 x 16 in LDS (pitch 65), x and acc in MFMA registers (register h of
// a result is the right operand of the next product's k = 4 h .. 4 h + 3)
__device__ inline v4d mul16(const double* L, v4d x, v4d acc, int lane) {
#pragma unroll
  for (int h = 0; h < 4; ++h)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(L[(lane & 15) * 65 + 4 * h + (lane >> 4)], x[h], acc, 0,
                                               0, 0);
  return acc;
}

// the block and its inverse by 256 threads; lds: PF_LDS doubles
constexpr int PF_LDS = 64 * 65 + 64 + 64;

__device__ __forceinline__ void potrf64(double* lds, double* Lblk, int ld, double* Dinv, int* flag, int k0) {
  auto a = reinterpret_cast<double (*)[65]>(lds);   // working lower triangle, becomes L
  double* bc = lds + 64 * 65;                       // a column of L (16-byte aligned)
  double* rd = bc + 64;                             // 1 / L[j][j]
  // the inverses of L's diagonal 16 x 16 blocks, above the block diagonal of a
  auto Xd = [&](int p) { return p < 3 ? &a[0][16 * p + 16] : &a[16][48]; };
  const int wave = threadIdx.x >> 6, k = wave - 1;
  int lane = threadIdx.x & 63, l15 = lane & 15, lg = lane >> 4;
  {
    double t[16];                   // all loads in flight at once
#pragma unroll
    for (int u = 0; u < 16; ++u) t[u] = Lblk[(size_t)(wave + 4 * u) * ld + lane];
#pragma unroll
    for (int u = 0; u < 16; ++u) a[wave + 4 * u][lane] = t[u];
  }
  __syncthreads();
  const v4d zero = (v4d){0.0, 0.0, 0.0, 0.0};
  v4d t0 = zero, t1 = zero, t2 = zero, t3 = zero;      // sum_j L_ij X_jk of rows i = p - 1 ..
  auto put = [&](int i, int kk, v4d y) {
#pragma unroll
    for (int r = 0; r < 4; ++r) Dinv[(16 * i + lg + 4 * r) * 64 + 16 * kk + l15] = y[r];
  };
  auto put_L = [&](int p) {                            // L's columns of panel p
    for (int r = 4 * k + lg; r < 64; r += 12)
      Lblk[(size_t)r * ld + 16 * p + l15] = 16 * p + l15 <= r ? a[r][16 * p + l15] : 0.0;
  };
  auto diag = [&](int p) {
    v4d y;
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = Xd(p)[(lg + 4 * r) * 65 + l15];
    return y;
  };
#pragma unroll 1
  for (int p = 0; p < 4; ++p) {
    const int p0 = 16 * p;
    asm("" : "+v"(lane));           // (keeps what follows from it out of registers between panels)
    l15 = lane & 15;
    lg = lane >> 4;
    if (wave == 0) {
      if (!potrf_panel<true>(a, bc, rd, p0, lane, flag, k0))
        potrf_panel<false>(a, bc, rd, p0, lane, flag, k0);
    } else if (p > 0) {
      // meanwhile: block row p - 1 of the inverse, by each wave its column k, from
      // the same inverse of the diagonal block
      invert16(a, rd, p0 - 16, lane, Xd(p - 1));
      if (k <= p - 1) {
        const v4d y = k == p - 1 ? diag(p - 1) : -mul16(Xd(p - 1), t0, zero, lane);
        t0 = mul16(&a[p0][p0 - 16], y, t1, lane);
        if (p < 3) t1 = mul16(&a[p0 + 16][p0 - 16], y, t2, lane);
        if (p < 2) t2 = mul16(&a[p0 + 32][p0 - 16], y, t3, lane);
        put(p - 1, k, y);
      } else {
        put(p - 1, k, zero);
      }
      put_L(p - 1);
    }
    __syncthreads();
    // blocks (I, J) right of the panel, row by row of the triangle
    const int nb = 3 - p;
    for (int e = wave; e < nb * (nb + 1) / 2; e += 4) {
      const int i = e < 1 ? 0 : e < 3 ? 1 : 2, j = e - i * (i + 1) / 2;
      const int I = p0 + 16 * (i + 1), J = p0 + 16 * (j + 1);
      v4d acc;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = a[I + lg + 4 * r][J + l15];
#pragma unroll
      for (int h = 0; h < 4; ++h)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[I + l15][p0 + 4 * h + lg],
                                                   a[J + l15][p0 + 4 * h + lg], acc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) a[I + lg + 4 * r][J + l15] = acc[r];
    }
    if (p < 3) __syncthreads();
  }
  if (wave > 0) put_L(3);
  invert16(a, rd, 48, lane, Xd(3));                    // (each wave the same values)
  if (wave > 0) {
    put(3, k, -mul16(Xd(3), t0, zero, lane));
  } else {
    put(3, 3, diag(3));
    for (int i = 0; i < 3; ++i) put(i, 3, zero);
  }
}

static_assert(PF_LDS <= GT_LDS64, "the block factors in the GEMM's LDS");

__global__ void __launch_bounds__(256) k_potrf_diag(double* Lblk, int ld, double* Dinv, int* flag,
                                                    int k0) {
  __shared__ __align__(16) double lds[PF_LDS];
  potrf64(lds, Lblk, ld, Dinv, flag, k0);
}

void launch_potrf_diag(hipStream_t st, double* Lblk, int ld, double* Dinv, int* flag, int k0) {
  hipLaunchKernelGGL(k_potrf_diag, dim3(1), dim3(256), 0, st, Lblk, ld, Dinv, flag, k0);
}

// ---------------------------------------------------------------------------
// The steps of the factorisation A = L L^T and, in the same launches, of X = L^-1 by
// forward substitution (X null: the factor alone).  A panel is 64 columns; r = the
// first row below it.
//   solve:  L_below <- L_below L_kk^-T, X_k <- L_kk^-1 X_k (columns that can be
//           non-zero), in place, a tile per workgroup.
//   update: L's tiles right of column c0 + K -= L L^T, rows of X below -= L X_c0.., by
//           the K columns from c0 on; the workgroup of the first tile, the next
//           diagonal block, then factors it while the others go on.
// Launches follow one another through the chain of diagonal blocks, so what is merged
// is hidden behind it: a panel at 2880 atoms took 51 us (block 12.4, solve and update
// of L 7.5 + 12, of X 7.2 + 12.5) and takes 30 (6.2 + 24, of which the first tile and
// its factor are the longest part).  The block factors in the GEMM's LDS and 128
// registers, so that four workgroups still share a CU in the large updates.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256, 4) k_chol_solve(double* L, double* X, const double* Dinv,
                                                       int ld, int k0, int nL) {
  __shared__ __align__(16) double lds[GT_LDS64];
  const int b = blockIdx.x;
  if (b < nL) {
    double* C = L + (size_t)(k0 + 64 + 64 * b) * ld + k0;
    gemm_tile64<false, true>(lds, C, ld, Dinv, 64, 64, 1.0, 0.0, C, ld, nullptr);
  } else {
    double* C = X + (size_t)k0 * ld + 64 * (b - nL);
    gemm_tile64<false, false>(lds, Dinv, 64, C, ld, 64, 1.0, 0.0, C, ld, nullptr);
  }
}

__global__ void __launch_bounds__(256, 4) k_chol_update(GtGeom g, double* L, double* X, double* Dinv,
                                                        int* flag, int ld, int c0, int ncX) {
  __shared__ __align__(16) double lds[GT_LDS64];
  const int nL = g.tm * g.tn - g.tn * (g.tn - 1) / 2, b = blockIdx.x, r0 = c0 + g.K;
  if (b < nL) {
    int bm, bn;
    g.tile(b, bm, bn);
    const size_t m = r0 + 64 * bm, n = r0 + 64 * bn;
    gemm_tile64<false, true>(lds, L + m * ld + c0, ld, L + n * ld + c0, ld, g.K, -1.0, 1.0,
                             L + m * ld + n, ld, nullptr);
    if (b == 0) {
      __syncthreads();
      potrf64(lds, L + m * ld + n, ld, Dinv, flag, r0);
    }
  } else {
    const size_t m = r0 + 64 * ((b - nL) / ncX), n = 64 * ((b - nL) % ncX);
    gemm_tile64<false, false>(lds, L + m * ld + c0, ld, X + (size_t)c0 * ld + n, ld, g.K, -1.0, 1.0,
                              X + m * ld + n, ld, nullptr);
  }
}

void launch_chol_solve(hipStream_t st, int npad, double* L, double* X, const double* Dinv, int k0) {
  const int nL = (npad - k0) / 64 - 1, nX = X ? k0 / 64 + 1 : 0;
  if (nL + nX > 0)
    hipLaunchKernelGGL(k_chol_solve, dim3(nL + nX), dim3(256), 0, st, L, X, Dinv, npad, k0, nL);
}

void launch_chol_update(hipStream_t st, int npad, double* L, double* X, double* Dinv, int* flag,
                        int c0, int K, int cols, int rowsX, int colsX) {
  const int r0 = c0 + K, tm = (npad - r0) / 64, tn = cols / 64;
  const GtGeom g{npad - r0, cols, K, 1, 0, tm, tn, 0};
  const int nX = X ? rowsX / 64 * (colsX / 64) : 0;
  hipLaunchKernelGGL(k_chol_update, dim3(g.tiles() + nX), dim3(256), 0, st, g, L, X, Dinv, flag, npad,
                     c0, colsX / 64);
}

__global__ void k_set_identity(int npad, double* X) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)npad * npad) return;
  const int i = (int)(e / npad), j = (int)(e % npad);
  X[e] = (i == j) ? 1.0 : 0.0;
}

void launch_set_identity(hipStream_t st, int npad, double* X) {
  const size_t tot = (size_t)npad * npad;
  hipLaunchKernelGGL(k_set_identity, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, npad,
                     X);
}

// ---------------------------------------------------------------------------
// wave64 helpers
// ---------------------------------------------------------------------------
__device__ inline double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// block-wide sum of 256 threads in a fixed order; result valid in every thread
__device__ inline double block_sum256(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  const double t = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  __syncthreads();
  return t;
}

// sum over a 1024-thread workgroup: wave sums, then the 16 in wave order
__device__ inline double block_sum1024(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) t += sh[w];
  __syncthreads();
  return t;
}

// out[i] = sum_{j<n} M[i][j] for i < n (one wave per row, fixed order)
__global__ void k_row_sums(int n, int npad, const double* __restrict__ M, double* out) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n) return;
  double s = 0.0;
  for (int j = lane; j < n; j += 64) s += M[(size_t)row * npad + j];
  s = wave_sum(s);
  if (lane == 0) out[row] = s;
}

void launch_row_sums(hipStream_t st, int n, int npad, const double* M, double* out) {
  hipLaunchKernelGGL(k_row_sums, dim3((n + 3) / 4), dim3(256), 0, st, n, npad, M, out);
}

__global__ void k_sum_vector(int n, const double* __restrict__ v, double* out) {
  __shared__ double sh[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += v[i];
  s = block_sum256(s, sh);
  if (threadIdx.x == 0) *out = s;
}

void launch_sum_vector(hipStream_t st, int n, const double* v, double* out) {
  hipLaunchKernelGGL(k_sum_vector, dim3(1), dim3(256), 0, st, n, v, out);
}

// S = A^-1 - u u^T / s on the n x n block (Eq. 4); zero in the padding.
__global__ void k_make_S(int n, int npad, const double* __restrict__ Ainv,
                         const double* __restrict__ u, const double* __restrict__ s_dev,
                         double* __restrict__ S) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)npad * npad) return;
  const int i = (int)(e / npad), j = (int)(e % npad);
  double v = 0.0;
  if (i < n && j < n) v = Ainv[e] - u[i] * u[j] / (*s_dev);
  S[e] = v;
}

void launch_make_S(hipStream_t st, int n, int npad, const double* Ainv, const double* u,
                   const double* s_dev, double* S) {
  const size_t tot = (size_t)npad * npad;
  hipLaunchKernelGGL(k_make_S, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, npad,
                     Ainv, u, s_dev, S);
}

// round-to-nearest-even FP32 -> BF16
__device__ inline uint16_t f32_to_bf16(float f) {
  uint32_t x = __float_as_uint(f);
  if ((x & 0x7f800000u) == 0x7f800000u) return (uint16_t)(x >> 16);
  x += 0x7fffu + ((x >> 16) & 1u);
  return (uint16_t)(x >> 16);
}

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// FP32 copy and split-BF16 pair of S (hi = bf16(S), lo = bf16(S - hi)).
__global__ void k_convert_S(size_t tot, const double* __restrict__ S, float* S32, uint16_t* hi,
                            uint16_t* lo) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= tot) return;
  const double v = S[e];
  if (S32) S32[e] = (float)v;
  if (hi) {
    const uint16_t h = f32_to_bf16((float)v);
    hi[e] = h;
    lo[e] = f32_to_bf16((float)(v - (double)bf16_to_f32(h)));
  }
}

// x ~ hi + lo: hi = bf16(x), lo = bf16(x - hi) through FP32, as for S
__global__ void k_split_bf16(size_t count, const double* __restrict__ x, uint16_t* __restrict__ hi,
                             uint16_t* __restrict__ lo) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count) return;
  const float f = (float)x[e];
  const uint16_t h = f32_to_bf16(f);
  hi[e] = h;
  lo[e] = f32_to_bf16(f - bf16_to_f32(h));
}

void launch_split_bf16(hipStream_t st, size_t count, const double* x, uint16_t* hi, uint16_t* lo) {
  hipLaunchKernelGGL(k_split_bf16, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, count,
                     x, hi, lo);
}

void launch_convert_S(hipStream_t st, int npad, const double* S, float* S32, uint16_t* hi,
                      uint16_t* lo) {
  const size_t tot = (size_t)npad * npad;
  hipLaunchKernelGGL(k_convert_S, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, tot, S,
                     S32, hi, lo);
}

// ---------------------------------------------------------------------------
// Matrix-vector product y[b] = sign * M x[b] + addscale * add, streaming the
// npad x npad matrix M (FP64 or FP32) once per vector.  x is FP64, npad
// apart per vector and zero beyond n, so every load is an aligned 16-byte
// vector with no bounds test.  One wave per R consecutive rows: 16-byte
// coalesced loads of each row, every x element read once per wave (through
// the cache) for all R rows, FP64 accumulation, wave reductions in a fixed
// order.  Matrices larger than the last-level cache are read with
// nontemporal loads (streamed past the caches, which the x vector keeps).
// ---------------------------------------------------------------------------
typedef float f4v __attribute__((ext_vector_type(4)));

template <typename TM, int R, bool NT>
__global__ void __launch_bounds__(256) k_matvec(int npad, const TM* __restrict__ M,
                                                const double* __restrict__ x,
                                                const double* __restrict__ add, int add_ld,
                                                double addscale, double* __restrict__ y, int ldy,
                                                int negate) {
  const int lane = threadIdx.x & 63;
  const int row0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * R;   // R consecutive rows per wave
  const int b = blockIdx.y;
  if (row0 >= npad) return;                  // npad is a multiple of 64, so all R rows exist
  constexpr int VEC = 16 / sizeof(TM);
  const TM* mrow = M + (size_t)row0 * npad;
  const double* xb = x + (size_t)b * npad;
  double acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0;
#pragma unroll 2
  for (int j0 = lane * VEC; j0 < npad; j0 += 64 * VEC) {
    // the R row segments first (R x 16 B in flight per lane), then x once for all rows
    TM mv[R][VEC];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const TM* src = mrow + (size_t)r * npad + j0;
      if constexpr (VEC == 2) {
        const d2v t = NT ? __builtin_nontemporal_load(reinterpret_cast<const d2v*>(src))
                         : *reinterpret_cast<const d2v*>(src);
        mv[r][0] = t.x; mv[r][1] = t.y;
      } else {
        const f4v t = NT ? __builtin_nontemporal_load(reinterpret_cast<const f4v*>(src))
                         : *reinterpret_cast<const f4v*>(src);
        mv[r][0] = t.x; mv[r][1] = t.y; mv[r][2] = t.z; mv[r][3] = t.w;
      }
    }
    double xj[VEC];
#pragma unroll
    for (int t = 0; t < VEC; t += 2) {
      const d2v v = *reinterpret_cast<const d2v*>(xb + j0 + t);
      xj[t] = v.x; xj[t + 1] = v.y;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < VEC; ++t) acc[r] += (double)mv[r][t] * xj[t];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = wave_sum(acc[r]);
  if (lane < R) {
    double s = acc[0];
#pragma unroll
    for (int r = 1; r < R; ++r)
      if (lane == r) s = acc[r];
    const int row = row0 + lane;
    double v = negate ? -s : s;
    if (add) v += addscale * add[(size_t)b * add_ld + row];
    y[(size_t)b * ldy + row] = v;
  }
}

template <typename TM>
void launch_matvec_t(hipStream_t st, int npad, const TM* M, int batch, const double* x,
                     const double* add, int add_ld, double addscale, double* y, int ldy,
                     int negate) {
  // rows per wave: 4 rows share each x load from npad = 2048 on (measured
  // best both where S stays in the last-level cache, n ~ 3k, and where it
  // streams from HBM, n ~ 20k); nontemporal loads from 128 MiB of matrix on
  // (20096^2: FP32 84%, FP64 87% of the HBM peak against 75%, 78% with
  // ordinary loads; a matrix that fits the 256 MB cache loses by them)
  int R = npad >= 2048 ? 4 : npad >= 1024 ? 2 : 1;
  bool nt = (double)npad * npad * sizeof(TM) >= 128.0 * 1024 * 1024;
  if (const char* ev = std::getenv("CPM_MV_ROWS")) {
    const int r = std::atoi(ev);
    if (r == 1 || r == 2 || r == 4 || r == 8) R = r;
  }
  if (const char* ev = std::getenv("CPM_MV_NT")) nt = std::atoi(ev) != 0;
  dim3 grid((npad / R + 3) / 4, batch), block(256);
#define CPM_MV(RR, NN)                                                                     \
  hipLaunchKernelGGL((k_matvec<TM, RR, NN>), grid, block, 0, st, npad, M, x, add, add_ld,  \
                     addscale, y, ldy, negate)
  if (nt) {
    if (R == 8) CPM_MV(8, true); else if (R == 4) CPM_MV(4, true);
    else if (R == 2) CPM_MV(2, true); else CPM_MV(1, true);
  } else {
    if (R == 8) CPM_MV(8, false); else if (R == 4) CPM_MV(4, false);
    else if (R == 2) CPM_MV(2, false); else CPM_MV(1, false);
  }
#undef CPM_MV
}

// One matrix-vector product per right-hand side: y = M x (+ add), M npad x
// npad row-major (FP64 or FP32), x FP64 padded (npad apart, zero beyond n),
// streamed once per vector with 16-byte coalesced loads; R rows per wave
// share each x load; fixed-order wave reductions.
void launch_matvec(hipStream_t st, int which, int npad, const void* M, int batch, const double* x,
                   const double* add, int add_ld, double addscale, double* y, int ldy, int negate) {
  if (which == 0)
    launch_matvec_t(st, npad, (const double*)M, batch, x, add, add_ld, addscale, y, ldy, negate);
  else
    launch_matvec_t(st, npad, (const float*)M, batch, x, add, add_ld, addscale, y, ldy, negate);
}

// dst[b] (npad apart, FP64) = src[b] (ldx apart, FP64 or FP32) minus its mean
// over i < n when `center` (the same fixed-order sum as k_row_means), zero
// for n <= i < npad: the padded right-hand side of the streaming solve.
// Grid (batch, parts): every workgroup of a vector forms the same mean (the
// same order; four loads per thread in flight) and writes its own part, so a
// single vector is not left to one workgroup.
template <typename TX>
__global__ void __launch_bounds__(1024) k_center_pad(int n, int npad, const TX* __restrict__ x,
                                                     int ldx, int center,
                                                     double* __restrict__ dst) {
  __shared__ double sh[16];
  const TX* xb = x + (size_t)blockIdx.x * ldx;
  double mean = 0.0;
  if (center) {
    double s = 0.0;
    for (int i0 = threadIdx.x; i0 < n; i0 += 4096) {
      double v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (double)xb[min(i0 + 1024 * j, n - 1)];
#pragma unroll
      for (int j = 0; j < 4; ++j) s += i0 + 1024 * j < n ? v[j] : 0.0;
    }
    mean = block_sum1024(s, sh) / n;
  }
  double* out = dst + (size_t)blockIdx.x * npad;
  for (int i = blockIdx.y * 1024 + threadIdx.x; i < npad; i += 1024 * gridDim.y)
    out[i] = i < n ? (double)xb[i] - mean : 0.0;
}

// workgroups per vector of the two per-vector passes: all of the vector's
// 1024-element parts for small batches, one otherwise
static int vector_parts(int batch, int len) {
  return batch < 16 ? std::max(1, (len + 1023) / 1024) : 1;
}

void launch_center_pad(hipStream_t st, int n, int npad, int batch, const void* x, int x_is_f32,
                       int ldx, int center, double* dst) {
  const dim3 grid(batch, vector_parts(batch, npad));
  if (x_is_f32)
    hipLaunchKernelGGL(k_center_pad<float>, grid, dim3(1024), 0, st, n, npad,
                       static_cast<const float*>(x), ldx, center, dst);
  else
    hipLaunchKernelGGL(k_center_pad<double>, grid, dim3(1024), 0, st, n, npad,
                       static_cast<const double*>(x), ldx, center, dst);
}

// means[b] = (1/n) sum_{i<n} x[b][i]: the uniform part of a right-hand side.
// S e = 0, so S x = S (x - mean e); removing it first keeps the rounding of a
// low-precision S from acting on the (large) uniform potential.
__global__ void __launch_bounds__(1024) k_row_means(int n, const void* __restrict__ x, int x_is_f32,
                                                    int ldx, double* __restrict__ means) {
  __shared__ double sh[16];
  const int b = blockIdx.x;
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024)
    s += x_is_f32 ? (double)reinterpret_cast<const float*>(x)[(size_t)b * ldx + i]
                  : reinterpret_cast<const double*>(x)[(size_t)b * ldx + i];
  s = block_sum1024(s, sh);
  if (threadIdx.x == 0) means[b] = s / n;
}

void launch_row_means(hipStream_t st, int n, int batch, const void* x, int x_is_f32, int ldx,
                      double* means) {
  hipLaunchKernelGGL(k_row_means, dim3(batch), dim3(1024), 0, st, n, x, x_is_f32, ldx, means);
}

// x[b][i] -= mean_b over i < n (in place, FP64, stride ld)
__global__ void __launch_bounds__(1024) k_center_rows(int n, int ld, double* __restrict__ x) {
  __shared__ double sh[16];
  double* row = x + (size_t)blockIdx.x * ld;
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) s += row[i];
  s = block_sum1024(s, sh) / n;
  for (int i = threadIdx.x; i < n; i += 1024) row[i] -= s;
}

void launch_center_rows(hipStream_t st, int n, int ld, int batch, double* x) {
  hipLaunchKernelGGL(k_center_rows, dim3(batch), dim3(1024), 0, st, n, ld, x);
}

// c[b] = b[b] + v (FP64, npad stride, zero padding): the right-hand side of
// A q = b + v used by the refinement residual.
__global__ void k_make_rhs(int n, int npad, const void* __restrict__ bsrc, int b_is_f32,
                           const double* __restrict__ v, double* __restrict__ c) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x, b = blockIdx.y;
  if (i >= npad) return;
  double x = 0.0;
  if (i < n)
    x = (b_is_f32 ? (double)reinterpret_cast<const float*>(bsrc)[(size_t)b * n + i]
                  : reinterpret_cast<const double*>(bsrc)[(size_t)b * n + i]) + v[i];
  c[(size_t)b * npad + i] = x;
}

void launch_make_rhs(hipStream_t st, int n, int npad, int batch, const void* bsrc, int b_is_f32,
                     const double* v, double* c) {
  hipLaunchKernelGGL(k_make_rhs, dim3((npad + 255) / 256, batch), dim3(256), 0, st, n, npad, bsrc,
                     b_is_f32, v, c);
}

// ---------------------------------------------------------------------------
// Neutrality projection and electrode totals (FP64):
//   mu = e^T qt / s,  q = qt - mu u,  Q_alpha = T_alpha - mu U_alpha,
// with T_alpha and U_alpha the sums of qt and u over electrode alpha (equal
// to the sum of q over alpha).  Grid (batch, parts): every workgroup of a
// vector forms the same e^T qt (one fixed-order workgroup sum) and writes its
// own part of q; workgroup 0 also forms the electrode sums, four electrodes
// per pass, the first four in the pass that sums e^T qt.
// ---------------------------------------------------------------------------
template <bool ADD>
__global__ void __launch_bounds__(1024) k_finalize(int n, const double* __restrict__ qt, int ldqt,
                                                   const double* __restrict__ add,
                                                   const double* __restrict__ u,
                                                   const double* __restrict__ s_dev,
                                                   const int* __restrict__ eid, int n_e,
                                                   double* __restrict__ q, int ldq,
                                                   double* __restrict__ Qe) {
  __shared__ double sh[16];
  __shared__ double shq[8][16];
  const int b = blockIdx.x;
  const double* x = qt + (size_t)b * ldqt;
  auto val = [&](int i) { return ADD ? x[i] + add[i] : x[i]; };
  const bool totals = Qe && blockIdx.y == 0;
  double s = 0.0, t[4] = {0.0, 0.0, 0.0, 0.0}, w[4] = {0.0, 0.0, 0.0, 0.0};
  // four elements per thread in flight: i0 + 1024 j, in increasing order
  for (int i0 = threadIdx.x; i0 < n; i0 += 4096) {
    double v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = val(min(i0 + 1024 * j, n - 1));
    if (totals) {
      double uu[4];
      int e[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = min(i0 + 1024 * j, n - 1);
        uu[j] = u[i];
        e[j] = i0 + 1024 * j < n ? eid[i] : -1;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          t[k] += e[j] == k ? v[j] : 0.0;
          w[k] += e[j] == k ? uu[j] : 0.0;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) s += i0 + 1024 * j < n ? v[j] : 0.0;
  }
  s = block_sum1024(s, sh);
  const double mu = s / (*s_dev);
  double* qo = q + (size_t)b * ldq;
  for (int i = blockIdx.y * 1024 + threadIdx.x; i < n; i += 1024 * gridDim.y)
    qo[i] = val(i) - mu * u[i];
  if (!totals) return;
#pragma unroll 1
  for (int a0 = 0; a0 < n_e; a0 += 4) {
    if (a0 > 0) {                   // electrodes beyond the first four
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = w[k] = 0.0;
#pragma unroll 1
      for (int i = threadIdx.x; i < n; i += 1024) {
        const int e = eid[i] - a0;
        const double v = val(i), ui = u[i];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          t[k] += e == k ? v : 0.0;
          w[k] += e == k ? ui : 0.0;
        }
      }
    }
    // wave sums, then thread k < 4 adds electrode a0 + k's 16 wave sums in order
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (a0 + k < n_e) {
        t[k] = wave_sum(t[k]);
        w[k] = wave_sum(w[k]);
      }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        shq[k][wave] = t[k];
        shq[4 + k][wave] = w[k];
      }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < 4 && a0 + k < n_e) {
      double tt = 0.0, ww = 0.0;
      for (int v = 0; v < 16; ++v) {
        tt += shq[k][v];
        ww += shq[4 + k][v];
      }
      Qe[(size_t)b * n_e + a0 + k] = tt - mu * ww;
    }
    __syncthreads();
  }
}

void launch_finalize(hipStream_t st, int n, int batch, const double* qt, int ldqt, const double* add,
                     const double* u, const double* s_dev, const int* eid, int n_e, double* q,
                     int ldq, double* Qe) {
  const dim3 grid(batch, vector_parts(batch, n));
  if (add)
    hipLaunchKernelGGL(k_finalize<true>, grid, dim3(1024), 0, st, n, qt, ldqt, add, u, s_dev, eid,
                       n_e, q, ldq, Qe);
  else
    hipLaunchKernelGGL(k_finalize<false>, grid, dim3(1024), 0, st, n, qt, ldqt, add, u, s_dev, eid,
                       n_e, q, ldq, Qe);
}

// ---------------------------------------------------------------------------
// One vector's solve in one launch: x = b - mean(b) in LDS (every workgroup forms
// it), rows of S x + d as k_matvec, and by the workgroup that ends last the
// neutrality projection and electrode totals as k_finalize.  For matrices that stay
// in the caches, whose product takes less time than the three launches' latencies
// (centre 4 us, product 12, finalize 9 at 2880 atoms): a step of
// 288 atoms 50 -> 45 us, of 2880 75 -> 69.5 (with a release fence per workgroup, which
// writes back its L2, 81).
// y is exchanged by stores and loads at device scope; *count is zero between
// launches.  Sums in a fixed order.
// ---------------------------------------------------------------------------
constexpr int MQ_MAX = 4096;                         // npad: x in 32 KiB of LDS

template <typename TM, typename TX, int R>
__global__ void __launch_bounds__(256) k_matvec_q(int n, int npad, const TM* __restrict__ M,
                                                  const TX* __restrict__ bx,
                                                  const double* __restrict__ d,
                                                  const double* __restrict__ u,
                                                  const double* __restrict__ s_dev,
                                                  const int* __restrict__ eid, int n_e, double* y,
                                                  double* __restrict__ q, double* __restrict__ Qe,
                                                  int* count) {
  constexpr int PT = MQ_MAX / 256, VEC = 16 / sizeof(TM);
  __shared__ __align__(16) double xs[MQ_MAX];
  __shared__ double sh[8][4];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.y;
  {
    const TX* xb = bx + (size_t)b * n;
    double v[PT], t = 0.0;
#pragma unroll
    for (int k = 0; k < PT; ++k) v[k] = tid + 256 * k < n ? (double)xb[tid + 256 * k] : 0.0;
#pragma unroll
    for (int k = 0; k < PT; ++k) t += v[k];
    const double mean = block_sum256(t, sh[0]) / n;
#pragma unroll
    for (int k = 0; k < PT; ++k)
      if (tid + 256 * k < npad) xs[tid + 256 * k] = tid + 256 * k < n ? v[k] - mean : 0.0;
  }
  const int row0 = (blockIdx.x * 4 + wave) * R;
  double* yb = y + (size_t)b * npad;
  __syncthreads();
  if (row0 < npad) {
    const TM* mrow = M + (size_t)row0 * npad;
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
#pragma unroll 2
    for (int j0 = lane * VEC; j0 < npad; j0 += 64 * VEC) {
      TM mv[R][VEC];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const TM* src = mrow + (size_t)r * npad + j0;
        if constexpr (VEC == 2) {
          const d2v t = *reinterpret_cast<const d2v*>(src);
          mv[r][0] = t.x; mv[r][1] = t.y;
        } else {
          const f4v t = *reinterpret_cast<const f4v*>(src);
          mv[r][0] = t.x; mv[r][1] = t.y; mv[r][2] = t.z; mv[r][3] = t.w;
        }
      }
      double xj[VEC];
#pragma unroll
      for (int t = 0; t < VEC; ++t) xj[t] = xs[j0 + t];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int t = 0; t < VEC; ++t) acc[r] += (double)mv[r][t] * xj[t];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = wave_sum(acc[r]);
    if (lane < R) {
      double t = acc[0];
#pragma unroll
      for (int r = 1; r < R; ++r)
        if (lane == r) t = acc[r];
      __hip_atomic_store(&yb[row0 + lane], t + d[row0 + lane], __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // only y is exchanged, by device-scope accesses past the XCD's L2: the stores have
  // to be complete before the count, no cache has to be written back
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0)
    last = __hip_atomic_fetch_add(&count[b], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           (int)gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  if (tid == 0) __hip_atomic_store(&count[b], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // this thread's values of y and u
  double v[PT], uu[PT], t = 0.0;
#pragma unroll
  for (int k = 0; k < PT; ++k) {
    const int i = tid + 256 * k;
    v[k] = i < n ? __hip_atomic_load(&yb[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
    uu[k] = i < n ? u[i] : 0.0;
  }
#pragma unroll
  for (int k = 0; k < PT; ++k) t += v[k];
  const double mu = block_sum256(t, sh[0]) / (*s_dev);
#pragma unroll
  for (int k = 0; k < PT; ++k)
    if (tid + 256 * k < n) q[(size_t)b * n + tid + 256 * k] = v[k] - mu * uu[k];
  if (!Qe) return;
  int e[PT];
#pragma unroll
  for (int k = 0; k < PT; ++k) e[k] = tid + 256 * k < n ? eid[tid + 256 * k] : -1;
  for (int a0 = 0; a0 < n_e; a0 += 4) {
    double tt[4] = {0.0, 0.0, 0.0, 0.0}, ww[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < PT; ++k)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        tt[a] += e[k] == a0 + a ? v[k] : 0.0;
        ww[a] += e[k] == a0 + a ? uu[k] : 0.0;
      }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      tt[a] = wave_sum(tt[a]);
      ww[a] = wave_sum(ww[a]);
      if (lane == 0) {
        sh[a][wave] = tt[a];
        sh[4 + a][wave] = ww[a];
      }
    }
    __syncthreads();
    if (tid < 4 && a0 + tid < n_e)
      Qe[(size_t)b * n_e + a0 + tid] =
          ((sh[tid][0] + sh[tid][1]) + (sh[tid][2] + sh[tid][3])) -
          mu * ((sh[4 + tid][0] + sh[4 + tid][1]) + (sh[4 + tid][2] + sh[4 + tid][3]));
  }
}

bool matvec_q_fits(int npad) { return npad <= MQ_MAX; }

template <typename TM, typename TX>
static void matvec_q_launch(hipStream_t st, int n, int npad, const TM* M, int batch, const TX* b,
                            const double* d, const double* u, const double* s_dev, const int* eid,
                            int n_e, double* y, double* q, double* Qe, int* count) {
  const int R = npad >= 2048 ? 4 : npad >= 1024 ? 2 : 1;
  hipLaunchKernelGGL((R == 4 ? k_matvec_q<TM, TX, 4> : R == 2 ? k_matvec_q<TM, TX, 2>
                                                               : k_matvec_q<TM, TX, 1>),
                     dim3((npad / R + 3) / 4, batch), dim3(256), 0, st, n, npad, M, b, d, u, s_dev,
                     eid, n_e, y, q, Qe, count);
}

void launch_matvec_q(hipStream_t st, int which, int n, int npad, const void* M, int batch,
                     const void* b, int b_is_f32, const double* d, const double* u,
                     const double* s_dev, const int* eid, int n_e, double* y, double* q, double* Qe,
                     int* count) {
  auto go = [&](auto m, auto x) {
    matvec_q_launch(st, n, npad, m, batch, x, d, u, s_dev, eid, n_e, y, q, Qe, count);
  };
  if (which == 0) {
    if (b_is_f32) go((const double*)M, (const float*)b); else go((const double*)M, (const double*)b);
  } else {
    if (b_is_f32) go((const float*)M, (const float*)b); else go((const float*)M, (const double*)b);
  }
}


// ---------------------------------------------------------------------------
// Inverse kept as the Cholesky factor (the solves are GEMMs with the factor's
// panels, driven from the host).  Electrode indicators as right-hand-side
// rows, and the quantities of Eqs. 4 and 6 from their solutions
// Y_a = g_a^T A^-1 (A symmetric): u = A^-1 e = sum_a Y_a^T (every atom is in
// one electrode), s = e^T u, and S g_a = Y_a^T - u (e^T Y_a^T) / s, since
// u^T g_a = e^T A^-1 g_a.  One workgroup; every sum in a fixed order.
// ---------------------------------------------------------------------------
__global__ void k_group_indicator(int n, int npad, int rows, const int* __restrict__ eid, int n_e,
                                  double* __restrict__ X) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)rows * npad) return;
  const int r = (int)(e / npad), j = (int)(e % npad);
  X[e] = (r < n_e && j < n && eid[j] == r) ? 1.0 : 0.0;
}

void launch_group_indicator(hipStream_t st, int n, int npad, int rows, const int* eid, int n_e,
                            double* X) {
  const size_t tot = (size_t)rows * npad;
  hipLaunchKernelGGL(k_group_indicator, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n,
                     npad, rows, eid, n_e, X);
}

__global__ void __launch_bounds__(1024) k_factor_response(int n, int npad, int n_e,
                                                          const double* __restrict__ Y, int ldy,
                                                          double* __restrict__ u,
                                                          double* __restrict__ s_out,
                                                          double* __restrict__ sg) {
  __shared__ double sh[16];
  __shared__ double tot[CCM_MAXE];
  for (int a = 0; a < n_e; ++a) {
    double t = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) t += Y[(size_t)a * ldy + i];
    t = block_sum1024(t, sh);
    if (threadIdx.x == 0) tot[a] = t;
  }
  __syncthreads();
  double s = 0.0;
  for (int a = 0; a < n_e; ++a) s += tot[a];           // e^T u
  for (int i = threadIdx.x; i < npad; i += 1024) {
    double ui = 0.0;
    if (i < n)
      for (int a = 0; a < n_e; ++a) ui += Y[(size_t)a * ldy + i];
    u[i] = ui;
    for (int a = 0; a < n_e; ++a)
      sg[(size_t)i * n_e + a] = i < n ? Y[(size_t)a * ldy + i] - ui * (tot[a] / s) : 0.0;
  }
  if (threadIdx.x == 0) *s_out = s;
}

void launch_factor_response(hipStream_t st, int n, int npad, int n_e, const double* Y, int ldy,
                            double* u, double* s, double* sg) {
  hipLaunchKernelGGL(k_factor_response, dim3(1), dim3(1024), 0, st, n, npad, n_e, Y, ldy, u, s, sg);
}

// ---------------------------------------------------------------------------
// Row sums of a symmetric npad x npad matrix over each electrode's columns,
// U = M G (npad x n_e, row-major; rows i >= n are zero), in one pass over M:
// one wave per row, lane-strided columns, one register per electrode and a
// fixed-order wave sum each.  M = A^-1 gives the constrained-charge response
// of Eq. 7; M = S gives the cached potential response S G of Eq. 6.
// ---------------------------------------------------------------------------
template <int NE>
__global__ void __launch_bounds__(256) k_group_row_sums(int n, int npad, const double* __restrict__ M,
                                                        const int* __restrict__ eid, int n_e,
                                                        double* __restrict__ U) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= npad) return;
  double acc[NE];
#pragma unroll
  for (int a = 0; a < NE; ++a) acc[a] = 0.0;
  if (i < n) {
    const double* row = M + (size_t)i * npad;
    for (int j = lane; j < n; j += 64) {
      const double v = row[j];
      const int e = eid[j];
#pragma unroll
      for (int a = 0; a < NE; ++a)
        if (e == a) acc[a] += v;
    }
  }
#pragma unroll
  for (int a = 0; a < NE; ++a) {
    const double s = wave_sum(acc[a]);
    if (lane == 0 && a < n_e) U[(size_t)i * n_e + a] = s;
  }
}

void launch_ccm_response(hipStream_t st, int n, int npad, const double* M, const int* eid,
                         int n_e, double* U) {
  dim3 grid((npad + 3) / 4), block(256);
  if (n_e <= 2)
    hipLaunchKernelGGL(k_group_row_sums<2>, grid, block, 0, st, n, npad, M, eid, n_e, U);
  else if (n_e <= 4)
    hipLaunchKernelGGL(k_group_row_sums<4>, grid, block, 0, st, n, npad, M, eid, n_e, U);
  else if (n_e <= 8)
    hipLaunchKernelGGL(k_group_row_sums<8>, grid, block, 0, st, n, npad, M, eid, n_e, U);
  else
    hipLaunchKernelGGL(k_group_row_sums<CCM_MAXE>, grid, block, 0, st, n, npad, M, eid, n_e, U);
}

// Applied potential from the cached response (Eqs. 5, 6): v_i = v~_e(i) and
// d_i = sum_a (S G)_ia v~_a (fixed electrode order), for i < npad (zero
// padding); d is left alone when SG is NULL (the operator has no S).
__global__ void k_apply_potential(int n, int npad, int n_e, const int* __restrict__ eid,
                                  const double* __restrict__ SG, ElectrodeValues vt,
                                  double* __restrict__ vat, double* __restrict__ d) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npad) return;
  double v = 0.0, di = 0.0;
  if (i < n) {
    v = vt.v[eid[i]];
    if (SG)
      for (int a = 0; a < n_e; ++a) di += SG[(size_t)i * n_e + a] * vt.v[a];
  }
  vat[i] = v;
  if (SG) d[i] = di;
}

void launch_apply_potential(hipStream_t st, int n, int npad, int n_e, const int* eid,
                            const double* SG, const ElectrodeValues& vt, double* vat, double* d) {
  hipLaunchKernelGGL(k_apply_potential, dim3((npad + 255) / 256), dim3(256), 0, st, n, npad, n_e,
                     eid, SG, vt, vat, d);
}

// Finite-field potential (Eqs. 13, 14) from its cached pieces: v = -dv0 zeta
// and d = S v = -dv0 (S zeta) (szeta NULL: d untouched).
__global__ void k_scale_field(int npad, double dv0, const double* __restrict__ zeta,
                              const double* __restrict__ szeta, double* __restrict__ vat,
                              double* __restrict__ d) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npad) return;
  vat[i] = -dv0 * zeta[i];
  if (szeta) d[i] = -dv0 * szeta[i];
}

void launch_scale_field(hipStream_t st, int npad, double dv0, const double* zeta,
                        const double* szeta, double* vat, double* d) {
  hipLaunchKernelGGL(k_scale_field, dim3((npad + 255) / 256), dim3(256), 0, st, npad, dv0, zeta,
                     szeta, vat, d);
}

// Per configuration b (one workgroup): y = A^-1 b is given (row b of yt);
// q~_b = G^T y, v~ = C~^-1 (Q - q~_b), q = y + U v~, Qe = G^T q.  Sums per
// electrode in a fixed order; n_e <= CCM_MAXE.
__global__ void __launch_bounds__(256) k_ccm_finalize(int n, const double* __restrict__ yt, int ldy,
                                                      const double* __restrict__ U,
                                                      const double* __restrict__ Cinv,
                                                      const double* __restrict__ Qt,
                                                      const int* __restrict__ eid, int n_e,
                                                      double* __restrict__ q, int ldq,
                                                      double* __restrict__ Qe) {
  __shared__ double sh[4];
  __shared__ double s_v[CCM_MAXE];
  __shared__ double s_g[CCM_MAXE];
  const int b = blockIdx.x;
  const double* y = yt + (size_t)b * ldy;
  for (int a = 0; a < n_e; ++a) {
    double t = 0.0;
    for (int i = threadIdx.x; i < n; i += 256)
      if (eid[i] == a) t += y[i];
    t = block_sum256(t, sh);
    if (threadIdx.x == 0) s_g[a] = t;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int a = 0; a < n_e; ++a) {
      double v = 0.0;
      for (int c = 0; c < n_e; ++c) v += Cinv[a * n_e + c] * (Qt[c] - s_g[c]);
      s_v[a] = v;
    }
  __syncthreads();
  double* qo = q + (size_t)b * ldq;
  for (int i = threadIdx.x; i < n; i += 256) {
    double v = y[i];
    for (int a = 0; a < n_e; ++a) v += U[(size_t)i * n_e + a] * s_v[a];
    qo[i] = v;
  }
  if (Qe) {
    __syncthreads();
    for (int a = 0; a < n_e; ++a) {
      double t = 0.0;
      for (int i = threadIdx.x; i < n; i += 256)
        if (eid[i] == a) t += qo[i];
      t = block_sum256(t, sh);
      if (threadIdx.x == 0) Qe[(size_t)b * n_e + a] = t;
    }
  }
}

void launch_ccm_finalize(hipStream_t st, int n, int batch, const double* yt, int ldy,
                         const double* U, const double* Cinv, const double* Qt, const int* eid,
                         int n_e, double* q, int ldq, double* Qe) {
  hipLaunchKernelGGL(k_ccm_finalize, dim3(batch), dim3(256), 0, st, n, yt, ldy, U, Cinv, Qt, eid,
                     n_e, q, ldq, Qe);
}

// p[0 .. count) = 0 (a kernel, so it can sit inside a captured graph)
__global__ void k_fill_zero(size_t count, float* p) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < count) p[e] = 0.0f;
}

void launch_fill_zero(hipStream_t st, size_t count, float* p) {
  if (count == 0) return;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, count, p);
}

// dst (rows x npad, FP64) = src (batch x n) zero-padded in both directions
__global__ void k_pad_rows(int n, int npad, int batch, int rows, const void* __restrict__ src,
                           int src_is_f32, const double* __restrict__ shift,
                           double* __restrict__ dst) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)rows * npad) return;
  const int r = (int)(e / npad), j = (int)(e % npad);
  double v = 0.0;
  if (r < batch && j < n)
    v = (src_is_f32 ? (double)reinterpret_cast<const float*>(src)[(size_t)r * n + j]
                    : reinterpret_cast<const double*>(src)[(size_t)r * n + j]) -
        (shift ? shift[r] : 0.0);
  dst[e] = v;
}

void launch_pad_rows(hipStream_t st, int n, int npad, int batch, int rows, const void* src,
                     int src_is_f32, const double* shift, double* dst) {
  const size_t tot = (size_t)rows * npad;
  hipLaunchKernelGGL(k_pad_rows, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, npad,
                     batch, rows, src, src_is_f32, shift, dst);
}

// ---------------------------------------------------------------------------
// Batched solve on BF16 matrix cores: C (+)= X S with both operands split as
// x ~ hi + lo (BF16 pairs) and three products hi*hi + hi*lo + lo*hi
// accumulated in FP32 (the lo*lo term is below FP32 resolution of the sum).
// S is symmetric, so its rows serve as the columns of the right operand and
// both operands are read K-contiguous.
//
// One persistent kernel serves a group of up to GB_MAXP independent
// problems (contexts of different sizes): the tiles of all problems form one
// list that the workgroups walk with a stride of the grid size.  Tile shape
// BM x 64 (BM = 32, 64 or 128 rows of X) and the split of K into ks parts
// are chosen per problem size by the autotuner; with ks > 1 each part
// writes its own slice of a partial buffer and k_sum_ksplit adds the slices
// in a fixed order.  4 waves in a 2 x 2 layout, v_mfma_f32_16x16x32_bf16,
// K slabs of 32 through LDS with the next slab prefetched into registers.
//   operand layout (lane l): A (row l%16, k 8(l/16)..+7); B (k 8(l/16)..+7,
//   col l%16); result register r: (row 4(l/16) + r, col l%16).
// ---------------------------------------------------------------------------
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <int BM>
__global__ void __launch_bounds__(256) k_gemm_bf16x3(GemmGroupBf grp) {
  constexpr int P = 40;                 // LDS row pitch in BF16 elements (32 + 8)
  constexpr int FM = BM / 32;           // 16-row blocks per wave
  __shared__ __attribute__((aligned(16))) uint16_t Ah[BM * P], Al[BM * P], Bh[64 * P], Bl[64 * P];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * 32;
  for (int t = blockIdx.x; t < grp.total; t += gridDim.x) {
    int p = 0;
    while (p + 1 < grp.nprob && t >= grp.start[p + 1]) ++p;
    const GemmProbBf& pr = grp.p[p];
    const int local = t - grp.start[p];
    const int kpart = local % pr.ks, rest = local / pr.ks;
    const int m0 = (rest / pr.tiles_n) * BM, n0 = (rest % pr.tiles_n) * 64;
    const int kchunk = ((pr.K + pr.ks - 1) / pr.ks + 31) / 32 * 32;
    const int kb = kpart * kchunk, ke = min(pr.K, kb + kchunk);
    v4f acc[FM][2];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b] = (v4f){0.f, 0.f, 0.f, 0.f};
    // loader slots: X rows (BM x 32 BF16 hi and lo per slab), S rows (64 x 32)
    const int sr = tid >> 2, sc = (tid & 3) * 8;
    constexpr int XR = BM >= 64 ? BM / 64 : 1;        // 8-element X groups per thread
    uint4 xh[XR], xl[XR];
    uint2 xh2, xl2;                                    // BM = 32: 4 elements per thread
    uint4 sh, sl;
    auto load = [&](int k0) {
      if constexpr (BM >= 64) {
#pragma unroll
        for (int u = 0; u < XR; ++u) {
          const size_t xo = (size_t)(m0 + sr + 64 * u) * pr.ldx + k0 + sc;
          xh[u] = *reinterpret_cast<const uint4*>(pr.Xhi + xo);
          xl[u] = *reinterpret_cast<const uint4*>(pr.Xlo + xo);
        }
      } else {
        const size_t xo = (size_t)(m0 + (tid >> 3)) * pr.ldx + k0 + (tid & 7) * 4;
        xh2 = *reinterpret_cast<const uint2*>(pr.Xhi + xo);
        xl2 = *reinterpret_cast<const uint2*>(pr.Xlo + xo);
      }
      const size_t so = (size_t)(n0 + sr) * pr.lds + k0 + sc;
      sh = *reinterpret_cast<const uint4*>(pr.Shi + so);
      sl = *reinterpret_cast<const uint4*>(pr.Slo + so);
    };
    auto store = [&]() {
      if constexpr (BM >= 64) {
#pragma unroll
        for (int u = 0; u < XR; ++u) {
          *reinterpret_cast<uint4*>(&Ah[(sr + 64 * u) * P + sc]) = xh[u];
          *reinterpret_cast<uint4*>(&Al[(sr + 64 * u) * P + sc]) = xl[u];
        }
      } else {
        const int r = tid >> 3, c4 = (tid & 7) * 4;
        *reinterpret_cast<uint2*>(&Ah[r * P + c4]) = xh2;
        *reinterpret_cast<uint2*>(&Al[r * P + c4]) = xl2;
      }
      *reinterpret_cast<uint4*>(&Bh[sr * P + sc]) = sh;
      *reinterpret_cast<uint4*>(&Bl[sr * P + sc]) = sl;
    };
    if (kb < ke) load(kb);
    for (int k0 = kb; k0 < ke; k0 += 32) {
      __syncthreads();                 // the previous slab (or tile) is no longer read
      store();
      __syncthreads();
      if (k0 + 32 < ke) load(k0 + 32);
      const int kk = 8 * (lane >> 4), rr = lane & 15;
      v8bf ah[FM], al[FM], bh[2], bl[2];
#pragma unroll
      for (int a = 0; a < FM; ++a) {
        ah[a] = *reinterpret_cast<const v8bf*>(&Ah[(wm + a * 16 + rr) * P + kk]);
        al[a] = *reinterpret_cast<const v8bf*>(&Al[(wm + a * 16 + rr) * P + kk]);
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        bh[b] = *reinterpret_cast<const v8bf*>(&Bh[(wn + b * 16 + rr) * P + kk]);
        bl[b] = *reinterpret_cast<const v8bf*>(&Bl[(wn + b * 16 + rr) * P + kk]);
      }
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[a], bh[b], acc[a][b], 0, 0, 0);
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[a], bl[b], acc[a][b], 0, 0, 0);
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[a], bh[b], acc[a][b], 0, 0, 0);
        }
    }
    // ks == 1: C (+)= result; ks > 1: slice kpart of the partial buffer
    double* out = pr.ks > 1 ? pr.part + (size_t)kpart * pr.M * pr.ldc : pr.C;
    const bool acc_c = pr.ks == 1 && pr.accumulate;
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = m0 + wm + a * 16 + 4 * (lane >> 4) + r;
          const int col = n0 + wn + b * 16 + (lane & 15);
          double* cp = out + (size_t)row * pr.ldc + col;
          const double v = (double)acc[a][b][r];
          *cp = acc_c ? *cp + v : v;
        }
  }
}

// C (+)= sum over ks slices of part, in slice order (fixed), M x ldc elements
__global__ void k_sum_ksplit(size_t count, int ks, const double* __restrict__ part,
                             double* __restrict__ C, int accumulate) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count) return;
  double s = part[e];
  for (int k = 1; k < ks; ++k) s += part[(size_t)k * count + e];
  C[e] = accumulate ? C[e] + s : s;
}

void launch_gemm_bf16x3_group(hipStream_t st, const GemmGroupBf& grp, int bm, int grid) {
  if (grp.total <= 0) return;
  const int g = std::max(1, std::min(grid, grp.total));
  if (bm == 32)
    hipLaunchKernelGGL(k_gemm_bf16x3<32>, dim3(g), dim3(256), 0, st, grp);
  else if (bm == 128)
    hipLaunchKernelGGL(k_gemm_bf16x3<128>, dim3(g), dim3(256), 0, st, grp);
  else
    hipLaunchKernelGGL(k_gemm_bf16x3<64>, dim3(g), dim3(256), 0, st, grp);
  for (int p = 0; p < grp.nprob; ++p) {
    const GemmProbBf& pr = grp.p[p];
    if (pr.ks > 1) {
      const size_t count = (size_t)pr.M * pr.ldc;
      hipLaunchKernelGGL(k_sum_ksplit, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st,
                         count, pr.ks, pr.part, pr.C, pr.accumulate);
    }
  }
}

// Fill one problem of a group: X (M x K, ld ldx), S hi/lo (N x K, ld lds),
// C (M x ldc); part: ks x M x ldc doubles when ks > 1.
GemmProbBf gemm_bf16x3_problem(int M, int N, int K, const uint16_t* Xhi, const uint16_t* Xlo,
                               int ldx, const uint16_t* Shi, const uint16_t* Slo, int lds,
                               double* C, int ldc, int accumulate, int bm, int ks, double* part) {
  GemmProbBf pr{};
  pr.Xhi = Xhi; pr.Xlo = Xlo; pr.Shi = Shi; pr.Slo = Slo; pr.C = C; pr.part = part;
  pr.M = M; pr.N = N; pr.K = K; pr.ldx = ldx; pr.lds = lds; pr.ldc = ldc;
  pr.tiles_m = M / bm; pr.tiles_n = N / 64; pr.ks = ks; pr.accumulate = accumulate;
  return pr;
}

void group_finish(GemmGroupBf& grp) {
  grp.start[0] = 0;
  for (int p = 0; p < grp.nprob; ++p)
    grp.start[p + 1] = grp.start[p] + grp.p[p].tiles_m * grp.p[p].tiles_n * grp.p[p].ks;
  grp.total = grp.start[grp.nprob];
}

}  // namespace cpm
