// The k-space part of b for planar electrodes from charges sorted by z
// (Sec. II.A: b is recomputed for every configuration).
//
// For a column c = (k_x, k_y) of the k set and a plane L the projection needs
//   T(c, L) = sum_n 2W(c, n) S(c, n) e^{-i n kz1 z_L}
//           = sum_j q_j e^{i theta_c(r_j)} G_c(z_j - z_L),
//   G_c(z)  = sum_{n >= 0} w(c, n) cos(n kz1 z)
// (the column holds n and -n with equal weights, folded into w; of the column
// (0, 0) only the real part of T is used).  G_c is band-limited by the k-space
// cutoff and its weights fall as e^{-k^2 / 4 alpha^2}, so on a z bin of half
// width hw ~ 0.4 / alpha its Chebyshev series ends at FP64 rounding after
// ZB_P = 16 terms.  With the charges sorted into such bins,
//   T(c, L) = sum_bins sum_{p < 16} H(c, L, bin, p) D(c, bin, p),
//   D(c, bin, p) = sum_{j in bin} q_j e^{i theta_c(r_j)} T_p(t_j),
// where t_j in [-1, 1] is z_j in its bin and H the Chebyshev coefficients of
// G_c(z - z_L) on the bin, fixed while the electrodes are.  The charges then
// meet 16 functions of z instead of the 2 n_z of the plane waves (158 at 2880
// atoms, 98 at 20064), the sums over k_z leave the per-charge work, and no
// phase tables or structure factors go through memory.  Measured (k_zb_sums
// against tables, structure factors and their reduction, kernels alone):
// b in FP64, 37 configurations of 7176 atoms (72k charges): 4.3 against about
// 17 ms; b in FP32, 64 configurations of 2880 atoms (6128 charges): 0.12
// against 0.42 ms; one configuration of 20064 atoms in FP64: 0.62 against
// 1.3 ms.
#include <algorithm>
#include <cmath>
#include <vector>

#include "cpm_internal.h"
#include "rs_plane.hpp"

namespace cpm {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Sorting: every configuration's charges by z, in nsort equal sort bins of
// [0, Lz) (each z bin of the expansion is `sub` of them), stable, so the
// order is fixed by the data.  A block of 16 waves places ZS_BLK charges,
// wave w a contiguous quarter-thousand of them, 64 at a time with ranks from
// ballots.  A charge's first position needs the counts of all blocks: with at
// most two blocks each counts every charge itself (SELF, one launch), else
// k_zb_count leaves the blocks' counts first.
// ---------------------------------------------------------------------------
constexpr int ZS_W = 16;
constexpr int ZS_BLK = 4096;           // charges per block
constexpr int ZS_ITERS = ZS_BLK / (64 * ZS_W);

__device__ inline double wrap_z(double z, double Lz, double invLz) {
  return z - Lz * floor(z * invLz);
}

__device__ inline int sort_bin(double zw, double scale, int nsort) {
  return min(nsort - 1, max(0, (int)(zw * scale)));
}

// counts[((s nblk) + blk) nsort + bin] of block blk's charges
__global__ void __launch_bounds__(64 * ZS_W) k_zb_count(int m, int nsort, double Lz,
                                                        const double* __restrict__ xyz,
                                                        int* __restrict__ counts) {
  __shared__ int h[ZB_MAXSORT];
  const int blk = blockIdx.x, s = blockIdx.y, nblk = gridDim.x;
  const double invLz = 1.0 / Lz, scale = nsort / Lz;
  xyz += (size_t)s * m * 3;
  for (int b = threadIdx.x; b < nsort; b += blockDim.x) h[b] = 0;
  __syncthreads();
  for (int j = blk * ZS_BLK + threadIdx.x; j < min(m, (blk + 1) * ZS_BLK); j += blockDim.x)
    atomicAdd(&h[sort_bin(wrap_z(xyz[3 * (size_t)j + 2], Lz, invLz), scale, nsort)], 1);
  __syncthreads();
  int* out = counts + ((size_t)s * nblk + blk) * nsort;
  for (int b = threadIdx.x; b < nsort; b += blockDim.x) out[b] = h[b];
}

// cq: the sorted charges (x wrapped, y wrapped, z, q), rows mpad64 apart; zr:
// z range of each block of 64 of them (edges of its sort bins); binoff
// [s (nbins + 1)]: first position of every z bin; dip: dipole partials of the
// block's charges (raw coordinates)
template <bool SELF>
__global__ void __launch_bounds__(64 * ZS_W) k_zb_scatter(
    int m, int mpad64, int nsort, int nbits, int sub, int nbins, double Lx, double Ly, double Lz,
    const double* __restrict__ xyz, const double* __restrict__ q, const int* __restrict__ counts,
    double4* __restrict__ cq, double2* __restrict__ zr, int* __restrict__ binoff,
    double* __restrict__ dip) {
  __shared__ int hist[ZS_W][ZB_MAXSORT];           // per wave: counts, then next positions
  __shared__ int before[ZB_MAXSORT], tot[ZB_MAXSORT];
  __shared__ double sd[3][ZS_W];
  const int blk = blockIdx.x, s = blockIdx.y, nblk = gridDim.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double invLx = 1.0 / Lx, invLy = 1.0 / Ly, invLz = 1.0 / Lz, scale = nsort / Lz;
  xyz += (size_t)s * m * 3;
  const int j0 = blk * ZS_BLK + wave * (ZS_BLK / ZS_W);
  // this thread's charges, all loads in flight at once
  double x[ZS_ITERS], y[ZS_ITERS], z[ZS_ITERS], qq[ZS_ITERS];
  int bin[ZS_ITERS];
#pragma unroll
  for (int it = 0; it < ZS_ITERS; ++it) {
    const int j = j0 + 64 * it + lane;
    const size_t jc = j < m ? j : 0;
    x[it] = xyz[3 * jc];
    y[it] = xyz[3 * jc + 1];
    z[it] = xyz[3 * jc + 2];
    qq[it] = j < m ? q[jc] : 0.0;
  }
  for (int b = lane; b < nsort; b += 64) hist[wave][b] = 0;
  for (int b = tid; b < nsort; b += 64 * ZS_W) before[b] = tot[b] = 0;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ZS_ITERS; ++it) {
    bin[it] = j0 + 64 * it + lane < m ? sort_bin(wrap_z(z[it], Lz, invLz), scale, nsort) : nsort;
    if (bin[it] < nsort) atomicAdd(&hist[wave][bin[it]], 1);
  }
  if (SELF) {
    // the other block's charges
    for (int j = (1 - blk) * ZS_BLK + tid; j < min(m, (2 - blk) * ZS_BLK); j += 64 * ZS_W) {
      const int b = sort_bin(wrap_z(xyz[3 * (size_t)j + 2], Lz, invLz), scale, nsort);
      atomicAdd(blk == 1 ? &before[b] : &tot[b], 1);
    }
  } else {
    const int* cs = counts + (size_t)s * nblk * nsort;
    for (int e = tid; e < nsort; e += 64 * ZS_W) {
      int bf = 0, af = 0;
#pragma unroll 8
      for (int k = 0; k < nblk; ++k) {
        const int c = cs[(size_t)k * nsort + e];
        bf += k < blk ? c : 0;
        af += k > blk ? c : 0;
      }
      before[e] = bf;
      tot[e] = af;
    }
  }
  // dipole partials, in a fixed order
  {
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int it = 0; it < ZS_ITERS; ++it) {
      v[0] += qq[it] * x[it];
      v[1] += qq[it] * y[it];
      v[2] += qq[it] * z[it];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      for (int o = 32; o > 0; o >>= 1) v[d] += __shfl_xor(v[d], o, 64);
      if (lane == 0) sd[d][wave] = v[d];
    }
  }
  __syncthreads();
  if (tid < 3) {
    double t = 0.0;
    for (int w = 0; w < ZS_W; ++w) t += sd[tid][w];
    dip[((size_t)s * nblk + blk) * 3 + tid] = t;
  }
  for (int b = tid; b < nsort; b += 64 * ZS_W) {
    int t = tot[b] + before[b];
    for (int w = 0; w < ZS_W; ++w) t += hist[w][b];
    tot[b] = t;
  }
  __syncthreads();
  if (wave == 0) {                                   // exclusive scan of the totals
    int running = 0;
    for (int k0 = 0; k0 < nsort; k0 += 64) {
      const int k = k0 + lane;
      const int c = k < nsort ? tot[k] : 0;
      int incl = c;
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
      }
      if (k < nsort) tot[k] = running + incl - c;
      running += __shfl(incl, 63, 64);
    }
  }
  __syncthreads();
  if (blk == 0) {
    int* bo = binoff + (size_t)s * (nbins + 1);
    for (int b = tid; b <= nbins; b += 64 * ZS_W) bo[b] = b < nbins ? tot[b * sub] : m;
  }
  for (int b = tid; b < nsort; b += 64 * ZS_W) {      // first position of each wave's run
    int p = tot[b] + before[b];
    for (int w = 0; w < ZS_W; ++w) {
      const int c = hist[w][b];
      hist[w][b] = p;
      p += c;
    }
  }
  __syncthreads();
  cq += (size_t)s * mpad64;
  zr += (size_t)s * (mpad64 / 64);
  const double width = Lz / nsort;
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int it = 0; it < ZS_ITERS; ++it) {
    const int key = bin[it];
    unsigned long long same = ~0ull;
    for (int t = 0; t < nbits; ++t) {
      const bool bit = (key >> t) & 1;
      const unsigned long long bal = __ballot(bit);
      same &= bit ? bal : ~bal;
    }
    const int rank = __popcll(same & below);
    if (key < nsort) {
      const int pos = hist[wave][key] + rank;
      if (pos < m) {                                 // always: the counts sum to m
        cq[pos] = make_double4(x[it] - Lx * floor(x[it] * invLx), y[it] - Ly * floor(y[it] * invLy),
                               z[it], qq[it]);
        if ((pos & 63) == 0) zr[pos >> 6].x = key * width;
        if ((pos & 63) == 63 || pos == m - 1) zr[pos >> 6].y = (key + 1) * width;
      }
    }
    wave_sync();
    if (key < nsort && rank == 0) hist[wave][key] += __popcll(same);
    wave_sync();
  }
}

// ---------------------------------------------------------------------------
// H: Chebyshev coefficients of G_c(z - z_L) on every bin.  One block per
// (bin, plane).  With z = z_b + hw t, A = n kz1 (z_b - z_L) and B = n kz1 hw,
//   cos(A + B t) = sum_p K(p, n) T_p(t),
//   K(p, n) = (2 - delta_p0) (-1)^floor((p + 1) / 2) J_p(B) (cos A, or sin A for odd p)
// (Jacobi and Anger), n in pieces of ZB_NC, and H(c, p) = sum_n w(c, n) K(p, n) for
// every column pair c = (n_x, n_y >= 0), the largest n and smallest weights first (J and
// w are stored in that order).  J: the factors of K without A, from zb_bessel_factors.  The
// coefficients fall with p like J_p, and so does their rounding: taken from values at
// the Chebyshev nodes, all p had the rounding of G_c itself, which the charges' uneven
// T_p sums carried into b (largest error of FP64 b against long double, relative to its
// largest entry, at 2880 and 4000 atoms: 2.3e-15 to 3.7e-15, now 1.0e-15 to 2.1e-15,
// explicit structure factors 1.1e-15 to 2.0e-15).  Once per rebuild and output type:
// 35 us (FP64) and 31 us (FP32) at 2880 atoms, 67 and 58 at 7176, 53 and 46 at 20064.
// Layout H[((bin ncu + c) nlayers + L) P + i], i the position of p in the
// matrix-core result layout of the consuming kernel (4 consecutive i per lane
// group).
// ---------------------------------------------------------------------------
constexpr int ZB_NC = 64;

// a charge's distance from the centre (bin + 0.5) width of its z bin, the centre not
// rounded (k_zb_response forms the bins' phases from the same centres)
__device__ inline double from_centre(double z, double Lz, double invLz, int bin, double width) {
  return fma(-(bin + 0.5), width, fma(-Lz, floor(z * invLz), z));
}

template <int P>
__global__ void __launch_bounds__(256) k_zb_response(int ncu, int nzt, int nbins, int nlayers,
                                                     const double* __restrict__ w,
                                                     const double* __restrict__ J,
                                                     const double* __restrict__ layer_z,
                                                     double Lz, double* __restrict__ H) {
  __shared__ double E[2][ZB_NC];                     // cos A, sin A
  __shared__ double K[P][ZB_NC];
  const int bin = blockIdx.x, L = blockIdx.y, tid = threadIdx.x;
  // the bin's centre minus the plane in cells, f + flo: a rounding of f alone would shift
  // all charges of the bin
  double f, flo;
  {
#pragma clang fp contract(off)
    const double width = Lz / nbins, zc = (bin + 0.5) * width, zl = layer_z[L];
    const double d = zc - zl, back = d + zl;
    const double dlo = (zc - back) + ((back - d) - zl) + fma(bin + 0.5, width, -zc);
    f = d / Lz;
    flo = (fma(-f, Lz, d) + dlo) / Lz;
    f -= rint(f);
  }
  for (int i0 = 0; i0 < nzt; i0 += ZB_NC) {          // n = nzt - 1 - i
    const int ni = min(ZB_NC, nzt - i0);
    __syncthreads();
    if (tid < ni) {
#pragma clang fp contract(off)
      const double n = nzt - 1 - i0 - tid, th = n * f;
      const double lo = fma(n, f, -th) + n * flo;
      double sn, cs;
      sincospi(2.0 * ((th - rint(th)) + lo), &sn, &cs);
      E[0][tid] = cs;
      E[1][tid] = sn;
    }
    __syncthreads();
    for (int e = tid; e < P * ZB_NC; e += 256) {
      const int p = e / ZB_NC, i = e % ZB_NC;
      if (i < ni) K[p][i] = J[p * nzt + i0 + i] * E[p & 1][i];
    }
    __syncthreads();
    // a thread per column pair; FP64 results (P = 16) hold row g + 4 r in
    // register r of lane group g
    for (int c = tid; c < ncu; c += 256) {
      double a[P];
      double* o = H + (((size_t)bin * ncu + c) * nlayers + L) * P;
#pragma unroll
      for (int p = 0; p < P; ++p) a[p] = i0 ? o[P == 16 ? (p & 3) * 4 + (p >> 2) : p] : 0.0;
#pragma unroll 2
      for (int i = 0; i < ni; ++i) {
        const double wn = w[(size_t)(i0 + i) * ncu + c];
#pragma unroll
        for (int p = 0; p < P; ++p) a[p] += wn * K[p][i];
      }
#pragma unroll
      for (int p = 0; p < P; ++p) o[P == 16 ? (p & 3) * 4 + (p >> 2) : p] = a[p];
    }
  }
}

// ---------------------------------------------------------------------------
// D and its contraction with H.  The matrix-core product of rows (T_p q cos
// kx x, T_p q sin kx x) with columns (cos ky y, sin ky y) over the charges, in
// FP64 with P = 16, or in FP32 (b stored in FP32) with P = 8 on narrower bins:
// one 16-row block then holds both cos and sin rows.  A workgroup takes one
// item (NC <= 2 blocks of 8 n_y and up to 8 NU <= 16 values of n_x) and one part
// of the sorted charges.  Its eight waves share tiles of 64 (FP32: 128) charges
// in LDS (powers of e^{2 pi i fx} and e^{2 pi i fy} in FP64 from one sincospi
// each, T_p by the recurrence, stored as T); every wave runs NU values of n_x
// against the 16 NC columns.  Two tiles alternate: while one is multiplied the
// next is formed, half of the waves forming first and half multiplying first,
// so that each SIMD has vector and matrix work at any time, and one barrier per
// tile is enough.  Where the part crosses a bin boundary the sums are
// contracted with the bin's H in FP64; a transposing reduction over the lane
// groups that share a result leaves each group planes of its own.
//
// FP32 sums run over ZB_CHAIN charges (16 for the lowest n_x, whose weights are
// the largest), then go to FP64; all sums are contracted after ZB_SEG charges at
// the latest.  The column (0, 0) has the largest weights of all and unit phases (the same few charge values are added
// over and over, so the rounding of its sums does not average out): its D is
// summed in FP64 on the vector units by the threads that form T_p.
//
// What bounds it: the matrix cores in FP64 (3.6 of 4.3 ms of the 7176-atom case
// with the forming taken out, at 46 of the 67 TFLOP/s that FP64 products reach
// with two waves per SIMD; the forming shares the FP64 units), latency and the
// forming in FP32 (0.07 of 0.12 ms without the products at 2880 atoms).
//
//   part[(s nparts + part) ppart + ((unit nlayers + L) 2 + a) 16 + col],
// unit: (n_x, 8 consecutive n_y); a = 0: cos kx x, 1: sin kx x;
// col = 2 (n_y - n_y0) + (0: cos ky y, 1: sin ky y).
// ---------------------------------------------------------------------------
constexpr int ZB_W = 8;                // waves per workgroup
constexpr int ZB_CHAIN = 128;          // charges summed in FP32
constexpr int ZB_SEG = 1024;           // charges summed before a contraction (rounding of long sums)

__device__ inline double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ inline double2 zpow(double2 z, int n) {
  double2 r = make_double2(1.0, 0.0);
  while (true) {
    if (n & 1) r = zmul(r, z);
    n >>= 1;
    if (!n) return r;
    z = zmul(z, z);
  }
}

// v of lane l ^ o
__device__ inline double xor_lane(double v, int o) { return __shfl_xor(v, o, 64); }

struct ZbArgs {
  int g, m, mpad64, nparts, nbins, ncu, nlayers, ppart, lgroups;
  const ZbItem* items;
  const int4* cu_of;
  const double4* cq;
  const int* binoff;
  double Lx, Ly, Lz;
  const double* H;
  double* part;
};

template <typename T> struct Zb;
template <> struct Zb<double> {
  // RB: row blocks (cos, sin); pitch: rows 8 banks apart
  static constexpr int P = 16, RB = 2, TJ = 64, PITCH = TJ + 4;
  typedef v4d acc;
  double X[ZB_NX][TJ][2];
  double B[P][PITCH];
  double Y[32][PITCH];
  static __device__ inline v4d mma(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <> struct Zb<float> {
  // one row block: rows 8 a + p; pitch: rows 4 banks apart
  static constexpr int P = 8, RB = 1, TJ = 128, PITCH = TJ + 4;
  typedef v4f acc;
  float X[ZB_NX][2][PITCH];
  float B[P][PITCH];
  float Y[32][PITCH];
  static __device__ inline v4f mma(float a, float b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

template <typename T, int NU, int NC, int NK>
__device__ inline void zb_item(const ZbArgs& A, const ZbItem it, int pt, int s, int lgroup, Zb<T>* W,
                               const int* bo, double* red) {
  typedef Zb<T> Z;
  typedef typename Z::acc acc_t;
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int P = Z::P, RB = Z::RB, TJ = Z::TJ;
  constexpr int NG = 64 * ZB_W / TJ;                         // thread groups that form a tile
  constexpr int HG = NG / 2;                                 // one half forms Y, one X
  constexpr int QB = P / NG, QY = 8 * NC / HG, QX = 8 * NU / HG;   // rows of each
  constexpr int NL = F32 ? 2 : 4;                            // planes per reduction
  constexpr int UB = F32 ? NU : 1;                           // units whose H is loaded together
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l15 = lane & 15, lg = lane >> 4;
  const int jl = tid & (TJ - 1), grp = wave / (TJ / 64);     // charge and group when forming
  const bool up = lane & 32, mid = lane & 16;
  const int nlayers = A.nlayers, nbins = A.nbins;
  const int L0 = lgroup * NL * NK;
  const double4* cq = A.cq + (size_t)s * A.mpad64;
  const bool col00 = F32 && it.nxa == 0 && it.ny0 == 0;
  // byte offsets of this lane's H (32 bits: a bin's H stays below 2^31 bytes)
  unsigned ho[NU][NC];
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int4 cu = A.cu_of[it.nxa + min(wave * NU + u, it.nxn - 1)];
      ho[u][c] = (unsigned)((cu.x + min(it.ny0 + 8 * c + (l15 >> 1), cu.y - 1)) * nlayers) *
                     (unsigned)(P * sizeof(double)) + 32u * (F32 ? lg & 1 : lg);
    }
  acc_t acc[NU][NC][RB];
  v4d dac[F32 ? NU : 1][NC];
  double tac[NU][NC][RB][NK];
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (F32) dac[F32 ? u : 0][c] = (v4d){0, 0, 0, 0};
#pragma unroll
      for (int a = 0; a < RB; ++a) {
        acc[u][c][a] = (acc_t){0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < NK; ++k) tac[u][c][a][k] = 0.0;
      }
    }
  const int ja = (int)((long long)A.m * pt / A.nparts);
  const int je = (int)((long long)A.m * (pt + 1) / A.nparts);
  const double invLx = 1.0 / A.Lx, invLy = 1.0 / A.Ly, invLz = 1.0 / A.Lz;
  const double bw = A.Lz / nbins, ihw = 2.0 * nbins / A.Lz;
  double s00[QB] = {}, t00[F32 ? NL * NK : 1] = {};
  // a tile: charges j .. j + nt of one bin (the tile after it starts at j + nt)
  struct Tile { int j, nt, bin, seg; };                      // seg: where its sums began
  auto tile_at = [&](int j, int bin, int seg) {
    if (bin + 1 < nbins && bo[bin + 1] <= j) {
      seg = j;
      do ++bin; while (bin + 1 < nbins && bo[bin + 1] <= j);
    }
    if (j - seg >= ZB_SEG) seg = j;
    const int jb = bin + 1 < nbins ? min(je, bo[bin + 1]) : je;
    return Tile{j, min(TJ, jb - j), bin, seg};
  };
  double4 v = make_double4(0.0, 0.0, 0.0, 0.0);
  auto load = [&](int j) {
    if (j + jl < je) v = cq[j + jl];
  };
  double d00[QB];                                            // the tile's share of D(0, 0)
  auto form = [&](Zb<T>& B, const Tile& t) {
    const bool in = jl < t.nt;                               // charges of the next bin: zero
    const double qj = in ? v.w : 0.0;
    {
      const bool isy = grp < HG;
      const int g2 = isy ? grp : grp - HG;
      double sn, cs;
      sincospi(2.0 * (isy ? v.y * invLy : v.x * invLx), &sn, &cs);
      const double2 e1 = make_double2(cs, sn);
      double2 p = zpow(e1, isy ? it.ny0 + QY * g2 : it.nxa + QX * g2);
      if (isy) {
#pragma unroll
        for (int k = 0; k < QY; ++k) {
          B.Y[2 * (QY * g2 + k)][jl] = (T)p.x;
          B.Y[2 * (QY * g2 + k) + 1][jl] = (T)p.y;
          if (k + 1 < QY) p = zmul(p, e1);
        }
      } else {
        p.x *= qj;
        p.y *= qj;
#pragma unroll
        for (int k = 0; k < QX; ++k) {
          if constexpr (F32) {
            B.X[QX * g2 + k][0][jl] = (T)p.x;
            B.X[QX * g2 + k][1][jl] = (T)p.y;
          } else {
            *reinterpret_cast<double2*>(B.X[QX * g2 + k][jl]) = p;
          }
          if (k + 1 < QX) p = zmul(p, e1);
        }
      }
    }
    {
      const double tz = in ? from_centre(v.z, A.Lz, invLz, t.bin, bw) * ihw : 0.0;
      double a = 1.0, b = tz;                                // T_0, T_1
      for (int k = 0; k < grp * QB; ++k) {
        const double c = 2.0 * tz * b - a;
        a = b;
        b = c;
      }
#pragma unroll
      for (int k = 0; k < QB; ++k) {
        B.B[grp * QB + k][jl] = (T)a;
        d00[k] = qj * a;
        const double c = 2.0 * tz * b - a;
        a = b;
        b = c;
      }
    }
    load(t.j + t.nt);
  };
  // products of 16 charges per round, in two halves: one half's operands are
  // read while the other half is multiplied
  struct Ops { T y[2][NC], b[2], x[2][NU][F32 ? 1 : 2]; };
  auto read = [&](const Zb<T>& B, int k0) {
    Ops o;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int kc = k0 + 4 * ks + lg;
#pragma unroll
      for (int c = 0; c < NC; ++c) o.y[ks][c] = B.Y[16 * c + l15][kc];
      o.b[ks] = B.B[F32 ? l15 & 7 : l15][kc];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if constexpr (F32) {
          o.x[ks][u][0] = B.X[wave * NU + u][l15 >> 3][kc];
        } else {
          const double2 x = *reinterpret_cast<const double2*>(B.X[wave * NU + u][kc]);
          o.x[ks][u][0] = x.x;
          o.x[ks][u][RB - 1] = x.y;
        }
      }
    }
    return o;
  };
  auto mma = [&](const Ops& o) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int a = 0; a < RB; ++a) {
          const T r = o.b[ks] * o.x[ks][u][a];
#pragma unroll
          for (int c = 0; c < NC; ++c) acc[u][c][a] = Z::mma(r, o.y[ks][c], acc[u][c][a]);
        }
  };
  // FP32 sums to FP64
  auto flush = [&]() {
    if constexpr (F32)
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
          for (int r = 0; r < 4; ++r) dac[u][c][r] += (double)acc[u][c][0][r];
          acc[u][c][0] = (acc_t){0, 0, 0, 0};
        }
  };
  const bool low = F32 && it.nxa + wave * NU < 2;            // largest weights: short chains
  auto multiply = [&](const Zb<T>& B, int nt) {
    Ops o = read(B, 0);
    for (int k0 = 0; k0 < nt; k0 += 16) {
      const Ops e = read(B, k0 + 8);
      mma(o);
      o = read(B, min(k0 + 16, TJ - 8));
      mma(e);
      if (low) flush();
    }
  };
  auto contract = [&](int bin) {
    const char* hb = reinterpret_cast<const char*>(A.H + (size_t)bin * A.ncu * nlayers * P);
    constexpr int HS = P * sizeof(double);
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
      for (int u0 = 0; u0 < NU; u0 += UB) {
        double2 h[UB][NC][NL][2];
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int i = 0; i < NL; ++i) {
              const char* hl = hb + min(L0 + NL * k + i, nlayers - 1) * HS;
              const double2* hp = reinterpret_cast<const double2*>(hl + ho[u0 + u][c]);
              h[u][c][i][0] = hp[0];
              h[u][c][i][1] = hp[1];
            }
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int a = 0; a < RB; ++a) {
              double d[4], t[NL];
#pragma unroll
              for (int r = 0; r < 4; ++r)
                d[r] = F32 ? dac[F32 ? u0 + u : 0][c][r] : (double)acc[u0 + u][c][a][r];
#pragma unroll
              for (int i = 0; i < NL; ++i)
                t[i] = h[u][c][i][0].x * d[0] + h[u][c][i][0].y * d[1] + h[u][c][i][1].x * d[2] +
                       h[u][c][i][1].y * d[3];
              if constexpr (F32) {
                tac[u0 + u][c][a][k] += (mid ? t[1] : t[0]) + xor_lane(mid ? t[0] : t[1], 16);
              } else {
                const double e = (up ? t[2] : t[0]) + xor_lane(up ? t[0] : t[2], 32);
                const double f = (up ? t[3] : t[1]) + xor_lane(up ? t[1] : t[3], 32);
                tac[u0 + u][c][a][k] += (mid ? f : e) + xor_lane(mid ? e : f, 16);
              }
            }
        __builtin_amdgcn_sched_barrier(0);                   // one group's H in flight: registers
      }
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (F32) dac[F32 ? u : 0][c] = (v4d){0, 0, 0, 0};
#pragma unroll
        for (int a = 0; a < RB; ++a) acc[u][c][a] = (acc_t){0, 0, 0, 0};
      }
    if (F32 && col00) {
      // column (0, 0): this lane's charges, p = grp QB ..
#pragma unroll
      for (int i = 0; i < (F32 ? NL * NK : 1); ++i) {
        const double* h =
            reinterpret_cast<const double*>(hb + min(L0 + i, nlayers - 1) * HS) + grp * QB;
#pragma unroll
        for (int k = 0; k < QB; ++k) t00[i] += h[k] * s00[k];
      }
    }
  };
  if (ja < je) {
    // the bin of charge ja: the last with bo <= ja (empty bins share offsets)
    int bin = -1;
    for (int b0 = 0; b0 < nbins; b0 += 64)
      bin += __popcll(__ballot(b0 + lane < nbins && bo[min(b0 + lane, nbins - 1)] <= ja));
    load(ja);
    Tile cur = tile_at(ja, bin, ja);
    form(W[0], cur);
#pragma unroll
    for (int k = 0; k < QB; ++k) s00[k] = d00[k];
    __syncthreads();
    int buf = 0, chain = 0;
    while (true) {
      const bool more = cur.j + cur.nt < je;
      const Tile nxt = more ? tile_at(cur.j + cur.nt, cur.bin, cur.seg) : cur;
      if (more && wave < ZB_W / 2) form(W[buf ^ 1], nxt);
      multiply(W[buf], cur.nt);
      if (more && wave >= ZB_W / 2) form(W[buf ^ 1], nxt);
      const bool end = !more || nxt.seg != cur.seg;
      if constexpr (F32) {
        chain += cur.nt;
        if (end || chain >= ZB_CHAIN) {
          chain = 0;
          flush();
        }
      }
      if (end) contract(cur.bin);
      if (!more) break;
#pragma unroll
      for (int k = 0; k < QB; ++k) s00[k] = end ? d00[k] : s00[k] + d00[k];
      __syncthreads();
      cur = nxt;
      buf ^= 1;
    }
  }
  double* out = A.part + ((size_t)s * A.nparts + pt) * A.ppart;
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    if (wave * NU + u >= it.nxn) continue;
    const int4 cu = A.cu_of[it.nxa + wave * NU + u];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int ny = it.ny0 + 8 * c;
      if (ny >= cu.y) continue;
#pragma unroll
      for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int a = 0; a < RB; ++a) {
          const int L = L0 + NL * k + (F32 ? lg & 1 : lg), ai = F32 ? lg >> 1 : a;
          if (L < nlayers)
            out[(((size_t)(cu.z + ny / 8) * nlayers + L) * 2 + ai) * 16 + l15] = tac[u][c][a][k];
        }
    }
  }
  if (col00) {                                               // unit 0, a = 0, col = 0
#pragma unroll
    for (int i = 0; i < (F32 ? NL * NK : 1); ++i) {
      double d = t00[i];
      for (int o = 32; o > 0; o >>= 1) d += xor_lane(d, o);
      if (lane == i) red[wave * 64 + lane] = d;
    }
    __syncthreads();
    if (wave == 0 && lane < min(nlayers - L0, NL * NK)) {
      double t = 0.0;
      for (int w = 0; w < ZB_W; ++w) t += red[64 * w + lane];
      out[(size_t)(L0 + lane) * 32] = t;
    }
  }
}

template <typename T>
struct ZbLds {
  Zb<T> W[2];
  int bo[ZB_MAXSORT];
  double red[sizeof(T) == 4 ? 64 * ZB_W : 1];
};

// The sums of nsum workgroups; WITH_RS: and after them the real-space pair sums of
// R.nx * R.ny * R.nz.  For few configurations, whose sums leave CUs idle: on a
// second stream beside the sums the pair sums cost two event waits, and a single
// configuration of 2880 atoms takes 75 us per step instead of 90 (replayed, where the
// streams cannot overlap, 85 instead of 105).
template <typename T, int NK, bool WITH_RS>
__global__ void __launch_bounds__(64 * ZB_W) k_zb_sums(const ZbArgs A, int nsum, const RpArgs R) {
  constexpr size_t lds = WITH_RS && sizeof(RpLds) > sizeof(ZbLds<T>) ? sizeof(RpLds) : sizeof(ZbLds<T>);
  __shared__ __align__(16) char raw[lds];
  if constexpr (WITH_RS) {
    static_assert(RP_WAVES == ZB_W, "one workgroup size");
    if ((int)blockIdx.x >= nsum) {
      const int b = blockIdx.x - nsum, by = b / R.nx % R.ny, bz = b / (R.nx * R.ny);
      RpLds& l = *reinterpret_cast<RpLds*>(raw);
      if (R.Lx >= 2.0 * R.rc && R.Ly >= 2.0 * R.rc)
        rp_body<false>(R, b % R.nx, by, bz, l);
      else
        rp_body<true>(R, b % R.nx, by, bz, l);
      return;
    }
  }
  ZbLds<T>& S = *reinterpret_cast<ZbLds<T>*>(raw);
  // the item varies slowest (consecutive workgroups go to different XCDs: an
  // item index that varies fastest would give each XCD one kind of item), the
  // largest items first
  const int per = nsum / A.lgroups, b0 = blockIdx.x % per, lgroup = blockIdx.x / per;
  const int pt = b0 % A.nparts, rest = b0 / A.nparts;
  const int s = rest % A.g, wg = rest / A.g;
  const ZbItem it = A.items[wg];
  for (int b = threadIdx.x; b < A.nbins; b += 64 * ZB_W)
    S.bo[b] = A.binoff[(size_t)s * (A.nbins + 1) + b];
  __syncthreads();
  switch (it.shape) {                                        // NU + 2 (NC - 1)
    case 1: zb_item<T, 1, 1, NK>(A, it, pt, s, lgroup, S.W, S.bo, S.red); break;
    case 2: zb_item<T, 2, 1, NK>(A, it, pt, s, lgroup, S.W, S.bo, S.red); break;
    case 3: zb_item<T, 1, 2, NK>(A, it, pt, s, lgroup, S.W, S.bo, S.red); break;
    default: zb_item<T, 2, 2, NK>(A, it, pt, s, lgroup, S.W, S.bo, S.red); break;
  }
}

// T(c, L) of both signs of n_y from the parts (added in order): with
// D_ab = sum q G a(kx x) b(ky y), a, b in {cos, sin},
//   T(n_x, +n_y) = (D_cc - D_ss) + i (D_cs + D_sc),
//   T(n_x, -n_y) = (D_cc + D_ss) + i (D_sc - D_cs).
// Written as the right-hand operand of the projection,
// Tcat[(L M2 + 2 c + (0: Re, 1: Im)) 64 + s].  One workgroup per (unit, plane);
// with few configurations the parts are split over the thread groups.  The
// workgroups (unit = nunits, plane 0) sum the dipole partials instead.
constexpr int ZR_S = 16;               // configurations per workgroup

__global__ void __launch_bounds__(256) k_zb_reduce(int g, int nunits, int nlayers, int nparts,
                                                   int ppart, const int2* __restrict__ units,
                                                   const int4* __restrict__ cu_of,
                                                   const int2* __restrict__ cols,
                                                   const double* __restrict__ part, int M2,
                                                   double* __restrict__ Tcat, int dblk,
                                                   const double* __restrict__ dip,
                                                   double* __restrict__ dtot) {
  const int unit = blockIdx.x, L = blockIdx.y, tid = threadIdx.x;
  if (unit == nunits) {
    if (L || blockIdx.z) return;
    const int lane = tid & 63;
    for (int s = tid >> 6; s < g; s += 4) {
      double v[3] = {0.0, 0.0, 0.0};
      for (int b = lane; b < dblk; b += 64)
#pragma unroll
        for (int d = 0; d < 3; ++d) v[d] += dip[((size_t)s * dblk + b) * 3 + d];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        for (int o = 32; o > 0; o >>= 1) v[d] += __shfl_xor(v[d], o, 64);
        if (lane == 0) dtot[s * 3 + d] = v[d];
      }
    }
    return;
  }
  // this workgroup's configurations sb .. sb + ns (ns <= ZR_S)
  const int sb = blockIdx.z * ZR_S, ns = min(ZR_S, g - sb);
  __shared__ double sm[32][ZR_S + 1];
  __shared__ double sl_sum[8][32];
  const int val = tid & 31, k = tid >> 5;
  const double* src = part + ((size_t)unit * nlayers + L) * 32 + val + (size_t)sb * nparts * ppart;
  const int nsl = ns < 8 ? 8 / ns : 1;                       // part slices per configuration
  if (nsl > 1) {
    const int s = k % ns, sl = k / ns;
    double a = 0.0;
    if (sl < nsl) {
      const int p0 = nparts * sl / nsl, p1 = nparts * (sl + 1) / nsl;
#pragma unroll 8
      for (int p = p0; p < p1; ++p) a += src[((size_t)s * nparts + p) * ppart];
    }
    sl_sum[k][val] = a;
    __syncthreads();
    if (sl == 0) {
      for (int i = 1; i < nsl; ++i) a += sl_sum[s + i * ns][val];
      sm[val][s] = a;
    }
  } else {
    for (int s = k; s < ns; s += 8) {
      double a = 0.0;
#pragma unroll 8
      for (int p = 0; p < nparts; ++p) a += src[((size_t)s * nparts + p) * ppart];
      sm[val][s] = a;
    }
  }
  __syncthreads();
  const int2 un = units[unit];
  const int4 cu = cu_of[un.x];
  const int s = tid % ZR_S;
  if (s >= ns) return;
  for (int i = tid / ZR_S; i < 8; i += 256 / ZR_S) {
    const int ny = un.y * 8 + i;
    if (ny >= cu.y) break;
    const double cc = sm[2 * i][s], cs = sm[2 * i + 1][s], sc = sm[16 + 2 * i][s],
                 ss = sm[16 + 2 * i + 1][s];
    const int2 c = cols[cu.x + ny];                          // sorted columns of +n_y, -n_y
    if (c.x >= 0) {
      double* o = Tcat + ((size_t)L * M2 + 2 * c.x) * 64 + sb + s;
      o[0] = cc - ss;
      o[64] = cs + sc;
    }
    if (c.y >= 0) {
      double* o = Tcat + ((size_t)L * M2 + 2 * c.y) * 64 + sb + s;
      o[0] = cc + ss;
      o[64] = sc - cs;
    }
  }
}

}  // namespace

// half width of the z bins: the largest for which the Chebyshev remainder of
// G_c after P terms stays below tol of its largest weight,
//   max_{k <= k_c} e^{-k^2 / 4 alpha^2} 2 (k hw / 2)^P / P! <= tol
double zb_half_width(double alpha, double kc, int P, double tol) {
  const double k = std::min(kc, alpha * std::sqrt(2.0 * P));
  double lf = 0.0;
  for (int i = 2; i <= P; ++i) lf += std::log((double)i);
  return 2.0 / k * std::exp((std::log(0.5 * tol) + lf + k * k / (4.0 * alpha * alpha)) / P);
}

// factors (2 - delta_p0) (-1)^floor((p + 1) / 2) J_p(pi n / nbins) at [p nzt + i], p < P,
// n = nzt - 1 - i (pi n / nbins = n kz1 hw); J_p by Miller's downward recurrence, normalised by
// J_0 + 2 (J_2 + J_4 + ..) = 1
void zb_bessel_factors(int nzt, int nbins, int P, std::vector<double>& out) {
  out.assign((size_t)nzt * P, 0.0);
  out[nzt - 1] = 1.0;                                // n = 0: J_0 alone
  std::vector<double> j;
  for (int n = 1; n < nzt; ++n) {
    const double x = M_PI * n / nbins;
    const int top = 2 * (((int)x + P + 40) / 2);     // J_top / J_P below 1e-30 for P <= 16
    j.assign(top + 2, 0.0);
    j[top] = 1e-300;
    double norm = 0.0;
    for (int k = top; k > 0; --k) {
      j[k - 1] = 2.0 * k / x * j[k] - j[k + 1];
      if (std::fabs(j[k - 1]) > 1e200) {             // keep within range
        for (int i = k - 1; i <= top; ++i) j[i] *= 1e-300;
        norm *= 1e-300;
      }
      if (k - 1 > 0 && (k - 1) % 2 == 0) norm += 2.0 * j[k - 1];
    }
    norm += j[0];
    for (int p = 0; p < P; ++p)
      out[(size_t)p * nzt + nzt - 1 - n] = (p ? 2.0 : 1.0) * ((p + 1) / 2 % 2 ? -1.0 : 1.0) * j[p] / norm;
  }
}

int zb_sort_blocks(int m) { return std::max(1, (m + ZS_BLK - 1) / ZS_BLK); }

void launch_zb_sort(hipStream_t st, int g, int m, int mpad64, const ZbTable& t, double Lx,
                    double Ly, double Lz, const double* xyz, const double* q, int* counts,
                    double4* cq, double2* zr, int* binoff, double* dip) {
  const int nblk = zb_sort_blocks(m);
  int nbits = 1;
  while ((1 << nbits) <= t.nsort) ++nbits;
  const dim3 grid(nblk, g), block(64 * ZS_W);
  if (nblk <= 2) {
    hipLaunchKernelGGL(k_zb_scatter<true>, grid, block, 0, st, m, mpad64, t.nsort, nbits, t.sub,
                       t.nbins, Lx, Ly, Lz, xyz, q, counts, cq, zr, binoff, dip);
    return;
  }
  hipLaunchKernelGGL(k_zb_count, grid, block, 0, st, m, t.nsort, Lz, xyz, counts);
  hipLaunchKernelGGL(k_zb_scatter<false>, grid, block, 0, st, m, mpad64, t.nsort, nbits, t.sub,
                     t.nbins, Lx, Ly, Lz, xyz, q, counts, cq, zr, binoff, dip);
}

void launch_zb_response(hipStream_t st, int ncu, int nzt, int nbins, int nlayers, int P,
                        const double* w, const double* J, const double* layer_z, double Lz, double* H) {
  hipLaunchKernelGGL((P == 16 ? k_zb_response<16> : k_zb_response<8>), dim3(nbins, nlayers),
                     dim3(256), 0, st, ncu, nzt, nbins, nlayers, w, J, layer_z, Lz, H);
}

template <bool WITH_RS>
static void zb_sums_launch(hipStream_t st, bool f32, int nk, int grid, const ZbArgs& a, int nsum,
                           const RpArgs& r) {
  const dim3 block(64 * ZB_W);
  if (f32)
    hipLaunchKernelGGL((nk == 1 ? k_zb_sums<float, 1, WITH_RS> : nk == 2 ? k_zb_sums<float, 2, WITH_RS>
                        : nk == 3 ? k_zb_sums<float, 3, WITH_RS> : k_zb_sums<float, 4, WITH_RS>),
                       dim3(grid), block, 0, st, a, nsum, r);
  else
    hipLaunchKernelGGL((nk == 1 ? k_zb_sums<double, 1, WITH_RS> : k_zb_sums<double, 2, WITH_RS>),
                       dim3(grid), block, 0, st, a, nsum, r);
}

void launch_zb_sums(hipStream_t st, int g, bool f32, const ZbPlan& z, const ZbTable& t,
                    const ZbItems& I, int m, int mpad64, int nparts, int nlayers,
                    const double4* cq, const int* binoff, double Lx, double Ly, double Lz,
                    double* part, const RpArgs* rs) {
  // planes kept per lane: up to 4 pairs (FP32) or 2 quadruples per workgroup
  const int nl = f32 ? 2 : 4, nk = std::min(f32 ? 4 : 2, (nlayers + nl - 1) / nl);
  const int lgroups = (nlayers + nl * nk - 1) / (nl * nk);
  const ZbArgs a{g, m, mpad64, nparts, t.nbins, z.ncu, nlayers, z.nunits * nlayers * 32, lgroups,
                 I.d_items, z.d_cu_of, cq, binoff, Lx, Ly, Lz, t.H, part};
  const int nsum = I.nwg * nparts * g * lgroups;
  if (rs)
    zb_sums_launch<true>(st, f32, nk, nsum + rs->nx * rs->ny * rs->nz, a, nsum, *rs);
  else
    zb_sums_launch<false>(st, f32, nk, nsum, a, nsum, RpArgs{});
}

void launch_zb_reduce(hipStream_t st, int g, const ZbPlan& z, int nlayers, int nparts,
                      const double* part, int M2, double* Tcat, int dblk, const double* dip,
                      double* dtot) {
  hipLaunchKernelGGL(k_zb_reduce, dim3(z.nunits + 1, nlayers, (g + ZR_S - 1) / ZR_S), dim3(256), 0, st, g, z.nunits,
                     nlayers, nparts, z.nunits * nlayers * 32, z.d_units, z.d_cu_of, z.d_cols,
                     part, M2, Tcat, dblk, dip, dtot);
}

}  // namespace cpm
