// Real-space pair sum of planar electrodes (device code of the kernels that run
// it: alone, or beside the k-space sums of few configurations).
#pragma once

#include "cpm_internal.h"

namespace cpm {

// One wave per 64 atom-map slots of one z plane (slot tiles are compact in
// x and y).  The charges of a chunk arrive 64 at a time (z-sorted blocks; a
// block whose z range misses [z_p - rc, z_p + rc] is skipped unread).  A
// charge within rc of the plane in z is taken relative to the tile centre,
// in each image that can come within rc of the tile's bounding box (x, y
// shifted by at most one cell length; MULTI, for cells shorter than 2 rc: every
// x and y image in reach; the general kernel tries all of them for every atom,
// 150 us against 19 us for one configuration of 288 atoms and 100 charges), and
// appended to the wave's ring of 128 entries:
//   FP32  (-2 dx, -2 dy) and W = dx^2 + dy^2 - (rc^2 - dz^2) - margin, so that
//         an atom at (ax, ay) from the centre is within rc when
//         ax (-2 dx) + ay (-2 dy) + W + (ax^2 + ay^2) < 0  (screen, margin
//         above its rounding error);
//   FP64  (dx, dy, dz^2, q) for the exact test and g.
// Every 64 entries each lane screens them into a 64-bit mask and evaluates
// the marked ones in FP64 (s < rc^2 exactly; the others take the zero polynomial
// after the table's last).  The summation order of an atom is fixed by the data
// (deterministic).
// What bounds it: LDS broadcasts and the vector issue slots together (the FP64 step
// of a wave is about 41 instructions, of whose lanes 64 to 78 % have a pair left),
// at 2.6 of 4 possible waves per SIMD.  So the screen, a 64 x 64 product of depth 3,
// is taken on the matrix cores (32x32x2 FP32 twice per quarter: the entries arrive
// as operands instead of as one broadcast per entry and lane; sign bits become each
// lane's mask), and the other images of a block are looked at only where one of them
// can reach the tile.  The kernel alone: 20064 atoms, one configuration, 288 to
// 250 us (283 with the instructions cut but the broadcasts left); 2880 atoms, 64
// configurations, 78 to 70 us.
constexpr int RP_RING = 128, RP_WAVES = 8;
typedef float f16v __attribute__((ext_vector_type(16)));
struct RpWave {
  float c[2][RP_RING], w[RP_RING];
  double2 d[2][RP_RING];                             // (16-byte pitch: all banks)
};
struct RpLds {
  double tab[(RP_N + 1) * RP_REC];
  RpWave w[RP_WAVES];
};

// order LDS accesses of one wave (its lanes run in step; no workgroup barrier)
__device__ inline void rp_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <bool MULTI>
__device__ __forceinline__ void rp_body(const RpArgs& A, int bx, int by, int bz, RpLds& lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int slot = bx * (64 * RP_WAVES) + threadIdx.x;
  const int atom = slot < A.nmap ? A.amap[slot] : -1;
  const int m = A.m, chunk = by / A.sub, rchunks = A.ny / A.sub;
  const bool mine = lane / (64 / A.sub) == by % A.sub;   // this workgroup's part of a block
  const int nb64 = A.mpad64 / 64, nbt = (m + 63) / 64;
  for (int t = threadIdx.x; t < (RP_N + 1) * RP_REC / 2; t += 64 * RP_WAVES)
    reinterpret_cast<double2*>(lds.tab)[t] =
        t < RP_N * RP_REC / 2 ? reinterpret_cast<const double2*>(A.ptab)[t] : make_double2(0.0, 0.0);
  __syncthreads();
  const unsigned long long valid_atoms = __ballot(atom >= 0);
  if (!valid_atoms) return;                      // a wave of padding slots only
  const double Lx = A.Lx, Ly = A.Ly, Lz = A.Lz, rc = A.rc;
  const double invLx = 1.0 / Lx, invLy = 1.0 / Ly, invLz = 1.0 / Lz, rc2 = rc * rc;
  double xi = 0, yi = 0, zi = 0;
  if (atom >= 0) { xi = A.ex[atom]; yi = A.ey[atom]; zi = A.ez[atom]; }
  xi -= Lx * floor(xi * invLx);
  yi -= Ly * floor(yi * invLy);
  // the plane's z (every atom of the wave shares it) and the tile's box
  const int first = __ffsll((long long)valid_atoms) - 1;
  const double zp = __shfl(zi, first, 64);
  double xlo = atom >= 0 ? xi : 1e300, xhi = atom >= 0 ? xi : -1e300;
  double ylo = atom >= 0 ? yi : 1e300, yhi = atom >= 0 ? yi : -1e300;
  for (int o = 32; o > 0; o >>= 1) {
    xlo = fmin(xlo, __shfl_xor(xlo, o, 64));
    xhi = fmax(xhi, __shfl_xor(xhi, o, 64));
    ylo = fmin(ylo, __shfl_xor(ylo, o, 64));
    yhi = fmax(yhi, __shfl_xor(yhi, o, 64));
  }
  const double cx = 0.5 * (xlo + xhi), cy = 0.5 * (ylo + yhi);
  const double hx = 0.5 * (xhi - xlo), hy = 0.5 * (yhi - ylo);
  const double ax = xi - cx, ay = yi - cy;
  // screen by MFMA, rows = 32 entries (-2 dx, -2 dy, W, 1), columns = 32 atoms (ax, ay,
  // 1, ax^2 + ay^2): a lane's left operand is of ring entry e0 (+ 16 per tile of rows),
  // placed so that result register r of tile T is entry 32 (lane / 32) + 16 T + r
  const float axf = (float)ax, ayf = (float)ay, Af = (float)(ax * ax + ay * ay);
  const int l31 = lane & 31, e0 = 32 * ((l31 >> 2) & 1) + 4 * (l31 >> 3) + (l31 & 3);
  float b1[2], b2[2];
#pragma unroll
  for (int S = 0; S < 2; ++S) {
    const float x = __shfl(axf, 32 * S + l31, 64), y = __shfl(ayf, 32 * S + l31, 64);
    const float a = __shfl(Af, 32 * S + l31, 64);
    b1[S] = lane < 32 ? x : y;
    b2[S] = lane < 32 ? 1.f : a;
  }
  // FP32 screen margin: its rounding error is below 50 u M^2 (u = 2^-24,
  // M the largest coordinate magnitude, rc + the tile's half extent)
  const double M = rc + fmax(hx, hy);
  const double marg = 4e-6 * M * M;
  RpWave& W = lds.w[wave];
  const float inv_hf = (float)(RP_N / rc);
  const double hh = (rc / RP_N) * (rc / RP_N);   // s_mid of interval k: hh (k (k + 1) + 1/2)
  const int nblk = chunk < nbt ? (nbt - chunk + rchunks - 1) / rchunks : 0;
  const int nloc = bz < A.g ? (A.g - bz + A.nz - 1) / A.nz : 0;
  const double wlo = zp - rc, whi = zp + rc;
  const double ox = Lx - rc - hx - 1e-6, oy = Ly - rc - hy - 1e-6;   // |dx| beyond: a second image
  // does block blk of configuration snap reach the plane's z window?
  auto hit = [&](int snap, int blk) {
    const double2 r = A.zr[(size_t)snap * nb64 + chunk + rchunks * blk];
    const double a = r.x - Lz * floor((r.x - wlo) * invLz), w = r.y - r.x;
    return a < whi + 1e-9 || a + w >= wlo + Lz - 1e-9;
  };
  auto fetch = [&](int snap, int blk) {
    double4 v = make_double4(0, 0, 0, 0);
    if (blk >= 0) {
      const int j = (chunk + rchunks * blk) * 64 + lane;
      if (j < m) v = A.cq[(size_t)snap * A.mpad64 + j];
    }
    return v;
  };
  // screen entries [base, base + len) of the ring and add the marked pairs
  double acc = 0.0;
  auto process = [&](int base, int len) {
    unsigned P[2];                               // entries 32 h + b (h: this lane's half) at bit b
#pragma unroll
    for (int S = 0; S < 2; ++S) {                // for atom 32 S + lane % 32
      unsigned b = 0u;
#pragma unroll
      for (int T = 1; T >= 0; --T) {
        const float a1 = W.c[lane >> 5][base + e0 + 16 * T];
        const float a2 = lane < 32 ? W.w[base + e0 + 16 * T] : 1.f;
        f16v v = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1[S], (f16v){}, 0, 0, 0);
        v = __builtin_amdgcn_mfma_f32_32x32x2f32(a2, b2[S], v, 0, 0, 0);
#pragma unroll
        for (int r = 15; r >= 0; --r)
          b = __builtin_amdgcn_alignbit(b, __float_as_uint(v[r]), 31);   // b << 1 | sign
      }
      P[S] = b;
    }
    const auto lohi = __builtin_amdgcn_permlane32_swap(P[0], P[1], false, false);
    if (atom >= 0) {
      unsigned long long mk = (unsigned long long)lohi[1] << 32 | lohi[0];
      if (len < 64) mk &= (1ull << len) - 1ull;
      while (mk) {
        const int t = __builtin_ctzll(mk);
        mk &= mk - 1ull;
        const double2 exy = W.d[0][base + t], ezq = W.d[1][base + t];
        const double rx = ax - exy.x, ry = ay - exy.y;
        const double sv = fma(rx, rx, fma(ry, ry, ezq.x));
        const float rf = __builtin_amdgcn_sqrtf((float)sv);   // picks the interval only
        const int k = sv < rc2 ? min((int)(rf * inv_hf), RP_N - 1) : RP_N;
        const double* T = lds.tab + __umul24(k, RP_REC);
        const double2 c01 = *reinterpret_cast<const double2*>(T);
        const double2 c23 = *reinterpret_cast<const double2*>(T + 2);
        const float4 c46 = *reinterpret_cast<const float4*>(T + 4);
        const double x = sv - hh * ((double)(__umul24(k, k) + k) + 0.5);   // s - s_mid
        const float xf = (float)x;
        const float th = fmaf(fmaf(c46.z, xf, c46.y), xf, c46.x);       // a6 x^2 + a5 x + a4
        double p = fma((double)th, x, c23.y);
        p = fma(p, x, c23.x);
        p = fma(p, x, c01.y);
        p = fma(p, x, c01.x);
        acc = fma(ezq.y, p, acc);
      }
    }
    rp_lds_sync();                             // the ring's entries are reused next
  };
  // per configuration: the blocks that reach the window, found 64 at a time
  // (one z-range load per lane, no load waits on another), then taken in
  // order with the charges of the next two in flight
  int head = 0, tail = 0;                        // ring window [head, tail), head in {0, 64}
  for (int li = 0; li < nloc; ++li) {
    const int snap = bz + A.nz * li;
    for (int b0 = 0; b0 < nblk; b0 += 64) {
      unsigned long long hm = __ballot(b0 + lane < nblk && hit(snap, b0 + lane));
      auto pop = [&]() {
        if (!hm) return -1;
        const int t = __builtin_ctzll(hm);
        hm &= hm - 1ull;
        return b0 + t;
      };
      int bA = pop(), bB = pop();
      double4 fA = fetch(snap, bA), fB = fetch(snap, bB);
      while (bA >= 0) {
        const int blk = bA;
        const double4 cur = fA;
        bA = bB;
        fA = fB;
        bB = pop();
        fB = fetch(snap, bB);
        const bool valid = mine && (chunk + rchunks * blk) * 64 + lane < m;
        double dz = cur.z - zp;
        dz -= Lz * rint(dz * invLz);
        const double rho2 = rc2 - dz * dz;
        double dx = cur.x - cx, dy = cur.y - cy;
        dx -= Lx * rint(dx * invLx);
        dy -= Ly * rint(dy * invLy);
        // images whose distance from the tile's box can be below sqrt(rho2)
        auto near = [&](double px, double py) {
          const double ux = fmax(fabs(px) - hx, 0.0), uy = fmax(fabs(py) - hy, 0.0);
          return ux * ux + uy * uy < rho2 + marg;
        };
        // append the lanes' images (has), then screen and sum full batches
        auto append = [&](bool has, unsigned long long bal, double px, double py) {
          if (has) {
            const int pos = (tail + __popcll(bal & ((1ull << lane) - 1ull))) & (RP_RING - 1);
            W.c[0][pos] = (float)(-2.0 * px);
            W.c[1][pos] = (float)(-2.0 * py);
            W.w[pos] = (float)(px * px + py * py - rho2 - marg);
            W.d[0][pos] = make_double2(px, py);
            W.d[1][pos] = make_double2(dz * dz, cur.w);
          }
          tail += __popcll(bal);
          rp_lds_sync();
          if (tail - head >= 64) {
            process(head & (RP_RING - 1), 64);
            head += 64;
          }
        };
        if constexpr (MULTI) {
          // every (ia, ib) with |dx + ia Lx| <= reach + hx and the like
          int ia = 0, ib = 0, blo = 0, bhi = -1, ahi = -1;
          if (valid && fabs(dz) < rc) {
            const double reach = rc + 1e-3;
            ia = (int)ceil((-(reach + hx) - dx) * invLx);
            ahi = (int)floor(((reach + hx) - dx) * invLx);
            blo = (int)ceil((-(reach + hy) - dy) * invLy);
            bhi = (int)floor(((reach + hy) - dy) * invLy);
            ib = blo;
          }
          bool more = ia <= ahi && blo <= bhi;
          while (__ballot(more)) {
            const double px = dx + ia * Lx, py = dy + ib * Ly;
            const bool has = more && near(px, py);
            const unsigned long long bal = __ballot(has);
            if (more && ++ib > bhi) {
              ib = blo;
              more = ++ia <= ahi;
            }
            if (bal) append(has, bal, px, py);
          }
        } else {
          // the nearest image; the others are no nearer, and can be in reach only
          // past half a cell
          const bool c0 = valid && fabs(dz) < rc && near(dx, dy);
          const unsigned long long b0 = __ballot(c0);
          if (__ballot(c0 && (fabs(dx) > ox || fabs(dy) > oy))) {
            const double dx2 = dx - copysign(Lx, dx), dy2 = dy - copysign(Ly, dy);
            int cand = 0;
            if (c0)
              cand = 1 | (near(dx2, dy) ? 2 : 0) | (near(dx, dy2) ? 4 : 0) | (near(dx2, dy2) ? 8 : 0);
            while (true) {
              const bool has = cand != 0;
              const unsigned long long bal = __ballot(has);
              if (!bal) break;
              const int which = has ? __builtin_ctz(cand) : 0;
              cand &= cand - 1;
              append(has, bal, (which & 1) ? dx2 : dx, (which & 2) ? dy2 : dy);
            }
          } else if (b0) {
            append(c0, b0, dx, dy);
          }
        }
      }
    }
    if (tail > head) process(head & (RP_RING - 1), tail - head);
    head = tail = 0;
    if (atom >= 0) A.part[((size_t)snap * A.ny + by) * A.n + atom] = acc;
    acc = 0.0;
  }
}

}  // namespace cpm
