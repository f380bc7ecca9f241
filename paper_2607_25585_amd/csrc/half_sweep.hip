// Half sweep: H*v for 1, 2, 4, 8 or 16 columns of a spin-1/2 system (variant 5), over L2 windows
// of 2048-row tiles (Sec. 2.1, Eq. mce-hamop, with the flips of a site as XORs of row bits).
// Several columns are the lowest bits of the row number, which no term moves.
//
// A block of 256 threads holds a tile (row bits 0..10); a thread holds 8 rows, the values
// of three row bits, in one of four layouts:
//   layout            0          1          2          3
//   register bits     8,9,10     5,6,7      2,3,4      0,1,(2)
// A flip of a register bit moves to another register, with a coefficient that is the same
// for the whole block (scalar registers).  So a tile is written to LDS once and read once
// per layout, and each read serves the flips of three sites; every layout has its own
// sums, brought together at the end:
//   - pairs inside the tile: the pair's higher site is a register bit of the layout, the
//     other one a register bit too, or a bit of the lanes (read shifted, one read for up
//     to three pairs): 15 reads per row for the 55 pairs;
//   - pairs (tile site, outer site a): the partner tile (bit a flipped) is loaded once,
//     its layout-0 flips and a's single flip come from registers, the others from 3 reads;
//     the next partner tile loads while the three layouts are worked on, and two tile
//     buffers alternate, so that a site costs one barrier;
//   - pairs of two outer sites: straight from v (L2: both sites lie in the window).
// The single flips of the lanes' sites are read one by one: their coefficients depend on
// all other sites.
//
// LDS position of row r: a linear map of the row bits under which the lanes of every
// layout's read fall on different banks (conflicts: none at complex64, 0.2 % of the cycles at
// complex128).
//
// Measured (one product, all pairs coupled, complex128 / complex64), against a tile of the
// same size whose threads kept to layout 0 and read every flip of a lane's site from LDS:
//   2^19 rows  91 -> 52 / 73 -> 45 us      2^22 rows  571 -> 396 / 298 -> 207 us
//   2^20 rows  125 -> 77 / 90 -> 58 us     2^24 rows  2.67 -> 2.28 / 1.45 -> 1.18 ms
// and, with columns, against the direct gather: 2^19 rows x 4  375 -> 174 / 143 -> 107 us,
// 2^21 x 8  6.6 -> 2.6 / 1.9 -> 1.1 ms.
// What bounds it.  complex128: the partner tiles that come from beyond L2 (2^22 rows: 2.1 GB
// at 5.2 TB/s; 2^24 rows in five passes: 9.5 GB read and 1.7 GB written at 4.9 TB/s) at two
// waves per SIMD, whose registers the four layouts' sums take; vector units 47 % busy, LDS
// 16 %.  complex64: the vector units, 81 % busy (0.9 GB beyond L2 at 4.3 TB/s).
// Lists and coefficients read by scalar loads, with a wait each, and addresses that the
// compiler kept in scratch had made it 590 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <vector>

#include "device_reduce.hpp"
#include "ftlm_internal.hpp"
#include "half_win.hpp"
#include "hv_common.hpp"

namespace ftlm {

namespace {

constexpr int kRows = 8;               // rows per thread
constexpr int kTile = kRows * kBlock;  // rows per tile
static_assert(kTile == 1 << kTileBits, "tile rows");

__device__ __forceinline__ constexpr uint32_t lds_pos(uint32_t r) {
  const uint32_t b4 = (r >> 4) & 1, b5 = (r >> 5) & 1, b6 = (r >> 6) & 1, b7 = (r >> 7) & 1;
  return r ^ (b4 | (b6 << 1) | (b5 << 2) | (b6 << 3) | (b7 << 4));
}
// tile row of thread t / of register q in layout L
template <int L>
__device__ __forceinline__ constexpr uint32_t row_t(uint32_t t) {
  return L == 0 ? t : L == 1 ? (t & 31u) | ((t >> 5) << 8) : L == 2 ? (t & 3u) | ((t >> 2) << 5) : t << 3;
}
template <int L>
__device__ __forceinline__ constexpr uint32_t row_q(uint32_t q) {
  return L == 0 ? q << 8 : L == 1 ? q << 5 : L == 2 ? q << 2 : q;
}

// LDS position of register q for the thread's position pt (in layout 0 a sum: pt < 256)
template <int L>
__device__ __forceinline__ uint32_t at(uint32_t pt, int q) {
  return L == 0 ? pt + row_q<0>(q) : pt ^ lds_pos(row_q<L>(q));
}

template <typename R>
__device__ __forceinline__ void cfma(Cx<R> &a, const Cx<R> &c, const Cx<R> &x) {
  a.re = fma(c.re, x.re, fma(-c.im, x.im, a.re));
  a.im = fma(c.re, x.im, fma(c.im, x.re, a.im));
}

// what lane l holds, as a wave-uniform value (lists and coefficients that the block
// walks are held by the lanes: loaded once for the tile, with no wait per entry)
__device__ __forceinline__ uint32_t lane_u(uint32_t x, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, l);
}
__device__ __forceinline__ float lane_r(float x, int l) { return __uint_as_float(lane_u(__float_as_uint(x), l)); }
__device__ __forceinline__ double lane_r(double x, int l) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const uint32_t lo = lane_u((uint32_t)u, l), hi = lane_u((uint32_t)(u >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename R>
__device__ __forceinline__ Cx<R> lane_cx(const Cx<R> &x, int l) {
  return Cx<R>{lane_r(x.re, l), lane_r(x.im, l)};
}

template <int L, typename R>
__device__ __forceinline__ void lds_rows(Cx<R> (&y)[kRows], const Cx<R> *buf, uint32_t pt) {
#pragma unroll
  for (int q = 0; q < kRows; q++) y[q] = buf[at<L>(pt, q)];
}
template <int L, typename R>
__device__ __forceinline__ void lds_put(const Cx<R> (&y)[kRows], Cx<R> *buf, uint32_t pt) {
#pragma unroll
  for (int q = 0; q < kRows; q++) buf[at<L>(pt, q)] = y[q];
}

// acc[q] += (register bit M of q ? c1 : c0) * y[q with bit M flipped]
template <int M, typename R>
__device__ __forceinline__ void reg_flip(Cx<R> (&acc)[kRows], const Cx<R> (&y)[kRows], const Cx<R> &c0,
                                         const Cx<R> &c1) {
#pragma unroll
  for (int q = 0; q < kRows; q++) cfma(acc[q], (q >> M) & 1 ? c1 : c0, y[q ^ (1 << M)]);
}
// two register bits A < B: coefficient c[(bit A) << 1 | bit B]
template <int A, int B, typename R>
__device__ __forceinline__ void reg_pair(Cx<R> (&acc)[kRows], const Cx<R> (&y)[kRows], const Cx<R> *c) {
  const Cx<R> c00 = c[0], c01 = c[1], c10 = c[2], c11 = c[3];
#pragma unroll
  for (int q = 0; q < kRows; q++)
    cfma(acc[q], (q >> A) & 1 ? ((q >> B) & 1 ? c11 : c10) : ((q >> B) & 1 ? c01 : c00),
         y[q ^ (1 << A) ^ (1 << B)]);
}

// The in-tile pairs of layout L: groups [g0, g1); z: the tile in layout 0.
template <int L, typename R>
__device__ __forceinline__ void tile_groups(Cx<R> (&acc)[kRows], const Cx<R> (&z)[kRows], const Cx<R> *buf, uint32_t t,
                                            int g0, int g1, uint32_t heads, const Cx<R> *s_gc) {
  const uint32_t rt = row_t<L>(t);
  uint32_t pt = lds_pos(rt);
#pragma unroll 1
  for (int e = g0; e < g1; e++) {
    asm volatile("" : "+v"(pt));  // (its XORs made where they are used, not held)
    const int h = (int)lane_u(heads, e), i = (h >> 3) - 1, m = h & 7;
    Cx<R> y[kRows];
    if (i < 0) {
      if constexpr (L == 0) {
#pragma unroll
        for (int q = 0; q < kRows; q++) y[q] = z[q];
      } else {
        lds_rows<L>(y, buf, pt);
      }
      const Cx<R> *c = s_gc + 12 * e;
      if (m & 1) reg_pair<0, 1>(acc, y, c);
      if (m & 2) reg_pair<0, 2>(acc, y, c + 4);
      if (m & 4) reg_pair<1, 2>(acc, y, c + 8);
    } else {
      lds_rows<L>(y, buf, pt ^ lds_pos(1u << i));
      const Cx<R> *c = s_gc + 12 * e + 2 * ((rt >> i) & 1u);
      if (m & 1) reg_flip<0>(acc, y, c[0], c[1]);
      if (m & 2) reg_flip<1>(acc, y, c[4], c[5]);
      if (m & 4) reg_flip<2>(acc, y, c[8], c[9]);
    }
  }
}

// Three register sites' pairs with the outer site: mask bits; the coefficients
// [site][bit of the site] are held by the lanes from l on.
template <typename R>
__device__ __forceinline__ void mixed(Cx<R> (&acc)[kRows], const Cx<R> (&y)[kRows], uint32_t m, const Cx<R> &c,
                                      int l) {
  if (m & 1) reg_flip<0>(acc, y, lane_cx(c, l), lane_cx(c, l + 1));
  if (m & 2) reg_flip<1>(acc, y, lane_cx(c, l + 2), lane_cx(c, l + 3));
  if (m & 4) reg_flip<2>(acc, y, lane_cx(c, l + 4), lane_cx(c, l + 5));
}

template <typename R>
struct HalfLds {
  size_t buf, gc, fslot, fb, hd, phi, total;
  __host__ __device__ HalfLds(int n, int ngrp) {
    const size_t cs = sizeof(Cx<R>);
    size_t o = 0;
    auto take = [&](size_t b) {
      const size_t r = o;
      o += (b + 15) & ~size_t(15);
      return r;
    };
    buf = take(cs * 2 * kTile);
    gc = take(cs * 12 * (size_t)ngrp);
    fslot = take(cs * 16 * n);
    fb = take(cs * 2 * n);
    hd = take(sizeof(R) * 2 * n);
    phi = take(sizeof(R) * n);
    total = o;
  }
};

// The np <= 64 pairs of two outer sites whose partner tiles and coefficients the lanes
// hold (lane p: pair p), NB pairs' rows in flight.
template <int NB, typename R>
__device__ __forceinline__ void outer_pairs(Cx<R> (&acc)[kRows], uint32_t tile, const Cx<R> &coef, int np,
                                            const Cx<R> *v, uint32_t t) {
  Cx<R> x[NB][kRows];
  auto fetch = [&](int b, int p) {
    const Cx<R> *vb = v + lane_u(tile, p);
#pragma unroll
    for (int r = 0; r < kRows; r++) x[b][r] = vb[r * kBlock + t];
  };
#pragma unroll
  for (int b = 0; b < NB; b++) fetch(b, b);  // (lanes past np hold the own tile)
#pragma unroll 1
  for (int p = 0; p < np; p += NB) {
#pragma unroll
    for (int b = 0; b < NB; b++) {
      if (p + b < np) {
        const Cx<R> c = lane_cx(coef, p + b);
#pragma unroll
        for (int r = 0; r < kRows; r++) cfma(acc[r], c, x[b][r]);
      }
      if (p + b + NB < np) fetch(b, p + b + NB);
    }
  }
}

template <typename R, bool COLS>
__global__ __launch_bounds__(kBlock, sizeof(R) == 8 ? 2 : 3) void hv_half_sweep(
    HamGeom g, DevTables<R> tb, WinPass W, const uint32_t *__restrict__ grp, const Cx<R> *__restrict__ gco,
    const uint32_t *__restrict__ msk, const Cx<R> *__restrict__ mco, const R *__restrict__ tdiag,
    const int4 *__restrict__ plist, const Cx<R> *__restrict__ pcl, int log_cols, HvParams P) {
  extern __shared__ __align__(16) unsigned char smem[];
  // sites are named by their row bits: site k is bit k + f, the bits below f the column
  const int f = COLS ? log_cols : 0;
  const int ns = g.n, n = ns + f, ngrp = W.hg[4] - W.hg[0];
  const HalfLds<R> L(n, ngrp);
  Cx<R> *buf = reinterpret_cast<Cx<R> *>(smem + L.buf);
  Cx<R> *s_gc = reinterpret_cast<Cx<R> *>(smem + L.gc);        // [group][member][4]
  Cx<R> *s_fslot = reinterpret_cast<Cx<R> *>(smem + L.fslot);  // [site][bit][8]
  Cx<R> *s_fb = reinterpret_cast<Cx<R> *>(smem + L.fb);        // [site][bit]
  R *s_hd = reinterpret_cast<R *>(smem + L.hd);                // [site][bit]
  R *s_phi = reinterpret_cast<R *>(smem + L.phi);
  uint32_t t = threadIdx.x;
  const int4 *pl = plist + W.p0;
  const Cx<R> *__restrict__ pch = pcl + 4 * (size_t)W.p0;
  const int e_out = W.np_ll + W.np_lh, np_out = W.np - e_out;
  const int lane = threadIdx.x & 63;
  // held by the lanes: group heads, the outer sites' masks, the first outer pairs
  const uint32_t heads = lane < ngrp ? grp[W.hg[0] + lane] : 0u;
  const uint32_t masks = lane < __builtin_popcount(W.xmask) ? msk[W.hm0 + lane] : 0u;
  const int4 pair0 = lane < np_out ? pl[e_out + lane] : make_int4(0, 0, 0, 0);
  const Cx<R> *__restrict__ v = reinterpret_cast<const Cx<R> *>(P.v);
  for (int i = t; i < 12 * ngrp; i += kBlock) s_gc[i] = gco[12 * (size_t)W.hg[0] + i];
  for (int i = t; i < 2 * n; i += kBlock) s_hd[i] = i < 2 * f ? R(0) : tb.hdiag[((i >> 1) - f) * 16 + (i & 1)];
  if (W.smask) {
    // the field that the slot bits (8..10) put on each site's flip
    for (int i = t; i < 16 * n; i += kBlock) {
      const int k = i >> 4, sel = (i >> 3) & 1, sl = i & 7;
      Cx<R> fs{0, 0};
      for (int s = 0; s < 3; s++) {
        if (kLowBits + s == k || k < f) continue;
        const Cx<R> c = tb.cz_half[((k - f) * ns + kLowBits + s - f) * 2 + sel];
        const R m = (sl >> s) & 1 ? R(0.5) : R(-0.5);
        fs.re = fma(c.re, m, fs.re);
        fs.im = fma(c.im, m, fs.im);
      }
      s_fslot[i] = fs;
    }
  }
  double red[3][1] = {{0.0}, {0.0}, {0.0}};
  // does the pass read the tile's own rows / use the other layouts' sums
  const bool own = W.diag || ngrp || (W.smask & ((1u << kTileBits) - 1u)), sums = ngrp || W.xmask;

  // Tile walk: with a grid that is a multiple of 8, block b runs on XCD b % 8.  With 8
  // windows or more XCD x takes windows x, x + 8, ...; with fewer the tiles are dealt to
  // the XCDs in eight runs.  Either way the tiles an XCD works on at a time are
  // neighbours, whose partners (up to a shift by the higher sites) it shares in its L2.
  const bool xcd = (gridDim.x & 7u) == 0 && ((W.nwin * W.nin) & 7u) == 0;
  const uint32_t total = W.nwin * W.nin, per = xcd ? total >> 3 : total, xc = xcd ? blockIdx.x & 7u : 0u;
#pragma unroll 1
  for (uint32_t j = xcd ? blockIdx.x >> 3 : blockIdx.x; j < per; j += xcd ? gridDim.x >> 3 : gridDim.x) {
    const uint32_t wl = j / W.nin;
    const uint32_t win = !xcd ? wl : W.nwin >= 8 ? xc + 8u * wl : (xc * per + j) / W.nin;
    const uint32_t item = !xcd || W.nwin >= 8 ? j - wl * W.nin : (xc * per + j) % W.nin;
    const uint32_t base = __builtin_amdgcn_readfirstlane(scatter_bits(item, W.emask) | scatter_bits(win, W.omask));
    // (made anew for every tile: what the compiler derives from t ahead of the loop would
    // be kept in scratch)
    asm volatile("" : "+v"(t));
    const uint32_t p0 = lds_pos(t);
    const Cx<R> *vt = v + base;
    auto mz = [&](int j) -> R { return (base >> j) & 1 ? R(0.5) : R(-0.5); };
    Cx<R> z[kRows];
#pragma unroll
    for (int q = 0; q < kRows; q++) z[q] = own ? vt[q * kBlock + t] : Cx<R>{0, 0};
    __syncthreads();  // (the last tile's reads of the LDS)
    // per tile: the outer sites' field on every site's flip, and z-fields
    if (t < 2u * n) {
      if (W.smask && t >= 2u * f) {
        const int k = t >> 1, sel = t & 1;
        Cx<R> fd = tb.hflip[t - 2 * f];
        if (g.has_z)
          for (int j0 = kTileBits; j0 < n; j0 += 7) {  // seven loads in flight; weight 0 past n
            Cx<R> c[7];
#pragma unroll
            for (int u = 0; u < 7; u++) c[u] = tb.cz_half[((k - f) * ns + (j0 + u < n ? j0 + u : n - 1) - f) * 2 + sel];
#pragma unroll
            for (int u = 0; u < 7; u++) {
              const int j = j0 + u;
              const R m = j == k || j >= n ? R(0) : mz(j);
              fd.re = fma(c[u].re, m, fd.re);
              fd.im = fma(c[u].im, m, fd.im);
            }
          }
        s_fb[t] = fd;
      }
    } else if (W.diag && t >= 64 && t < 64u + n) {
      const int i = t - 64;
      R ph = 0;
      for (int j0 = i < f ? n : i < kTileBits ? kTileBits : i + 1; j0 < n; j0 += 7) {
        R c[7];
#pragma unroll
        for (int u = 0; u < 7; u++) c[u] = tb.zz[(i - f) * ns + (j0 + u < n ? j0 + u : n - 1) - f];
#pragma unroll
        for (int u = 0; u < 7; u++) ph = fma(c[u], j0 + u < n ? mz(j0 + u) : R(0), ph);
      }
      s_phi[i] = i < kTileBits ? ph : fma(mz(i), ph, s_hd[2 * i + ((base >> i) & 1)]);
    }
    if (own) lds_put<0>(z, buf, p0);
    __syncthreads();

    Cx<R> acc[kRows];
#pragma unroll
    for (int q = 0; q < kRows; q++) acc[q] = Cx<R>{0, 0};
    if (W.diag) {
      R dg = 0;
      for (int k = kTileBits; k < n; k++) dg += s_phi[k];
#pragma unroll
      for (int i = 0; i < kLowBits; i++) dg = fma((t >> i) & 1 ? R(0.5) : R(-0.5), s_phi[i], dg);
      const R f0 = R(0.5) * s_phi[8], f1 = R(0.5) * s_phi[9], f2 = R(0.5) * s_phi[10];
#pragma unroll
      for (int q = 0; q < kRows; q++) {
        const R d = tdiag[(q * kBlock + t) >> f] + (dg + ((q & 1 ? f0 : -f0) + ((q & 2 ? f1 : -f1) + (q & 4 ? f2 : -f2))));
        acc[q] = Cx<R>{d * z[q].re, d * z[q].im};
      }
    }
    // single flips: coefficient = field of the outer sites + of the low sites + of the slot bits
    auto single = [&](int k, int b, const Cx<R> &a2, int q) -> Cx<R> {
      const Cx<R> a1 = s_fb[2 * k + b], a3 = s_fslot[(2 * k + b) * 8 + q];
      return Cx<R>{a1.re + a2.re + a3.re, a1.im + a2.im + a3.im};
    };
    // The field of the sites on row bits f..7.  The table holds that of the sites 0..7;
    // the f highest of them, on bits 8 and up, drop out of the mean over both their values.
    auto field = [&](int k, int b) -> Cx<R> {
      const Cx<R> *e = tb.lowf + ((k - f) * 2 + b) * 256;
      if (f == 0) return e[t];
      const Cx<R> lo = e[t >> f], hi = e[(t >> f) | (255u & ~(255u >> f))];
      return Cx<R>{R(0.5) * (lo.re + hi.re), R(0.5) * (lo.im + hi.im)};
    };
    Cx<R> a2n{0, 0};  // (the next site's field is loaded ahead)
    if (const uint32_t sm = W.smask & ((1u << kLowBits) - 1u)) a2n = field(__builtin_ctz(sm), (t >> __builtin_ctz(sm)) & 1);
#pragma unroll 1
    for (uint32_t sm = W.smask & ((1u << kLowBits) - 1u); sm;) {
      const int k = __builtin_ctz(sm), b = (t >> k) & 1;
      sm &= sm - 1u;
      Cx<R> y[kRows];
      lds_rows<0>(y, buf, p0 ^ lds_pos(1u << k));
      const Cx<R> a2 = a2n;
      if (sm) a2n = field(__builtin_ctz(sm), (t >> __builtin_ctz(sm)) & 1);
#pragma unroll
      for (int q = 0; q < kRows; q++) cfma(acc[q], single(k, b, a2, q), y[q]);
    }
#pragma unroll
    for (int s = 0; s < 3; s++) {
      const int k = kLowBits + s;
      if (!((W.smask >> k) & 1u)) continue;
      const Cx<R> l0 = field(k, 0), l1 = field(k, 1);
#pragma unroll
      for (int q = 0; q < kRows; q++) {
        const int b = (q >> s) & 1;
        cfma(acc[q], single(k, b, b ? l1 : l0, q), z[q ^ (1 << s)]);
      }
    }
    tile_groups<0>(acc, z, buf, t, 0, W.hg[1] - W.hg[0], heads, s_gc);
    Cx<R> acc1[kRows], acc2[kRows], acc3[kRows];
#pragma unroll
    for (int q = 0; q < kRows; q++) acc1[q] = acc2[q] = acc3[q] = Cx<R>{0, 0};
    uint32_t xm = W.xmask;
    int rank = 0;
    Cx<R> cn{0, 0};  // the next outer site's coefficients
    auto load_next = [&]() {
      if (xm) {
        const Cx<R> *vb = v + (base ^ (1u << __builtin_ctz(xm)));
#pragma unroll
        for (int q = 0; q < kRows; q++) z[q] = vb[q * kBlock + t];
        const uint32_t ba = (base >> __builtin_ctz(xm)) & 1u;
        a2n = field(__builtin_ctz(xm), ba);
        cn = mco[(2 * (size_t)(W.hm0 + rank) + ba) * (2 * kTileBits) + (lane < 2 * kTileBits ? lane : 0)];
      }
    };
    load_next();
    tile_groups<1>(acc1, z, buf, t, W.hg[1] - W.hg[0], W.hg[2] - W.hg[0], heads, s_gc);
    tile_groups<2>(acc2, z, buf, t, W.hg[2] - W.hg[0], W.hg[3] - W.hg[0], heads, s_gc);
    tile_groups<3>(acc3, z, buf, t, W.hg[3] - W.hg[0], ngrp, heads, s_gc);
    uint32_t p1 = lds_pos(row_t<1>(t)), p2 = lds_pos(row_t<2>(t)), p3 = lds_pos(row_t<3>(t));
    uint32_t x = kTile;  // the buffer to write
#pragma unroll 1
    while (xm) {
      const int a = __builtin_ctz(xm);
      xm &= xm - 1u;
      asm volatile("" : "+v"(p1), "+v"(p2), "+v"(p3));  // (their XORs made where they are used)
      const uint32_t ba = (base >> a) & 1u, m = lane_u(masks, rank++);
      const Cx<R> c = cn;
      if ((W.smask >> a) & 1u) {
        const Cx<R> a2 = a2n;
#pragma unroll
        for (int q = 0; q < kRows; q++) cfma(acc[q], single(a, ba, a2, q), z[q]);
      }
      mixed(acc, z, m >> 8, c, 16);
      if (m & 255u) lds_put<0>(z, buf + x, p0);
      load_next();
      if (m & 255u) {
        __syncthreads();
        const Cx<R> *b = buf + x;
        Cx<R> y[kRows];
        if (m & 0xe0u) {
          lds_rows<1>(y, b, p1);
          mixed(acc1, y, m >> 5, c, 10);
        }
        if (m & 0x1cu) {
          lds_rows<2>(y, b, p2);
          mixed(acc2, y, m >> 2, c, 4);
        }
        if (m & 3u) {
          lds_rows<3>(y, b, p3);
          mixed(acc3, y, m & 3u, c, 0);
        }
        x ^= kTile;
      }
    }
    // the outer pairs' tiles and coefficients, by lane
    uint32_t otile = base;
    Cx<R> ocoef{0, 0};
    auto hold = [&](const int4 &q, int e, bool ok) {
      if (ok) {
        otile = base ^ (1u << q.y) ^ (1u << q.z);
        ocoef = pch[4 * e + ((((base >> q.y) & 1) << 1) | ((base >> q.z) & 1))];
      }
    };
    hold(pair0, e_out + lane, lane < np_out);
    // the layouts' sums, brought to layout 0
    if (sums) {
      __syncthreads();
      lds_put<1>(acc1, buf, p1);
      lds_put<2>(acc2, buf + kTile, p2);
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kRows; q++) {
        const Cx<R> u = buf[at<0>(p0, q)], w = buf[kTile + at<0>(p0, q)];
        acc[q].re += u.re + w.re;
        acc[q].im += u.im + w.im;
      }
      __syncthreads();
      lds_put<3>(acc3, buf, p3);
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kRows; q++) {
        const Cx<R> u = buf[at<0>(p0, q)];
        acc[q].re += u.re;
        acc[q].im += u.im;
      }
    }
    for (int e = 0; e < np_out; e += 64) {
      if (e) {
        const bool ok = e + lane < np_out;
        otile = base;
        hold(pl[e_out + (ok ? e + lane : 0)], e_out + e + lane, ok);
      }
      outer_pairs<3>(acc, otile, ocoef, np_out - e < 64 ? np_out - e : 64, v, t);
    }
    // the earlier passes' partial sums of these rows
    Cx<R> *wt = reinterpret_cast<Cx<R> *>(P.w) + base;
    Cx<R> wprev[kRows];
#pragma unroll
    for (int q = 0; q < kRows; q++) wprev[q] = W.first ? Cx<R>{0, 0} : ld_stream(wt + q * kBlock + t);
    if (W.last && P.lanczos) {
#pragma unroll
      for (int q = 0; q < kRows; q++) z[q] = vt[q * kBlock + t];
    }
#pragma unroll
    for (int q = 0; q < kRows; q++) {
      Acc<R, 1> a1;
      a1.re[0] = acc[q].re + wprev[q].re;
      a1.im[0] = acc[q].im + wprev[q].im;
      if (W.last) hv_epilogue<R, 1, true>(P, (base + q * kBlock + t) >> f, COLS ? (int)(t & (P.K - 1)) : 0, a1, &z[q], red);
      else st_stream(wt + q * kBlock + t, Cx<R>{a1.re[0], a1.im[0]});
    }
  }
  if (!W.last || !P.lanczos) return;
  if constexpr (!COLS) {
    hv_finish<1>(P, red);
    return;
  }
  // a thread's rows are of one column, its lowest f bits: sums over the other lane bits,
  // then over the four waves in order
  double *part = reinterpret_cast<double *>(smem);
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 3; a++) {
    double s = red[a][0];
    for (int m = 32; m >= P.K; m >>= 1) s += __shfl_xor(s, m);
    if (lane < P.K) part[((threadIdx.x >> 6) * 3 + a) * P.K + lane] = s;
  }
  __syncthreads();
  if ((int)threadIdx.x < 3 * P.K) {
    const int a = threadIdx.x / P.K, c = threadIdx.x % P.K;
    double s = 0;
    for (int wv = 0; wv < kBlock / 64; wv++) s += part[(wv * 3 + a) * P.K + c];
    P.part[((size_t)c * gridDim.x + blockIdx.x) * 3 + a] = s;
  }
}

template <typename R, bool COLS>
int launch_r(const HamGeom &g, const DevTables<R> &tb, const WinPlan &plan, int f, const HvParams &P, int cap,
             unsigned *last_gx, hipStream_t s) {
  static std::atomic<uint64_t> granted{0};
  const HalfTables &H = plan.half;
  if (!H.d_plist || !H.d_pcoef || !H.d_grp || plan.passes.empty()) return FTLM_EINVAL;
  // the blocks that are resident, but for a single pass of complex128 (2^22 rows: complex64
  // 213 us with 768 blocks, 226 with 2048; complex128 402 with 2048, 417 with 512; in
  // several passes, 2^24 rows: 2421 and 2275)
  cap = cap > 0 ? std::min(cap, 2048) : sizeof(R) == 4 ? 768 : plan.passes.size() > 1 ? 512 : 2048;
  for (const WinPass &W : plan.passes) {
    const uint64_t items = (uint64_t)W.nwin * W.nin;
    uint32_t gx = (uint32_t)(items < (uint64_t)cap ? items : (uint64_t)cap);
    if (W.nwin >= 8 && gx >= 8) gx &= ~7u;
    HvParams Pp = P;
    if (!W.last) Pp.lanczos = 0;
    const size_t sm = HalfLds<R>(g.n + f, W.hg[4] - W.hg[0]).total;
    const int rc = grant_lds(reinterpret_cast<const void *>(&hv_half_sweep<R, COLS>), 1024, sm, granted);  // (1 KB: the sums)
    if (rc) return rc;
    hipLaunchKernelGGL((hv_half_sweep<R, COLS>), dim3(gx), dim3(kBlock), sm, s, g, tb, W, H.d_grp,
                       reinterpret_cast<const Cx<R> *>(H.d_gco), H.d_msk, reinterpret_cast<const Cx<R> *>(H.d_mco),
                       reinterpret_cast<const R *>(H.d_tdiag), H.d_plist,
                       reinterpret_cast<const Cx<R> *>(H.d_pcoef), f, Pp);
    *last_gx = gx;
  }
  return FTLM_OK;
}

template <typename R>
int launch_f(const HamGeom &g, const DevTables<R> &tb, const WinPlan &plan, int f, const HvParams &P, int cap,
             unsigned *gx, hipStream_t s) {
  return f ? launch_r<R, true>(g, tb, plan, f, P, cap, gx, s) : launch_r<R, false>(g, tb, plan, 0, P, cap, gx, s);
}

int layout_of(int bit) { return bit >= 8 ? 0 : bit >= 5 ? 1 : bit >= 2 ? 2 : 3; }
int layout_base(int L) { return L == 0 ? 8 : L == 1 ? 5 : L == 2 ? 2 : 0; }

}  // namespace

// The in-tile pairs of every pass as groups (layout of the higher site j; the lower
// site i when it is not a register bit of that layout), and the mixed pairs by outer
// site; pcoef: four coefficients per list entry, by the row bits (i, j).
HalfLists plan_half(const std::vector<Cx<double>> &pcoef, WinPlan &plan) {
  HalfLists H;
  // (by j, then i, the tiles that an XCD works on share more partners: 2^22 rows, all pairs
  // coupled, complex128 399 us against 539 by i, then j; the tile kernel of the other column
  // counts keeps that order: 2^20 rows x 3 675 us, 853 by j, then i)
  H.plist = plan.plist;
  for (WinPass &W : plan.passes) {
    std::stable_sort(H.plist.begin() + W.p0 + W.np_ll + W.np_lh, H.plist.begin() + W.p0 + W.np,
                     [](const int4 &a, const int4 &b) { return a.z != b.z ? a.z < b.z : a.y < b.y; });
    for (int L = 0; L < 4; L++) {
      W.hg[L] = (int)H.grp.size();
      const int lo = layout_base(L), nr = L == 3 ? 2 : 3;
      for (int i = -1; i < lo; i++) {
        int mask = 0;
        Cx<double> c[12] = {};
        for (int e = 0; e < W.np_ll; e++) {
          const int4 q = plan.plist[W.p0 + e];  // q.y < q.z
          const int a = q.y - lo, b = q.z - lo;
          if (layout_of(q.z) != L) continue;
          int m;
          if (i < 0) {
            if (a < 0 || b >= nr) continue;
            m = a == 0 ? (b == 1 ? 0 : 1) : 2;
          } else {
            if (q.y != i) continue;
            m = b;
          }
          mask |= 1 << m;
          for (int u = 0; u < 4; u++) c[4 * m + u] = pcoef[4 * (size_t)(W.p0 + e) + u];
        }
        if (!mask) continue;
        H.grp.push_back((uint32_t)(mask | ((i + 1) << 3)));
        H.gco.insert(H.gco.end(), c, c + 12);
      }
    }
    W.hg[4] = (int)H.grp.size();
    W.hm0 = (int)H.msk.size();
    for (uint32_t xm = W.xmask; xm; xm &= xm - 1u) {
      const int a = __builtin_ctz(xm);
      uint32_t mask = 0;
      Cx<double> c[4 * kTileBits] = {};  // [bit of a][tile site][bit of the site]
      for (int e = W.np_ll; e < W.np_ll + W.np_lh; e++) {
        const int4 q = plan.plist[W.p0 + e];
        if (q.z != a) continue;
        mask |= 1u << q.y;
        for (int u = 0; u < 4; u++)
          c[(u & 1) * 2 * kTileBits + 2 * q.y + (u >> 1)] = pcoef[4 * (size_t)(W.p0 + e) + u];
      }
      H.msk.push_back(mask);
      H.mco.insert(H.mco.end(), c, c + 4 * kTileBits);
    }
  }
  return H;
}

// Built site by site: a value of site k adds its own element and its moment times the
// z-field of the sites below.  (From the row with every site down, each site adding what
// raising it changes, the table carried roundings of that row's size: products of 18 spins
// 1/2 with nn + nnn exchange were 1.3 times as far from 64 bits.)
std::vector<double> half_tile_diagonal(const HostHam &hh, int f) {
  const int n = hh.n, nt = kTileBits - f;
  std::vector<double> tdiag((size_t)1 << nt, 0.0), zf((size_t)1 << nt);
  for (int k = 0; k < nt; k++) {
    const double *z = &hh.zz[(size_t)k * n];
    const double dn = hh.h[(size_t)k * 256].re, up = hh.h[(size_t)k * 256 + 17].re;
    zf[0] = 0.0;
    for (int j = 0; j < k; j++)
      for (int r = 0; r < 1 << j; r++) {
        zf[r + (1 << j)] = zf[r] + 0.5 * z[j];
        zf[r] -= 0.5 * z[j];
      }
    for (int r = 0; r < 1 << k; r++) {
      tdiag[r + (1 << k)] = tdiag[r] + (up + 0.5 * zf[r]);
      tdiag[r] += dn - 0.5 * zf[r];
    }
  }
  return tdiag;
}

// One pass over all rows for 2^f columns: row bits (site k on bit k + f), pairs in the
// order of a window pass (both in the tile | one outer site, by that site | two outer).
void plan_columns(const HostHam &hh, const std::vector<int> &pi, const std::vector<int> &pj, int f, WinPlan &plan) {
  plan = WinPlan();
  const int nb = hh.n + f;
  if (hh.n < kTileBits || f < 1 || nb > 31) return;
  std::vector<int> prs(pi.size());
  for (size_t p = 0; p < prs.size(); p++) prs[p] = (int)p;
  auto cls = [&](int p) { return (pi[p] + f >= kTileBits) + (pj[p] + f >= kTileBits); };
  std::stable_sort(prs.begin(), prs.end(), [&](int a, int b) {
    if (cls(a) != cls(b)) return cls(a) < cls(b);
    return cls(a) > 0 && pj[a] < pj[b];
  });
  WinPass W;
  std::memset(&W, 0, sizeof(W));
  W.first = W.last = W.diag = 1;
  W.np = (int)prs.size();
  W.nwin = 1;
  W.nin = 1u << (nb - kTileBits);
  W.emask = (W.nin - 1u) << kTileBits;
  for (int k = 0; k < hh.n; k++)
    if (site_has_singles(hh, k)) W.smask |= 1u << (k + f);
  W.xmask = W.smask >> kTileBits << kTileBits;
  for (int p : prs) {
    plan.plist.push_back(make_int4(p, pi[p] + f, pj[p] + f, 0));
    if (cls(p) == 0) W.np_ll++;
    if (cls(p) == 1) {
      W.np_lh++;
      W.xmask |= 1u << (pj[p] + f);
    }
  }
  if (plan.plist.empty()) plan.plist.push_back(make_int4(0, 0, 0, 0));
  plan.passes.push_back(W);
}

int launch_half_sweep(const DevHam &dh, int precision, const HvParams &P, int cap, unsigned *gx, hipStream_t s) {
  const bool f32 = precision == FTLM_C64;
  const int f = P.K == 1 ? 0 : P.K == 2 ? 1 : P.K == 4 ? 2 : P.K == 8 ? 3 : P.K == 16 ? 4 : -1;
  if (f < 0) return FTLM_EINVAL;
  const WinPlan &plan = f ? dh.twc[f32][f - 1] : f32 ? dh.tw32 : dh.tw64;
  return f32 ? launch_f<float>(dh.geom, dh.t32, plan, f, P, cap, gx, s)
             : launch_f<double>(dh.geom, dh.t64, plan, f, P, cap, gx, s);
}

}  // namespace ftlm
