// Tile sweep: H*v for one column of a general-radix system without s+- s^z pair
// pieces (Sec. 2.1, Eq. mce-hamop, in the ladder form of ftlm_internal.hpp), in one
// pass over the rows.
//
// The low sites are tile sites; the rows that share the digits of every other
// ("outer") site are a tile, staged in LDS by one block.  Thread q owns the rows of
// one value of the lower tile sites' digits and ALL digits d of the top tile site:
// every digit but d is the thread's own for the whole launch, so a term's validity,
// ladder factors and partner are worked out once for RPT rows, and moves of the top
// site are moves between the thread's registers.  Terms:
//   - inside the tile: partners from LDS ([q][d], an odd number of values per q, so
//     that the lanes' 16-byte reads fall on different banks); one read of a lower
//     site's neighbour serves its single flip and its pair with the top site;
//   - one outer site j and one move of it: the partner tile's rows come straight from
//     v (coalesced, the same offset for every row) and serve j's single flip and its
//     pairs with the top site from registers; the pairs with lower sites read them
//     shifted, from LDS (the tile's own rows are not needed there any more; shifted
//     reads from v instead, for groups of up to two, gave 6.80 -> 7.24 ms on 3^17 rows
//     and 11.4 -> 11.5 on 5^12, nn + nnn);
//   - two outer sites, and single flips by two: one coefficient per tile, partners
//     from v, two terms in flight.
//
// Tile walk: with a grid that is a multiple of 8, block b runs on XCD b % 8; chunks of
// consecutive tiles go to the XCDs in turn and each XCD's blocks walk its chunks in
// order.  The default grid is the blocks that are resident at once: with more, the
// blocks of an XCD drift apart and the partner tiles leave its L2 in between.
//
// Measured (one product, complex128 / complex64), against the earlier mapping of rows to
// threads (row = thread + k * block: digits, validity and ladder factors per row):
//   6 x 5^8 rows, 20 pairs (51 per row)   223 -> 121 / 138 -> 74 us
//   5^12 rows, all pairs (204 per row)   71 -> 39.8 / 42.2 -> 21.6 ms
//   5^12 rows, nn + nnn (32 per row)     13.8 -> 10.9 / 9.6 -> 5.8 ms
// What bounds it now is the partner tiles that come from beyond L2 (8 % of the requests hit
// there): all pairs, complex128 / complex64, 282 / 144 GB at 7.1 / 6.7 TB/s, nn + nnn 79 GB
// at 7.2 TB/s, where a copy that stays in the last-level cache moves 6.7 to 7.1; vector units
// 28 / 51 % busy, LDS 20 / 29 %.  Passes over subsets of the sites whose windows fit an XCD's
// L2 read a third of that, but took longer (nn + nnn 12.1 -> 13.7 ms at complex128, all pairs
// 30 -> 35 at complex64): every pass pays the own tile, the tables and a read-add of w.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <vector>

#include "device_reduce.hpp"
#include "ftlm_internal.hpp"
#include "hv_common.hpp"

namespace ftlm {

namespace {

// Waves per SIMD that the registers are allocated for.  The kernel waits for partner
// tiles, so more waves help until the rows in flight spill: complex64 rows take half the
// registers.  5^12 rows, all pairs: complex128 3 waves 46.7 ms, 4 50.9; complex64
// 4 waves 30.4 ms, 6 25.3, 8 26.8.  4^13 rows, nn + nnn, complex64: 6 2.16 ms, 8 1.75.
constexpr int sweep_waves(size_t real_bytes, int rpt) {
  return rpt >= 5 ? (real_bytes == 8 ? 3 : 6) : real_bytes == 8 ? 4 : 8;
}
// Threads of a block at most: with RPT 5 and 6 (3 waves per SIMD) one block is what a CU holds.
constexpr int sweep_threads(int rpt) { return rpt >= 5 ? 768 : 1024; }

// Threads of a plan's block: the values below the top tile site in whole waves, and two
// waves at the least: per tile, the first lists the outer terms while the second makes
// the outer sites' fields.
inline int sweep_block(const SweepPass &G) { return std::max(128, (int)((G.Q + 63) / 64 * 64)); }

// LDS layout (offsets 16-byte aligned).
template <typename R>
struct SweepLds {
  size_t tile, hoff, pc, gp, gm, hd, zz, phi, pij, ooff, oc, cnt, total;
  __host__ __device__ SweepLds(const SweepPass &G) {
    const size_t cs = sizeof(Cx<R>), rs = sizeof(R), n = G.n, np = G.np;
    const size_t no = 4 * (size_t)G.np_out + 2 * (size_t)(G.n - G.t);
    size_t o = 0;
    auto take = [&](size_t b) {
      const size_t r = o;
      o += (b + 15) & ~size_t(15);
      return r;
    };
    tile = take(cs * G.Q * (G.rtop | 1));
    hoff = take(cs * 64 * n);
    pc = take(cs * 4 * np);
    gp = take(rs * 16 * n);
    gm = take(rs * 16 * n);
    hd = take(rs * 16 * n);
    zz = take(rs * n * n);
    phi = take(rs * n);
    pij = take(sizeof(int4) * np);
    ooff = take(sizeof(int64_t) * no);
    oc = take(cs * no);
    cnt = take(sizeof(int));
    total = o;
  }
};

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uni64(int64_t x) {
  const uint64_t u = (uint64_t)x;
  const uint32_t lo = (uint32_t)uni((int)(uint32_t)u), hi = (uint32_t)uni((int)(uint32_t)(u >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ float unir(float x) { return __int_as_float(uni(__float_as_int(x))); }
__device__ __forceinline__ double unir(double x) { return __longlong_as_double(uni64(__double_as_longlong(x))); }
template <typename R>
__device__ __forceinline__ Cx<R> unic(const Cx<R> &c) {
  return Cx<R>{unir(c.re), unir(c.im)};
}

template <typename R, bool CPLX>
__device__ __forceinline__ void cfma(Cx<R> &a, const Cx<R> &c, const Cx<R> &x) {
  a.re = fma(c.re, x.re, a.re);
  a.im = fma(c.re, x.im, a.im);
  if (CPLX) {
    a.re = fma(-c.im, x.im, a.re);
    a.im = fma(c.im, x.re, a.im);
  }
}

// The lanes of one wave append their valid candidates to an LDS list in lane order.
__device__ __forceinline__ int append(bool valid, int count, int *pos) {
  const unsigned long long m = __ballot(valid);
  *pos = count + __popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull));
  return count + __popcll(m);
}

template <typename R, int RPT, bool CPLX>
__global__ __launch_bounds__(sweep_threads(RPT), sweep_waves(sizeof(R), RPT)) void hv_sweep(
    SweepPass G, DevTables<R> tb, const int4 *__restrict__ pij, const Cx<R> *__restrict__ pcs,
    const R *__restrict__ tdiag, uint32_t chunk, HvParams P) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int SP = RPT | 1;
  const SweepLds<R> L(G);
  Cx<R> *tile = reinterpret_cast<Cx<R> *>(smem + L.tile);
  Cx<R> *s_hoff = reinterpret_cast<Cx<R> *>(smem + L.hoff);  // [site][4][16]
  Cx<R> *s_pc = reinterpret_cast<Cx<R> *>(smem + L.pc);      // [np][4]
  R *s_gp = reinterpret_cast<R *>(smem + L.gp);              // [site][16]
  R *s_gm = reinterpret_cast<R *>(smem + L.gm);
  R *s_hd = reinterpret_cast<R *>(smem + L.hd);
  R *s_zz = reinterpret_cast<R *>(smem + L.zz);              // [site][site]
  R *s_phi = reinterpret_cast<R *>(smem + L.phi);
  int4 *s_pij = reinterpret_cast<int4 *>(smem + L.pij);      // (site a, site b, non-zero types, 0)
  int64_t *s_ooff = reinterpret_cast<int64_t *>(smem + L.ooff);
  Cx<R> *s_oc = reinterpret_cast<Cx<R> *>(smem + L.oc);
  int *s_cnt = reinterpret_cast<int *>(smem + L.cnt);
  const int t = G.t, n = G.n, top = t - 1, tid = threadIdx.x, NT = blockDim.x;
  const uint32_t Q = G.Q;
  for (int i = tid; i < 64 * n; i += NT) s_hoff[i] = tb.hoff[i];
  for (int i = tid; i < 16 * n; i += NT) {
    s_gp[i] = tb.gp[i];
    s_gm[i] = tb.gm[i];
    s_hd[i] = tb.hdiag[i];
  }
  for (int i = tid; i < 4 * G.np; i += NT) s_pc[i] = pcs[i];
  for (int i = tid; i < G.np; i += NT) s_pij[i] = pij[i];
  for (int i = tid; i < n * n; i += NT) s_zz[i] = tb.zz[i];
  // the thread's lower digits (4 bits each, at most 8 lower tile sites) and the
  // offset of its rows within the basis; threads past Q repeat the last one's reads
  const bool act = (uint32_t)tid < Q;
  const uint32_t q = act ? (uint32_t)tid : Q - 1;
  uint32_t dig = 0, goff = 0;  // (goff in bytes, within the tile: its sites are the lowest digits)
  {
    uint32_t rem = q;
    for (int i = 0; i < top; i++) {
      const uint32_t rd = (uint32_t)G.radix[i], qq = rem / rd, d = rem - qq * rd;
      dig |= d << (4 * i);
      goff += d * G.st[i] * (uint32_t)sizeof(Cx<R>);
      rem = qq;
    }
  }
  auto digit = [&](int i) -> int { return (int)((dig >> (4 * i)) & 15u); };
  const uint32_t stt = G.st[top];
  const Cx<R> *__restrict__ v = reinterpret_cast<const Cx<R> *>(P.v);
  double red[3][1] = {{0.0}, {0.0}, {0.0}};
  __syncthreads();
  // the top site's ladder factors
  R gpt[RPT], gmt[RPT];
#pragma unroll
  for (int d = 0; d < RPT; d++) {
    gpt[d] = unir(s_gp[top * 16 + d]);
    gmt[d] = unir(s_gm[top * 16 + d]);
  }

  const bool xcd = gridDim.x >= 8 && (gridDim.x & 7u) == 0;
  const uint32_t nbx = xcd ? gridDim.x >> 3 : gridDim.x, x = xcd ? blockIdx.x & 7u : 0u;
  const uint32_t stride_c = xcd ? 8u : 1u;
  for (uint32_t l = xcd ? blockIdx.x >> 3 : blockIdx.x;; l += nbx) {
    const uint64_t c64 = ((uint64_t)(l / chunk) * stride_c + x) * chunk;
    if (c64 >= G.ntile) break;
    if (c64 + l % chunk >= G.ntile) continue;  // (a last chunk that is not full)
    const uint32_t tl = (uint32_t)(c64 + l % chunk);
    // outer digits, 4 bits each (at most 16 outer sites), and the tile's base row
    uint64_t od = 0;
    uint32_t base = 0;
    {
      uint32_t rem = tl;
      for (int k = t; k < n; k++) {
        const uint32_t rd = (uint32_t)G.radix[k], qq = rem / rd, d = rem - qq * rd;
        od |= (uint64_t)d << (4 * (k - t));
        base += d * G.st[k];
        rem = qq;
      }
    }
    auto odig = [&](int k) -> int { return (int)((od >> (4 * (k - t))) & 15u); };
    auto om = [&](int k) -> R { return (R)odig(k) - (R)G.s[k]; };
    const Cx<R> *vb = v + base;
    // RPT rows at a uniform offset from the tile, lower-site shift `off` per lane
    auto rows = [&](Cx<R> (&y)[RPT], int64_t shift, uint32_t off) {
      const Cx<R> *p = vb + shift;
#pragma unroll
      for (int d = 0; d < RPT; d++) {
        y[d] = *reinterpret_cast<const Cx<R> *>(reinterpret_cast<const char *>(p) + off);
        p += stt;
      }
    };
    Cx<R> own[RPT];
    rows(own, 0, goff);
    if (act)
#pragma unroll
      for (int d = 0; d < RPT; d++) tile[q * SP + d] = own[d];
    if (tid < 64) {
      // wave 0: the valid terms with one coefficient per tile
      int no = 0, pos;
      for (int c0 = 0; c0 < 2 * (n - t); c0 += 64) {  // single flips of outer sites by two
        const int c = c0 + tid, k = t + c / 2, di = (c & 1) * 3, D = (c & 1) ? 2 : -2;
        bool ok = c < 2 * (n - t) && ((G.smask2 >> k) & 1u);
        int d = 0;
        if (ok) {
          d = odig(k);
          ok = (unsigned)(d + D) < (unsigned)G.radix[k];
        }
        no = append(ok, no, &pos);
        if (ok) {
          s_ooff[pos] = (int64_t)D * (int64_t)G.st[k];
          s_oc[pos] = s_hoff[(k * 4 + di) * 16 + d];
        }
      }
      const int p0 = G.np - G.np_out;
      for (int c0 = 0; c0 < 4 * G.np_out; c0 += 64) {  // pairs of two outer sites
        const int c = c0 + tid, p = p0 + c / 4, qt = c & 3;
        bool ok = c < 4 * G.np_out;
        Cx<R> cf{0, 0};
        int64_t off = 0;
        if (ok) {
          const int4 ab = s_pij[p];
          const int da = odig(ab.x), db = odig(ab.y);
          const bool am = (qt >> 1) != 0, bm = (qt & 1) != 0;  // '-' ladder: the partner is one up
          const R f = (am ? s_gm : s_gp)[ab.x * 16 + da] * (bm ? s_gm : s_gp)[ab.y * 16 + db];
          ok = ((ab.z >> qt) & 1) && f != R(0);
          const Cx<R> cc = s_pc[4 * p + qt];
          cf = Cx<R>{cc.re * f, cc.im * f};
          const int64_t sa = (int64_t)G.st[ab.x], sb = (int64_t)G.st[ab.y];
          off = (am ? sa : -sa) + (bm ? sb : -sb);
        }
        no = append(ok, no, &pos);
        if (ok) {
          s_ooff[pos] = off;
          s_oc[pos] = cf;
        }
      }
      if (tid == 0) *s_cnt = no;
    } else if (tid < 64 + n) {
      // wave 1: for a tile site, the field of the outer sites' z-components; for an
      // outer site, its own diagonal element and its coupling to the later ones
      const int i = tid - 64;
      R ph = 0;
      for (int k = i < t ? t : i + 1; k < n; k++) ph = fma(s_zz[i * n + k], om(k), ph);
      s_phi[i] = i < t ? ph : fma(om(i), ph, s_hd[i * 16 + odig(i)]);
    }
    __syncthreads();
    Cx<R> acc[RPT];
#pragma unroll
    for (int d = 0; d < RPT; d++) acc[d] = Cx<R>{0, 0};
    {
      R dq = 0;
      for (int k = t; k < n; k++) dq += s_phi[k];
      for (int i = 0; i < top; i++) dq = fma((R)digit(i) - (R)G.s[i], s_phi[i], dq);
#pragma unroll
      for (int d = 0; d < RPT; d++) {
        const R dg = tdiag[q + (uint32_t)d * Q] + fma((R)d - (R)G.s[top], s_phi[top], dq);
        acc[d] = Cx<R>{dg * own[d].re, dg * own[d].im};
      }
    }
    // y shifted by one along the top site, times cc: the pair's top move up (the
    // partner is d + 1, '-' ladder) or down
    auto top_move = [&](const Cx<R> &cc, bool up, const Cx<R> (&y)[RPT]) {
      if (up) {
#pragma unroll
        for (int d = 0; d + 1 < RPT; d++) cfma<R, CPLX>(acc[d], cc, Cx<R>{gmt[d] * y[d + 1].re, gmt[d] * y[d + 1].im});
      } else {
#pragma unroll
        for (int d = 1; d < RPT; d++) cfma<R, CPLX>(acc[d], cc, Cx<R>{gpt[d] * y[d - 1].re, gpt[d] * y[d - 1].im});
      }
    };
    auto lds_rows = [&](Cx<R> (&y)[RPT], int qp) {
#pragma unroll
      for (int d = 0; d < RPT; d++) y[d] = tile[qp * SP + d];
    };
    // single flips of the top site: registers only
    if ((G.smask >> top) & 1u) {
#pragma unroll
      for (int di = 0; di < 4; di++) {
        const int D = (di < 2) ? di - 2 : di - 1;
        if ((D == 2 || D == -2) && !((G.smask2 >> top) & 1u)) continue;
#pragma unroll
        for (int d = 0; d < RPT; d++)
          if (d + D >= 0 && d + D < RPT) cfma<R, CPLX>(acc[d], s_hoff[(top * 4 + di) * 16 + d], own[d + D]);
      }
    }
    // lower sites: single flips and pairs with the top site
#pragma unroll 1
    for (int i = 0; i < top; i++) {
      const int pt = G.ptop[i];  // the pair (i, top), or -1
      const bool sg = (G.smask >> i) & 1u;
      if (!sg && pt < 0) continue;
      const int di = digit(i), rd = G.radix[i], ws = (int)G.st[i];
      const int nzt = pt < 0 ? 0 : uni(s_pij[pt].z);
#pragma unroll
      for (int up = 0; up < 2; up++) {
        const R fi = (up ? s_gm : s_gp)[i * 16 + di];
        const bool ok = fi != R(0);
        Cx<R> y[RPT];
        lds_rows(y, ok ? (int)q + (up ? ws : -ws) : (int)q);
        if (sg) {
          // (an invalid move has coefficient 0 in the table)
          const Cx<R> c = s_hoff[(i * 4 + (up ? 2 : 1)) * 16 + di];
#pragma unroll
          for (int d = 0; d < RPT; d++) cfma<R, CPLX>(acc[d], c, y[d]);
        }
#pragma unroll
        for (int tu = 0; tu < 2; tu++)
          if ((nzt >> (2 * up + tu)) & 1) {
            const Cx<R> c = s_pc[4 * pt + 2 * up + tu];
            top_move(Cx<R>{c.re * fi, c.im * fi}, tu != 0, y);
          }
      }
      if ((G.smask2 >> i) & 1u) {
#pragma unroll
        for (int up = 0; up < 2; up++) {
          const int D = up ? 2 : -2;
          const bool ok = (unsigned)(di + D) < (unsigned)rd;
          const Cx<R> c = s_hoff[(i * 4 + (up ? 3 : 0)) * 16 + di];
          Cx<R> y[RPT];
          lds_rows(y, ok ? (int)q + D * ws : (int)q);
#pragma unroll
          for (int d = 0; d < RPT; d++) cfma<R, CPLX>(acc[d], c, y[d]);
        }
      }
    }
    // pairs of two lower sites
#pragma unroll 1
    for (int p = 0; p < G.np_low; p++) {
      const int4 ab = s_pij[p];
      const int a = uni(ab.x), b = uni(ab.y), nz = uni(ab.z);
      const int da = digit(a), db = digit(b), wa = (int)G.st[a], wb = (int)G.st[b];
#pragma unroll
      for (int qt = 0; qt < 4; qt++) {
        if (!((nz >> qt) & 1)) continue;
        const bool am = (qt >> 1) != 0, bm = (qt & 1) != 0;
        const R f = (am ? s_gm : s_gp)[a * 16 + da] * (bm ? s_gm : s_gp)[b * 16 + db];
        const Cx<R> c = s_pc[4 * p + qt];
        Cx<R> y[RPT];
        lds_rows(y, f != R(0) ? (int)q + (am ? wa : -wa) + (bm ? wb : -wb) : (int)q);
        const Cx<R> cc{c.re * f, c.im * f};
#pragma unroll
        for (int d = 0; d < RPT; d++) cfma<R, CPLX>(acc[d], cc, y[d]);
      }
    }
    // groups: one outer site and one move of it
#pragma unroll 1
    for (int k = t; k < n; k++) {
      const int m0 = G.mx[k - t], m1 = G.mx[k - t + 1];
      const bool sg = (G.smask >> k) & 1u;
      if (!sg && m0 == m1) continue;
      const int dk = odig(k);
#pragma unroll 1
      for (int up = 0; up < 2; up++) {
        if (up ? dk + 1 >= G.radix[k] : dk < 1) continue;
        const int64_t shift = up ? (int64_t)G.st[k] : -(int64_t)G.st[k];
        const R fk = unir((up ? s_gm : s_gp)[k * 16 + dk]);
        Cx<R> z[RPT];
        rows(z, shift, goff);
        if (sg) {
          const Cx<R> c = unic(s_hoff[(k * 4 + (up ? 2 : 1)) * 16 + dk]);
#pragma unroll
          for (int d = 0; d < RPT; d++) cfma<R, CPLX>(acc[d], c, z[d]);
        }
        // pairs with the top site first, then with lower sites; coefficient index
        // [tile move up][outer move up]
        bool low = false;
        for (int p = m0; p < m1; p++) {
          const int4 ab = s_pij[p];
          const int a = uni(ab.x), nz = uni(ab.z);
          if (a != top) {
            low = low || ((nz >> up) & 5);
            continue;
          }
#pragma unroll
          for (int tu = 0; tu < 2; tu++)
            if ((nz >> (2 * tu + up)) & 1) {
              const Cx<R> c = unic(s_pc[4 * p + 2 * tu + up]);
              top_move(Cx<R>{c.re * fk, c.im * fk}, tu != 0, z);
            }
        }
        if (!low) continue;
        __syncthreads();
        if (act)
#pragma unroll
          for (int d = 0; d < RPT; d++) tile[q * SP + d] = z[d];
        __syncthreads();
#pragma unroll 1
        for (int p = m0; p < m1; p++) {
          const int4 ab = s_pij[p];
          const int a = uni(ab.x), nz = uni(ab.z);
          if (a == top) continue;
          const int da = digit(a);
#pragma unroll
          for (int au = 0; au < 2; au++) {
            if (!((nz >> (2 * au + up)) & 1)) continue;
            const R fa = (au ? s_gm : s_gp)[a * 16 + da];
            const Cx<R> c = unic(s_pc[4 * p + 2 * au + up]);
            Cx<R> y[RPT];
            const int ws = (int)G.st[a];
            lds_rows(y, fa != R(0) ? (int)q + (au ? ws : -ws) : (int)q);
            const R f = fa * fk;
            const Cx<R> cc{c.re * f, c.im * f};
#pragma unroll
            for (int d = 0; d < RPT; d++) cfma<R, CPLX>(acc[d], cc, y[d]);
          }
        }
      }
    }
    // one coefficient per tile: two terms' loads in flight
    const int no = uni(*s_cnt);
#pragma unroll 1
    for (int e = 0; e < no; e += 2) {
      const int e1 = e + 1 < no ? e + 1 : e;
      Cx<R> y0[RPT], y1[RPT];
      rows(y0, uni64(s_ooff[e]), goff);
      rows(y1, uni64(s_ooff[e1]), goff);
      const Cx<R> c0 = unic(s_oc[e]);
#pragma unroll
      for (int d = 0; d < RPT; d++) cfma<R, CPLX>(acc[d], c0, y0[d]);
      if (e1 != e) {
        const Cx<R> c1 = unic(s_oc[e1]);
#pragma unroll
        for (int d = 0; d < RPT; d++) cfma<R, CPLX>(acc[d], c1, y1[d]);
      }
    }
    if (act) {
      // (the own rows are read again: held through the terms they cost registers)
      Cx<R> x[RPT];
      if (P.lanczos) {
        rows(x, 0, goff);
      } else {
#pragma unroll
        for (int d = 0; d < RPT; d++) x[d] = Cx<R>{0, 0};
      }
#pragma unroll
      for (int d = 0; d < RPT; d++) {
        const uint32_t row = base + goff / (uint32_t)sizeof(Cx<R>) + (uint32_t)d * stt;
        Acc<R, 1> a;
        a.re[0] = acc[d].re;
        a.im[0] = acc[d].im;
        hv_epilogue<R, 1, true>(P, row, 0, a, &x[d], red);
      }
    }
    __syncthreads();  // the next tile overwrites the LDS
  }
  if (!P.lanczos) return;
  // (the block's size is the plan's: sum over its waves in order)
  __shared__ double part[16][3];
#pragma unroll
  for (int a = 0; a < 3; a++) {
    const double s = wave_sum(red[a][0]);
    if ((tid & 63) == 0) part[tid >> 6][a] = s;
  }
  __syncthreads();
  if (tid < 3) {
    double s = 0;
    for (int wv = 0; wv < NT / 64; wv++) s += part[wv][tid];
    P.part[(size_t)blockIdx.x * 3 + tid] = s;
  }
}

template <typename R, int RPT, bool CPLX>
int launch_t(const SweepPass &G, const SweepTables &S, const DevTables<R> &tb, const HvParams &P, unsigned gx,
             uint32_t chunk, hipStream_t s) {
  static std::atomic<uint64_t> granted{0};
  const size_t sm = SweepLds<R>(G).total;
  const int rc = grant_lds(reinterpret_cast<const void *>(&hv_sweep<R, RPT, CPLX>), 1024, sm, granted);  // (1 KB: the sums)
  if (rc) return rc;
  hipLaunchKernelGGL((hv_sweep<R, RPT, CPLX>), dim3(gx), dim3(sweep_block(G)), sm, s, G, tb,
                     S.d_pij, reinterpret_cast<const Cx<R> *>(S.d_pc), reinterpret_cast<const R *>(S.d_tdiag), chunk, P);
  return FTLM_OK;
}

template <typename R, bool CPLX>
int launch_rpt(const SweepPass &G, const SweepTables &S, const DevTables<R> &tb, const HvParams &P, unsigned gx,
               uint32_t chunk, hipStream_t s) {
  switch (G.rtop) {
    case 3: return launch_t<R, 3, CPLX>(G, S, tb, P, gx, chunk, s);
    case 4: return launch_t<R, 4, CPLX>(G, S, tb, P, gx, chunk, s);
    case 5: return launch_t<R, 5, CPLX>(G, S, tb, P, gx, chunk, s);
    case 6: return launch_t<R, 6, CPLX>(G, S, tb, P, gx, chunk, s);
    default: return FTLM_EINVAL;
  }
}

template <typename R>
int launch_r(const SweepPlan &sp, const DevTables<R> &tb, const HvParams &P, int cap, int kc, unsigned *gx_out,
             hipStream_t s) {
  if (!sp.ok || !sp.tab.d_pij) return FTLM_EINVAL;
  const SweepPass &G = sp.pass;
  if (cap <= 0) {
    // the blocks resident at once on 256 CUs, by registers and by LDS
    const int wv = sweep_block(G) / 64;
    const int regs = 4 * sweep_waves(sizeof(R), G.rtop) / wv;
    const int lds = (int)(160 * 1024 / (SweepLds<R>(G).total + 1024));
    cap = 256 * std::max(1, std::min(regs, lds));
  }
  cap = std::min(cap, 2048);
  uint32_t gx = G.ntile < (uint32_t)cap ? G.ntile : (uint32_t)cap;
  if (gx >= 8) gx &= ~7u;
  *gx_out = gx;
  const uint32_t chunk = 1u << ((kc >> 4) & 15);
  return sp.cplx ? launch_rpt<R, true>(G, sp.tab, tb, P, gx, chunk, s)
                 : launch_rpt<R, false>(G, sp.tab, tb, P, gx, chunk, s);
}

}  // namespace

// Host plan: the tile takes the low sites while its rows fit tile_rows and the values of
// the sites below the top one fit the block's threads.
void plan_sweep(const HostHam &hh, size_t es, uint32_t tile_rows, SweepPlan &pl) {
  const SweepTables keep = pl.tab;
  pl = SweepPlan();
  pl.tab = keep;
  const int n = hh.n;
  if (hh.has_z || hh.spin_half || hh.dim < (1u << 16)) return;
  int t = 0;
  uint64_t T = 1;
  while (t < n && t < 9 && T <= (uint64_t)sweep_threads(hh.radix[t]) && T * (uint64_t)hh.radix[t] <= tile_rows)
    T *= (uint64_t)hh.radix[t++];
  if (t < 2 || n - t > 16 || n - t < 1) return;
  const int rtop = hh.radix[t - 1];
  if (rtop < 3 || rtop > 6) return;  // the instantiated rows per thread
  SweepPass G{};
  G.n = n;
  G.t = t;
  G.rtop = rtop;
  G.Q = (uint32_t)(T / rtop);
  G.ntile = (uint32_t)(hh.dim / T);
  for (int k = 0; k < n; k++) {
    G.radix[k] = hh.radix[k];
    G.st[k] = hh.stride[k];
    G.s[k] = 0.5f * (float)hh.two_s[k];
    if (site_has_singles(hh, k)) G.smask |= 1u << k;
    for (int d = 0; d + 2 < hh.radix[k]; d++) {
      const Cx<double> up = hh.h[(size_t)k * 256 + d * 16 + d + 2], dn = hh.h[(size_t)k * 256 + (d + 2) * 16 + d];
      if (up.re != 0.0 || up.im != 0.0 || dn.re != 0.0 || dn.im != 0.0) G.smask2 |= 1u << k;
    }
  }
  // pairs of sites (a, b): both lower | lower a, top b | tile a, outer b (by b) | outer
  struct E {
    int cls, a, b, p;
  };
  std::vector<E> es_;
  for (int p = 0; p < hh.npair; p++) {
    int a = hh.pi[p], b = hh.pj[p];
    if (a > b) std::swap(a, b);
    es_.push_back({b >= t ? (a >= t ? 3 : 2) : (b == t - 1 ? 1 : 0), a, b, p});
  }
  std::stable_sort(es_.begin(), es_.end(), [](const E &x, const E &y) {
    if (x.cls != y.cls) return x.cls < y.cls;
    return x.cls == 2 && x.b < y.b;
  });
  for (int i = 0; i < kMaxSites; i++) G.ptop[i] = -1;
  G.np = (int)es_.size();
  bool cplx = false;
  for (int e = 0; e < G.np; e++) {
    const E &x = es_[e];
    const bool swapped = hh.pi[x.p] != x.a;
    int nz = 0;
    for (int qa = 0; qa < 2; qa++)
      for (int qb = 0; qb < 2; qb++) {
        const Cx<double> c = hh.pc[4 * x.p + (swapped ? 2 * qb + qa : 2 * qa + qb)];
        pl.pc.push_back(c);
        if (c.re != 0.0 || c.im != 0.0) nz |= 1 << (2 * qa + qb);
        cplx = cplx || c.im != 0.0;
      }
    pl.pij.push_back(make_int4(x.a, x.b, nz, 0));
    if (x.cls == 0) G.np_low++;
    if (x.cls == 1) G.ptop[x.a] = e;
    if (x.cls == 3) G.np_out++;
  }
  int e = 0;
  while (e < G.np && es_[e].cls < 2) e++;
  for (int k = t; k < n; k++) {
    G.mx[k - t] = e;
    while (e < G.np && es_[e].cls == 2 && es_[e].b == k) e++;
  }
  G.mx[n - t] = e;
  for (int k = 0; k < n; k++)
    for (int a = 0; a < hh.radix[k]; a++)
      for (int b = 0; b < hh.radix[k]; b++)
        if (a != b) cplx = cplx || hh.h[(size_t)k * 256 + a * 16 + b].im != 0.0;
  pl.cplx = cplx;
  // diagonal over the tile sites, per tile row, built site by site: a value d of site k adds
  // its own element and its moment times the z-field of the sites below (every row anew
  // took 87 us of each field change of the centred cube in either precision, and this 5)
  pl.tdiag.assign(T, 0.0);
  std::vector<double> zf(T);
  uint32_t below = 1;  // rows of the sites below k
  for (int k = 0; k < t; k++) {
    zf[0] = 0.0;
    uint32_t m = 1;
    for (int j = 0; j < k; j++) {
      const double z = hh.zz[(size_t)k * n + j];
      for (int d = G.radix[j] - 1; d >= 0; d--)
        for (uint32_t r = 0; r < m; r++) zf[r + d * m] = zf[r] + z * (d - 0.5 * hh.two_s[j]);
      m *= (uint32_t)G.radix[j];
    }
    for (int d = G.radix[k] - 1; d >= 0; d--) {
      const double own = hh.h[(size_t)k * 256 + d * 16 + d].re, mk = d - 0.5 * hh.two_s[k];
      for (uint32_t r = 0; r < below; r++) pl.tdiag[r + d * below] = pl.tdiag[r] + (own + mk * zf[r]);
    }
    below *= (uint32_t)G.radix[k];
  }
  // the block's tables and tile share the LDS
  const size_t lds = es == 16 ? SweepLds<double>(G).total : SweepLds<float>(G).total;
  if (lds > 159 * 1024) return;  // 1 KB for static LDS
  pl.pass = G;
  pl.ok = true;
}

int launch_sweep(const DevHam &dh, int precision, const HvParams &P, int cap, int kc, unsigned *gx, hipStream_t s) {
  if (P.K != 1) return FTLM_EINVAL;
  return precision == FTLM_C64 ? launch_r<float>(dh.sw32, dh.t32, P, cap, kc, gx, s)
                               : launch_r<double>(dh.sw64, dh.t64, P, cap, kc, gx, s);
}

}  // namespace ftlm
