// Krylov eigenpairs: implicit QL with shifts on symmetric tridiagonals, as
// published by Bowdler, Martin, Reinsch and Wilkinson, "The QR and QL algorithms
// for symmetric matrices", Numer. Math. 11 (1968) 293-306 (tql2).
//
//  * tridiag_kernel : two rows of the eigenvector matrix (what the thermal sums
//    of Eqs. (E-2-C) and (E-2-D) need), one wave per column; tridiag_lanes_kernel :
//    the same with a lane per column, for thousands of short columns;
//  * tridiag_full_kernel : the whole eigenvector matrix (the double sum of
//    Eq. (E-2-H)), one block per column.
//
// What bounds them is the serial chain of one plane rotation after the other
// (about 85 n of them for a Krylov tridiagonal of n = 100): nothing else in a
// column can start before it.  So a column has a wave of its own (no lane waits
// for another column's sweep), every lane carries the same scalars, the search
// for a negligible off-diagonal element takes 64 elements at a time with a
// ballot, and a rotation has no division and no guarded hypot in its chain: with
// T scaled by a power of two to norm about 1, f^2 + g^2 cannot overflow, and
// sqrt and its reciprocal come from one reciprocal square root refined by two
// coupled Newton steps, c and s from the reciprocal and the quotients' residuals.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ftlm_internal.hpp"

namespace ftlm {

namespace {

constexpr int kWave = 64;

// r = sqrt(x), ri = 1 / sqrt(x) for a normal positive x (coupled Newton steps:
// g -> sqrt x, h -> 1 / (2 sqrt x), the residual 1/2 - h g in one fma; then the residual
// of g itself, which rounds r to within half a unit and a little)
__device__ __forceinline__ void sqrt_pair(double x, double &r, double &ri) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
#pragma unroll
  for (int it = 0; it < 2; it++) {
    const double q = fma(-h, g, 0.5);
    g = fma(g, q, g);
    h = fma(h, q, h);
  }
  r = fma(fma(-g, g, x), h, g);
  ri = 2.0 * h;
}

// a / r by its reciprocal and the quotient's residual.  (Products with the reciprocal
// alone, and an r of one or two units, left c^2 + s^2 off 1 to one side: 100 steps of
// rotations moved every eigenvalue by up to 2e-15 of it, five times what divisions did.)
__device__ __forceinline__ double quot(double a, double r, double ri) {
  const double q = a * ri;
  return fma(fma(-q, r, a), ri, q);
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, kWave));
  return v;
}

// Power of two that brings the largest |d|, |e| of a column to [1/2, 1) (its
// exponent in *ex); 1 for a zero or non-finite column.
__device__ __forceinline__ double norm_scale(double big, int *ex) {
  *ex = 0;
  if (!(big > 0.0) || !(big < 1.7e308)) return 1.0;
  (void)frexp(big, ex);
  *ex = max(-1000, min(1000, *ex));
  return ldexp(1.0, -*ex);
}

// First m >= l whose off-diagonal element e[m] is negligible (n - 1 if none is);
// called by a whole wave, 64 elements per trip.
__device__ __forceinline__ int ql_block_end(const double *d, const double *e, size_t S, int l, int n) {
  const int lane = threadIdx.x & (kWave - 1);
  for (int base = l;; base += kWave) {
    const int i = base + lane;
    bool stop = i >= n - 1;
    if (!stop) {
      const double dd = fabs(d[(size_t)i * S]) + fabs(d[(size_t)(i + 1) * S]);
      stop = fabs(e[(size_t)i * S]) <= 2.220446049250313e-16 * dd;
    }
    const unsigned long long mask = __ballot(stop);
    if (mask) return base + __builtin_ctzll(mask);
  }
}

// One QL sweep over the block [l, m]; rot(i, c, s) for every rotation of columns
// i and i + 1, i = m - 1 down to the returned index (l, or above it when a
// rotation vanishes and the block splits).  Every lane runs it alike and writes
// the same values.
template <typename F>
__device__ __forceinline__ int ql_sweep(double *d, double *e, size_t S, int l, int m, F &&rot) {
#define AT(p, i) (p)[(size_t)(i)*S]
  const double el = AT(e, l), dl = AT(d, l);
  double gg = (AT(d, l + 1) - dl) / (2.0 * el);
  const double r0 = sqrt(fma(gg, gg, 1.0));
  gg = AT(d, m) - dl + el / (gg + copysign(r0, gg));
  double s = 1.0, c = 1.0, p = 0.0;
  // the next rotation's elements are read one step ahead, and d[i + 1] is the
  // previous step's d[i]
  double d_hi = AT(d, m), e_i = AT(e, m - 1), d_i = AT(d, m - 1);
  for (int i = m - 1; i >= l; i--) {
    const int in = max(i - 1, l);
    const double e_n = AT(e, in), d_n = AT(d, in);
    const double f = s * e_i, b = c * e_i;
    const double t = fma(gg, gg, f * f);
    const double g1 = d_hi - p;
    if (t <= 1e-280) {  // (a NaN goes on, as any other value)
      AT(e, i + 1) = 0.0;
      AT(d, i + 1) = g1;
      AT(e, m) = 0.0;
      return i + 1;
    }
    double r, ri;
    sqrt_pair(t, r, ri);
    AT(e, i + 1) = r;
    s = quot(f, r, ri);
    c = quot(gg, r, ri);
    const double r2 = fma(d_i - g1, s, 2.0 * c * b);
    p = s * r2;
    AT(d, i + 1) = g1 + p;
    gg = fma(c, r2, -b);
    rot(i, c, s);
    d_hi = d_i;
    e_i = e_n;
    d_i = d_n;
  }
  AT(d, l) = d_hi - p;
  AT(e, l) = gg;
  AT(e, m) = 0.0;
  return l;
#undef AT
}

// A sweep that carries the rows z1 = e_1^T Z and zy = y^T Z of Z, the product of the plane
// rotations; rotated entries stay in registers for the next rotation, the entries of
// index i - 1 are read one step ahead.
__device__ __forceinline__ void ql_sweep_rows(double *d, double *e, double *z1, double *zy, size_t S, int l, int m) {
  double a_hi = z1[(size_t)m * S], b_hi = zy[(size_t)m * S];
  double a_i = z1[(size_t)(m - 1) * S], b_i = zy[(size_t)(m - 1) * S];
  const int lo = ql_sweep(d, e, S, l, m, [&](int i, double c, double s) {
    const int in = max(i - 1, l);
    const double a_n = z1[(size_t)in * S], b_n = zy[(size_t)in * S];
    z1[(size_t)(i + 1) * S] = fma(s, a_i, c * a_hi);
    a_hi = fma(c, a_i, -s * a_hi);
    zy[(size_t)(i + 1) * S] = fma(s, b_i, c * b_hi);
    b_hi = fma(c, b_i, -s * b_hi);
    a_i = a_n;
    b_i = b_n;
  });
  z1[(size_t)lo * S] = a_hi;
  zy[(size_t)lo * S] = b_hi;
}

struct TriArgs {
  int n_cols, nl;
  const int *n_used;
  int used_stride, in_stride;
  const double *alpha, *beta, *y;
  double *eps, *q1, *qy;
  int out_stride, out_col0;
};

// Column col's elements i0, i0 + di, ...: their largest size; scaled into the work arrays;
// and the results.
__device__ __forceinline__ double tri_big(const TriArgs &A, int col, int n, int i0, int di) {
  double big = 0.0;
  for (int i = i0; i < n; i += di) {
    big = fmax(big, fabs(A.alpha[(size_t)i * A.in_stride + col]));
    if (i + 1 < n) big = fmax(big, fabs(A.beta[(size_t)i * A.in_stride + col]));
  }
  return big;
}
__device__ __forceinline__ void tri_load(const TriArgs &A, int col, int n, int i0, int di, double sc, double *d, double *e,
                                         double *z1, double *zy, size_t S) {
  for (int i = i0; i < n; i += di) {
    d[(size_t)i * S] = A.alpha[(size_t)i * A.in_stride + col] * sc;
    e[(size_t)i * S] = (i + 1 < n) ? A.beta[(size_t)i * A.in_stride + col] * sc : 0.0;
    z1[(size_t)i * S] = (i == 0) ? 1.0 : 0.0;
    zy[(size_t)i * S] = A.y ? A.y[(size_t)i * A.in_stride + col] : 0.0;
  }
}
__device__ __forceinline__ void tri_store(const TriArgs &A, int col, int n, int i0, int di, int ex, const double *d,
                                          const double *z1, const double *zy, size_t S) {
  for (int i = i0; i < A.nl; i += di) {
    const bool ok = i < n;
    const size_t o = (size_t)i * A.out_stride + A.out_col0 + col;
    A.eps[o] = ok ? ldexp(d[(size_t)i * S], ex) : 0.0;
    A.q1[o] = ok ? z1[(size_t)i * S] : 0.0;
    A.qy[o] = ok ? zy[(size_t)i * S] : 0.0;
  }
}

// One wave per column; the four work arrays of the column are in LDS, or in the global
// scratch [4][nl][n_cols].
// 100 steps, 20 columns: 6.2 ms as one lane per column with hypot and two
// divisions per rotation, 2.7 ms so (2.5 with c and s as products with the reciprocal).
template <bool LDS>
__global__ __launch_bounds__(kWave) void tridiag_kernel(TriArgs A, double *scratch) {
  extern __shared__ double tri_sh[];
  const int col = blockIdx.x, lane = threadIdx.x;
  const int n = A.n_used ? min(A.n_used[col * A.used_stride], A.nl) : A.nl;
  const size_t S = LDS ? 1 : (size_t)A.n_cols;
  double *d = LDS ? tri_sh : scratch + col;
  double *e = d + (size_t)A.nl * S, *z1 = e + (size_t)A.nl * S, *zy = z1 + (size_t)A.nl * S;
  int ex;
  const double sc = norm_scale(wave_max(tri_big(A, col, n, lane, kWave)), &ex);
  tri_load(A, col, n, lane, kWave, sc, d, e, z1, zy, S);
  __syncthreads();
  for (int l = 0; l < n; l++) {
    for (int iter = 0; iter < 100; iter++) {
      const int m = ql_block_end(d, e, S, l, n);
      if (m == l) break;
      ql_sweep_rows(d, e, z1, zy, S, l, m);
    }
  }
  __syncthreads();
  tri_store(A, col, n, lane, kWave, ex, d, z1, zy, S);
}

// One lane per column, for columns enough that the rotations are not waited for but
// issued: the work arrays [4][nl][blockDim] of a block's columns in LDS.  The same
// rotations as a wave per column, to the bit.
__global__ __launch_bounds__(kWave) void tridiag_lanes_kernel(TriArgs A) {
  extern __shared__ double tri_sh[];
  const int col = blockIdx.x * blockDim.x + threadIdx.x;
  if (col >= A.n_cols) return;
  const int n = A.n_used ? min(A.n_used[col * A.used_stride], A.nl) : A.nl;
  const size_t S = blockDim.x;
  double *d = tri_sh + threadIdx.x;
  double *e = d + (size_t)A.nl * S, *z1 = e + (size_t)A.nl * S, *zy = z1 + (size_t)A.nl * S;
  int ex;
  const double sc = norm_scale(tri_big(A, col, n, 0, 1), &ex);
  tri_load(A, col, n, 0, 1, sc, d, e, z1, zy, S);
  for (int l = 0; l < n; l++) {
    for (int iter = 0; iter < 100; iter++) {
      int m = l;
      for (double dm = fabs(d[(size_t)l * S]); m < n - 1; m++) {
        const double dm1 = fabs(d[(size_t)(m + 1) * S]);
        if (fabs(e[(size_t)m * S]) <= 2.220446049250313e-16 * (dm + dm1)) break;
        dm = dm1;
      }
      if (m == l) break;
      ql_sweep_rows(d, e, z1, zy, S, l, m);
    }
  }
  tri_store(A, col, n, 0, 1, ex, d, z1, zy, S);
}

// One block per column c: element j of alpha and beta at
// (c / group) nl group + j group + c % group, n_used[c].  Wave 0 runs the sweeps' scalar chain and leaves each sweep's
// rotations in LDS; the other waves apply them to their rows of Z (LDS,
// column-major Z[i][a]) while wave 0 runs the next sweep (nbuf = 2 rotation
// buffers; nbuf = 1, where LDS holds no second one, takes turns).  Output:
// eps[c][nl] and Qt[c][m][a] = Q[a][m] (one eigenvector after the other), zero
// beyond n.
__global__ __launch_bounds__(256) void tridiag_full_kernel(int nl, int nbuf, const int *__restrict__ n_used,
                                                           const double *__restrict__ alpha,
                                                           const double *__restrict__ beta, int group,
                                                           double *__restrict__ eps, double *__restrict__ Qt) {
  extern __shared__ double tri_sh[];
  double *d = tri_sh, *e = d + nl, *rot = e + nl, *Z = rot + (size_t)2 * nl * nbuf;  // rot: [nbuf][2][nl]
  __shared__ int s_lo[2], s_hi[2];
  const int t = threadIdx.x, col = blockIdx.x;
  const int n = min(n_used[col], nl);
  const size_t in0 = (size_t)(col / group) * nl * group + col % group;
  alpha += in0;
  beta += in0;
  eps += (size_t)col * nl;
  Qt += (size_t)col * nl * nl;
  double big = 0.0;
  for (int i = t & (kWave - 1); i < n; i += kWave) {  // every wave alike
    big = fmax(big, fabs(alpha[(size_t)i * group]));
    if (i + 1 < n) big = fmax(big, fabs(beta[(size_t)i * group]));
  }
  int ex;
  const double sc = norm_scale(wave_max(big), &ex);
  for (int i = t; i < nl; i += blockDim.x) {
    d[i] = i < n ? alpha[(size_t)i * group] * sc : 0.0;
    e[i] = (i + 1 < n) ? beta[(size_t)i * group] * sc : 0.0;
  }
  for (int idx = t; idx < nl * nl; idx += blockDim.x) Z[idx] = (idx / nl == idx % nl) ? 1.0 : 0.0;
  __syncthreads();
  int l = 0, iter = 0, buf = 0;  // l and iter: wave 0's
  while (true) {
    if (t < kWave) {
      double *rc = rot + (size_t)buf * 2 * nl, *rs = rc + nl;
      int m = l;
      while (l < n) {
        m = ql_block_end(d, e, 1, l, n);
        if (m != l && iter < 100) break;
        l++;
        iter = 0;
      }
      int lo = -1;  // -1: done
      if (l < n) {
        iter++;
        lo = ql_sweep(d, e, 1, l, m, [&](int i, double c, double s) {
          rc[i] = c;
          rs[i] = s;
        });
      }
      s_lo[buf] = lo;
      s_hi[buf] = m - 1;
    }
    __syncthreads();
    const int lo = s_lo[buf], hi = s_hi[buf];
    if (lo < 0) break;
    if (t >= kWave) {
      const double *rc = rot + (size_t)buf * 2 * nl, *rs = rc + nl;
      for (int a = t - kWave; a < nl; a += blockDim.x - kWave) {
        double z_hi = Z[(size_t)(hi + 1) * nl + a];
#pragma unroll 4
        for (int i = hi; i >= lo; i--) {
          const double c = rc[i], s = rs[i], z = Z[(size_t)i * nl + a];
          Z[(size_t)(i + 1) * nl + a] = fma(s, z, c * z_hi);
          z_hi = fma(c, z, -s * z_hi);
        }
        Z[(size_t)lo * nl + a] = z_hi;
      }
    }
    if (nbuf == 1) __syncthreads();
    else buf ^= 1;
  }
  for (int i = t; i < nl; i += blockDim.x) eps[i] = i < n ? ldexp(d[i], ex) : 0.0;
  for (int idx = t; idx < nl * nl; idx += blockDim.x) {
    const int m = idx / nl, a = idx % nl;
    Qt[idx] = (a < n && m < n) ? Z[idx] : 0.0;
  }
}

// A lane per column instead of a wave?  Its time does not grow until the columns that 64 KB
// of LDS hold are taken by every block that fits, the other's from about 2000 columns on.
// Measured (us, wave / lane per column):
//   steps   320 columns     4000            8000            32,000            128,000
//   10      49 / 100        91 / 106        157 / 112       543 / 112         1910 / 138
//   30      313 / 810       627 / 836       1099 / 823      3566 / 852        13115 / 3349
//   60      1129 / 3039     2175 / 3013     3682 / 2901     12850 / 5960      48277 / 23321
//   100     2916 / 8490     5583 / 8867     9726 / 8229     34128 / 29937     129038 / 96649
//   120     4157 / 11773    7881 / 12466    13991 / 11398   48848 / 42710     (64,000: 93667 / 83533)
//   160     7226 / 19730    13756 / 24366   24276 / 36687   85487 / 113997
bool lanes_per_column_pay(int n_cols, int nl) { return n_cols >= 7168 && nl <= 128; }

size_t full_smem(int nl, int nbuf) {
  return sizeof(double) * ((size_t)2 * nl + (size_t)2 * nl * nbuf + (size_t)nl * nl);
}

}  // namespace

int launch_tridiag(int n_cols, int n_lanczos, const int *n_used, int used_stride, int in_stride,
                   const double *alpha, const double *beta, const double *y, double *eps,
                   double *q1, double *qy, int out_stride, int out_col0, double *scratch,
                   hipStream_t s) {
  const size_t lds = (size_t)32 * n_lanczos;  // the four work arrays
  const TriArgs A{n_cols, n_lanczos, n_used, used_stride, in_stride, alpha, beta, y, eps, q1, qy, out_stride, out_col0};
  if (lanes_per_column_pay(n_cols, n_lanczos)) {
    const int cpb = (int)std::min<size_t>(kWave, 64 * 1024 / lds);  // as many columns as 64 KB hold
    hipLaunchKernelGGL(tridiag_lanes_kernel, dim3((n_cols + cpb - 1) / cpb), dim3(cpb), (size_t)cpb * lds, s, A);
  } else if (lds <= 64 * 1024) {
    hipLaunchKernelGGL(tridiag_kernel<true>, dim3(n_cols), dim3(kWave), lds, s, A, scratch);
  } else {
    hipLaunchKernelGGL(tridiag_kernel<false>, dim3(n_cols), dim3(kWave), 0, s, A, scratch);
  }
  return hipGetLastError() == hipSuccess ? FTLM_OK : FTLM_EHIP;
}

// (one rotation buffer is the least; a second one only where it fits too)
size_t tridiag_full_smem(int nl) { return full_smem(nl, 1); }

int launch_tridiag_full(int n_cols, int n_lanczos, const int *n_used, const double *alpha, const double *beta,
                        int group, double *eps, double *Qt, hipStream_t s) {
  constexpr size_t kLds = 160 * 1024 - 64;  // less the static words
  const int nbuf = full_smem(n_lanczos, 2) <= kLds ? 2 : 1;
  const size_t sm = full_smem(n_lanczos, nbuf);
  // (the same value from every host thread, whatever its length)
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(&tridiag_full_kernel),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds) != hipSuccess)
    return FTLM_EHIP;
  const int threads = kWave + std::min(192, (n_lanczos + kWave - 1) / kWave * kWave);
  hipLaunchKernelGGL(tridiag_full_kernel, dim3(n_cols), dim3(threads), sm, s, n_lanczos, nbuf, n_used, alpha, beta,
                     group, eps, Qt);
  return hipGetLastError() == hipSuccess ? FTLM_OK : FTLM_EHIP;
}

}  // namespace ftlm
