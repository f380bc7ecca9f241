// Symmetric FTLM (sFTLM) with pairs of mutually time-reversed random vectors,
// Sec. 2.2, Eqs. (E-2-G), (E-2-H).
//
// The R vectors (R/2 Gaussian vectors and their time reverses) iterate in waves
// of K interleaved columns.  A wave runs N_L Lanczos steps keeping every Krylov
// vector (slot j of the workspace holds the unnormalised X_j [dim][K] with scales
// sx_j), applies O = -sum_i g_i s_i.B_hat to every slot and forms Re(V^H O V) of
// every column (Gram kernel).  The tridiagonals of all R vectors are then
// diagonalised together with the full eigenvector matrices Q, and per temperature
//   den_r = sum_n exp(-(eps_n - E_min)/T) Q_1n^2                      (Eq. E-2-D)
//   num_r = z^T Re(O_K) z,  z_a = sum_n Q_an exp(-(eps_n - E_min)/2T) Q_1n
// (the double sum of Eq. E-2-H written as a quadratic form; z is real, so only
// the real part of O_K enters), and M = sum_r num_r / sum_r den_r.
// ln Z, E and C come from the Ritz values exactly as in the plain driver.
//
// Time reversal in the product basis (Condon-Shortley phases, site 0 fastest):
//   (Theta x)[dim-1-nu] = (-1)^{sum_i (2 s_i - d_i(nu))} conj(x[nu]).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "ftlm_internal.hpp"

namespace ftlm {

namespace {

struct ThetaGeom {
  int n;
  uint32_t dim;
  int radix[kMaxSites];
  int two_s_sum_parity;
};

// dst [dim][np]: np = 1: the time reverse of src [dim][1]; np = 2 P: columns 2p
// and 2p + 1 hold src's column p [dim][P] and its time reverse.  The scales of the
// P source columns are handed on to dst's (np >= 2).
template <typename R>
__global__ __launch_bounds__(256) void theta_kernel(ThetaGeom g, const Cx<R> *__restrict__ src, Cx<R> *__restrict__ dst,
                                                    int np, const double *__restrict__ sx_src, double *__restrict__ sx) {
  const int P = np > 1 ? np / 2 : 1;
  if (np > 1 && blockIdx.x == 0 && (int)threadIdx.x < np) sx[threadIdx.x] = sx_src[threadIdx.x / 2];
  const uint64_t total = (uint64_t)g.dim * P;
  for (uint64_t e = (uint64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (uint64_t)gridDim.x * 256) {
    const uint64_t nu = e / (unsigned)P;
    const int p = (int)(e - nu * P);
    uint32_t rem = (uint32_t)nu, dsum = 0;
    for (int k = 0; k < g.n; k++) {
      const uint32_t r = (uint32_t)g.radix[k], q = rem / r;
      dsum += rem - q * r;
      rem = q;
    }
    const bool neg = ((uint32_t)g.two_s_sum_parity + dsum) & 1u;  // parity of sum(2 s_i - d_i)
    const Cx<R> x = src[e];
    const Cx<R> th = neg ? Cx<R>{-x.re, x.im} : Cx<R>{x.re, -x.im};
    const uint64_t rev = (uint64_t)g.dim - 1 - nu;
    if (np == 1) {
      dst[rev] = th;
    } else {
      dst[nu * np + 2 * p] = x;
      dst[rev * np + 2 * p + 1] = th;
    }
  }
}

// Re(V^H W) of every column of a wave on the matrix cores: with a complex row
// read as two real ones, Re(conj(x) w) is the real product of length 2 dim, so one
// 16-byte load per lane feeds two v_mfma_f64_16x16x4f64 (real parts, imaginary
// parts; complex64 rows are widened first).  A wave owns a 32 x 32 block of (a, b)
// with a-block <= b-block (Re(V^H O V) is symmetric, the rest is mirrored) over
// the rows of its split: 4 loads feed 8 MFMAs.  blockIdx.x: block pair, y: column,
// z: group of 4 splits, one per wave; partial products at part[split][column].
// 100 x 100 over 7776 rows and 20 columns: 1.14 ms (16 x 16 tiles from LDS with
// vector FMAs, real and imaginary parts, one column per launch: 20 x 275 us).
constexpr int kGB = 32;
typedef double d4 __attribute__((ext_vector_type(4)));

template <typename R>
__global__ __launch_bounds__(256) void gram_kernel(const Cx<R> *__restrict__ X, const Cx<R> *__restrict__ Wv, int K,
                                                   int nl, uint32_t dim, uint32_t chunk, int nsplit,
                                                   const double *__restrict__ sx, int sstride, double *__restrict__ part) {
  const int lane = threadIdx.x & 63, c = blockIdx.y;
  const int split = blockIdx.z * 4 + (threadIdx.x >> 6);
  if (split >= nsplit) return;
  int bb = 0, ab = blockIdx.x;  // block pair index -> (ab <= bb)
  while (ab > bb) ab -= ++bb;
  const uint64_t lo = (uint64_t)split * chunk, hi = min((uint64_t)dim, lo + chunk);
  const int i = lane & 15, kr = lane >> 4;
  // slots past the last one read the last one; their products are not stored
  const Cx<R> *xa[2], *wb[2];
#pragma unroll
  for (int u = 0; u < 2; u++) {
    xa[u] = X + (size_t)min(ab * kGB + 16 * u + i, nl - 1) * dim * K + c;
    wb[u] = Wv + (size_t)min(bb * kGB + 16 * u + i, nl - 1) * dim * K + c;
  }
  d4 acc[2][2];
#pragma unroll
  for (int u = 0; u < 2; u++)
#pragma unroll
    for (int w = 0; w < 2; w++) acc[u][w] = d4{0, 0, 0, 0};
#pragma unroll 2
  for (uint64_t r0 = lo; r0 < hi; r0 += 4) {
    const bool ok = r0 + kr < hi;
    const size_t o = (size_t)(ok ? r0 + kr : lo) * K;
    Cx<R> x[2], w[2];
#pragma unroll
    for (int u = 0; u < 2; u++) {
      x[u] = xa[u][o];
      w[u] = wb[u][o];
    }
#pragma unroll
    for (int u = 0; u < 2; u++)
      if (!ok) x[u] = w[u] = Cx<R>{0, 0};
#pragma unroll
    for (int u = 0; u < 2; u++)
#pragma unroll
      for (int q = 0; q < 2; q++) {
        acc[u][q] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[u].re, (double)w[q].re, acc[u][q], 0, 0, 0);
        acc[u][q] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[u].im, (double)w[q].im, acc[u][q], 0, 0, 0);
      }
  }
  // D of each 16 x 16 tile: row 4 r + lane / 16, column lane % 16
  double *out = part + ((size_t)split * K + c) * nl * nl;
#pragma unroll
  for (int u = 0; u < 2; u++)
#pragma unroll
    for (int q = 0; q < 2; q++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int a = ab * kGB + 16 * u + 4 * r + kr, b = bb * kGB + 16 * q + i;
        if (a < nl && b < nl) out[(size_t)a * nl + b] = acc[u][q][r] * sx[(size_t)a * sstride + c];
      }
}

// Sums the partials over the splits in a fixed order; the blocks below the diagonal are
// mirrored.  PH threads share an element's splits (one after the other, each of its PHth
// splits, then the threads in order): with few columns and steps there are thousands of
// splits of few elements, and one thread's chain of loads took longer than the products
// (2^20 rows, 30 steps, one column: 4096 splits of 900 elements).
template <int PH>
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double *__restrict__ part, int nsplit, int nl, int K,
                                                          double *__restrict__ ok) {
  constexpr int NE = 256 / PH;  // elements per block
  __shared__ double sh[PH][NE];
  const int el = threadIdx.x % NE, ph = threadIdx.x / NE;
  const int idx = blockIdx.x * NE + el, c = blockIdx.y;
  double r = 0;
  if (idx < nl * nl) {
    int a = idx / nl, b = idx % nl;
    if (a / kGB > b / kGB) {
      const int t = a;
      a = b;
      b = t;
    }
#pragma unroll 4
    for (int s = ph; s < nsplit; s += PH) r += part[((size_t)s * K + c) * nl * nl + (size_t)a * nl + b];
  }
  if (PH > 1) {
    sh[ph][el] = r;
    __syncthreads();
    if (ph > 0) return;
    r = 0;
    for (int p = 0; p < PH; p++) r += sh[p][el];
  }
  if (idx < nl * nl) ok[(size_t)c * nl * nl + idx] = r;
}

// Lowest Ritz value over a field's vectors (the QL output is unsorted).
__global__ __launch_bounds__(256) void sftlm_emin_kernel(int R, int nl, const int *__restrict__ n_used,
                                                         const double *__restrict__ eps, double *E_min) {
  __shared__ double red[4];
  double lo = 1e300;
  for (int k = threadIdx.x; k < R * nl; k += 256)
    if (k % nl < n_used[k / nl]) lo = fmin(lo, eps[k]);
  for (int off = 32; off > 0; off >>= 1) lo = fmin(lo, __shfl_xor(lo, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lo;
  __syncthreads();
  if (threadIdx.x == 0) *E_min = fmin(fmin(red[0], red[1]), fmin(red[2], red[3]));
}

// num[it][r] = z^T Re(O_K) z of one (temperature, vector) per block: thread a
// holds z_a; eigenvectors and O_K's rows (symmetric) are read with the threads
// along a.
__global__ __launch_bounds__(192) void sftlm_moment_kernel(int R, int nl, const int *__restrict__ n_used,
                                                           const double *__restrict__ eps,
                                                           const double *__restrict__ Qt,
                                                           const double *__restrict__ OK,
                                                           const double *__restrict__ T,
                                                           const double *__restrict__ E_min,
                                                           double *__restrict__ num) {
  extern __shared__ double sh[];
  double *h = sh, *z = h + nl;
  __shared__ double red[3];
  const int t = threadIdx.x, r = blockIdx.y, n = n_used[r];
  const double temp = T[blockIdx.x], emin = *E_min;
  Qt += (size_t)r * nl * nl;
  OK += (size_t)r * nl * nl;
  for (int m = t; m < n; m += 192)
    h[m] = exp(-(eps[(size_t)r * nl + m] - emin) / (2.0 * temp)) * Qt[(size_t)m * nl];
  __syncthreads();
  for (int a = t; a < n; a += 192) {
    double s = 0;
#pragma unroll 8
    for (int m = 0; m < n; m++) s = fma(Qt[(size_t)m * nl + a], h[m], s);
    z[a] = s;
  }
  __syncthreads();
  double v = 0;
  for (int a = t; a < n; a += 192) {
    double s = 0;
#pragma unroll 8
    for (int b = 0; b < n; b++) s = fma(OK[(size_t)b * nl + a], z[b], s);
    v = fma(z[a], s, v);
  }
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((t & 63) == 0) red[t >> 6] = v;
  __syncthreads();
  if (t == 0) num[(size_t)blockIdx.x * R + r] = red[0] + red[1] + red[2];
}

// One block per temperature: ln Z, E, C and the symmetric M over the R vectors
// of one field.  eps [R][nl], Qt [R][nl][nl], num [n_T][R], n_used [R].
__global__ __launch_bounds__(256) void sftlm_boltzmann_kernel(int R, int nl, const int *__restrict__ n_used,
                                                              const double *__restrict__ eps,
                                                              const double *__restrict__ Qt,
                                                              const double *__restrict__ num,
                                                              const double *__restrict__ dims,
                                                              const double *__restrict__ T,
                                                              const double *__restrict__ E_min, double *lnZ,
                                                              double *E, double *C, double *M) {
  __shared__ double red[256 / 64];
  const int t = threadIdx.x;
  const double temp = T[blockIdx.x], emin = *E_min;
  auto block_sum = [&](double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((t & 63) == 0) red[t >> 6] = v;
    __syncthreads();
    double s = 0;
    for (int w = 0; w < 4; w++) s += red[w];
    __syncthreads();
    return s;
  };
  double den = 0, e1 = 0;
  for (int k = t; k < R * nl; k += 256) {
    if (k % nl >= n_used[k / nl]) continue;
    const double q = Qt[(size_t)k * nl], ev = eps[k];
    const double w = exp(-(ev - emin) / temp) * q * q;
    den += w;
    e1 += w * ev;
  }
  den = block_sum(den);
  e1 = block_sum(e1);
  const double em = e1 / den;
  double e2 = 0, mm = 0;
  for (int k = t; k < R * nl; k += 256) {
    if (k % nl >= n_used[k / nl]) continue;
    const double q = Qt[(size_t)k * nl], ev = eps[k];
    e2 += exp(-(ev - emin) / temp) * q * q * (ev - em) * (ev - em);
  }
  for (int r = t; r < R; r += 256) mm += num[(size_t)blockIdx.x * R + r];
  e2 = block_sum(e2);
  mm = block_sum(mm);
  if (t == 0) {
    const int k = blockIdx.x;
    lnZ[k] = log(dims[0] / R) - emin / temp + log(den);
    E[k] = em;
    C[k] = e2 / den / (temp * temp);
    M[k] = mm / den;
  }
}

struct SPlan {
  int R = 0, NL = 0, nT = 0, nF = 0, prec = 0, nsplit = 0;
  int K = 1, nwave = 0;  // columns per wave (1 or even), waves
  size_t es = 16;
  uint64_t dim = 0;
  size_t V, W, alpha, beta, yre, yim, sx, smax, done, nused, part, counter;
  size_t gpart, eps, Q, OK, num, sx0, nused_all, T, dims, lnZ, E, C, M, emin;
  size_t total = 0;
};

struct Carve2 {
  size_t off = 0;
  size_t take(size_t n) {
    size_t o = (off + 255) & ~size_t(255);
    off = o + n;
    return o;
  }
};

void make_splan(const ftlm_hamiltonian *h, const ftlm_run_params *p, SPlan &pl) {
  pl.R = p->R;
  pl.NL = p->n_lanczos;
  pl.nT = p->n_T;
  pl.nF = p->fields ? p->n_fields : 1;
  pl.prec = p->precision;
  pl.es = p->precision == FTLM_C64 ? 8 : 16;
  pl.dim = h->host.dim;
  const size_t vec = (size_t)pl.dim * pl.es;
  // Columns per wave: as many vectors together as plain runs take at the
  // dimension (small vectors are bound by launches and gather latency, which
  // columns share; one column from 2^20 rows, for the tile kernels), as far as
  // their Krylov bases fit 1 GiB; whole pairs, or a single vector.
  const size_t basis = vec * (2 * (size_t)pl.NL + 1);
  const int want = pl.dim >= (1ull << 20) ? 1 : pl.dim >= (1ull << 17) ? 4 : pl.dim >= (1ull << 14) ? 16 : 64;
  pl.K = (int)std::min<uint64_t>((uint64_t)std::min(want, pl.R), (1ull << 30) / basis) & ~1;
  if (pl.K < 2) pl.K = 1;
  pl.nwave = (pl.R + pl.K - 1) / pl.K;
  const int nb = (pl.NL + kGB - 1) / kGB, pairs = nb * (nb + 1) / 2 * pl.K;
  // about 4096 waves for the Gram products, each of at least 64 rows
  pl.nsplit = (int)std::max<uint64_t>(1, std::min<uint64_t>((4096 + pairs - 1) / pairs, pl.dim / 64));
  Carve2 c;
  pl.V = c.take(vec * pl.K * (pl.NL + 1));
  pl.W = c.take(vec * pl.K * pl.NL);
  const size_t sd = sizeof(double), sK = sd * pl.K;
  pl.alpha = c.take(sK * pl.NL * pl.nwave);
  pl.beta = c.take(sK * pl.NL * pl.nwave);
  pl.yre = c.take(sK * pl.NL);
  pl.yim = c.take(sK * pl.NL);
  pl.sx = c.take(sK * (pl.NL + 1));
  pl.sx0 = c.take(sK);
  pl.smax = c.take(sK);
  pl.done = c.take(sizeof(int) * pl.K);
  pl.nused = c.take(sizeof(int) * pl.K);
  pl.part = c.take(sK * 2048 * 3);
  pl.counter = c.take(sizeof(unsigned) * kCounterWords);
  pl.gpart = c.take(sd * (size_t)pl.nsplit * pl.K * pl.NL * pl.NL);
  pl.eps = c.take(sd * (size_t)pl.R * pl.NL);
  pl.Q = c.take(sd * (size_t)pl.R * pl.NL * pl.NL);
  pl.OK = c.take(sd * (size_t)pl.R * pl.NL * pl.NL);
  pl.num = c.take(sd * (size_t)pl.R * pl.nT);
  pl.nused_all = c.take(sizeof(int) * (size_t)pl.R * pl.nF);
  pl.T = c.take(sd * pl.nT);
  pl.dims = c.take(sd);
  const size_t res = sd * pl.nT * pl.nF;
  pl.lnZ = c.take(res);
  pl.E = c.take(res);
  pl.C = c.take(res);
  pl.M = c.take(res);
  pl.emin = c.take(sd * pl.nF);
  pl.total = (c.off + 255) & ~size_t(255);
}

template <typename T>
T *at2(void *ws, size_t off) {
  return reinterpret_cast<T *>(reinterpret_cast<char *>(ws) + off);
}

int validate_sftlm(const ftlm_hamiltonian *h, const ftlm_run_params *p, std::string &err) {
  if (!p) { err = "params is NULL"; return FTLM_EINVAL; }
  if (p->R < 2 || (p->R & 1)) { err = "R must be even and >= 2 (time-reversed pairs)"; return FTLM_EINVAL; }
  if (p->n_lanczos < 1) { err = "n_lanczos must be >= 1"; return FTLM_ERANGE; }
  if (tridiag_full_smem(p->n_lanczos) > 160 * 1024) { err = "n_lanczos too large for the sFTLM eigensolver (<= 141)"; return FTLM_ERANGE; }
  if (p->n_T < 1 || !p->T) { err = "a temperature grid is required"; return FTLM_EINVAL; }
  for (int i = 0; i < p->n_T; i++)
    if (!(p->T[i] > 0) || !std::isfinite(p->T[i])) { err = "temperatures must be positive"; return FTLM_EINVAL; }
  if (p->precision != FTLM_C128 && p->precision != FTLM_C64) { err = "bad precision"; return FTLM_EINVAL; }
  if (p->r_init) { err = "r_init is not supported by the sFTLM driver"; return FTLM_EINVAL; }
  if (p->fields) {
    if (p->n_fields < 1) { err = "n_fields must be >= 1"; return FTLM_EINVAL; }
    for (int i = 0; i < 3 * p->n_fields; i++)
      if (!std::isfinite(p->fields[i])) { err = "fields must be finite"; return FTLM_EINVAL; }
  } else if (p->n_fields > 1) {
    err = "n_fields > 1 needs a fields array";
    return FTLM_EINVAL;
  }
  if (h->host.dim > 0xFFFFFFFFull) { err = "dimension too large"; return FTLM_ERANGE; }
  return FTLM_OK;
}

}  // namespace
}  // namespace ftlm

using namespace ftlm;

extern "C" {

int ftlm_run_sftlm_workspace_size(const ftlm_hamiltonian *h, const ftlm_run_params *p, size_t *bytes) {
  std::string err;
  if (!h || !bytes) { set_error("NULL argument"); return FTLM_EINVAL; }
  int rc = validate_sftlm(h, p, err);
  if (rc) { set_error(err); return rc; }
  SPlan pl;
  make_splan(h, p, pl);
  *bytes = pl.total;
  return FTLM_OK;
}

int ftlm_run_sftlm(const ftlm_hamiltonian *hc, const ftlm_run_params *p, void *ws, size_t bytes,
                   void *stream_, ftlm_result *out) {
  std::string err;
  if (!hc || !ws || !out) { set_error("NULL argument"); return FTLM_EINVAL; }
  int rc = validate_sftlm(hc, p, err);
  if (rc) { set_error(err); return rc; }
  ftlm_hamiltonian *h = const_cast<ftlm_hamiltonian *>(hc);
  SPlan pl;
  make_splan(h, p, pl);
  if (bytes < pl.total) { set_error("workspace too small"); return FTLM_ENOMEM; }
  hipStream_t s = (hipStream_t)stream_;
  const double saved_B[3] = {h->host.B[0], h->host.B[1], h->host.B[2]};
  const double dimd = (double)pl.dim;
  if (hipMemcpyAsync(at2<double>(ws, pl.T), p->T, sizeof(double) * pl.nT, hipMemcpyHostToDevice, s) != hipSuccess ||
      hipMemcpyAsync(at2<double>(ws, pl.dims), &dimd, sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    set_error("copy of run inputs failed");
    return FTLM_EHIP;
  }
  auto fail = [&](int code, const std::string &m) {
    set_error(m);
    if (p->fields) (void)ftlm_hamiltonian_set_field(h, saved_B);
    return code;
  };
  ThetaGeom tg{};
  tg.n = h->host.n;
  tg.dim = (uint32_t)pl.dim;
  int ts = 0;
  for (int k = 0; k < tg.n; k++) {
    tg.radix[k] = h->host.radix[k];
    ts += h->host.two_s[k];
  }
  tg.two_s_sum_parity = ts & 1;
  const int NL = pl.NL, Kp = pl.K;
  const size_t vbytes = (size_t)pl.dim * pl.es;
  char *V = at2<char>(ws, pl.V), *Wb = at2<char>(ws, pl.W);
  const uint32_t tgrid = (uint32_t)std::min<uint64_t>(4096, (pl.dim + 255) / 256);
  double *sx = at2<double>(ws, pl.sx), *sx0 = at2<double>(ws, pl.sx0);
  for (int f = 0; f < pl.nF; f++) {
    if (p->fields) {
      rc = ftlm_hamiltonian_set_field(h, p->fields + 3 * f);
      if (rc) return fail(rc, std::string("set_field: ") + ftlm_last_error());
    }
    int *nused_f = at2<int>(ws, pl.nused_all) + (size_t)f * pl.R;
    for (int wave = 0; wave < pl.nwave; wave++) {
      const int r0 = wave * Kp, K = std::min(Kp, pl.R - r0);
      const size_t slot = vbytes * K;  // one Krylov vector of every column, [dim][K]
      double *alpha = at2<double>(ws, pl.alpha) + (size_t)wave * NL * Kp;
      double *beta = at2<double>(ws, pl.beta) + (size_t)wave * NL * Kp;
      if (launch_zero_state(at2<double>(ws, pl.smax), at2<int>(ws, pl.done), at2<int>(ws, pl.nused),
                            at2<unsigned>(ws, pl.counter), kCounterWords, K, s))
        return fail(FTLM_EHIP, "zero_state launch failed");
      // start vectors: the Gaussian vectors of the wave's pairs (pair index as the
      // vector index) go to slot 1 and from there, each with its time reverse,
      // to slot 0; a wave of one vector makes either of them
      const bool pairs = K > 1, direct = !pairs && !(r0 & 1);
      rc = launch_gaussian(p->seed, p->instance, (uint32_t)f, (uint32_t)(r0 >> 1), pairs ? K / 2 : 1,
                           (uint32_t)pl.dim, pl.prec, direct ? V : V + slot, at2<double>(ws, pl.part),
                           at2<unsigned>(ws, pl.counter), pairs ? sx0 : sx, 0, s);
      if (rc) return fail(rc, "start-vector launch failed");
      if (!direct) {
        if (pl.prec == FTLM_C64)
          hipLaunchKernelGGL(theta_kernel<float>, dim3(tgrid), dim3(256), 0, s, tg,
                             reinterpret_cast<const Cx<float> *>(V + slot), reinterpret_cast<Cx<float> *>(V), K, sx0, sx);
        else
          hipLaunchKernelGGL(theta_kernel<double>, dim3(tgrid), dim3(256), 0, s, tg,
                             reinterpret_cast<const Cx<double> *>(V + slot), reinterpret_cast<Cx<double> *>(V), K, sx0,
                             sx);
        if (hipGetLastError() != hipSuccess) return fail(FTLM_EHIP, "theta launch failed");
      }
      // Lanczos: X_j in slot j, u_j written into slot j+1
      for (int j = 0; j < NL; j++) {
        EpiLanczos lz{};
        lz.xprev = j > 0 ? V + (size_t)(j - 1) * slot : nullptr;
        lz.ov1 = nullptr;
        lz.sx_cur = sx + (size_t)j * Kp;
        lz.sx_prev = j > 0 ? sx + (size_t)(j - 1) * Kp : nullptr;
        lz.beta_prev = j > 0 ? beta + (size_t)(j - 1) * Kp : nullptr;
        lz.part = at2<double>(ws, pl.part);
        lz.counter = at2<unsigned>(ws, pl.counter);
        lz.alpha_out = alpha + (size_t)j * Kp;
        lz.yre_out = at2<double>(ws, pl.yre) + (size_t)j * Kp;
        lz.yim_out = at2<double>(ws, pl.yim) + (size_t)j * Kp;
        HvLaunch L{};
        L.precision = pl.prec;
        L.K = K;
        L.v = V + (size_t)j * slot;
        L.w = V + (size_t)(j + 1) * slot;
        L.lz = &lz;
        rc = launch_hv(h->dev, L, s);
        if (rc) return fail(rc, "H*v launch failed");
        UpdateArgs u{};
        u.precision = pl.prec;
        u.K = K;
        u.step = j;
        u.n_lanczos = NL;
        u.dim = (uint32_t)pl.dim;
        u.w = L.w;
        u.x = L.v;
        u.sx_cur = lz.sx_cur;
        u.alpha = lz.alpha_out;
        u.beta = beta + (size_t)j * Kp;
        u.sx_next = sx + (size_t)(j + 1) * Kp;
        u.scale_max = at2<double>(ws, pl.smax);
        u.done = at2<int>(ws, pl.done);
        u.n_used = at2<int>(ws, pl.nused);
        u.part = at2<double>(ws, pl.part);
        u.counter = at2<unsigned>(ws, pl.counter);
        rc = launch_update(u, s);
        if (rc) return fail(rc, "update launch failed");
      }
      // W_b = O (sx_b X_b)
      for (int b = 0; b < NL; b++) {
        HvLaunch L{};
        L.precision = pl.prec;
        L.K = K;
        L.v = V + (size_t)b * slot;
        L.w = Wb + (size_t)b * slot;
        L.scale = sx + (size_t)b * Kp;
        if (launch_hv(h->mom_dev, L, s)) return fail(FTLM_EHIP, "O V launch failed");
      }
      // Re(O_K) = Re(V^H W) of every column
      const uint32_t chunk = (uint32_t)((pl.dim + pl.nsplit - 1) / pl.nsplit);
      const int nb = (NL + kGB - 1) / kGB;
      const dim3 gg(nb * (nb + 1) / 2, K, (pl.nsplit + 3) / 4);
      double *gpart = at2<double>(ws, pl.gpart);
      if (pl.prec == FTLM_C64)
        hipLaunchKernelGGL(gram_kernel<float>, gg, dim3(256), 0, s, reinterpret_cast<const Cx<float> *>(V),
                           reinterpret_cast<const Cx<float> *>(Wb), K, NL, (uint32_t)pl.dim, chunk, pl.nsplit, sx, Kp,
                           gpart);
      else
        hipLaunchKernelGGL(gram_kernel<double>, gg, dim3(256), 0, s, reinterpret_cast<const Cx<double> *>(V),
                           reinterpret_cast<const Cx<double> *>(Wb), K, NL, (uint32_t)pl.dim, chunk, pl.nsplit, sx, Kp,
                           gpart);
      double *okr = at2<double>(ws, pl.OK) + (size_t)r0 * NL * NL;
      if (pl.nsplit >= 64)
        hipLaunchKernelGGL(gram_reduce_kernel<16>, dim3((NL * NL + 15) / 16, K), dim3(256), 0, s, gpart, pl.nsplit, NL,
                           K, okr);
      else
        hipLaunchKernelGGL(gram_reduce_kernel<1>, dim3((NL * NL + 255) / 256, K), dim3(256), 0, s, gpart, pl.nsplit, NL,
                           K, okr);
      if (hipGetLastError() != hipSuccess) return fail(FTLM_EHIP, "sFTLM kernel launch failed");
      if (hipMemcpyAsync(nused_f + r0, at2<int>(ws, pl.nused), sizeof(int) * K, hipMemcpyDeviceToDevice, s) != hipSuccess)
        return fail(FTLM_EHIP, "copy of n_used failed");
    }
    // full eigenpairs of every vector's tridiagonal in one launch: they are
    // serial chains, and side by side they cost one chain
    double *eps = at2<double>(ws, pl.eps), *Qt = at2<double>(ws, pl.Q), *num = at2<double>(ws, pl.num);
    if (launch_tridiag_full(pl.R, NL, nused_f, at2<double>(ws, pl.alpha), at2<double>(ws, pl.beta), Kp, eps, Qt, s))
      return fail(FTLM_EHIP, "tridiagonal launch failed");
    const size_t ro = (size_t)f * pl.nT;
    const double *Td = at2<double>(ws, pl.T);
    double *emin = at2<double>(ws, pl.emin) + f;
    hipLaunchKernelGGL(sftlm_emin_kernel, dim3(1), dim3(256), 0, s, pl.R, NL, nused_f, eps, emin);
    hipLaunchKernelGGL(sftlm_moment_kernel, dim3(pl.nT, pl.R), dim3(192), sizeof(double) * 2 * (size_t)NL, s, pl.R, NL,
                       nused_f, eps, Qt, at2<double>(ws, pl.OK), Td, emin, num);
    hipLaunchKernelGGL(sftlm_boltzmann_kernel, dim3(pl.nT), dim3(256), 0, s, pl.R, NL, nused_f, eps, Qt, num,
                       at2<double>(ws, pl.dims), Td, emin, at2<double>(ws, pl.lnZ) + ro, at2<double>(ws, pl.E) + ro,
                       at2<double>(ws, pl.C) + ro, at2<double>(ws, pl.M) + ro);
    if (hipGetLastError() != hipSuccess) return fail(FTLM_EHIP, "sFTLM Boltzmann launch failed");
  }
  const size_t res = sizeof(double) * pl.nT * pl.nF;
  struct { double *dst; size_t off; size_t n; } outs[] = {
      {out->lnZ, pl.lnZ, res}, {out->E, pl.E, res}, {out->C, pl.C, res}, {out->M, pl.M, res},
      {out->E_min, pl.emin, sizeof(double) * pl.nF}};
  for (auto &o : outs)
    if (o.dst && hipMemcpyAsync(o.dst, at2<char>(ws, o.off), o.n, hipMemcpyDeviceToHost, s) != hipSuccess)
      return fail(FTLM_EHIP, "copy of results failed");
  if (out->n_lanczos_used &&
      hipMemcpyAsync(out->n_lanczos_used, at2<int>(ws, pl.nused_all), sizeof(int) * pl.R * pl.nF,
                     hipMemcpyDeviceToHost, s) != hipSuccess)
    return fail(FTLM_EHIP, "copy of n_used failed");
  if (hipStreamSynchronize(s) != hipSuccess) return fail(FTLM_EHIP, "stream synchronise failed");
  if (p->fields) {
    rc = ftlm_hamiltonian_set_field(h, saved_B);
    if (rc) return rc;
  }
  return FTLM_OK;
}

}  // extern "C"
