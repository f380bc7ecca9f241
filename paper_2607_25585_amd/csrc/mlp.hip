// Surrogate MLP kernels (gfx950): 7 -> 256 -> 256 -> 256 -> 3 with SiLU,
// BF16 weights and activations feeding MFMA (v_mfma_f32_16x16x16_bf16) with FP32
// accumulation; FP32 pre-activations, gradients of the biases and Adam master
// weights.  Layer k computes z_k = a_{k-1} W_k + b_k (W_k stored [fan_in][fan_out]),
// a_k = silu(z_k) for the hidden layers; the output layer is linear.  Loss
// L = 1/(3B) sum (y - t)^2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <string>

#include "ftlm_internal.hpp"

namespace ftlm {

namespace {

constexpr int kIn = 7, kHid = 256, kOut = 3;

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// C[m][n] = sum_k A(m,k) B(k,n), A(m,k) = A[m*sam + k*sak], B(k,n) = B[k*sbk + n*sbn]
// (bf16), FP32 accumulation.  Block = 4 waves on a 64x64 tile of C; each wave owns
// 32x32 = 2x2 MFMA 16x16 tiles; K advances kStep at a time through LDS, where both
// operands lie k-contiguous (a lane's four k of a fragment are one 8-byte read).
// Epilogue modes:
//   0: hidden forward:  Z = C + bias -> zf (fp32, ld N) and a = silu(Z) -> ob (bf16, ld N)
//   1: output forward:  Y = C + bias -> zf and, unless NULL, zf2 (fp32, ld N)
//   2: plain:           zf = C (fp32, ld N)
//   3: backward:        g = C * silu'(zin[m][n]) -> ob (bf16), and the tile's column
//                       sums of g -> csum[m-tile][n] (the bias gradient's partials)
// What bounds them at a batch of 4096 is latency: 256 blocks, one per CU, of eight
// k-steps each.  So a thread fetches 16 bytes of each operand per k-step, and the
// next step's are in flight during this step's MFMAs (2-byte loads, 16 k at a time and
// no prefetch: 25 us per product on average, 13 us so).
struct GemmArgs {
  int M, N, K;
  int ksplit;  // mode 2: K split over blockIdx.z, partial products at zf + z*M*N (0 or 1: none)
  const uint16_t *A;
  long sam, sak;
  const uint16_t *B;
  long sbk, sbn;
  int mode;
  const float *bias;
  const float *zin;
  float *zf, *zf2;
  uint16_t *ob;
  float *csum;
};

constexpr int kStep = 64, kLd = kStep + 8;  // rows of 144 bytes: 16-byte aligned, banks spread
constexpr int kFr = kStep / 32;             // 16-byte fragments per thread and operand

// 64 (rows) x kStep (k) of an operand with element (r, k) at p[r * sr + k * sk]: thread t
// holds kFr fragments of 8, along k (sk == 1) or along the rows (else), unpacked only
// when they are put to LDS, so that the loads stay in flight; elements outside
// rows x ke are 0.  16-byte loads where the 8 are contiguous and aligned.
__device__ __forceinline__ void frag_at(int u, bool along_k, int &r, int &k) {
  const int e = threadIdx.x + 256 * u;
  r = along_k ? e / (kStep / 8) : (e & 7) * 8;
  k = along_k ? e % (kStep / 8) * 8 : e >> 3;
}
__device__ __forceinline__ void fetch(uint4 (&f)[kFr], const uint16_t *p, long sr, long sk, int r0, int rows, int k0,
                                      int ke) {
  const bool along_k = sk == 1;
  const bool aligned = (along_k || sr == 1) && ((along_k ? sr : sk) & 7) == 0 &&
                       ((reinterpret_cast<uintptr_t>(p) + (uintptr_t)(along_k ? k0 : r0) * 2) & 15) == 0;
#pragma unroll
  for (int u = 0; u < kFr; u++) {
    int r, k;
    frag_at(u, along_k, r, k);
    r += r0;
    k += k0;
    const bool whole = aligned && (along_k ? (r < rows && k + 8 <= ke) : (r + 8 <= rows && k < ke));
    if (whole) {
      f[u] = *reinterpret_cast<const uint4 *>(p + (long)r * sr + (long)k * sk);
    } else {
      uint32_t x[8];
#pragma unroll
      for (int h = 0; h < 8; h++) {
        const int rh = along_k ? r : r + h, kh = along_k ? k + h : k;
        x[h] = 0;
        if (rh < rows && kh < ke) x[h] = p[(long)rh * sr + (long)kh * sk];
      }
      f[u] = make_uint4(x[0] | x[1] << 16, x[2] | x[3] << 16, x[4] | x[5] << 16, x[6] | x[7] << 16);
    }
  }
}
__device__ __forceinline__ void put(uint16_t (*lds)[kLd], const uint4 (&f)[kFr], bool along_k) {
#pragma unroll
  for (int u = 0; u < kFr; u++) {
    int r, k;
    frag_at(u, along_k, r, k);
    if (along_k) {
      *reinterpret_cast<uint4 *>(&lds[r][k]) = f[u];
    } else {
      const uint32_t w[4] = {f[u].x, f[u].y, f[u].z, f[u].w};
#pragma unroll
      for (int h = 0; h < 8; h++) lds[r + h][k] = (uint16_t)(w[h >> 1] >> (16 * (h & 1)));
    }
  }
}

// Two products in one launch: blocks [0, n0) take g0, the others g1 (the weight
// gradient and the next layer's gradient need the same inputs, and each alone
// leaves CUs idle).
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmArgs g0, GemmArgs g1, int n0) {
  __shared__ __align__(16) uint16_t As[2][64][kLd];
  __shared__ __align__(16) uint16_t Bs[2][64][kLd];
  const bool second = (int)blockIdx.x >= n0;
  const GemmArgs &g = second ? g1 : g0;
  const int bid = (int)blockIdx.x - (second ? n0 : 0);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int nx = (g.N + 63) / 64, ny = (g.M + 63) / 64;
  const int bx = bid % nx, by = bid / nx % ny, bz = bid / nx / ny;
  const int m0 = by * 64, n0t = bx * 64;
  // K range of this block (all of K unless split)
  const int ks = g.ksplit > 1 ? g.ksplit : 1;
  const int kchunk = ((g.K + ks - 1) / ks + 15) & ~15;
  const int kb = bz * kchunk, ke = min(g.K, kb + kchunk);
  float *zf = g.zf + (ks > 1 ? (long)bz * g.M * g.N : 0L);
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const bool ak = g.sak == 1, bk = g.sbk == 1;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint4 fa[kFr], fb[kFr];
  fetch(fa, g.A, g.sam, g.sak, m0, g.M, kb, ke);
  fetch(fb, g.B, g.sbn, g.sbk, n0t, g.N, kb, ke);
  int buf = 0;
  for (int k0 = kb; k0 < ke; k0 += kStep, buf ^= 1) {
    put(As[buf], fa, ak);
    put(Bs[buf], fb, bk);
    __syncthreads();  // (the buffer written next was last read before this barrier)
    if (k0 + kStep < ke) {
      fetch(fa, g.A, g.sam, g.sak, m0, g.M, k0 + kStep, ke);
      fetch(fb, g.B, g.sbn, g.sbk, n0t, g.N, k0 + kStep, ke);
    }
    const int kq = 4 * (lane >> 4), rl = lane & 15;
#pragma unroll
    for (int kk = 0; kk < kStep; kk += 16) {
      bf16x4 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; i++) {
        a[i] = *reinterpret_cast<const bf16x4 *>(&As[buf][wm + 16 * i + rl][kk + kq]);
        b[i] = *reinterpret_cast<const bf16x4 *>(&Bs[buf][wn + 16 * i + rl][kk + kq]);
      }
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int jj = 0; jj < 2; jj++)
          acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[i], b[jj], acc[i][jj], 0, 0, 0);
    }
  }
  // D[row = 4*(lane/16) + j][col = lane % 16] of each 16x16 tile
  float cs[2] = {0.f, 0.f};
#pragma unroll
  for (int jj = 0; jj < 2; jj++)
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int m = m0 + wm + 16 * i + 4 * (lane >> 4) + j;
        const int n = n0t + wn + 16 * jj + (lane & 15);
        if (m >= g.M || n >= g.N) continue;
        float c = acc[i][jj][j];
        const long o = (long)m * g.N + n;
        if (g.mode == 0) {
          c += g.bias[n];
          g.zf[o] = c;
          g.ob[o] = f2bf(silu(c));
        } else if (g.mode == 1) {
          c += g.bias[n];
          g.zf[o] = c;
          if (g.zf2) g.zf2[o] = c;
        } else if (g.mode == 2) {
          zf[o] = c;
        } else {
          c *= dsilu(g.zin[o]);
          g.ob[o] = f2bf(c);
          cs[jj] += c;
        }
      }
  if (g.mode != 3) return;
  // column sums of the tile in a fixed order: the lanes of a column, then the two
  // waves above each other
  __shared__ float cpart[2][64];
#pragma unroll
  for (int jj = 0; jj < 2; jj++) {
    cs[jj] += __shfl_xor(cs[jj], 16, 64);
    cs[jj] += __shfl_xor(cs[jj], 32, 64);
    if (lane < 16) cpart[wave >> 1][wn + 16 * jj + lane] = cs[jj];
  }
  __syncthreads();
  if (t < 64 && n0t + t < g.N) g.csum[(long)by * g.N + n0t + t] = cpart[0][t] + cpart[1][t];
}

int gemm_blocks(const GemmArgs &a) {
  return ((a.N + 63) / 64) * ((a.M + 63) / 64) * (a.ksplit > 1 ? a.ksplit : 1);
}

void gemm(const GemmArgs &a, hipStream_t s) {
  const int n = gemm_blocks(a);
  hipLaunchKernelGGL(gemm_bf16_kernel, dim3(n), dim3(256), 0, s, a, a, n);
}

void gemm2(const GemmArgs &a, const GemmArgs &b, hipStream_t s) {
  const int n = gemm_blocks(a);
  hipLaunchKernelGGL(gemm_bf16_kernel, dim3(n + gemm_blocks(b)), dim3(256), 0, s, a, b, n);
}

// The weight gradients have a long K (the batch) and few output tiles: K is split
// over up to kMaxSplit blocks per tile, and the partial products are summed in
// split order by grad_sum_kernel.
constexpr int kMaxSplit = 16;
int grad_splits(const GemmArgs &a) {
  const int tiles = ((a.N + 63) / 64) * ((a.M + 63) / 64);
  return tiles >= 256 ? 1 : std::min(kMaxSplit, std::max(1, (a.K + 255) / 256));
}

// One launch for every sum over partials of a backward pass: out[i] = scale
// sum_z part[z][i] in order of z, for up to kSums arrays, whose elements follow each
// other over the threads.  Long sums of few elements (the biases') are split over
// the 16 lanes of a row of lanes, added in a fixed order.
constexpr int kSums = 9;
struct GradSums {
  const float *part[kSums];
  float *out[kSums];
  int parts[kSums], n[kSums], block0[kSums + 1], wide[kSums];
  float scale[kSums];
};
__global__ __launch_bounds__(256) void grad_sum_kernel(GradSums S) {
  int k = 0;
  while ((int)blockIdx.x >= S.block0[k + 1]) k++;
  const int t = threadIdx.x, b = (int)blockIdx.x - S.block0[k], n = S.n[k], parts = S.parts[k];
  const float *part = S.part[k];
  if (S.wide[k]) {  // 16 lanes per element
    const int i = b * 16 + (t >> 4), ph = t & 15;
    float s = 0.f;
    if (i < n)
      for (int z = ph; z < parts; z += 16) s += part[(long)z * n + i];
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) s += __shfl_xor(s, m, 64);
    if (i < n && ph == 0) S.out[k][i] = s * S.scale[k];
  } else {
    const int i = b * 256 + t;
    if (i >= n) return;
    float s = 0.f;
#pragma unroll 4
    for (int z = 0; z < parts; z++) s += part[(long)z * n + i];
    S.out[k][i] = s * S.scale[k];
  }
}

__global__ void to_bf16_kernel(const float *x, uint16_t *y, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = f2bf(x[i]);
}

// dY = 2 (y - t) / (3B) (bf16), and per block of 64 rows the sums of dY's columns and of
// (y - t)^2: part[block][3] and lpart[block].
constexpr int kLossRows = 64;
__global__ __launch_bounds__(256) void loss_kernel(const float *y, const float *tg, int B, uint16_t *dyb, float *part,
                                                   float *lpart) {
  const int t = threadIdx.x, r = t & 63, c = t >> 6, row = blockIdx.x * kLossRows + r;
  const float sc = 2.0f / (float)(B * kOut);
  float g = 0.f, s = 0.f;
  if (row < B) {
    if (c < kOut) {
      g = sc * (y[(long)row * kOut + c] - tg[(long)row * kOut + c]);
      dyb[(long)row * kOut + c] = f2bf(g);
    } else {
#pragma unroll
      for (int q = 0; q < kOut; q++) {
        const float d = y[(long)row * kOut + q] - tg[(long)row * kOut + q];
        s += d * d;
      }
    }
  }
  float v = c < kOut ? g : s;  // wave c sums its quantity over the rows
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
  if (r == 0) {
    if (c < kOut) part[blockIdx.x * kOut + c] = v;
    else lpart[blockIdx.x] = v;
  }
}

__global__ void adam_kernel(long n, float *p, const float *g, float *m, float *v, uint16_t *pb,
                            float lr, float b1, float b2, float eps, float c1, float c2) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    if (pb) pb[i] = f2bf(pi);
  }
}

struct MlpWs {
  uint16_t *xb;          // [B][7]
  float *z[3];           // [B][256] pre-activations
  uint16_t *a[3];        // [B][256] activations (bf16)
  float *y;              // [B][3] output copy
  uint16_t *gb[2];       // [B][256] gradient (bf16), ping-pong
  uint16_t *dyb;         // [B][3]
  float *splitk[4];      // [kMaxSplit][fan_in][fan_out] partial weight gradients
  float *csum[4];        // [ceil(B / 64)][fan_out] partial bias gradients
  float *lpart;          // [ceil(B / 64)] partial losses
  size_t bytes;
};

const int kFanIn[4] = {kIn, kHid, kHid, kHid};
const int kFanOut[4] = {kHid, kHid, kHid, kOut};

MlpWs layout(int B, void *base) {
  MlpWs w{};
  size_t off = 0;
  auto take = [&](size_t n) {
    const size_t o = (off + 255) & ~size_t(255);
    off = o + n;
    return reinterpret_cast<unsigned char *>(base) + o;
  };
  const size_t tiles = ((size_t)B + 63) / 64;
  w.xb = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * B * kIn));
  for (int k = 0; k < 3; k++) w.z[k] = reinterpret_cast<float *>(take(sizeof(float) * B * kHid));
  for (int k = 0; k < 3; k++) w.a[k] = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * B * kHid));
  w.y = reinterpret_cast<float *>(take(sizeof(float) * B * kOut));
  for (int k = 0; k < 2; k++) w.gb[k] = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * B * kHid));
  w.dyb = reinterpret_cast<uint16_t *>(take(sizeof(uint16_t) * B * kOut));
  for (int k = 0; k < 4; k++)
    w.splitk[k] = reinterpret_cast<float *>(take(sizeof(float) * kMaxSplit * kFanIn[k] * kFanOut[k]));
  for (int k = 0; k < 4; k++) w.csum[k] = reinterpret_cast<float *>(take(sizeof(float) * tiles * kFanOut[k]));
  w.lpart = reinterpret_cast<float *>(take(sizeof(float) * tiles));
  w.bytes = (off + 255) & ~size_t(255);
  return w;
}

}  // namespace
}  // namespace ftlm

using namespace ftlm;

extern "C" {

int ftlm_mlp_workspace_size(int32_t batch, size_t *bytes) {
  if (batch < 1 || !bytes) {
    set_error("batch must be >= 1 and bytes non-NULL");
    return FTLM_EINVAL;
  }
  *bytes = layout(batch, nullptr).bytes;
  return FTLM_OK;
}

int ftlm_mlp_forward(const ftlm_mlp_weights *w, int32_t B, const float *x, float *y, void *ws,
                     size_t bytes, void *stream) {
  if (!w || !x || !y || !ws || B < 1) {
    set_error("NULL argument or bad batch");
    return FTLM_EINVAL;
  }
  MlpWs L = layout(B, ws);
  if (bytes < L.bytes) {
    set_error("MLP workspace too small");
    return FTLM_ENOMEM;
  }
  for (int k = 0; k < 4; k++)
    if (!w->W[k] || !w->b[k]) {
      set_error("NULL weight");
      return FTLM_EINVAL;
    }
  hipStream_t s = (hipStream_t)stream;
  const long nx = (long)B * kIn;
  hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)((nx + 255) / 256 < 4096 ? (nx + 255) / 256 : 4096)),
                     dim3(256), 0, s, x, L.xb, nx);
  const uint16_t *in = L.xb;
  for (int k = 0; k < 4; k++) {
    GemmArgs g{};
    g.M = B;
    g.N = kFanOut[k];
    g.K = kFanIn[k];
    g.A = in;
    g.sam = kFanIn[k];
    g.sak = 1;
    g.B = w->W[k];
    g.sbk = kFanOut[k];
    g.sbn = 1;
    g.bias = w->b[k];
    if (k < 3) {
      g.mode = 0;
      g.zf = L.z[k];
      g.ob = L.a[k];
      in = L.a[k];
    } else {
      g.mode = 1;
      g.zf = L.y;
      g.zf2 = y;
    }
    gemm(g, s);
  }
  if (hipGetLastError() != hipSuccess) {
    set_error("MLP forward launch failed");
    return FTLM_EHIP;
  }
  return FTLM_OK;
}

int ftlm_mlp_backward(const ftlm_mlp_weights *w, int32_t B, const float *t, float *loss,
                      float *const dW[4], float *const db[4], void *ws, size_t bytes, void *stream) {
  if (!w || !t || !dW || !db || !ws || B < 1) {
    set_error("NULL argument or bad batch");
    return FTLM_EINVAL;
  }
  MlpWs L = layout(B, ws);
  if (bytes < L.bytes) {
    set_error("MLP workspace too small");
    return FTLM_ENOMEM;
  }
  hipStream_t s = (hipStream_t)stream;
  const int tiles = (B + 63) / 64;
  hipLaunchKernelGGL(loss_kernel, dim3(tiles), dim3(256), 0, s, L.y, t, B, L.dyb, L.csum[3], L.lpart);
  GradSums S{};
  int ns = 0;
  auto sum = [&](const float *part, int parts, int n, float *out, bool wide, float scale) {
    S.part[ns] = part;
    S.out[ns] = out;
    S.parts[ns] = parts;
    S.n[ns] = n;
    S.wide[ns] = wide;
    S.scale[ns] = scale;
    S.block0[ns + 1] = S.block0[ns] + (n + (wide ? 15 : 255)) / (wide ? 16 : 256);
    ns++;
  };
  // output layer
  const uint16_t *gin = L.dyb;  // gradient w.r.t. z of the current layer (bf16)
  int cur = 0;
  for (int k = 3; k >= 0; k--) {
    // dW_k = a_{k-1}^T g  ([fan_in][fan_out])
    GemmArgs gw{};
    gw.M = kFanIn[k];
    gw.N = kFanOut[k];
    gw.K = B;
    gw.A = k > 0 ? L.a[k - 1] : L.xb;
    gw.sam = 1;
    gw.sak = kFanIn[k];
    gw.B = gin;
    gw.sbk = kFanOut[k];
    gw.sbn = 1;
    gw.mode = 2;
    gw.ksplit = grad_splits(gw);
    gw.zf = L.splitk[k];
    sum(L.splitk[k], gw.ksplit, gw.M * gw.N, dW[k], false, 1.0f);
    sum(L.csum[k], tiles, kFanOut[k], db[k], true, 1.0f);
    if (k == 0) {
      gemm(gw, s);
      break;
    }
    // g_{k-1} = (g W_k^T) * silu'(z_{k-1})
    GemmArgs ga{};
    ga.M = B;
    ga.N = kFanIn[k];
    ga.K = kFanOut[k];
    ga.A = gin;
    ga.sam = kFanOut[k];
    ga.sak = 1;
    ga.B = w->W[k];
    ga.sbk = 1;
    ga.sbn = kFanOut[k];
    ga.mode = 3;
    ga.zin = L.z[k - 1];
    ga.ob = L.gb[cur];
    ga.csum = L.csum[k - 1];
    gemm2(ga, gw, s);
    gin = L.gb[cur];
    cur ^= 1;
  }
  if (loss) sum(L.lpart, tiles, 1, loss, true, 1.0f / (float)(B * kOut));
  hipLaunchKernelGGL(grad_sum_kernel, dim3(S.block0[ns]), dim3(256), 0, s, S);
  if (hipGetLastError() != hipSuccess) {
    set_error("MLP backward launch failed");
    return FTLM_EHIP;
  }
  return FTLM_OK;
}

int ftlm_adam_step(int64_t n, float *p, const float *grad, float *m, float *v, uint16_t *pb, float lr,
                   float beta1, float beta2, float eps, int32_t step, void *stream) {
  if (n < 1 || !p || !grad || !m || !v || step < 1) {
    set_error("bad Adam arguments");
    return FTLM_EINVAL;
  }
  const float c1 = 1.0f - std::pow(beta1, (float)step), c2 = 1.0f - std::pow(beta2, (float)step);
  const long blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, (long)n, p, grad,
                     m, v, pb, lr, beta1, beta2, eps, c1, c2);
  if (hipGetLastError() != hipSuccess) {
    set_error("Adam launch failed");
    return FTLM_EHIP;
  }
  return FTLM_OK;
}

}  // extern "C"
