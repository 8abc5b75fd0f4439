// Learned initial amplitudes: features, forward, backward, Adam, guess.
//
// Network (parameters FP64 in device memory, 17153 values in this order):
//   W1[128][3], b1[128], W2[128][128], b2[128], W3[1][128], b3[1]
//   g(z) = W3 relu(W2 relu(W1 z + b1) + b2) + b3,   f(z) = (g(z) - g(z~)) / 2
// where z~ is z with its first component (the scaled integral <ij||ab>)
// negated, so f is odd in <ij||ab> and the predicted t2 is antisymmetric.
// A batch of c samples is evaluated as 2c rows (the + and - branches).  The
// three dense layers are MFMA GEMMs (FP64, or FP32 MFMA with FP32
// accumulation); the elementwise parts below are FP64.
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "plan.hpp"

namespace ccmi {
namespace {

constexpr int HID = 128;
constexpr int64_t NPAR = HID * 3 + HID + HID * HID + HID + HID + 1;  // 17153
constexpr int64_t OFF_W1 = 0, OFF_B1 = HID * 3, OFF_W2 = OFF_B1 + HID, OFF_B2 = OFF_W2 + HID * HID,
                  OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + HID;

// k-th pair i < j of n, in row order (row r starts at r (2n - 1 - r) / 2)
__device__ __forceinline__ void tri(int64_t k, int n, int &i, int &j) {
  const double m = 2.0 * n - 1.0;
  int r = max(0, int(0.5 * (m - sqrt(m * m - 8.0 * double(k)))));
  auto first = [n](int q) { return int64_t(q) * (2 * n - 1 - q) / 2; };
  while (first(r + 1) <= k) ++r;  // (the root is off by one at most)
  while (first(r) > k) --r;
  i = r;
  j = r + 1 + int(k - first(r));
}

// e_ij = sum_{a<b} <ij||ab>^2 / D_ij^ab for every i < j (one workgroup each).
// Bound by the latency of its loads and the FP64 divisions (50 of each per
// thread at v = 160).  Walking the rows and loading eight at a time, instead of
// a search from row 0 for every pair: 170 -> 39 us at o = 32, v = 160.
__global__ __launch_bounds__(256) void pair_energy_kernel(int o, int v, const double *__restrict__ oovv,
                                                          const double *__restrict__ d_oo,
                                                          const double *__restrict__ d_vv,
                                                          double *__restrict__ epair) {
  __shared__ double sh[256];
  int i, j;
  tri(blockIdx.x, o, i, j);
  const int64_t base = (int64_t(i) * o + j) * v * v;
  double s = 0.0;
  const int64_t nab = int64_t(v) * (v - 1) / 2;
  // eight pairs per round, their loads in flight together
  constexpr int U = 8;
  int a = 0, b = 1;
  if (threadIdx.x < nab) tri(threadIdx.x, v, a, b);
  for (int64_t u0 = threadIdx.x; u0 < nab; u0 += 256 * U) {
    double x[U], D[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      x[q] = 0.0;
      D[q] = 1.0;
      if (u0 + 256 * q < nab) {
        x[q] = oovv[base + int64_t(a) * v + b];
        D[q] = (d_oo[i] + d_oo[j]) - (d_vv[a] + d_vv[b]);
        b += 256;  // the pair 256 further on
        while (b >= v && a < v - 2) {
          ++a;
          b += a + 1 - v;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (u0 + 256 * q < nab) s += x[q] * x[q] / D[q];
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) epair[blockIdx.x] = sh[0];
}

// Raw (x, D, e) or standardised features of unique amplitudes, (ij, ab) order
// (bound by HBM: 200 MB at o = 32, v = 160, 47 us; 100 with a search for the pairs).
__global__ __launch_bounds__(256) void features_kernel(int o, int v, const double *__restrict__ oovv,
                                                       const double *__restrict__ d_oo,
                                                       const double *__restrict__ d_vv,
                                                       const double *__restrict__ epair, cc_mlp_stats st,
                                                       int standardise, double *__restrict__ z) {
  const int64_t nab = int64_t(v) * (v - 1) / 2, n = nab * (int64_t(o) * (o - 1) / 2);
  for (int64_t u = blockIdx.x * int64_t(256) + threadIdx.x; u < n; u += int64_t(gridDim.x) * 256) {
    int i, j, a, b;
    const int64_t ij = idiv(u, nab);
    tri(ij, o, i, j);
    tri(u - ij * nab, v, a, b);
    const double x = oovv[(int64_t(i) * o + j) * v * v + int64_t(a) * v + b];
    const double D = (d_oo[i] + d_oo[j]) - (d_vv[a] + d_vv[b]);
    const double e = epair[ij];
    if (standardise) {
      z[3 * u] = x / st.sx;
      z[3 * u + 1] = (D - st.mD) / st.sD;
      z[3 * u + 2] = (e - st.me) / st.se;
    } else {
      z[3 * u] = x;
      z[3 * u + 1] = D;
      z[3 * u + 2] = e;
    }
  }
}

__global__ __launch_bounds__(256) void standardise_kernel(const double *__restrict__ raw, const double *__restrict__ y,
                                                          int64_t n, cc_mlp_stats st, double *__restrict__ z,
                                                          double *__restrict__ ys) {
  for (int64_t r = blockIdx.x * int64_t(256) + threadIdx.x; r < n; r += int64_t(gridDim.x) * 256) {
    z[3 * r] = raw[3 * r] / st.sx;
    z[3 * r + 1] = (raw[3 * r + 1] - st.mD) / st.sD;
    z[3 * r + 2] = (raw[3 * r + 2] - st.me) / st.se;
    if (y) ys[r] = y[r] / st.st;
  }
}

// unique amplitudes of t2 (scaled by 1/st) -> y
__global__ __launch_bounds__(256) void gather_targets_kernel(int o, int v, const double *__restrict__ t2,
                                                             double inv_st, double *__restrict__ y) {
  const int64_t nab = int64_t(v) * (v - 1) / 2, n = nab * (int64_t(o) * (o - 1) / 2);
  for (int64_t u = blockIdx.x * int64_t(256) + threadIdx.x; u < n; u += int64_t(gridDim.x) * 256) {
    int i, j, a, b;
    const int64_t ij = idiv(u, nab);
    tri(ij, o, i, j);
    tri(u - ij * nab, v, a, b);
    y[u] = t2[(int64_t(i) * o + j) * v * v + int64_t(a) * v + b] * inv_st;
  }
}

// predictions f (scaled by st) -> antisymmetric t2 (four images, zero diagonals).
// Bound by HBM (f read once, t2 written): one workgroup takes an i < j and a
// pair of 32-wide tiles of (a, b) and writes the images through LDS, each
// coalesced; the (i, i) blocks are zeros, by workgroups of their own.  One element
// per thread, with the transposed images gathered, took 160 us at o = 32,
// v = 160; this 48 (260 MB, 5.4 TB/s).
constexpr int64_t CH_ZERO = 4096;  // zeros per workgroup
__global__ __launch_bounds__(256) void scatter_t2_kernel(int o, int v, const double *__restrict__ f, double st,
                                                         double *__restrict__ t2) {
  __shared__ double T[32][33];
  const int64_t vv = int64_t(v) * v, nab = int64_t(v) * (v - 1) / 2;
  const uint32_t nt = (v + 31) / 32, ntp = nt * (nt + 1) / 2, npair = uint32_t(o) * (o - 1) / 2, nval = npair * ntp;
  if (blockIdx.x >= nval) {
    const uint32_t nch = uint32_t((vv + CH_ZERO - 1) / CH_ZERO), z = blockIdx.x - nval, i = z / nch;
    double *p = t2 + int64_t(i) * (o + 1) * vv;
    const int64_t e0 = int64_t(z - i * nch) * CH_ZERO;
    for (int64_t e = e0 + threadIdx.x; e < e0 + CH_ZERO && e < vv; e += 256) p[e] = 0.0;
    return;
  }
  const uint32_t pij = blockIdx.x / ntp;
  int i, j, ta, tb;
  tri(pij, o, i, j);
  tri(blockIdx.x - pij * ntp, nt + 1, ta, tb);
  --tb;  // ta <= tb
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5, a0 = ta * 32, b0 = tb * 32;
  const double *F = f + int64_t(pij) * nab;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int a = a0 + ty + 8 * k, b = b0 + tx;
    T[ty + 8 * k][tx] = a < b && b < v ? st * F[int64_t(a) * (2 * v - a - 1) / 2 + (b - a - 1)] : 0.0;
  }
  __syncthreads();
  double *ij = t2 + (int64_t(i) * o + j) * vv, *ji = t2 + (int64_t(j) * o + i) * vv;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int la = ty + 8 * k, a = a0 + la, b = b0 + tx;
    if (a < v && b < v) {
      const bool up = a < b;
      const double x = up ? T[la][tx] : T[tx][la];
      const double y = a == b ? 0.0 : -x;
      ij[int64_t(a) * v + b] = up ? x : y;
      ji[int64_t(a) * v + b] = up ? y : x;
    }
  }
  if (ta == tb) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int lb = ty + 8 * k, b = b0 + lb, a = a0 + tx;
    if (a < v && b < v) {
      const double x = T[tx][lb];
      ij[int64_t(b) * v + a] = -x;
      ji[int64_t(b) * v + a] = x;
    }
  }
}

// rows [0,c): z[order[r]], rows [c,2c): same with the first component negated
__global__ __launch_bounds__(256) void build_z2_kernel(const double *__restrict__ z, const int64_t *__restrict__ order,
                                                       int64_t r0, int64_t c, double *__restrict__ z2) {
  for (int64_t r = blockIdx.x * int64_t(256) + threadIdx.x; r < c; r += int64_t(gridDim.x) * 256) {
    const int64_t src = order ? order[r0 + r] : r0 + r;
    const double a = z[3 * src], b = z[3 * src + 1], d = z[3 * src + 2];
    z2[3 * r] = a;
    z2[3 * r + 1] = b;
    z2[3 * r + 2] = d;
    z2[3 * (c + r)] = -a;
    z2[3 * (c + r) + 1] = b;
    z2[3 * (c + r) + 2] = d;
  }
}

__global__ __launch_bounds__(256) void bias_relu_kernel(double *__restrict__ A, const double *__restrict__ b,
                                                        int64_t rows) {
  const int64_t n = rows * HID;
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256) {
    const double x = A[e] + b[e % HID];
    A[e] = x > 0.0 ? x : 0.0;
  }
}

// f = (g+ - g-)/2 (g includes b3, which cancels); optional loss terms.
__global__ __launch_bounds__(256) void head_kernel(const double *__restrict__ g, int64_t c,
                                                   const double *__restrict__ y, const int64_t *__restrict__ order,
                                                   int64_t r0, double *__restrict__ f, double *__restrict__ dg,
                                                   double *__restrict__ lpart) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t r = blockIdx.x * int64_t(256) + threadIdx.x; r < c; r += int64_t(gridDim.x) * 256) {
    const double fv = 0.5 * (g[r] - g[c + r]);
    if (f) f[r0 + r] = fv;
    if (y) {
      const double res = fv - y[order ? order[r0 + r] : r0 + r];
      s += res * res;
      // d loss / d f = 2 res / c ; d f / d g+- = +-1/2
      dg[r] = res / double(c);
      dg[c + r] = -res / double(c);
    }
  }
  if (lpart) {
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) lpart[blockIdx.x] = sh[0];
  }
}

// dA2[r][j] = dg[r] W3[j] (H2[r][j] > 0)
__global__ __launch_bounds__(256) void da2_kernel(const double *__restrict__ dg, const double *__restrict__ W3,
                                                  const double *__restrict__ H2, int64_t rows,
                                                  double *__restrict__ dA2) {
  const int64_t n = rows * HID;
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256)
    dA2[e] = H2[e] > 0.0 ? dg[e / HID] * W3[e % HID] : 0.0;
}

__global__ __launch_bounds__(256) void relu_mask_kernel(double *__restrict__ d, const double *__restrict__ H,
                                                        int64_t n) {
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256)
    if (!(H[e] > 0.0)) d[e] = 0.0;
}

__global__ __launch_bounds__(256) void fill_kernel(double *p, double v, int64_t n) {
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256) p[e] = v;
}

// loss = sum of the nb <= 4096 partials / c, in order, written to out[idx]
// (staged in LDS first: one thread adding from device memory took 15 us)
__global__ __launch_bounds__(256) void loss_sum_kernel(const double *__restrict__ lpart, int nb, int64_t c,
                                                       double *__restrict__ out, int64_t idx) {
  __shared__ double sh[4096];
  for (int k = threadIdx.x; k < nb; k += 256) sh[k] = lpart[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int k = 0; k < nb; ++k) s += sh[k];
    out[idx] = s / double(c);
  }
}

__global__ __launch_bounds__(256) void adam_kernel(double *__restrict__ p, const double *__restrict__ g,
                                                   double *__restrict__ m, double *__restrict__ vv, int64_t n,
                                                   double lr, double b1, double b2, double eps, double c1,
                                                   double c2) {
  for (int64_t e = blockIdx.x * int64_t(256) + threadIdx.x; e < n; e += int64_t(gridDim.x) * 256) {
    const double gi = g[e];
    const double mi = b1 * m[e] + (1.0 - b1) * gi;
    const double vi = b2 * vv[e] + (1.0 - b2) * gi * gi;
    m[e] = mi;
    vv[e] = vi;
    p[e] -= lr * (mi / c1) / (sqrt(vi / c2) + eps);
  }
}

// column moments of raw features: [sum x^2, sum D, sum D^2, sum e, sum e^2] partials
__global__ __launch_bounds__(256) void moments_kernel(const double *__restrict__ raw, const double *__restrict__ y,
                                                      int64_t n, double *__restrict__ part) {
  __shared__ double sh[256];
  double acc[7] = {0, 0, 0, 0, 0, 0, 0};
  for (int64_t r = blockIdx.x * int64_t(256) + threadIdx.x; r < n; r += int64_t(gridDim.x) * 256) {
    const double x = raw[3 * r], D = raw[3 * r + 1], e = raw[3 * r + 2];
    acc[0] += x * x;
    acc[1] += D;
    acc[2] += D * D;
    acc[3] += e;
    acc[4] += e * e;
    if (y) acc[5] += y[r] * y[r];
    acc[6] += 1.0;
  }
  for (int q = 0; q < 7; ++q) {
    sh[threadIdx.x] = acc[q];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) part[7 * blockIdx.x + q] = sh[0];
    __syncthreads();
  }
}

int64_t grid_of(int64_t n) { return std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096)); }

// ---- fused FP32 forward (inference) ----------------------------------------
// f[u] = (g(z_u) - g(z~_u)) / 2 without writing activations anywhere: one
// wave takes 16 samples at a time as two 16-row blocks (the + branch and the
// branch with z0 negated) against all 128 hidden units.  Layer 1 is formed in
// registers directly in the MFMA operand layout, layer 2 runs on
// v_mfma_f32_16x16x4_f32 with W2 (rounded to FP32) staged once per workgroup
// in LDS, and bias, ReLU and the 128 -> 1 layer are applied to the
// accumulators, summed over the 16 lanes that share output rows.
//   MFMA 16x16x4 operands: lane l = 16 q + r supplies A[row r][k q] and
//   B[k q][col r] and holds D[4 q + t][r], t = 0..3.  Step s of chunk c uses
//   hidden unit k = 16 c + 4 q + s for lane group q (a permutation of the
//   128 units, the same on both operands).
typedef float f4v __attribute__((ext_vector_type(4)));
constexpr int FW_WAVES = 4;
constexpr int W2_LD = HID + 4;  // padded LDS row: the 16 lanes of a read phase hit distinct banks

__global__ __launch_bounds__(FW_WAVES * 64) void mlp_forward_fused_kernel(const double *__restrict__ P,
                                                                          const double *__restrict__ z, int64_t n,
                                                                          double *__restrict__ f) {
  __shared__ __attribute__((aligned(16))) float sW2[HID * W2_LD];
  __shared__ __attribute__((aligned(16))) float sW1[HID * 4];  // (w1 x, w1 y, w1 z, b1) per hidden unit
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int e = tid; e < HID * HID; e += FW_WAVES * 64) sW2[(e / HID) * W2_LD + e % HID] = float(P[OFF_W2 + e]);
  for (int k = tid; k < HID; k += FW_WAVES * 64) {
    sW1[4 * k] = float(P[OFF_W1 + 3 * k]);
    sW1[4 * k + 1] = float(P[OFF_W1 + 3 * k + 1]);
    sW1[4 * k + 2] = float(P[OFF_W1 + 3 * k + 2]);
    sW1[4 * k + 3] = float(P[OFF_B1 + k]);
  }
  __syncthreads();
  const int r = lane & 15, q = lane >> 4;
  float b2r[8], w3r[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    b2r[j] = float(P[OFF_B2 + 16 * j + r]);
    w3r[j] = float(P[OFF_W3 + 16 * j + r]);
  }
  const int64_t nblk = (n + 15) / 16;
  for (int64_t blk = int64_t(blockIdx.x) * FW_WAVES + wave; blk < nblk; blk += int64_t(gridDim.x) * FW_WAVES) {
    const int64_t u = std::min<int64_t>(blk * 16 + r, n - 1);
    const float z0 = float(z[3 * u]), z1 = float(z[3 * u + 1]), z2 = float(z[3 * u + 2]);
    f4v acc[2][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[0][j] = acc[1][j] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int c = 0; c < 8; ++c) {
      float a0[4], a1[4];
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        const f4v w = *reinterpret_cast<const f4v *>(&sW1[4 * (16 * c + 4 * q + st)]);
        const float common = w[1] * z1 + w[2] * z2 + w[3];
        const float hp = common + w[0] * z0, hm = common - w[0] * z0;
        a0[st] = hp > 0.f ? hp : 0.f;
        a1[st] = hm > 0.f ? hm : 0.f;
      }
      f4v bf[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) bf[j] = *reinterpret_cast<const f4v *>(&sW2[(16 * j + r) * W2_LD + 16 * c + 4 * q]);
#pragma unroll
      for (int st = 0; st < 4; ++st)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[st], bf[j][st], acc[0][j], 0, 0, 0);
          acc[1][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[st], bf[j][st], acc[1][j], 0, 0, 0);
        }
    }
    // g (without b3, which cancels in f) for rows 4 q + t of both branches
    float g[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float h = acc[i][j][t] + b2r[j];
          sum += (h > 0.f ? h : 0.f) * w3r[j];
        }
        g[i][t] = sum;
      }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) g[i][t] += __shfl_xor(g[i][t], off, 64);
    if (r == 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t uu = blk * 16 + 4 * q + t;
        if (uu < n) f[uu] = 0.5 * (double(g[0][t]) - double(g[1][t]));
      }
    }
  }
}

void forward_fused(const double *P, const double *z, int64_t n, double *f, hipStream_t s) {
  if (n <= 0) return;
  const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((n + 16 * FW_WAVES - 1) / (16 * FW_WAVES), 512));
  hipLaunchKernelGGL(mlp_forward_fused_kernel, dim3(blocks), dim3(FW_WAVES * 64), 0, s, P, z, n, f);
  CC_HIP_CHECK(hipGetLastError());
}

// ---- fused FP32 training passes ---------------------------------------------
// One minibatch of c samples is R = 2c rows (the + branch, then the - branch).
// The dense layers take FP32 operands on v_mfma_f32_16x16x4_f32 with FP32
// sums, bias, ReLU and the output layer's gradient in FP64 from those sums:
// every product, its place in its sum and every rounding is that of the
// layer-by-layer GEMMs (dense() below), so the results are theirs bit for bit.
// What is gone are the FP64 activations in device memory, written and read
// once per layer and elementwise pass (13 passes of 134 MB per minibatch of
// 65536, 970 us): the forward pass writes the second hidden layer once, in FP32
// and with its ReLU mask in the sign of zero, and the backward pass forms
// everything else from it and z in registers and LDS (both bound by MFMA).
// Minibatch of 65536: 970 -> 211 us (forward 70, backward 113: 61 and 76 TFLOP/s
// of the work that has to be done, the FP32 MFMA peak being 157).
//   MFMA 16x16x4 operands: lane l = 16 q + r supplies A[row r][k q] and
//   B[k q][col r] and holds D[4 q + t][r], t = 0..3 ("D form").  Step s of a
//   16-long chunk of k uses k = 4 q + s.  So a D-form block of 16 rows is,
//   value for value, the operand of a sum over those rows.
// Eight waves; wave w owns hidden units 16 w .. 16 w + 15.  Rows go by in
// blocks of 64.
constexpr int TW = 8, TROWS = 64;
constexpr int RM_LD = HID + 4;    // row-major LDS rows: 16-byte reads spread over the banks
constexpr int TR_LD = TROWS + 4;  // the same for unit-major rows

__device__ __forceinline__ int64_t mb_source(const int64_t *order, int64_t r0, int64_t c, int64_t row) {
  const int64_t u = r0 + (row < c ? row : row - c);
  return order ? order[u] : u;
}

// (1, z0, z1, z2) of a row in FP32; zeros past the last row
__device__ __forceinline__ f4v mb_row(const double *z, const int64_t *order, int64_t r0, int64_t c, int64_t row) {
  if (row >= 2 * c) return f4v{0.f, 0.f, 0.f, 0.f};
  const double *p = z + 3 * mb_source(order, r0, c, row);
  const float z0 = float(p[0]);
  return f4v{1.f, row < c ? z0 : -z0, float(p[1]), float(p[2])};
}

// FP64 bias and ReLU of an FP32 sum, rounded to FP32; -0 where the unit is off
__device__ __forceinline__ float bias_relu_f32(float acc, double bias) {
  const double x = double(acc) + bias;
  return x > 0.0 ? float(x) : -0.f;
}
__device__ __forceinline__ bool unit_on(float h) { return __float_as_uint(h) != 0x80000000u; }

// H1 of this wave's 16 units for the rows zl holds, D form per 16-row block
__device__ __forceinline__ void layer1(const f4v *zl, const float (&w1)[3], double b1, int q, int r, f4v (&h)[4]) {
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const f4v zr = zl[16 * b + r];
    f4v acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 3; ++s)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(q == 0 ? zr[1 + s] : 0.f, q == 0 ? w1[s] : 0.f, acc, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) h[b][t] = bias_relu_f32(acc[t], b1);
  }
}

__global__ __launch_bounds__(TW * 64, 4) void mlp_train_forward_kernel(const double *__restrict__ P,
                                                                    const double *__restrict__ z,
                                                                    const int64_t *__restrict__ order, int64_t r0,
                                                                    int64_t c, float *__restrict__ H2f,
                                                                    double *__restrict__ g) {
  __shared__ __attribute__((aligned(16))) float sH1[TROWS * RM_LD], sH2[TROWS * RM_LD];
  __shared__ f4v zl[TROWS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, r = lane & 15;
  const int64_t R = 2 * c;
  const int u = 16 * w + r;  // this lane's unit in D form
  float w1[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) w1[s] = float(P[OFF_W1 + 3 * u + s]);
  const double b1 = P[OFF_B1 + u], b2 = P[OFF_B2 + u];
  f4v w2[8], w3[8];  // B operands: W2[unit][16 kc + 4 q + s], W3 in column 0
#pragma unroll
  for (int kc = 0; kc < 8; ++kc)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      w2[kc][s] = float(P[OFF_W2 + u * HID + 16 * kc + 4 * q + s]);
      w3[kc][s] = r == 0 ? float(P[OFF_W3 + 16 * kc + 4 * q + s]) : 0.f;
    }
  for (int64_t row0 = int64_t(blockIdx.x) * TROWS; row0 < R; row0 += int64_t(gridDim.x) * TROWS) {
    if (w == 0) zl[lane] = mb_row(z, order, r0, c, row0 + lane);
    __syncthreads();
    f4v h[4];
    layer1(zl, w1, b1, q, r, h);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) sH1[(16 * b + 4 * q + t) * RM_LD + u] = h[b][t];
    __syncthreads();
    f4v acc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) {
      f4v a[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) a[b] = *reinterpret_cast<const f4v *>(&sH1[(16 * b + r) * RM_LD + 16 * kc + 4 * q]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][s], w2[kc][s], acc[b], 0, 0, 0);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) sH2[(16 * b + 4 * q + t) * RM_LD + u] = bias_relu_f32(acc[b][t], b2);
    __syncthreads();
    // the whole block in 16-byte stores, and g = H2 W3 by one wave per 16 rows
    for (int e = tid; e < TROWS * HID / 4; e += TW * 64) {
      const int row = e / (HID / 4), col = (e % (HID / 4)) * 4;
      if (row0 + row < R)
        *reinterpret_cast<f4v *>(H2f + (row0 + row) * HID + col) =
            *reinterpret_cast<const f4v *>(&sH2[row * RM_LD + col]);
    }
    if (w < 4) {
      f4v gs{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < 8; ++kc) {
        const f4v a = *reinterpret_cast<const f4v *>(&sH2[(16 * w + r) * RM_LD + 16 * kc + 4 * q]);
#pragma unroll
        for (int s = 0; s < 4; ++s) gs = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], w3[kc][s], gs, 0, 0, 0);
      }
      if (r == 0)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int64_t row = row0 + 16 * w + 4 * q + t;
          if (row < R) g[row] = double(gs[t]);
        }
    }
    // the next block's zl and sH1 writes come behind its first barrier; sH2 is
    // written behind its second
  }
}

struct GradSplits {
  int64_t kw, kv;  // rows per slice: dW2, sums over rows with a vector
  int nw, nv;      // slices of each kind
};

// Partial sums of the gradients.  Workgroup s sums rows [s kw, (s + 1) kw) of
// dW2 into slice s of ws_w2; the sums over rows with a vector (biases, W1,
// W3) go out every kv rows (kw a multiple of kv), slice by slice.
struct GradSlices {
  double *w2, *w1, *b1, *b2, *w3, *b3;  // [split][...]
  int64_t kw, kv;
  int nw, nv;  // slices of each kind
};

__global__ __launch_bounds__(TW * 64) void mlp_train_backward_kernel(const double *__restrict__ P,
                                                                     const double *__restrict__ z,
                                                                     const int64_t *__restrict__ order, int64_t r0,
                                                                     int64_t c, const float *__restrict__ H2f,
                                                                     const double *__restrict__ dg, GradSlices G) {
  // two buffers each: the next block is formed while slower waves still read
  __shared__ __attribute__((aligned(16))) float sH1[2][HID * TR_LD];    // [unit][row]
  __shared__ __attribute__((aligned(16))) float sD2[2][TROWS * RM_LD];  // dA2 [row][unit]
  __shared__ f4v zl[3][TROWS];
  __shared__ double dgl[3][TROWS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, r = lane & 15;
  const int64_t R = 2 * c;
  const int u = 16 * w + r;
  float w1[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) w1[s] = float(P[OFF_W1 + 3 * u + s]);
  const double b1 = P[OFF_B1 + u], w3 = P[OFF_W3 + u];
  f4v w2t[8];  // B operand of dA1: W2[16 kc + 4 q + s][unit]
#pragma unroll
  for (int kc = 0; kc < 8; ++kc)
#pragma unroll
    for (int s = 0; s < 4; ++s) w2t[kc][s] = float(P[OFF_W2 + (16 * kc + 4 * q + s) * HID + u]);

  const int64_t begin = int64_t(blockIdx.x) * G.kw, end = begin + G.kw;
  auto load_rows = [&](int64_t row0, f4v &zr, double &d) {
    const int64_t row = row0 + lane;
    const bool in = row < end && row < R;
    zr = in ? mb_row(z, order, r0, c, row) : f4v{0.f, 0.f, 0.f, 0.f};
    d = in ? dg[row] : 0.0;
  };
  auto load_h2 = [&](int64_t row0, f4v (&h)[4]) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t row = row0 + 16 * b + 4 * q + t;
        h[b][t] = row < end && row < R ? H2f[row * HID + u] : -0.f;
      }
  };
  const f4v zero4{0.f, 0.f, 0.f, 0.f};
  f4v accw[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) accw[i] = zero4;
  f4v accv1 = zero4, accv2 = zero4, accv3 = zero4, accv0 = zero4;
  int slice = int(begin / G.kv);
  int64_t left = G.kv;  // rows until the vector sums go out

  f4v zn;
  double dn = 0.0;
  if (w == 0) {
    load_rows(begin, zn, dn);
    zl[0][lane] = zn;
    dgl[0][lane] = dn;
    load_rows(begin + TROWS, zn, dn);
  }
  f4v h2n[4];
  load_h2(begin, h2n);
  __syncthreads();
  int it = 0;
  for (int64_t row0 = begin; row0 < end; row0 += TROWS, ++it) {
    const int buf = it & 1, zb = it % 3;
    // -- form H1 and dA2 of the wave's units
    if (w == 0) {  // the next block's rows (read behind the barrier below)
      zl[(it + 1) % 3][lane] = zn;
      dgl[(it + 1) % 3][lane] = dn;
    }
    f4v h1[4], h2[4], d2[4];
    layer1(zl[zb], w1, b1, q, r, h1);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      *reinterpret_cast<f4v *>(&sH1[buf][u * TR_LD + 16 * b + 4 * q]) = h1[b];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        h2[b][t] = h2n[b][t];
        const double dgr = dgl[zb][16 * b + 4 * q + t];
        d2[b][t] = unit_on(h2[b][t]) ? float(dgr * w3) : 0.f;
        sD2[buf][(16 * b + 4 * q + t) * RM_LD + u] = d2[b][t];
      }
    }
    __syncthreads();
    if (row0 + TROWS < end) load_h2(row0 + TROWS, h2n);
    if (w == 0) load_rows(row0 + 2 * TROWS, zn, dn);
    // -- dA1 = dA2 W2, units of this wave
    f4v d1[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) d1[b] = zero4;
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) {
      f4v a[4];
#pragma unroll
      for (int b = 0; b < 4; ++b)
        a[b] = *reinterpret_cast<const f4v *>(&sD2[buf][(16 * b + r) * RM_LD + 16 * kc + 4 * q]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int b = 0; b < 4; ++b)
          d1[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][s], w2t[kc][s], d1[b], 0, 0, 0);
    }
    // -- sums over the rows, block by block
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (row0 + 16 * b >= end) break;
      f4v hb[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        hb[i] = *reinterpret_cast<const f4v *>(&sH1[buf][(16 * i + r) * TR_LD + 16 * b + 4 * q]);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          accw[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(d2[b][s], hb[i][s], accw[i], 0, 0, 0);
        // A rows 0..3: 1, z0, z1, z2 (bias and W1), 1 (b2), dg (W3, b3)
        const int row = 16 * b + 4 * q + s;
        const f4v zr = zl[zb][row];
        const float one = zr[0];
        const float av = r == 0 ? one : r == 1 ? zr[1] : r == 2 ? zr[2] : r == 3 ? zr[3] : 0.f;
        const float ad = r == 0 ? float(dgl[zb][row]) : 0.f;
        const float dd = unit_on(h1[b][s]) ? d1[b][s] : 0.f;
        accv1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av, dd, accv1, 0, 0, 0);
        accv2 = __builtin_amdgcn_mfma_f32_16x16x4f32(r == 0 ? one : 0.f, d2[b][s], accv2, 0, 0, 0);
        accv3 = __builtin_amdgcn_mfma_f32_16x16x4f32(ad, h2[b][s], accv3, 0, 0, 0);
        if (w == 0) accv0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ad, r == 0 ? one : 0.f, accv0, 0, 0, 0);
      }
      left -= 16;
      if (left == 0) {
        if (q == 0 && slice < G.nv) {
          const int64_t v = int64_t(slice) * HID + u;
          G.b1[v] = double(accv1[0]);
          G.w1[3 * v] = double(accv1[1]);
          G.w1[3 * v + 1] = double(accv1[2]);
          G.w1[3 * v + 2] = double(accv1[3]);
          G.b2[v] = double(accv2[0]);
          G.w3[v] = double(accv3[0]);
          if (w == 0 && r == 0) G.b3[slice] = double(accv0[0]);
        }
        accv0 = accv1 = accv2 = accv3 = zero4;
        ++slice;
        left = G.kv;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int t = 0; t < 4; ++t)
      G.w2[(int64_t(blockIdx.x) * HID + 16 * w + 4 * q + t) * HID + 16 * i + r] = double(accw[i][t]);
  // vector slices that lie wholly past the workgroups' rows
  if (blockIdx.x == gridDim.x - 1)
    for (int sl = int(int64_t(G.nw) * (G.kw / G.kv)); sl < G.nv; ++sl)
      if (w == 0) {
        for (int e = lane; e < HID; e += 64) G.b1[int64_t(sl) * HID + e] = G.b2[int64_t(sl) * HID + e] =
            G.w3[int64_t(sl) * HID + e] = 0.0;
        for (int e = lane; e < 3 * HID; e += 64) G.w1[int64_t(sl) * 3 * HID + e] = 0.0;
        if (lane == 0) G.b3[sl] = 0.0;
      }
}

// Dense layer helper: C[M][N] = alpha * A' B'^T + beta C (GemmDesc conventions)
void dense(int prec, int64_t M, int64_t N, int64_t K, const double *A, int64_t sam, int64_t sak, const double *B,
           int64_t sbn, int64_t sbk, double *C, double beta, double *ws, int64_t ws_elems, hipStream_t s) {
  GemmDesc d{M, N, K, A, sam, sak, B, sbn, sbk, C, N, 1.0, beta};
  // the split-K factor the library picks, down to what the workspace holds
  // (the weight gradients, K = rows of a minibatch, run on a handful of
  // output tiles and need the split)
  int64_t split = gemm_split_pick(M, N, K, -1);
  if (ws) split = std::min<int64_t>(split, ws_elems / (M * N));
  if (split > 1 && ws) {
    d.split = int(split);
    d.ws = ws;
  }
  if (prec == PREC_F64) gemm_f64(d, s, -1);
  else gemm_lowp(d, prec, s, -1);
}

// Slices of the fused backward pass: those of the layer-by-layer gradient
// GEMMs (their split-K factors, whole 16-row chunks), so that the partial sums
// are the same.  The sums over rows with a vector go out several times per
// dW2 slice; minibatches whose slice lengths do not fit each other that way run
// layer by layer, at the times of those passes.  Up to 32,768 samples all fit,
// above one size in sixteen (32769 to 34815 but for multiples of 128, and the
// multiples of 128 from 63616 to the default of 65536).
constexpr int64_t WS_ELEMS = 256 * int64_t(HID) * HID;
bool fused_slices(int64_t R, GradSplits *g) {
  auto pick = [R](int64_t M, int64_t N, int *split, int64_t *kc) {
    *split = int(std::min<int64_t>(gemm_split_pick(M, N, R, -1), WS_ELEMS / (M * N)));
    *kc = ((R + *split - 1) / *split + 15) / 16 * 16;
  };
  int64_t k1 = 0, k3 = 0;
  int s1 = 0, s3 = 0;
  pick(HID, HID, &g->nw, &g->kw);
  pick(1, HID, &g->nv, &g->kv);  // b1, b2, W3
  pick(HID, 3, &s1, &k1);        // W1
  pick(1, 1, &s3, &k3);          // b3
  return s1 == g->nv && s3 == g->nv && k1 == g->kv && k3 == g->kv && g->kw % g->kv == 0;
}

struct MlpWork {
  int64_t cap = 0;  // rows per chunk (samples)
  double *z2 = nullptr, *H1 = nullptr, *H2 = nullptr, *dH = nullptr, *g = nullptr, *dg = nullptr,
         *grad = nullptr, *ones = nullptr, *lpart = nullptr, *ws = nullptr, *wsv = nullptr;
  float *H2f = nullptr;
  void *red = nullptr;  // grouped reductions of the fused pass: entries and offsets for up to two R
  int64_t red_R[2] = {0, 0}, red_blocks[2] = {0, 0};
  std::vector<unsigned char> red_host[2];
  int64_t ws_elems = 0;
  static constexpr int64_t kMaxVec = 1024;  // vector slices (the largest split-K factor)
  static void A(void **p, int64_t bytes) {
    if (*p) return;
    if (hipMalloc(p, std::max<int64_t>(bytes, 16)) != hipSuccess) {
      (void)hipGetLastError();
      *p = nullptr;
      throw CCError(CC_ENOMEM, "MLP workspace allocation failed");
    }
  }
  static void A(double **p, int64_t n) { A(reinterpret_cast<void **>(p), n * int64_t(sizeof(double))); }
  void alloc(int64_t c) {
    cap = c;
    A(&g, 2 * c);
    A(&dg, 2 * c);
    A(&grad, NPAR);
    A(&lpart, 4096);
    ws_elems = WS_ELEMS;
    A(&ws, ws_elems);
  }
  void layers(hipStream_t s) {  // FP64 activations of the layer-by-layer passes
    if (ones) return;
    A(&z2, 2 * cap * 3);
    A(&H1, 2 * cap * HID);
    A(&H2, 2 * cap * HID);
    A(&dH, 2 * cap * HID);
    A(&ones, 2 * cap);
    hipLaunchKernelGGL(fill_kernel, dim3(grid_of(2 * cap)), dim3(256), 0, s, ones, 1.0, 2 * cap);
  }
  void fused() {
    A(reinterpret_cast<void **>(&H2f), 2 * cap * HID * int64_t(sizeof(float)));
    A(&wsv, kMaxVec * (6 * HID + 1));
    A(&red, 2 * kRedBytes);
  }
  static constexpr int kRed = 6;
  static constexpr int64_t kRedBytes = 1024;
  ~MlpWork() {
    for (double *p : {z2, H1, H2, dH, g, dg, grad, ones, lpart, ws, wsv})
      if (p) (void)hipFree(p);
    if (H2f) (void)hipFree(H2f);
    if (red) (void)hipFree(red);
  }
};

// Fused FP32 forward and backward of one minibatch; its gradient into w.grad.
void fused_chunk(const double *P, const double *z, const double *y, const int64_t *order, int64_t r0, int64_t c,
                 const GradSplits &sp, MlpWork &w, double *loss_out, int64_t loss_idx, hipStream_t s) {
  const int64_t R = 2 * c;
  w.fused();
  GradSlices G{};
  G.w2 = w.ws;
  G.b1 = w.wsv;
  G.b2 = G.b1 + MlpWork::kMaxVec * HID;
  G.w3 = G.b2 + MlpWork::kMaxVec * HID;
  G.w1 = G.w3 + MlpWork::kMaxVec * HID;
  G.b3 = G.w1 + MlpWork::kMaxVec * 3 * HID;
  G.kw = sp.kw;
  G.kv = sp.kv;
  G.nw = sp.nw;
  G.nv = sp.nv;
  // the six reductions as one grouped launch (tables kept for the full and
  // the last minibatch)
  int set = w.red_R[0] == R ? 0 : w.red_R[1] == R ? 1 : w.red_R[0] == 0 ? 0 : 1;
  if (w.red_R[set] != R) {
    const SplitkEntry es[MlpWork::kRed] = {
        make_splitk_entry(G.w2, sp.nw, HID, HID, w.grad + OFF_W2, HID, 1.0, 0.0),
        make_splitk_entry(G.w1, sp.nv, HID, 3, w.grad + OFF_W1, 3, 1.0, 0.0),
        make_splitk_entry(G.b1, sp.nv, 1, HID, w.grad + OFF_B1, HID, 1.0, 0.0),
        make_splitk_entry(G.b2, sp.nv, 1, HID, w.grad + OFF_B2, HID, 1.0, 0.0),
        make_splitk_entry(G.w3, sp.nv, 1, HID, w.grad + OFF_W3, HID, 1.0, 0.0),
        make_splitk_entry(G.b3, sp.nv, 1, 1, w.grad + OFF_B3, 1, 1.0, 0.0)};
    int64_t off[MlpWork::kRed + 1] = {0};
    for (int k = 0; k < MlpWork::kRed; ++k) off[k + 1] = off[k] + es[k].units;
    static_assert(sizeof(es) + sizeof(off) <= MlpWork::kRedBytes, "reduction tables");
    if (w.red_R[set] != 0) CC_HIP_CHECK(hipStreamSynchronize(s));  // an older table may still be read
    w.red_host[set].resize(MlpWork::kRedBytes);
    std::memcpy(w.red_host[set].data(), es, sizeof(es));
    std::memcpy(w.red_host[set].data() + sizeof(es), off, sizeof(off));
    CC_HIP_CHECK(hipMemcpyAsync(static_cast<char *>(w.red) + set * MlpWork::kRedBytes, w.red_host[set].data(),
                                MlpWork::kRedBytes, hipMemcpyHostToDevice, s));
    w.red_R[set] = R;
    w.red_blocks[set] = off[MlpWork::kRed];
  }
  const int64_t nblk = (R + TROWS - 1) / TROWS;
  hipLaunchKernelGGL(mlp_train_forward_kernel, dim3(std::min<int64_t>(nblk, 512)), dim3(TW * 64), 0, s, P, z, order,
                     r0, c, w.H2f, w.g);
  const int nb = int(grid_of(c));
  hipLaunchKernelGGL(head_kernel, dim3(nb), dim3(256), 0, s, w.g, c, y, order, r0, (double *)nullptr, w.dg, w.lpart);
  if (loss_out) hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(256), 0, s, w.lpart, nb, c, loss_out, loss_idx);
  hipLaunchKernelGGL(mlp_train_backward_kernel, dim3(sp.nw), dim3(TW * 64), 0, s, P, z, order, r0, c, w.H2f, w.dg, G);
  CC_HIP_CHECK(hipGetLastError());
  const char *tab = static_cast<const char *>(w.red) + set * MlpWork::kRedBytes;
  launch_splitk_grouped(reinterpret_cast<const SplitkEntry *>(tab),
                        reinterpret_cast<const int64_t *>(tab + MlpWork::kRed * sizeof(SplitkEntry)), MlpWork::kRed,
                        w.red_blocks[set], false, s);
}

// Forward of rows [r0, r0+c): leaves H1, H2, g in the workspace.
void forward_chunk(int prec, const double *P, const double *z, const int64_t *order, int64_t r0, int64_t c,
                   MlpWork &w, hipStream_t s) {
  const int64_t R = 2 * c;
  hipLaunchKernelGGL(build_z2_kernel, dim3(grid_of(c)), dim3(256), 0, s, z, order, r0, c, w.z2);
  dense(prec, R, HID, 3, w.z2, 3, 1, P + OFF_W1, 3, 1, w.H1, 0.0, nullptr, 0, s);
  hipLaunchKernelGGL(bias_relu_kernel, dim3(grid_of(R * HID)), dim3(256), 0, s, w.H1, P + OFF_B1, R);
  dense(prec, R, HID, HID, w.H1, HID, 1, P + OFF_W2, HID, 1, w.H2, 0.0, nullptr, 0, s);
  hipLaunchKernelGGL(bias_relu_kernel, dim3(grid_of(R * HID)), dim3(256), 0, s, w.H2, P + OFF_B2, R);
  dense(prec, R, 1, HID, w.H2, HID, 1, P + OFF_W3, HID, 1, w.g, 0.0, nullptr, 0, s);
  CC_HIP_CHECK(hipGetLastError());
}

// Gradient of the chunk's mean squared error into w.grad (overwritten).
void backward_chunk(int prec, const double *P, const double *z, const double *y, const int64_t *order, int64_t r0,
                    int64_t c, MlpWork &w, double *loss_out, int64_t loss_idx, hipStream_t s) {
  const int64_t R = 2 * c;
  GradSplits sp;
  if (prec == PREC_F32 && fused_slices(R, &sp)) {
    fused_chunk(P, z, y, order, r0, c, sp, w, loss_out, loss_idx, s);
    return;
  }
  w.layers(s);
  forward_chunk(prec, P, z, order, r0, c, w, s);
  const int nb = int(grid_of(c));
  hipLaunchKernelGGL(head_kernel, dim3(nb), dim3(256), 0, s, w.g, c, y, order, r0, (double *)nullptr, w.dg,
                     w.lpart);
  if (loss_out) hipLaunchKernelGGL(loss_sum_kernel, dim3(1), dim3(256), 0, s, w.lpart, nb, c, loss_out, loss_idx);
  double *G = w.grad;
  // W3 (1 x 128) = dg^T H2 ; b3 = sum dg
  dense(prec, 1, HID, R, w.dg, R, 1, w.H2, 1, HID, G + OFF_W3, 0.0, w.ws, w.ws_elems, s);
  dense(prec, 1, 1, R, w.dg, R, 1, w.ones, R, 1, G + OFF_B3, 0.0, w.ws, w.ws_elems, s);
  // dA2 in place of H2 (H2 is needed for the mask first)
  hipLaunchKernelGGL(da2_kernel, dim3(grid_of(R * HID)), dim3(256), 0, s, w.dg, P + OFF_W3, w.H2, R, w.H2);
  dense(prec, HID, HID, R, w.H2, 1, HID, w.H1, 1, HID, G + OFF_W2, 0.0, w.ws, w.ws_elems, s);
  dense(prec, 1, HID, R, w.ones, R, 1, w.H2, 1, HID, G + OFF_B2, 0.0, w.ws, w.ws_elems, s);
  // dA1 = (dA2 W2) * (H1 > 0)
  dense(prec, R, HID, HID, w.H2, HID, 1, P + OFF_W2, 1, HID, w.dH, 0.0, nullptr, 0, s);
  hipLaunchKernelGGL(relu_mask_kernel, dim3(grid_of(R * HID)), dim3(256), 0, s, w.dH, w.H1, R * HID);
  dense(prec, HID, 3, R, w.dH, 1, HID, w.z2, 1, 3, G + OFF_W1, 0.0, w.ws, w.ws_elems, s);
  dense(prec, 1, HID, R, w.ones, R, 1, w.dH, 1, HID, G + OFF_B1, 0.0, w.ws, w.ws_elems, s);
  CC_HIP_CHECK(hipGetLastError());
}

// Scratch of the features: pair energies and the two Fock diagonals.
int64_t features_scratch(int o, int v) { return int64_t(o) * (o - 1) / 2 + o + v; }

// Enqueue the features of a system; scratch holds features_scratch() doubles.
void features(const cc_system *sys, const cc_mlp_stats *stats, double *z, double *scratch, hipStream_t s) {
  const int o = sys->o, v = sys->v;
  const int64_t npair = int64_t(o) * (o - 1) / 2, n = npair * (int64_t(v) * (v - 1) / 2);
  double *ep = scratch, *d_oo = ep + npair, *d_vv = d_oo + o;
  fock_diag(false, o, v, sys->f_oo, sys->f_vv, d_oo, d_vv, s);
  const cc_mlp_stats st = stats ? *stats : cc_mlp_stats{1, 0, 1, 0, 1, 1};
  hipLaunchKernelGGL(pair_energy_kernel, dim3(npair), dim3(256), 0, s, o, v, static_cast<const double *>(sys->oovv),
                     d_oo, d_vv, ep);
  hipLaunchKernelGGL(features_kernel, dim3(grid_of(n)), dim3(256), 0, s, o, v, static_cast<const double *>(sys->oovv),
                     d_oo, d_vv, ep, st, stats ? 1 : 0, z);
  CC_HIP_CHECK(hipGetLastError());
}

// Device scratch of one call.
struct Scratch {
  double *p = nullptr;
  explicit Scratch(int64_t n) { CC_HIP_CHECK(hipMalloc(&p, sizeof(double) * n)); }
  ~Scratch() { (void)hipFree(p); }
  Scratch(const Scratch &) = delete;
  Scratch &operator=(const Scratch &) = delete;
};

}  // namespace
}  // namespace ccmi

// ================================================================ C ABI ====
using ccmi::CCError;
namespace {
int mfail(cc_ctx *ctx, int st, const std::string &m) {
  if (ctx) ctx->last_error = m;
  return st;
}
template <class F>
int mguard(cc_ctx *ctx, F &&f) {
  try {
    return f();
  } catch (const CCError &e) {
    return mfail(ctx, e.status, e.what());
  } catch (const std::exception &e) {
    return mfail(ctx, CC_EINTERNAL, e.what());
  }
}
void check_sys_real(const cc_system *sys) {
  if (!sys || sys->o < 2 || sys->v < 2) throw CCError(CC_EINVAL, "MLP features need o >= 2 and v >= 2");
  if (sys->scalar != CC_R64) throw CCError(CC_EUNSUPPORTED, "the amplitude-guess network is real-valued");
  if (!sys->oovv || !sys->f_oo || !sys->f_vv) throw CCError(CC_EINVAL, "system pointers are NULL");
}
void check_prec(int prec) {
  if (prec != CC_PREC_F64 && prec != CC_PREC_F32) throw CCError(CC_EINVAL, "MLP precision must be F64 or F32");
}
}  // namespace

extern "C" {

int64_t cc_mlp_num_params(void) { return ccmi::NPAR; }

int64_t cc_mlp_num_samples(int o, int v) {
  if (o < 2 || v < 2) return 0;
  return (int64_t(o) * (o - 1) / 2) * (int64_t(v) * (v - 1) / 2);
}

int cc_mlp_features(cc_ctx *ctx, const cc_system *sys, const cc_mlp_stats *stats, double *z_out) {
  if (!ctx) return mfail(nullptr, CC_EINVAL, "ctx is NULL");
  return mguard(ctx, [&] {
    check_sys_real(sys);
    if (!z_out) throw CCError(CC_EINVAL, "z_out is NULL");
    CC_HIP_CHECK(hipSetDevice(ctx->device));
    ccmi::Scratch w(ccmi::features_scratch(sys->o, sys->v));
    ccmi::features(sys, stats, z_out, w.p, ctx->stream);
    CC_HIP_CHECK(hipStreamSynchronize(ctx->stream));
    return CC_OK;
  });
}

int cc_mlp_targets(cc_ctx *ctx, int o, int v, const double *t2, double scale, double *y_out) {
  if (!ctx) return mfail(nullptr, CC_EINVAL, "ctx is NULL");
  return mguard(ctx, [&] {
    if (!t2 || !y_out || o < 2 || v < 2 || !(scale != 0.0)) throw CCError(CC_EINVAL, "bad arguments");
    const int64_t n = cc_mlp_num_samples(o, v);
    hipLaunchKernelGGL(ccmi::gather_targets_kernel, dim3(ccmi::grid_of(n)), dim3(256), 0, ctx->stream, o, v, t2,
                       1.0 / scale, y_out);
    CC_HIP_CHECK(hipGetLastError());
    CC_HIP_CHECK(hipStreamSynchronize(ctx->stream));
    return CC_OK;
  });
}

int cc_mlp_standardise(cc_ctx *ctx, const double *raw, const double *y, int64_t n, const cc_mlp_stats *stats,
                       double *z_out, double *y_out) {
  if (!ctx) return mfail(nullptr, CC_EINVAL, "ctx is NULL");
  return mguard(ctx, [&] {
    if (!raw || !stats || !z_out || n < 1 || (y && !y_out)) throw CCError(CC_EINVAL, "bad arguments");
    hipLaunchKernelGGL(ccmi::standardise_kernel, dim3(ccmi::grid_of(n)), dim3(256), 0, ctx->stream, raw, y, n,
                       *stats, z_out, y_out);
    CC_HIP_CHECK(hipGetLastError());
    CC_HIP_CHECK(hipStreamSynchronize(ctx->stream));
    return CC_OK;
  });
}

int cc_mlp_moments(cc_ctx *ctx, const double *raw, const double *y, int64_t n, double *out7) {
  if (!ctx) return mfail(nullptr, CC_EINVAL, "ctx is NULL");
  return mguard(ctx, [&] {
    if (!raw || n < 1 || !out7) throw CCError(CC_EINVAL, "bad arguments");
    const int nb = int(ccmi::grid_of(n));
    double *part = nullptr;
    CC_HIP_CHECK(hipMalloc(&part, sizeof(double) * 7 * nb));
    hipLaunchKernelGGL(ccmi::moments_kernel, dim3(nb), dim3(256), 0, ctx->stream, raw, y, n, part);
    std::vector<double> h(7 * nb);
    CC_HIP_CHECK(hipMemcpyAsync(h.data(), part, sizeof(double) * 7 * nb, hipMemcpyDeviceToHost, ctx->stream));
    CC_HIP_CHECK(hipStreamSynchronize(ctx->stream));
    (void)hipFree(part);
    for (int q = 0; q < 7; ++q) {
      double s = 0.0;
      for (int b = 0; b < nb; ++b) s += h[7 * b + q];
      out7[q] = s;
    }
    return CC_OK;
  });
}

int cc_mlp_forward(cc_ctx *ctx, int prec, const double *params, const double *z, int64_t n, double *f_out) {
  if (!ctx) return mfail(nullptr, CC_EINVAL, "ctx is NULL");
  return mguard(ctx, [&] {
    check_prec(prec);
    if (!params || !z || !f_out || n < 1) throw CCError(CC_EINVAL, "bad arguments");
    CC_HIP_CHECK(hipSetDevice(ctx->device));
    if (prec == CC_PREC_F32) {  // inference in one fused launch
      ccmi::forward_fused(params, z, n, f_out, ctx->stream);
      CC_HIP_CHECK(hipStreamSynchronize(ctx->stream));
      return CC_OK;
    }
    ccmi::MlpWork w;
    const int64_t cap = std::min<int64_t>(n, 1 << 18);
    w.alloc(cap);
    w.layers(ctx->stream);
    for (int64_t r0 = 0; r0 < n; r0 += cap) {
      const int64_t c = std::min(cap, n - r0);
      ccmi::forward_chunk(prec, params, z, nullptr, r0, c, w, ctx->stream);
      hipLaunchKernelGGL(ccmi::head_kernel, dim3(ccmi::grid_of(c)), dim3(256), 0, ctx->stream, w.g, c,
                         (const double *)nullptr, (const int64_t *)nullptr, r0, f_out, (double *)nullptr,
                         (double *)nullptr);
    }
    CC_HIP_CHECK(hipStreamSynchronize(ctx->stream));
    return CC_OK;
  });
}

int cc_mlp_loss_grad(cc_ctx *ctx, int prec, const double *params, const double *z, const double *y, int64_t n,
                     double *loss, double *grad_out) {
  if (!ctx) return mfail(nullptr, CC_EINVAL, "ctx is NULL");
  return mguard(ctx, [&] {
    check_prec(prec);
    if (!params || !z || !y || !grad_out || n < 1) throw CCError(CC_EINVAL, "bad arguments");
    CC_HIP_CHECK(hipSetDevice(ctx->device));
    ccmi::MlpWork w;
    w.alloc(n);
    hipStream_t s = ctx->stream;
    double *dl = nullptr;
    CC_HIP_CHECK(hipMalloc(&dl, sizeof(double)));
    ccmi::backward_chunk(prec, params, z, y, nullptr, 0, n, w, dl, 0, s);
    CC_HIP_CHECK(hipMemcpyAsync(grad_out, w.grad, sizeof(double) * ccmi::NPAR, hipMemcpyDeviceToDevice, s));
    double hl = 0.0;
    CC_HIP_CHECK(hipMemcpyAsync(&hl, dl, sizeof(double), hipMemcpyDeviceToHost, s));
    CC_HIP_CHECK(hipStreamSynchronize(s));
    (void)hipFree(dl);
    if (loss) *loss = hl;
    return CC_OK;
  });
}

int cc_mlp_train(cc_ctx *ctx, int prec, double *params, double *adam_m, double *adam_v, const double *z,
                 const double *y, int64_t n, const int64_t *order, int64_t batch, int32_t epochs, double lr,
                 int64_t *adam_t, double *loss_hist, int32_t hist_cap) {
  if (!ctx) return mfail(nullptr, CC_EINVAL, "ctx is NULL");
  return mguard(ctx, [&] {
    check_prec(prec);
    if (!params || !adam_m || !adam_v || !z || !y || !adam_t || n < 1 || batch < 1 || epochs < 1 || !(lr > 0))
      throw CCError(CC_EINVAL, "bad arguments");
    CC_HIP_CHECK(hipSetDevice(ctx->device));
    hipStream_t s = ctx->stream;
    const int64_t c = std::min(batch, n);
    ccmi::MlpWork w;
    w.alloc(c);
    const int64_t steps_per_epoch = (n + c - 1) / c;
    double *dl = nullptr;
    CC_HIP_CHECK(hipMalloc(&dl, sizeof(double) * steps_per_epoch));
    const double b1 = 0.9, b2 = 0.999, eps = 1e-8;
    for (int ep = 0; ep < epochs; ++ep) {
      for (int64_t st = 0; st < steps_per_epoch; ++st) {
        const int64_t r0 = st * c, cc = std::min(c, n - r0);
        ccmi::backward_chunk(prec, params, z, y, order, r0, cc, w, dl, st, s);
        const int64_t t = ++(*adam_t);
        hipLaunchKernelGGL(ccmi::adam_kernel, dim3(ccmi::grid_of(ccmi::NPAR)), dim3(256), 0, s, params, w.grad,
                           adam_m, adam_v, ccmi::NPAR, lr, b1, b2, eps, 1.0 - std::pow(b1, double(t)),
                           1.0 - std::pow(b2, double(t)));
      }
      std::vector<double> h(steps_per_epoch);
      CC_HIP_CHECK(hipMemcpyAsync(h.data(), dl, sizeof(double) * steps_per_epoch, hipMemcpyDeviceToHost, s));
      CC_HIP_CHECK(hipStreamSynchronize(s));
      double mean = 0.0;
      for (double x : h) mean += x;
      mean /= double(steps_per_epoch);
      if (loss_hist && ep < hist_cap) loss_hist[ep] = mean;
    }
    (void)hipFree(dl);
    return CC_OK;
  });
}

int cc_guess_mlp(cc_ctx *ctx, const cc_system *sys, int prec, const double *params, const cc_mlp_stats *stats,
                 cc_amps *t_out) {
  if (!ctx) return mfail(nullptr, CC_EINVAL, "ctx is NULL");
  return mguard(ctx, [&]() -> int {
    check_sys_real(sys);
    check_prec(prec);
    if (!params || !stats || !t_out || !t_out->t2) throw CCError(CC_EINVAL, "bad arguments");
    const int o = sys->o, v = sys->v;
    const int64_t n = cc_mlp_num_samples(o, v);
    CC_HIP_CHECK(hipSetDevice(ctx->device));
    hipStream_t s = ctx->stream;
    ccmi::Scratch w(4 * n + ccmi::features_scratch(o, v));
    double *z = w.p, *f = z + 3 * n;
    ccmi::features(sys, stats, z, f + n, s);
    if (prec == CC_PREC_F32) {
      ccmi::forward_fused(params, z, n, f, s);
    } else {
      const int st = cc_mlp_forward(ctx, prec, params, z, n, f);
      if (st != CC_OK) return st;
    }
    const int64_t nt = (v + 31) / 32, vv = int64_t(v) * v;
    const int64_t blocks = (int64_t(o) * (o - 1) / 2) * (nt * (nt + 1) / 2) + o * ((vv + ccmi::CH_ZERO - 1) / ccmi::CH_ZERO);
    CC_REQUIRE(blocks < (int64_t(1) << 31), -1, "grid too large");
    hipLaunchKernelGGL(ccmi::scatter_t2_kernel, dim3(blocks), dim3(256), 0, s, o, v, f, stats->st,
                       static_cast<double *>(t_out->t2));
    if (t_out->t1)
      hipLaunchKernelGGL(ccmi::fill_kernel, dim3(ccmi::grid_of(int64_t(o) * v)), dim3(256), 0, s,
                         static_cast<double *>(t_out->t1), 0.0, int64_t(o) * v);
    CC_HIP_CHECK(hipGetLastError());
    CC_HIP_CHECK(hipStreamSynchronize(s));
    return CC_OK;
  });
}

}  // extern "C"
