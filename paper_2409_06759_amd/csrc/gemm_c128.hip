// Complex128 GEMM on FP64 MFMA:  C = alpha * sum_k A(m,k) B(n,k) + beta * C,
// interleaved (re, im) storage, real alpha and beta.
//
// Each complex product is four real products on v_mfma_f64_16x16x4_f64:
//   re += ar*br - ai*bi,  im += ar*bi + ai*br
// with separate real and imaginary accumulators (8 real flop per complex
// multiply-add, the algorithmic count of the complex residual).  Tiles are
// staged into planar real/imaginary LDS panels, double buffered; split-K and
// the XCD-aware tile order follow the real FP64 kernel.  The LDS-direct
// configurations load K-contiguous operands straight into two or three
// interleaved (re, im) LDS stages.  Conjugated operands
// never reach this kernel: the contraction planner materialises them as
// conjugated views.
#include "common.hpp"

#include <algorithm>
#include <cmath>

namespace ccmi {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC>
struct ZCfg {
  static constexpr int NT = WM * WN * kWave;
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int FM = WTM / 16, FN = WTN / 16;
  static constexpr int PAD = 2;
  static constexpr int A_ROWS = AKC ? BM : BK, A_LD = AKC ? BK + PAD : BM + PAD;
  static constexpr int B_ROWS = BKC ? BN : BK, B_LD = BKC ? BK + PAD : BN + PAD;
  static constexpr int A_ELEMS = A_ROWS * A_LD, B_ELEMS = B_ROWS * B_LD;
  static constexpr int LA = BM * BK / NT, LB = BN * BK / NT;
  static_assert(BM % (16 * WM) == 0 && BN % (16 * WN) == 0, "tile/wave mismatch");
  static_assert(BK % 16 == 0 && (BM * BK) % NT == 0 && (BN * BK) % NT == 0, "tile");
};

template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC>
__global__ __launch_bounds__(WM *WN *kWave) void gemm_c128_kernel(GemmDesc d, int64_t tilesM,
                                                                   int64_t tilesN) {
  using C = ZCfg<BM, BN, BK, WM, WN, AKC, BKC>;
  // per buffer: A re, A im, B re, B im
  constexpr int BUF = 2 * C::A_ELEMS + 2 * C::B_ELEMS;
  __shared__ double smem[2 * BUF];

  const int64_t tiles = tilesM * tilesN, total = tiles * d.split;
  const int64_t L0 = xcd_remap(blockIdx.x, total);
  const int64_t ks = L0 / tiles, L = L0 % tiles;
  const int64_t m0 = (L % tilesM) * BM, n0 = (L / tilesM) * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WN) * C::WTM, wn0 = (wave % WN) * C::WTN;
  const int q = lane >> 4, r = lane & 15;

  const double2 *__restrict__ A = static_cast<const double2 *>(d.A);
  const double2 *__restrict__ B = static_cast<const double2 *>(d.B);
  const int64_t M = d.M, N = d.N;
  const int64_t kchunk = ((d.K + d.split - 1) / d.split + BK - 1) / BK * BK;
  const int64_t kb = ks * kchunk;
  const int64_t K = std::max<int64_t>(0, std::min<int64_t>(d.K - kb, kchunk));
  A += kb * d.sak;
  B += kb * d.sbk;

  double2 ra[C::LA], rb[C::LB];
  auto gload = [&](int64_t k0) {
#pragma unroll
    for (int i = 0; i < C::LA; ++i) {
      const int e = tid + i * C::NT;
      int mm, kk;
      if (AKC) { mm = e / BK; kk = e % BK; } else { kk = e / BM; mm = e % BM; }
      const int64_t gm = m0 + mm, gk = k0 + kk;
      ra[i] = (gm < M && gk < K) ? A[gm * d.sam + gk * d.sak] : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int i = 0; i < C::LB; ++i) {
      const int e = tid + i * C::NT;
      int nn, kk;
      if (BKC) { nn = e / BK; kk = e % BK; } else { kk = e / BN; nn = e % BN; }
      const int64_t gn = n0 + nn, gk = k0 + kk;
      rb[i] = (gn < N && gk < K) ? B[gn * d.sbn + gk * d.sbk] : make_double2(0.0, 0.0);
    }
  };
  auto sstore = [&](int buf) {
    double *ar = smem + buf * BUF, *ai = ar + C::A_ELEMS;
    double *br = ai + C::A_ELEMS, *bi = br + C::B_ELEMS;
#pragma unroll
    for (int i = 0; i < C::LA; ++i) {
      const int e = tid + i * C::NT;
      const int idx = AKC ? (e / BK) * C::A_LD + (e % BK) : (e / BM) * C::A_LD + (e % BM);
      ar[idx] = ra[i].x;
      ai[idx] = ra[i].y;
    }
#pragma unroll
    for (int i = 0; i < C::LB; ++i) {
      const int e = tid + i * C::NT;
      const int idx = BKC ? (e / BK) * C::B_LD + (e % BK) : (e / BN) * C::B_LD + (e % BN);
      br[idx] = rb[i].x;
      bi[idx] = rb[i].y;
    }
  };

  d4 acr[C::FM][C::FN], aci[C::FM][C::FN];
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
      acr[i][j] = d4{0.0, 0.0, 0.0, 0.0};
      aci[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    }

  const int64_t nk = (K + BK - 1) / BK;
  gload(0);
  sstore(0);
  __syncthreads();
  for (int64_t kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) gload((kt + 1) * BK);
    const double *ar = smem + buf * BUF, *ai = ar + C::A_ELEMS;
    const double *br = ai + C::A_ELEMS, *bi = br + C::B_ELEMS;
#pragma unroll
    for (int kc = 0; kc < BK; kc += 16) {
      double far_[C::FM][4], fai[C::FM][4], fbr[C::FN][4], fbi[C::FN][4];
#pragma unroll
      for (int i = 0; i < C::FM; ++i) {
        const int mm = wm0 + i * 16 + r;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int idx = AKC ? mm * C::A_LD + kc + 4 * q + s : (kc + 4 * q + s) * C::A_LD + mm;
          far_[i][s] = ar[idx];
          fai[i][s] = ai[idx];
        }
      }
#pragma unroll
      for (int j = 0; j < C::FN; ++j) {
        const int nn = wn0 + j * 16 + r;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int idx = BKC ? nn * C::B_LD + kc + 4 * q + s : (kc + 4 * q + s) * C::B_LD + nn;
          fbr[j][s] = br[idx];
          fbi[j][s] = bi[idx];
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
          for (int j = 0; j < C::FN; ++j) {
            acr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(far_[i][s], fbr[j][s], acr[i][j], 0, 0, 0);
            acr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-fai[i][s], fbi[j][s], acr[i][j], 0, 0, 0);
            aci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(far_[i][s], fbi[j][s], aci[i][j], 0, 0, 0);
            aci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fai[i][s], fbr[j][s], aci[i][j], 0, 0, 0);
          }
    }
    if (kt + 1 < nk) sstore(buf ^ 1);
    __syncthreads();
  }

  // accumulator t of lane l is row (l >> 4) + 4t, column l & 15 (f64 MFMA layout)
  double2 *__restrict__ Cp = static_cast<double2 *>(d.C);
  double alpha = d.alpha, beta = d.beta;
  int64_t ldc = d.ldc;
  if (d.split > 1) {
    Cp = static_cast<double2 *>(d.ws) + ks * M * N;
    alpha = 1.0;
    beta = 0.0;
    ldc = N;
  }
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
      const int64_t gn = n0 + wn0 + j * 16 + r;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t gm = m0 + wm0 + i * 16 + q + 4 * t;
        if (gm < M && gn < N) {
          double2 *p = Cp + gm * ldc + gn;
          double2 v = make_double2(alpha * acr[i][j][t], alpha * aci[i][j][t]);
          if (beta != 0.0) {
            const double2 o = *p;
            v.x += beta * o.x;
            v.y += beta * o.y;
          }
          *p = v;
        }
      }
    }
}

// ---- LDS-direct configurations (K chunk 16) ---------------------------------
// Both operands K-contiguous (the complex ladder's layout).  Each lane's 16
// bytes (one complex element) go straight into LDS with
// global_load_lds_dwordx4: two or three stages, one or two chunks of K in
// flight, no staging registers; elements past K load a zero in device memory.
// A 16-row block of a stage is four quarters of 64 slots; slot L of quarter s
// holds element (row L & 15, k = 4 (L >> 4) + s), the value lane L feeds the
// f64 MFMAs at step s (as in the staged kernel), so each quarter is read
// contiguously across the wave.  Rows past M or N load the last valid row
// instead: they only reach outputs that are never stored.  The products and
// their order are those of the staged kernels, so results are bitwise the
// same.  Waits as in the real LDS-direct kernel: "vmcnt <= LOADS" after the
// next chunk's loads, a barrier, and "lgkmcnt == 0" before it for the stage
// being overwritten.
__device__ __attribute__((aligned(16))) const double kZeroElement[2] = {0.0, 0.0};

template <int BM, int BN, int WM, int WN, int NST>
__global__ __launch_bounds__(WM *WN *kWave) void gemm_c128_dma_kernel(GemmDesc d, int64_t tilesM, int64_t tilesN) {
  constexpr int BK = 16, FM = BM / WM / 16, FN = BN / WN / 16;
  constexpr int A_EL = BM * BK, STAGE = (BM + BN) * BK;  // complex elements
  constexpr int LOADS = 4 * (BM / 16 + BN / 16) / (WM * WN);
  static_assert(4 * (BM / 16 + BN / 16) % (WM * WN) == 0, "whole loads per wave");
  static_assert(NST == 2 || NST == 3, "the explicit waits are written for one or two chunks in flight");
  __shared__ __attribute__((aligned(16))) double2 S[NST * STAGE];

  const int64_t tiles = tilesM * tilesN, total = tiles * d.split;
  const int64_t L0 = xcd_remap(blockIdx.x, total);
  const int64_t ks = L0 / tiles, L = L0 % tiles;
  const int64_t m0 = (L % tilesM) * BM, n0 = (L / tilesM) * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  const int q = lane >> 4, r = lane & 15;
  const int64_t M = d.M, N = d.N;
  const int64_t kchunk = ((d.K + d.split - 1) / d.split + BK - 1) / BK * BK;
  const int64_t kb = ks * kchunk;
  const int64_t K = std::max<int64_t>(0, std::min<int64_t>(d.K - kb, kchunk));
  // chunks, and whole ones (32-bit scalars, and running pointers advanced behind
  // the MFMAs, as in the real kernel: formed at the loads, the addresses cost
  // 1600 x 8000 x 8000 15.4 instead of 13.8 ms on 64 x 128, 400 x 2000 x 2001 360
  // instead of 313 us on 64 x 64)
  const int nk = __builtin_amdgcn_readfirstlane(int((K + BK - 1) / BK)), nf = __builtin_amdgcn_readfirstlane(int(K / BK));

  // load j of this wave (j = LOADS wave + u): block j >> 2 of the stage (A
  // before B), quarter j & 3; a block-quarter sits at elements
  // (blk * 4 + quarter) * 64 of the stage
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(S));
  const double2 *src[LOADS];  // of the next chunk to load
  uint32_t dst[LOADS];
  const double2 *Ag = static_cast<const double2 *>(d.A) + kb;
  const double2 *Bg = static_cast<const double2 *>(d.B) + kb;
  const int wv = __builtin_amdgcn_readfirstlane(wave);  // wave-uniform, so the choice below is too
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int j = LOADS * wv + u, blk = j >> 2;
    const bool isa = blk < BM / 16;
    const int64_t lim = isa ? M : N, want = isa ? m0 + blk * 16 + r : n0 + (blk - BM / 16) * 16 + r;
    const int64_t row = want < lim ? want : lim - 1;
    src[u] = (isa ? Ag + row * d.sam : Bg + row * d.sbn) + 4 * q + (j & 3);
    dst[u] = __builtin_amdgcn_readfirstlane(lds0 + 16u * uint32_t(j * 64));
  }
  auto issue = [&](int stage, int kt) {
    if (kt < nf) {
#pragma unroll
      for (int u = 0; u < LOADS; ++u) lds_load16(src[u], dst[u] + uint32_t(stage) * uint32_t(16 * STAGE));
    } else {  // the last, partial chunk: zeros past K
      const int left = int(K - int64_t(nf) * BK);
#pragma unroll
      for (int u = 0; u < LOADS; ++u)
        lds_load16(4 * q + ((LOADS * wv + u) & 3) < left ? static_cast<const void *>(src[u]) : kZeroElement,
                   dst[u] + uint32_t(stage) * uint32_t(16 * STAGE));
    }
  };
  auto advance = [&] {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) src[u] += BK;
  };

  d4 acr[FM][FN], aci[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      acr[i][j] = d4{0.0, 0.0, 0.0, 0.0};
      aci[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    }

  if (nk > 0) issue(0, 0);
  advance();
  if (NST == 3 && nk > 1) {
    issue(1, 1);
    advance();
  }
  int cur = 0, nxt = NST - 1;
  for (int kt = 0; kt < nk; ++kt) {
    if (NST == 3 && kt + 1 < nk) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (kt + NST - 1 < nk) issue(nxt, kt + NST - 1);
    const double2 *St = S + cur * STAGE;
    // steps 0-1 are read first and steps 2-3 behind the MFMAs of step 0, so
    // those reads overlap them (at most eight LDS reads in flight)
    double2 fa[FM][4], fb[FN][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (s == 0 || s == 2) {
        // the fragments of steps s and s + 1
#pragma unroll
        for (int t = s; t < s + 2; ++t) {
#pragma unroll
          for (int i = 0; i < FM; ++i) fa[i][t] = St[(((wm0 >> 4) + i) * 4 + t) * 64 + lane];
#pragma unroll
          for (int j = 0; j < FN; ++j) fb[j][t] = St[A_EL + (((wn0 >> 4) + j) * 4 + t) * 64 + lane];
        }
      }
      if (s <= 1) __builtin_amdgcn_sched_barrier(0);
      // (a branch in the 64 x 64 kernel: without it 1 to 8% slower; with one, 64 x 128 is 3%)
      if (s == 1 && (NST == 3 || FM * FN == 1 || kt + NST - 1 < nk)) advance();
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          acr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i][s].x, fb[j][s].x, acr[i][j], 0, 0, 0);
          acr[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-fa[i][s].y, fb[j][s].y, acr[i][j], 0, 0, 0);
          aci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i][s].x, fb[j][s].y, aci[i][j], 0, 0, 0);
          aci[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i][s].y, fb[j][s].x, aci[i][j], 0, 0, 0);
        }
      if (s == 0) __builtin_amdgcn_sched_barrier(0);
    }
    cur = cur == NST - 1 ? 0 : cur + 1;
    nxt = nxt == NST - 1 ? 0 : nxt + 1;
  }

  // epilogue (as the staged kernel): accumulator t of lane l is row (l >> 4) + 4t, column l & 15
  double2 *__restrict__ Cp = static_cast<double2 *>(d.C);
  double alpha = d.alpha, beta = d.beta;
  int64_t ldc = d.ldc;
  if (d.split > 1) {
    Cp = static_cast<double2 *>(d.ws) + ks * M * N;
    alpha = 1.0;
    beta = 0.0;
    ldc = N;
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int64_t gn = n0 + wn0 + j * 16 + r;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t gm = m0 + wm0 + i * 16 + q + 4 * t;
        if (gm < M && gn < N) {
          double2 *p = Cp + gm * ldc + gn;
          double2 v = make_double2(alpha * acr[i][j][t], alpha * aci[i][j][t]);
          if (beta != 0.0) {
            const double2 o = *p;
            v.x += beta * o.x;
            v.y += beta * o.y;
          }
          *p = v;
        }
      }
    }
}

bool c128_dma_ok(const GemmDesc &d) {
  return d.sak == 1 && d.sbk == 1 && d.K > 0 && (reinterpret_cast<uintptr_t>(d.A) & 15) == 0 &&
         (reinterpret_cast<uintptr_t>(d.B) & 15) == 0;
}

struct ZTile {
  const char *name;
  int BM, BN, BK;
  void (*launch[4])(const GemmDesc &, int64_t, int64_t, hipStream_t);
};

template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC>
void launch_z(const GemmDesc &d, int64_t tm, int64_t tn, hipStream_t s) {
  hipLaunchKernelGGL((gemm_c128_kernel<BM, BN, BK, WM, WN, AKC, BKC>), dim3(tm * tn * d.split),
                     dim3(WM * WN * kWave), 0, s, d, tm, tn);
}

#define CC_ZTILE(BM, BN, BK, WM, WN)                                                              \
  ZTile {                                                                                         \
    #BM "x" #BN "x" #BK "_w" #WM "x" #WN, BM, BN, BK,                                             \
        {&launch_z<BM, BN, BK, WM, WN, false, false>, &launch_z<BM, BN, BK, WM, WN, false, true>, \
         &launch_z<BM, BN, BK, WM, WN, true, false>, &launch_z<BM, BN, BK, WM, WN, true, true>}   \
  }

template <int BM, int BN, int WM, int WN, int NST>
void launch_z_dma(const GemmDesc &d, int64_t tm, int64_t tn, hipStream_t s) {
  if (c128_dma_ok(d))
    hipLaunchKernelGGL((gemm_c128_dma_kernel<BM, BN, WM, WN, NST>), dim3(tm * tn * d.split), dim3(WM * WN * kWave), 0,
                       s, d, tm, tn);
  else
    launch_z<BM, BN, 16, WM, WN, true, true>(d, tm, tn, s);
}

// LDS-direct where the layout allows, else the staged kernel of the tile
#define CC_ZTILE_DMA(BM, BN, WM, WN, NST, NAME)                                                   \
  ZTile {                                                                                         \
    #BM "x" #BN "x16_w" #WM "x" #WN NAME, BM, BN, 16,                                             \
        {&launch_z<BM, BN, 16, WM, WN, false, false>, &launch_z<BM, BN, 16, WM, WN, false, true>, \
         &launch_z<BM, BN, 16, WM, WN, true, false>, &launch_z_dma<BM, BN, WM, WN, NST>}          \
  }

const ZTile kZTiles[] = {CC_ZTILE(64, 64, 16, 2, 2), CC_ZTILE(32, 32, 16, 2, 2), CC_ZTILE(128, 64, 16, 2, 2),
                         CC_ZTILE(64, 128, 16, 2, 2),
                         CC_ZTILE_DMA(64, 128, 2, 4, 3, "_lds"),
                         CC_ZTILE_DMA(64, 64, 4, 2, 2, "_lds2"),
                         CC_ZTILE_DMA(32, 32, 2, 2, 2, "_lds2")};
constexpr int kNumZ = sizeof(kZTiles) / sizeof(kZTiles[0]);

// The same kind of model as the real FP64 one (F64Tile), fitted to the
// timings of every configuration and split-K factor on the 139 GEMM shapes of
// complex CCSD at o = 4..20, v = 20..90: on them its choice is 1.3% slower
// than the fastest, and 1.33 times faster than the rule it replaced (rounds of
// 512 workgroups x tile area over a split chosen for 64 x 64 tiles):
// 1600 x 8000 x 8000 17.1 -> 12.4 ms, 256 x 6400 x 6400 1.55 -> 1.33 ms,
// 1280^3 359 -> 291 us.
constexpr int kZBig = 5, kZSmall = 6;  // 64x64 and 32x32 (LDS-direct, or their staged kernels)
// per operand form (0: M/N-contiguous, 1: LDS-direct): MFMA share of the 64x64
// and the 32x32 tile, cycles of one chunk alone, cycles per workgroup set
// (fixed; per 1,024 outputs), HBM TB/s, microseconds and TB/s of the partial
// sums, share of the shorter time that is not hidden
constexpr double kZConst[2][9] = {{0.80, 0.70, 2493, 32, 595, 5.28, 4.94, 13.5, 0.35},
                                  {0.77, 0.71, 1584, 353, 60, 8.09, 3.02, 8.7, 0.23}};

double c128_model_us(int tile, int form, int64_t M, int64_t N, int64_t K, int64_t split) {
  const ZTile &ti = kZTiles[tile];
  const double *c = kZConst[form];
  const bool big = tile == kZBig;
  const int64_t n = ((K + split - 1) / split + 15) / 16;
  const double area = double(ti.BM) * ti.BN;
  const double wgs = double((M + ti.BM - 1) / ti.BM) * double((N + ti.BN - 1) / ti.BN) * double(split);
  const double w = std::ceil(wgs / 256.0), conc = std::min(w, big ? 2.0 : form ? 5.0 : 4.0);
  const double chunk = std::max(conc * area / c[big ? 0 : 1], c[2]);
  const double mfma = (w / conc) * (double(n) * chunk + c[3] + c[4] * area / 1024.0 * conc) / 2400.0;
  const double mem = (double(M) * K + double(N) * K + (split == 1 ? 2.0 * double(M) * N : 0.0)) * 16.0 / c[5] * 1e-6;
  const double red = split > 1 ? c[6] + 32.0 * double(split) * double(M) * N / c[7] * 1e-6 : 0.0;
  return 3.0 + std::max(mfma, mem) + c[8] * std::min(mfma, mem) + red;
}

}  // namespace

int gemm_c128_num_tiles() { return kNumZ; }
const char *gemm_c128_tile_name(int id) { return (id >= 0 && id < kNumZ) ? kZTiles[id].name : "?"; }

F64Choice gemm_c128_choose(int64_t M, int64_t N, int64_t K, bool lds_direct, int64_t ws_elems) {
  static constexpr int kSplits[] = {1, 2, 3, 4, 5, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512};
  F64Choice best{kZSmall, 1};
  double best_us = 1e300;
  for (int t : {kZBig, kZSmall}) {
    const ZTile &ti = kZTiles[t];
    const int64_t tiles = ((M + ti.BM - 1) / ti.BM) * ((N + ti.BN - 1) / ti.BN);
    for (int s : kSplits) {
      if (s > 1 && (int64_t(s) * 64 > K || tiles * s > 4096 || int64_t(s) * M * N > ws_elems)) break;
      const double us = c128_model_us(t, lds_direct ? 1 : 0, M, N, K, s);
      if (us < best_us) {
        best_us = us;
        best = F64Choice{t, s};
      }
    }
  }
  return best;
}

void gemm_c128(const GemmDesc &d0, hipStream_t s, int tile_id) {
  GemmDesc d = d0;
  if (d.M <= 0 || d.N <= 0) return;
  const bool akc = (d.sak == 1), bkc = (d.sbk == 1);
  CC_REQUIRE(akc || d.sam == 1, -1, "gemm: A needs a unit stride in m or k");
  CC_REQUIRE(bkc || d.sbn == 1, -1, "gemm: B needs a unit stride in n or k");
  CC_REQUIRE(d.conj_a == 0 && d.conj_b == 0, -7, "gemm_c128: conjugated operands are planned as views");
  if (d.K <= 0) {
    PermDesc p{};
    p.rank = 2;
    p.out_dims[0] = d.M;
    p.out_dims[1] = d.N;
    p.out_strides[0] = d.ldc;
    p.out_strides[1] = 1;
    p.in_strides[0] = d.ldc;
    p.in_strides[1] = 1;
    p.alpha = d.beta;
    permute_c128(p, d.C, d.C, s);
    return;
  }
  if (tile_id < 0 || tile_id >= kNumZ) {
    const F64Choice ch = gemm_c128_choose(
        d.M, d.N, d.K, c128_dma_ok(d), d.split > 1 && d.ws ? (d.ws_elems > 0 ? d.ws_elems : d.split * d.M * d.N) : 0);
    tile_id = ch.tile;
    d.split = ch.split;
  }
  const ZTile &ti = kZTiles[tile_id];
  const int64_t tm = (d.M + ti.BM - 1) / ti.BM, tn = (d.N + ti.BN - 1) / ti.BN;
  CC_REQUIRE(d.split >= 1 && (d.split == 1 || d.ws != nullptr), -1, "gemm: split-K workspace");
  CC_REQUIRE(tm * tn * d.split < (int64_t(1) << 31), -1, "gemm: too many tiles");
  ti.launch[(akc ? 2 : 0) + (bkc ? 1 : 0)](d, tm, tn, s);
  CC_HIP_CHECK(hipGetLastError());
  if (d.split > 1) splitk_reduce(true, d.ws, d.split, d.M, d.N, d.C, d.ldc, d.alpha, d.beta, s);
}

}  // namespace ccmi
