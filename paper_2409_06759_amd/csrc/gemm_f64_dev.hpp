// Device bodies of the FP64 MFMA GEMM (register-staged and LDS-direct tiles),
// shared by its own kernels and by the merged launches of small systems.
#pragma once

#include "common.hpp"

#include <algorithm>
#include <type_traits>

namespace ccmi {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC>
struct Cfg {
  static constexpr int NT = WM * WN * kWave;
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int FM = WTM / 16, FN = WTN / 16;
  static constexpr int PAD = 2;
  // LDS panel shapes (rows x row-stride) per operand
  static constexpr int A_ROWS = AKC ? BM : BK, A_LD = AKC ? BK + PAD : BM + PAD;
  static constexpr int B_ROWS = BKC ? BN : BK, B_LD = BKC ? BK + PAD : BN + PAD;
  static constexpr int A_ELEMS = A_ROWS * A_LD, B_ELEMS = B_ROWS * B_LD;
  static constexpr int LA = BM * BK / NT, LB = BN * BK / NT;  // global loads per thread
  static_assert(BM % (16 * WM) == 0 && BN % (16 * WN) == 0, "tile/wave mismatch");
  static_assert(BK % 16 == 0, "BK must be a multiple of 16");
  static_assert((BM * BK) % NT == 0 && (BN * BK) % NT == 0, "load split");
};

// One workgroup's share of a GEMM: logical tile L0 in [0, tiles * split).
template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC>
__device__ __forceinline__ void gemm_f64_body(const GemmDesc &d, int64_t tilesM, int64_t tilesN,
                                              int64_t L0, double *smem) {
  using C = Cfg<BM, BN, BK, WM, WN, AKC, BKC>;
  // buffer b of A at smem + b*A_ELEMS, of B at smem + 2*A_ELEMS + b*B_ELEMS

  const TileAt at = tile_at(L0, tilesM, tilesN, d.split);
  const int64_t ks = at.ks, m0 = at.m * BM, n0 = at.n * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WN) * C::WTM, wn0 = (wave % WN) * C::WTN;
  const int q = lane >> 4, r = lane & 15;

  const double *__restrict__ A = static_cast<const double *>(d.A);
  const double *__restrict__ B = static_cast<const double *>(d.B);
  const int64_t M = d.M, N = d.N;
  // split-K: this workgroup covers k in [kb, kb + K) of the full range
  const int64_t kchunk = k_slice(d.K, d.split, BK);
  const int64_t kb = ks * kchunk;
  const int64_t K = std::max<int64_t>(0, std::min<int64_t>(d.K - kb, kchunk));
  A += kb * d.sak;
  B += kb * d.sbk;

  // Global -> register staging in 16-byte vectors (two doubles along the
  // unit-stride dimension; global loads need only 8-byte alignment), the last
  // element of an odd row on its own.  Out-of-range elements are 0.
  constexpr int AR = AKC ? BM : BK, AC = AKC ? BK : BM, BR = BKC ? BN : BK, BC = BKC ? BK : BN;
  constexpr int ANV = AR * AC / 2, BNV = BR * BC / 2;
  constexpr int AVT = (ANV + C::NT - 1) / C::NT, BVT = (BNV + C::NT - 1) / C::NT;
  typedef double d2 __attribute__((ext_vector_type(2)));
  typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
  d2 ra[AVT], rb[BVT];

  auto vload = [&](const double *base, int64_t rstride, int64_t r_lim, int64_t c_lim, int64_t r0, int64_t c0, int v,
                   int ncolv) -> d2 {
    const int rr = v / ncolv, cc = (v % ncolv) * 2;
    const int64_t gr = r0 + rr, gc = c0 + cc;
    const double *src = base + gr * rstride + gc;
    if (gr < r_lim && gc + 2 <= c_lim) return *reinterpret_cast<const d2u *>(src);
    d2 t;
    t.x = (gr < r_lim && gc < c_lim) ? src[0] : 0.0;
    t.y = 0.0;
    return t;
  };
  auto gload = [&](int64_t k0) {
#pragma unroll
    for (int i = 0; i < AVT; ++i) {
      const int v = tid + i * C::NT;
      if (ANV % C::NT == 0 || v < ANV)
        ra[i] = AKC ? vload(A, d.sam, M, K, m0, k0, v, AC / 2) : vload(A, d.sak, K, M, k0, m0, v, AC / 2);
    }
#pragma unroll
    for (int i = 0; i < BVT; ++i) {
      const int v = tid + i * C::NT;
      if (BNV % C::NT == 0 || v < BNV)
        rb[i] = BKC ? vload(B, d.sbn, N, K, n0, k0, v, BC / 2) : vload(B, d.sbk, K, N, k0, n0, v, BC / 2);
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < AVT; ++i) {
      const int v = tid + i * C::NT;
      if (ANV % C::NT == 0 || v < ANV) {
        const int rr = v / (AC / 2), cc = (v % (AC / 2)) * 2;
        *reinterpret_cast<d2 *>(smem + buf * C::A_ELEMS + rr * C::A_LD + cc) = ra[i];
      }
    }
#pragma unroll
    for (int i = 0; i < BVT; ++i) {
      const int v = tid + i * C::NT;
      if (BNV % C::NT == 0 || v < BNV) {
        const int rr = v / (BC / 2), cc = (v % (BC / 2)) * 2;
        *reinterpret_cast<d2 *>(smem + 2 * C::A_ELEMS + buf * C::B_ELEMS + rr * C::B_LD + cc) = rb[i];
      }
    }
  };

  d4 acc[C::FM][C::FN];
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  const int64_t nk = (K + BK - 1) / BK;
  gload(0);
  sstore(0);
  __syncthreads();
  for (int64_t kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) gload((kt + 1) * BK);
    const double *as = smem + buf * C::A_ELEMS, *bs = smem + 2 * C::A_ELEMS + buf * C::B_ELEMS;
#pragma unroll
    for (int kc = 0; kc < BK; kc += 16) {
      double fa[C::FM][4], fb[C::FN][4];
#pragma unroll
      for (int i = 0; i < C::FM; ++i) {
        const int mm = wm0 + i * 16 + r;
#pragma unroll
        for (int s = 0; s < 4; ++s)
          fa[i][s] = AKC ? as[mm * C::A_LD + kc + 4 * q + s] : as[(kc + 4 * q + s) * C::A_LD + mm];
      }
#pragma unroll
      for (int j = 0; j < C::FN; ++j) {
        const int nn = wn0 + j * 16 + r;
#pragma unroll
        for (int s = 0; s < 4; ++s)
          fb[j][s] = BKC ? bs[nn * C::B_LD + kc + 4 * q + s] : bs[(kc + 4 * q + s) * C::B_LD + nn];
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
          for (int j = 0; j < C::FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i][s], fb[j][s], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) sstore(buf ^ 1);
    __syncthreads();
  }

  // epilogue: accumulator t of lane l holds row (l >> 4) + 4t, column l & 15
  // of its 16x16 block (f64 MFMA output layout, checked on the device)
  double *__restrict__ Cp = static_cast<double *>(d.C);
  double alpha = d.alpha, beta = d.beta;
  int64_t ldc = d.ldc;
  if (d.split > 1) {  // raw partial sums; splitk_reduce applies alpha and beta
    Cp = static_cast<double *>(d.ws) + ks * M * N;
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
          double *p = Cp + gm * ldc + gn;
          const double v = alpha * acc[i][j][t];
          *p = (beta == 0.0) ? v : v + beta * *p;
        }
      }
    }
}

// ---- LDS-direct configurations (K chunk 16) ---------------------------------
// Both operands K-contiguous (the particle-particle ladder's layout); the
// rows need no alignment beyond their elements' (global loads take any dword
// address).  Rows past M or N load the last valid row instead, which only
// reaches outputs that are never stored, and k pairs past K load zeros from a
// zero pair in device memory.  The last k of an odd K has no pair: its lanes
// load zeros too, and write the element over the first of them once the chunk
// has landed.  Odd K took the staged kernels before: 169 x 3721 x 3721
// went from 188 to 113 us (41 TF, as at K = 3720).  Each lane's 16
// bytes go straight from HBM/L2 into LDS (global_load_lds_dwordx4): no
// staging registers, two or three LDS stages, one or two chunks of K in flight.  A 16-row
// block of a stage is two halves of 64 slots of 16 bytes; slot L of half h
// holds row (L & 15), k = 4 (L >> 4) + 2h + {0, 1}, so lane L reads the four
// k values it feeds the f64 MFMA (k = 4q + s, as in the staged kernel) as
// two 16-byte reads, each contiguous across the wave (no bank conflicts).  The
// products and their order are those of the staged kernel of the same tile,
// so results are bitwise the same.  Waits: "vmcnt <= LOADS" after the loads
// of chunk kt+1 means chunk kt has landed (in-order completion), the barrier
// behind it makes that so for every wave, and "lgkmcnt == 0" before it
// means every wave has finished reading the stage the next loads overwrite.
__device__ __attribute__((aligned(16))) const double kZeroPair[2] = {0.0, 0.0};

template <int BM, int BN, int WM, int WN, int NST>
struct Dma64 {
  static constexpr int BK = 16, NT = WM * WN * kWave;
  static constexpr int FM = BM / WM / 16, FN = BN / WN / 16;
  static constexpr int A_EL = BM * BK, STAGE = (BM + BN) * BK;  // doubles
  static constexpr int NSTAGE = NST, ELEMS = NSTAGE * STAGE;
  static constexpr int LOADS = 2 * (BM / 16 + BN / 16) / (WM * WN);  // 1 KiB loads per wave and chunk
  static_assert(2 * (BM / 16 + BN / 16) % (WM * WN) == 0, "whole loads per wave");
  static_assert(BM % (16 * WM) == 0 && BN % (16 * WN) == 0, "tile/wave mismatch");
};

// ODD: K may be odd (of its own: the element's registers cost the 256 x 128
// tile 3% of its rate).
template <int BM, int BN, int WM, int WN, int NST, bool ODD>
__device__ __forceinline__ void gemm_f64_dma_body(const GemmDesc &d, int64_t tilesM, int64_t tilesN, int64_t L0,
                                                  double *S) {
  using C = Dma64<BM, BN, WM, WN, NST>;
  constexpr int BK = C::BK, FM = C::FM, FN = C::FN, A_EL = C::A_EL, STAGE = C::STAGE, NSTAGE = C::NSTAGE,
                LOADS = C::LOADS;
  const TileAt at = tile_at(L0, tilesM, tilesN, d.split);
  const int64_t ks = at.ks, m0 = at.m * BM, n0 = at.n * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  const int q = lane >> 4, r = lane & 15;
  const int64_t M = d.M, N = d.N;
  const int64_t kchunk = k_slice(d.K, d.split, BK);
  const int64_t kb = ks * kchunk;
  const int64_t K = std::max<int64_t>(0, std::min<int64_t>(d.K - kb, kchunk));
  constexpr bool RUN = FM * FN > 1;
  using Int = std::conditional_t<RUN, int, int64_t>;
  const Int nk = RUN ? Int(__builtin_amdgcn_readfirstlane(int((K + BK - 1) / BK))) : Int((K + BK - 1) / BK);
  const int nf = RUN ? __builtin_amdgcn_readfirstlane(int(K / BK)) : 0;

  // this wave's loads: LOADS of the stage's half blocks (16 rows x 8 k),
  // numbered with the A blocks first; lane l of half h loads row (l & 15),
  // k = 4 (l >> 4) + 2h + {0, 1}
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(S));
  const double *src[LOADS];  // of the next chunk to load (RUN), else of the first
  uint32_t dst[LOADS];
  const double *Ag = static_cast<const double *>(d.A) + kb;
  const double *Bg = static_cast<const double *>(d.B) + kb;
  auto kof = [&](int u) { return 4 * q + 2 * ((wave * LOADS + u) & 1); };
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int x = wave * LOADS + u, blk = x >> 1, h = x & 1;
    src[u] = (blk < BM / 16 ? Ag + std::min<int64_t>(m0 + blk * 16 + r, M - 1) * d.sam
                            : Bg + std::min<int64_t>(n0 + (blk - BM / 16) * 16 + r, N - 1) * d.sbn) +
             kof(u);
    dst[u] = __builtin_amdgcn_readfirstlane(lds0 + 8u * uint32_t(blk * 256 + h * 128));
  }
  auto issue = [&](int stage, Int kt) {
    const int64_t k0 = RUN ? 0 : int64_t(kt) * BK;
    if (RUN ? kt < nf : k0 + BK <= K) {
#pragma unroll
      for (int u = 0; u < LOADS; ++u) lds_load16(src[u] + k0, dst[u] + uint32_t(stage) * uint32_t(8 * STAGE));
    } else {  // the last, partial chunk: zeros past K
      const int64_t left = RUN ? K - int64_t(nf) * BK : K - k0;
#pragma unroll
      for (int u = 0; u < LOADS; ++u)
        lds_load16(kof(u) + 1 < left ? src[u] + k0 : kZeroPair, dst[u] + uint32_t(stage) * uint32_t(8 * STAGE));
    }
  };
  auto advance = [&] {
    if (!RUN) return;
#pragma unroll
    for (int u = 0; u < LOADS; ++u) src[u] += BK;
  };

  d4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  static_assert(NST == 2 || NST == 3, "the explicit waits are written for one or two chunks in flight");
  // odd K: the last element of the rows this lane loads, fetched up front
  const bool oddk = ODD && (K & 1) != 0;
  const int64_t kl = int64_t(nk - 1) * BK;  // its chunk
  const int odd_at = int(K - 1 - kl);       // its place there
  double last[LOADS];
  if (oddk) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) last[u] = kof(u) == odd_at ? src[u][kl] : 0.0;
  }
  if (nk > 0) issue(0, 0);
  advance();
  if (NST == 3 && nk > 1) {
    issue(1, 1);
    advance();
  }
  int cur = 0, nxt = NST - 1;
  for (Int kt = 0; kt < nk; ++kt) {
    if (NST == 3 && kt + 1 < nk) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (kt + NST - 1 < nk) issue(nxt, kt + NST - 1);
    if (oddk && kt == nk - 1) {
#pragma unroll
      for (int u = 0; u < LOADS; ++u)
        if (kof(u) == odd_at) S[cur * STAGE + ((dst[u] - lds0) >> 3) + 2 * lane] = last[u];
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    const double *St = S + cur * STAGE;
    // the k pair of steps 0-1 of every fragment is read first; the pair of
    // steps 2-3 is read behind the MFMAs of step 0, so it overlaps them (at
    // most eight LDS reads in flight, within what lgkmcnt can count)
    typedef double d2 __attribute__((ext_vector_type(2)));
    d2 fa[2][FM], fb[2][FN];
    auto read_pair = [&](int h) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[h][i] = *reinterpret_cast<const d2 *>(St + ((wm0 >> 4) + i) * 256 + h * 128 + lane * 2);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        fb[h][j] = *reinterpret_cast<const d2 *>(St + A_EL + ((wn0 >> 4) + j) * 256 + h * 128 + lane * 2);
    };
    auto mfma_step = [&](int s) {
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[s >> 1][i][s & 1], fb[s >> 1][j][s & 1], acc[i][j],
                                                           0, 0, 0);
    };
    read_pair(0);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step(0);
    __builtin_amdgcn_sched_barrier(0);
    read_pair(1);
    __builtin_amdgcn_sched_barrier(0);
    advance();
    mfma_step(1);
    mfma_step(2);
    mfma_step(3);
    cur = cur == NSTAGE - 1 ? 0 : cur + 1;
    nxt = nxt == NSTAGE - 1 ? 0 : nxt + 1;
  }

  // epilogue (as the staged kernel): accumulator t of lane l holds row
  // (l >> 4) + 4t, column l & 15 of its 16x16 block
  double *__restrict__ Cp = static_cast<double *>(d.C);
  double alpha = d.alpha, beta = d.beta;
  int64_t ldc = d.ldc;
  if (d.split > 1) {
    Cp = static_cast<double *>(d.ws) + ks * M * N;
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
          double *p = Cp + gm * ldc + gn;
          const double v = alpha * acc[i][j][t];
          *p = (beta == 0.0) ? v : v + beta * *p;
        }
      }
    }
}

}  // namespace
}  // namespace ccmi
