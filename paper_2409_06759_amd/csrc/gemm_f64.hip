// FP64 MFMA GEMM for gfx950:  C[m][n] = alpha * sum_k A(m,k) B(n,k) + beta * C[m][n].
//
// This is the GEMM step of the transpose-transpose-GEMM-transpose evaluation
// of a binary tensor contraction (paper, Sec. "Tensor contractions"); the
// particle-particle ladder R_ij^ab += 1/2 sum_ef tau_ij^ef <ab||ef> is one call
// with A = tau[(ij)][(ef)] and B = vvvv[(ab)][(ef)], both K-contiguous.
//
// Design (CDNA4):
// * v_mfma_f64_16x16x4_f64: each lane holds one A and one B value and four
//   accumulators.  Lane l covers row (l & 15) of A / column (l & 15) of B and
//   k-slot (l >> 4); accumulator t of lane l is C[(l >> 4) + 4t][l & 15].
//   Four consecutive MFMAs consume 16 k values: in MFMA s lane group
//   q = l >> 4 supplies logical k = 4q + s, identically for A and B, so each
//   lane reads 4 consecutive k of its row when the operand is K-contiguous.
// * Staged configurations: block tile BM x BN, K chunk BK, staged through LDS
//   with two buffers; the next chunk's global loads are in flight (in
//   registers) while the current one is multiplied.  Operands may be
//   K-contiguous or M/N-contiguous; the LDS layout follows the global one so
//   both the HBM reads and the LDS fragment reads stay unit-stride.
// * The LDS-direct configurations take K-contiguous operands with
//   global_load_lds_dwordx4 into two or three LDS stages (see their kernel).
// * Workgroup ids are remapped so that the M tiles sharing one N tile are
//   dispatched to the same XCD (shared L2 for the B panel).
// * A launch whose last round of resident workgroups would be at most half
//   full runs as whole rounds plus a K-split tail (gemm_tail_cut).  Tile and
//   split-K factor come from a model of the time (gemm_f64_choose); a tile the
//   autotuner finds faster gets its factor from gemm_split_refine.
#include "common.hpp"
#include "gemm_f64_dev.hpp"
#include "kernels.hpp"

#include <algorithm>
#include <atomic>
#include <mutex>

#include <cmath>

namespace ccmi {
namespace {

template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC, int TAG>
__global__ __launch_bounds__(WM *WN *kWave) void gemm_f64_kernel(GemmDesc d, int64_t tilesM,
                                                                  int64_t tilesN) {
  using C = Cfg<BM, BN, BK, WM, WN, AKC, BKC>;
  __shared__ __attribute__((aligned(16))) double smem[2 * (C::A_ELEMS + C::B_ELEMS)];
  const int64_t total = tilesM * tilesN * d.split;
  gemm_f64_body<BM, BN, BK, WM, WN, AKC, BKC>(d, tilesM, tilesN, xcd_remap(blockIdx.x, total), smem);
}

// Grouped launch: one workgroup range per system; system b owns logical
// tiles [g.off[b], g.off[b+1]).  Same arithmetic as the single launch.
template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC>
__global__ __launch_bounds__(WM *WN *kWave) void gemm_f64_grouped(const GemmGroupEntry *__restrict__ e,
                                                                   const int64_t *__restrict__ off, int n) {
  using C = Cfg<BM, BN, BK, WM, WN, AKC, BKC>;
  __shared__ __attribute__((aligned(16))) double smem[2 * (C::A_ELEMS + C::B_ELEMS)];
  const int b = group_find(off, n, blockIdx.x);
  const GemmGroupEntry &g = e[b];
  gemm_f64_body<BM, BN, BK, WM, WN, AKC, BKC>(g.d, g.tilesM, g.tilesN, int64_t(blockIdx.x) - off[b], smem);
}

template <int BM, int BN, int WM, int WN, int NST, int TAG, bool ODD>
__global__ __launch_bounds__(WM *WN *kWave) void gemm_f64_dma_kernel(GemmDesc d, int64_t tilesM, int64_t tilesN) {
  __shared__ __attribute__((aligned(16))) double S[Dma64<BM, BN, WM, WN, NST>::ELEMS];
  gemm_f64_dma_body<BM, BN, WM, WN, NST, ODD>(d, tilesM, tilesN, xcd_remap(blockIdx.x, tilesM * tilesN * d.split), S);
}

template <int BM, int BN, int WM, int WN, int NST>
__global__ __launch_bounds__(WM *WN *kWave) void gemm_f64_dma_grouped(const GemmGroupEntry *__restrict__ e,
                                                                      const int64_t *__restrict__ off, int n) {
  __shared__ __attribute__((aligned(16))) double S[Dma64<BM, BN, WM, WN, NST>::ELEMS];
  const int b = group_find(off, n, blockIdx.x);
  const GemmGroupEntry &g = e[b];
  gemm_f64_dma_body<BM, BN, WM, WN, NST, true>(g.d, g.tilesM, g.tilesN, int64_t(blockIdx.x) - off[b], S);
}

struct TileInfo {
  const char *name;
  int BM, BN, BK, threads;
  void (*launch[4])(const GemmDesc &, int64_t, int64_t, hipStream_t);  // [akc*2 + bkc]
  void (*launch_ladder)(const GemmDesc &, int64_t, int64_t, hipStream_t);  // both K-contiguous
  void (*launch_ladder_tail)(const GemmDesc &, int64_t, int64_t, hipStream_t);
  void (*launch_grouped[4])(const GemmGroupEntry *, const int64_t *, int, int64_t, hipStream_t);
  int (*occupancy[4])();  // resident workgroups per CU, [akc*2 + bkc]
};

// Workgroups of one configuration that fit on a CU at once (registers, LDS,
// waves), as the runtime computes it for the compiled kernel; 0 if unknown.
template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC>
int occupancy_cfg() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f64_kernel<BM, BN, BK, WM, WN, AKC, BKC, 0>,
                                                   WM * WN * kWave, 0) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return nb;
}

template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC>
void launch_grp(const GemmGroupEntry *e, const int64_t *off, int n, int64_t blocks, hipStream_t s) {
  hipLaunchKernelGGL((gemm_f64_grouped<BM, BN, BK, WM, WN, AKC, BKC>), dim3(blocks), dim3(WM * WN * kWave),
                     0, s, e, off, n);
}

// TAG only changes the kernel's symbol name: TAG 1 is the particle-particle
// ladder and TAG 2 the K-split tail of a cut ladder launch, so that profilers
// report them on lines of their own.
template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC, int TAG = 0>
void launch_cfg(const GemmDesc &d, int64_t tm, int64_t tn, hipStream_t s) {
  hipLaunchKernelGGL((gemm_f64_kernel<BM, BN, BK, WM, WN, AKC, BKC, TAG>), dim3(tm * tn * d.split),
                     dim3(WM * WN * kWave), 0, s, d, tm, tn);
}

#define CC_TILE(BM, BN, BK, WM, WN)                                                          \
  TileInfo {                                                                                 \
    #BM "x" #BN "x" #BK "_w" #WM "x" #WN, BM, BN, BK, WM *WN * kWave, {                      \
      &launch_cfg<BM, BN, BK, WM, WN, false, false>, &launch_cfg<BM, BN, BK, WM, WN, false, true>, \
          &launch_cfg<BM, BN, BK, WM, WN, true, false>, &launch_cfg<BM, BN, BK, WM, WN, true, true> \
    }, &launch_cfg<BM, BN, BK, WM, WN, true, true, 1>, &launch_cfg<BM, BN, BK, WM, WN, true, true, 2>, \
    {&launch_grp<BM, BN, BK, WM, WN, false, false>, &launch_grp<BM, BN, BK, WM, WN, false, true>, \
     &launch_grp<BM, BN, BK, WM, WN, true, false>, &launch_grp<BM, BN, BK, WM, WN, true, true>},  \
    {&occupancy_cfg<BM, BN, BK, WM, WN, false, false>, &occupancy_cfg<BM, BN, BK, WM, WN, false, true>, \
     &occupancy_cfg<BM, BN, BK, WM, WN, true, false>, &occupancy_cfg<BM, BN, BK, WM, WN, true, true>} \
  }

template <int BM, int BN, int WM, int WN, int NST, int TAG>
void launch_f64_dma(const GemmDesc &d, int64_t tm, int64_t tn, hipStream_t s) {
  const dim3 grid(tm * tn * d.split), block(WM * WN * kWave);
  if (d.K & 1) hipLaunchKernelGGL((gemm_f64_dma_kernel<BM, BN, WM, WN, NST, TAG, true>), grid, block, 0, s, d, tm, tn);
  else hipLaunchKernelGGL((gemm_f64_dma_kernel<BM, BN, WM, WN, NST, TAG, false>), grid, block, 0, s, d, tm, tn);
}
template <int BM, int BN, int WM, int WN, int NST>
int occ_f64_dma() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f64_dma_kernel<BM, BN, WM, WN, NST, 0, false>, WM * WN * kWave, 0) !=
      hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return nb;
}
template <int BM, int BN, int WM, int WN, int NST>
void launch_grp_dma(const GemmGroupEntry *e, const int64_t *off, int n, int64_t blocks, hipStream_t s) {
  hipLaunchKernelGGL((gemm_f64_dma_grouped<BM, BN, WM, WN, NST>), dim3(blocks), dim3(WM * WN * kWave), 0, s, e, off, n);
}

// LDS-direct where both operands are K-contiguous, else the staged kernel of the tile
#define CC_TILE_DMA(BM, BN, WM, WN, NST, NAME)                                                                              \
  TileInfo {                                                                                                     \
    #BM "x" #BN "x16_w" #WM "x" #WN NAME, BM, BN, 16, WM *WN * kWave, {                                        \
      &launch_cfg<BM, BN, 16, WM, WN, false, false>, &launch_cfg<BM, BN, 16, WM, WN, false, true>,               \
          &launch_cfg<BM, BN, 16, WM, WN, true, false>, &launch_f64_dma<BM, BN, WM, WN, NST, 0>                       \
    }, &launch_f64_dma<BM, BN, WM, WN, NST, 1>, &launch_f64_dma<BM, BN, WM, WN, NST, 2>,                                   \
    {&launch_grp<BM, BN, 16, WM, WN, false, false>, &launch_grp<BM, BN, 16, WM, WN, false, true>,                \
     &launch_grp<BM, BN, 16, WM, WN, true, false>, &launch_grp_dma<BM, BN, WM, WN, NST>},                             \
    {&occupancy_cfg<BM, BN, 16, WM, WN, false, false>, &occupancy_cfg<BM, BN, 16, WM, WN, false, true>,          \
     &occupancy_cfg<BM, BN, 16, WM, WN, true, false>, &occ_f64_dma<BM, BN, WM, WN, NST>}                              \
  }

const TileInfo kTiles[] = {
    CC_TILE(128, 128, 16, 2, 2),
    CC_TILE(128, 160, 16, 2, 2),
    CC_TILE(64, 64, 16, 2, 2),
    CC_TILE(32, 32, 16, 2, 2),
    CC_TILE(256, 128, 16, 4, 2),
    CC_TILE(128, 64, 16, 2, 2),
    CC_TILE(64, 128, 16, 2, 2),
    CC_TILE(128, 128, 32, 2, 2),
    CC_TILE(64, 64, 32, 2, 2),
    CC_TILE(128, 64, 32, 2, 2),
    CC_TILE(64, 128, 32, 2, 2),
    CC_TILE(128, 128, 16, 4, 2),
    CC_TILE(128, 64, 16, 4, 2),
    CC_TILE(64, 128, 16, 2, 4),
    CC_TILE(128, 128, 16, 4, 4),
    CC_TILE(256, 64, 16, 8, 2),
    CC_TILE_DMA(256, 128, 4, 2, 3, "_lds"),
    CC_TILE_DMA(64, 128, 2, 4, 2, "_lds2"),
    CC_TILE_DMA(32, 32, 2, 2, 3, "_lds"),
    CC_TILE_DMA(64, 64, 4, 2, 3, "_lds"),
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// resident slots of a configuration on the whole device (cached per process,
// which assumes every device it uses is the same GPU model; -1 = not yet asked)
std::atomic<int64_t> g_slots[kNumTiles][4];
std::once_flag g_slots_once;

int64_t tile_slots(int tile_id, int variant) {
  std::call_once(g_slots_once, [] {
    for (auto &row : g_slots)
      for (auto &x : row) x.store(-1);
  });
  int64_t v = g_slots[tile_id][variant].load();
  if (v < 0) {
    v = int64_t(kTiles[tile_id].occupancy[variant]()) * gpu_cu_count();
    g_slots[tile_id][variant].store(v);
  }
  return v;
}

TailCut f64_cut(const GemmDesc &d, int tile_id) {
  const bool akc = (d.sak == 1), bkc = (d.sbk == 1);
  const TileInfo &ti = kTiles[tile_id];
  if (d.split != 1 || d.K <= 0) return TailCut{};
  return gemm_tail_cut(d.M, d.N, d.K, ti.BM, ti.BN, ti.BK, tile_slots(tile_id, (akc ? 2 : 0) + (bkc ? 1 : 0)));
}

}  // namespace

int gpu_cu_count() {
  static std::atomic<int> cus{0};
  int c = cus.load();
  if (c == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0) {
      (void)hipGetLastError();
      c = 256;
    }
    cus.store(c);
  }
  return c;
}

// A round must carry enough work to pay for the two extra launches (the tail
// and its reduction), about 0.2 ms at the FP64 rate.
constexpr double kTailMinRoundFlops = 1.2e10;

TailCut gemm_tail_cut(int64_t M, int64_t N, int64_t K, int BM, int BN, int BK, int64_t slots) {
  TailCut best;
  if (slots <= 0 || M <= 0 || N <= 0 || K <= 0) return best;
  const int64_t tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN, tiles = tm * tn;
  if (tiles <= slots || 2.0 * double(slots) * BM * BN * double(K) < kTailMinRoundFlops) return best;
  const int64_t full = tiles / slots, rem = tiles - full * slots;
  if (rem == 0 || 2 * rem > slots) return best;  // the last round is full enough
  double best_rounds = double(full + 1);
  for (int axis = 1; axis <= 2; ++axis) {
    const int64_t per = axis == 1 ? tm : tn;  // tiles per panel
    const int64_t np = axis == 1 ? tn : tm;   // panels
    const int64_t mainp = (full * slots) / per;
    if (mainp <= 0 || mainp >= np) continue;
    const int64_t tail_tiles = (np - mainp) * per;
    int64_t split = std::min<int64_t>({slots / tail_tiles, 16, K / (8 * int64_t(BK))});
    if (split < 2) continue;
    const double rounds = std::ceil(double(mainp * per) / double(slots)) + 1.0 / double(split);
    if (rounds < best_rounds) {
      best_rounds = rounds;
      best.axis = axis;
      best.main = mainp * (axis == 1 ? BN : BM);
      best.split = int(split);
      const int64_t tr = axis == 1 ? M : M - best.main, tc = axis == 1 ? N - best.main : N;
      best.ws_elems = split * tr * tc;
    }
  }
  return best;
}

int gemm_split_refine(int64_t M, int64_t N, int64_t K, int BM, int BN, int BK, int64_t slots, int split,
                      int64_t ws_elems) {
  if (split <= 1 || slots <= 0 || M <= 0 || N <= 0 || K <= 0) return split;
  const int64_t tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  if (2.0 * double(std::min(tiles, slots)) * BM * BN * double(K) < kTailMinRoundFlops) return split;
  const int64_t smax = std::min<int64_t>({16, std::max<int64_t>(1, K / (8 * int64_t(BK))), ws_elems / (M * N)});
  // full-K rounds the launch takes with s splits, plus a small charge per
  // split for its partial sums (written once, read once by the reduction)
  auto cost = [&](int64_t s) { return std::ceil(double(tiles * s) / double(slots)) / double(s) + 0.02 * double(s); };
  int best = split <= smax ? split : 1;
  double best_cost = cost(best);
  for (int64_t s = 1; s <= smax; ++s)
    if (cost(s) < best_cost - 1e-9) {
      best_cost = cost(s);
      best = int(s);
    }
  return best;
}

int64_t gemm_tail_ws_bound(int64_t M, int64_t N, int64_t K) {
  if (M <= 0 || N <= 0 || K <= 0 || 2.0 * double(M) * double(N) * double(K) < kTailMinRoundFlops) return 0;
  // split x tail elements <= slots x BM x BN = every resident workgroup's
  // accumulators, bounded by the register file (256 CUs x 512 KiB of 4-byte
  // accumulators); the launch checks the exact figure against ws_elems
  return std::min<int64_t>(16 * M * N, int64_t(1) << 25);
}

int64_t gemm_f64_tail_ws(const GemmDesc &d, int tile_id) {
  if (d.M <= 0 || d.N <= 0 || d.K <= 0) return 0;
  if (tile_id < 0 || tile_id >= kNumTiles) tile_id = gemm_f64_choose(d.M, d.N, d.K, d.sak == 1 && d.sbk == 1, 0).tile;
  return f64_cut(d, tile_id).ws_elems;
}

int gemm_f64_num_tiles() { return kNumTiles; }
const char *gemm_f64_tile_name(int id) { return (id >= 0 && id < kNumTiles) ? kTiles[id].name : "?"; }

// ---- static choice of tile and split-K factor --------------------------------
// Time of one launch (and its split-K reduction), in microseconds, from a
// model whose constants were fitted to 15,000 timings on the MI355X: every
// configuration and a grid of split-K factors on the 404 GEMM shapes of the
// CCSD, packed CCSD and CCSDT lists at o = 4..32, v = 20..160.  A compute unit
// runs min(resident, w) of its w workgroups at a time; a K chunk of those takes
// their MFMA cycles over the tile's efficiency, or the latency of one chunk
// when there are too few of them to hide it.  That time competes with the
// operands' and outputs' HBM traffic and with the tiles' operand traffic from
// the L2s; the shorter of the two is partly hidden.  Over those shapes the
// choice was 2.5% (geometric mean) slower than the fastest configuration when
// fitted; the rule it replaced (rounds of 256 workgroups x tile area, staged tiles
// first) was 37% slower, on launches over 50 us: ladder 1024 x 25600 x 25600
// 28.3 -> 19.6 ms, 2000^3 394 -> 258 us, 160000 x 400 x 400 1.97 -> 1.28 ms,
// 10 x 6400000 x 10 0.61 -> 0.46 ms.  The autotuner refines it by timing.
// A launch that is cut into whole rounds and a K-split tail (gemm_tail_cut) counts as
// such, and among choices within 5% the one with the least operand traffic through
// its tiles is taken once the operands exceed 1 GB, four times the last-level
// cache: at 1024 x 25600 x 25600 the 64 x 128 tile reads three times as much from
// HBM as 256 x 128 (20.8 against 19.6 ms).  Over 62 shapes of 2e9 flops and more the
// choice is 4.0% slower than the fastest configuration, 4.9% without the two.
// The 64x64 configuration was fitted to 4,000 timings of 160 small and middle
// shapes; it is the fastest one at 1024^3 (64 x 128 50, 64 x 64 45 us) and 1280^3 (93,
// 88 us), and on long contractions (400 x 2000 x 10000 309, 299 us).
struct F64Model {
  int tile;       // kTiles index
  int resident;   // workgroups per CU
  // operand forms: [0] an M/N-contiguous one, [1] both K-contiguous
  double eff[2];    // share of the MFMA rate (0: not this form)
  double alone[2];  // cycles of one chunk when nothing hides its latency
};
constexpr F64Model kF64Models[] = {
    {3, 6, {0.78, 0.32}, {1044, 702}},   // 32x32 staged: launches bound by memory
    {11, 2, {0.74, 0.0}, {1044, 702}},   // 128x128 staged
    {16, 1, {0.0, 0.89}, {1044, 702}},   // 256x128 LDS-direct
    {17, 3, {0.74, 0.92}, {1044, 702}},  // 64x128 LDS-direct, two stages
    {18, 6, {0.0, 0.57}, {1044, 702}},   // 32x32 LDS-direct (staged: the first line)
    {19, 3, {0.0, 0.83}, {1044, 1100}},  // 64x64 LDS-direct
};
// per operand form: cycles per workgroup set besides its chunks (fixed; per
// 1,024 outputs), HBM TB/s, microseconds and TB/s of the split-K partial sums,
// L2 TB/s, share of the shorter time that is not hidden
constexpr double kF64Const[2][7] = {{159, 454, 5.24, 2.9, 7.6, 10.0, 0.54}, {359, 417, 5.9, 2.3, 3.4, 26.5, 0.14}};

// A plan of 25 GEMMs asks for some 5,000 times: the terms that do not depend on
// the split-K factor are formed once per tile.
struct F64Tile {
  const F64Model &m;
  const TileInfo &ti;
  int64_t tm, tn, tiles;
  double us = 1e300;  // with its best factor
  F64Choice choice;

  F64Tile(const F64Model &model, int64_t M, int64_t N)
      : m(model), ti(kTiles[m.tile]), tm((M + ti.BM - 1) / ti.BM), tn((N + ti.BN - 1) / ti.BN), tiles(tm * tn),
        choice{m.tile, 1} {}

  void best(int form, int64_t M, int64_t N, int64_t K, int64_t ws_elems) {
    static constexpr int kSplits[] = {1,  2,  3,  4,  5,   6,   8,   12,  16,  24,  32,
                                      48, 64, 96, 128, 192, 256, 384, 512, 768, 1024};
    const double *c = kF64Const[form];
    const double area = double(ti.BM) * ti.BN, cyc = area / 4.0 / m.eff[form];  // 128 flop per cycle and CU
    const double setup = c[1] * area / 1024.0, res = m.resident, mn = double(M) * double(N);
    const double l2s = double(tiles) * double(ti.BM + ti.BN) * 128.0 / c[5] * 1e-6;
    const double ins = (double(M) + double(N)) * double(K) * 8.0 / c[2] * 1e-6, outs = 16.0 * mn / c[2] * 1e-6;
    const double sums = 16.0 * mn / c[4] * 1e-6;
    for (int s : kSplits) {
      if (s > 1 && (int64_t(s) * 64 > K || tiles * s > 4096 || double(s) * mn > double(ws_elems))) break;
      const int64_t per = s == 1 ? K : K >> 31 ? (K + s - 1) / s : int64_t((uint32_t(K) + uint32_t(s) - 1) / uint32_t(s));
      const double n = double((per + 15) >> 4);  // chunks per workgroup
      double w = double((tiles * s + 255) >> 8);
      if (s == 1) {  // whole rounds and a K-split tail, where the launch is cut that way
        const int64_t slots = 256 * m.resident;
        const TailCut cut = gemm_tail_cut(M, N, K, ti.BM, ti.BN, ti.BK, slots);
        if (cut.axis) {
          const int64_t main = cut.axis == 1 ? tm * (cut.main / ti.BN) : tn * (cut.main / ti.BM);
          w = std::min(w, res * (double((main + slots - 1) / slots) + 1.0 / cut.split));
        }
      }
      const double conc = std::min(w, res);
      const double chunk = std::max(conc * cyc, m.alone[form]);
      const double mfma = (w > res ? w / res : 1.0) * (n * chunk + c[0] + setup * conc) * (1.0 / 2400.0);
      const double mem = s == 1 ? ins + outs : ins, work = std::max(mfma, l2s * double(s) * n);
      const double red = s > 1 ? c[3] + sums * double(s) : 0.0;
      const double t = 3.0 + std::max(work, mem) + c[6] * std::min(work, mem) + red;
      if (t < us) {
        us = t;
        choice.split = s;
      }
    }
  }
};

bool gemm_f64_tile_merged(int tile_id) { return tile_id == 3 || tile_id == 18; }

F64Choice gemm_f64_choose(int64_t M, int64_t N, int64_t K, bool lds_direct, int64_t ws_elems, F64Choice *merged) {
  const int form = lds_direct ? 1 : 0;
  const bool huge = 8.0 * double(M + N) * double(K) > 1e9;
  F64Choice best{3, 1}, own{3, 1}, near{3, 1};
  double best_us = 1e300, own_us = 1e300;
  double us[sizeof(kF64Models) / sizeof(kF64Models[0])];
  int q = 0;
  for (const F64Model &m : kF64Models) {
    us[q] = 1e300;
    if (m.eff[form] > 0.0) {
      F64Tile t(m, M, N);
      t.best(form, M, N, K, ws_elems);
      us[q] = t.us;
      if (t.us < best_us) {
        best_us = t.us;
        best = t.choice;
      }
      if (gemm_f64_tile_merged(m.tile) && t.us < own_us) {
        own_us = t.us;
        own = t.choice;
      }
    }
    ++q;
  }
  if (huge) {
    double least = 1e300;
    q = 0;
    for (const F64Model &m : kF64Models)
      if (us[q++] <= best_us * 1.05) {
        F64Tile t(m, M, N);
        const double traffic = double(t.tiles) * (t.ti.BM + t.ti.BN);
        if (traffic >= least) continue;
        least = traffic;
        t.best(form, M, N, K, ws_elems);
        near = t.choice;
      }
    best = near;
  }
  // A merged launch saves the step its own, about 3 us of the model's time, so
  // the small tiles are taken unless another tile is faster by more than that.
  if (merged) *merged = own_us <= best_us + 3.0 ? own : best;
  return best;
}

// Split-K factor: about 2048 workgroups (eight per CU) when the output has
// few tiles and the contraction is long (e.g. M = N = o, K = o v^2), each
// split covering at least 256 of K.
// Independent of the tile so that the autotuner can change tiles freely.
int gemm_split_pick(int64_t M, int64_t N, int64_t K, int) {
  const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);
  if (tiles >= 2048) return 1;  // eight 64x64 tiles per CU or more
  int64_t split = (2048 + tiles - 1) / tiles;
  split = std::min<int64_t>(split, std::max<int64_t>(1, K / 256));
  return int(std::max<int64_t>(1, std::min<int64_t>(split, 1024)));
}

void gemm_f64_grouped_launch(const GemmGroupEntry *dev_entries, const int64_t *dev_off, int n,
                             int64_t blocks, bool akc, bool bkc, int tile_id, hipStream_t s) {
  if (blocks <= 0) return;
  CC_REQUIRE(tile_id >= 0 && tile_id < kNumTiles, -7, "grouped gemm: tile");
  CC_REQUIRE(blocks < (int64_t(1) << 31), -1, "grouped gemm: too many tiles");
  kTiles[tile_id].launch_grouped[(akc ? 2 : 0) + (bkc ? 1 : 0)](dev_entries, dev_off, n, blocks, s);
  CC_HIP_CHECK(hipGetLastError());
}

void gemm_f64_tile_shape(int tile_id, int *bm, int *bn) {
  *bm = kTiles[tile_id].BM;
  *bn = kTiles[tile_id].BN;
}

int gemm_f64_refined_split(const GemmDesc &d, int tile_id, int64_t ws_elems) {
  const TileInfo &ti = kTiles[tile_id];
  return gemm_split_refine(d.M, d.N, d.K, ti.BM, ti.BN, ti.BK,
                           tile_slots(tile_id, (d.sak == 1 ? 2 : 0) + (d.sbk == 1 ? 1 : 0)), d.split, ws_elems);
}

void gemm_f64(const GemmDesc &d0, hipStream_t s, int tile_id) {
  GemmDesc d = d0;
  if (d.M <= 0 || d.N <= 0) return;
  const bool akc = (d.sak == 1), bkc = (d.sbk == 1);
  CC_REQUIRE(akc || d.sam == 1, -1, "gemm: A needs a unit stride in m or k");
  CC_REQUIRE(bkc || d.sbn == 1, -1, "gemm: B needs a unit stride in n or k");
  if (d.K <= 0) {
    // C = beta * C: a GEMM with an empty contraction still scales C (an
    // in-place, element-by-element identity permutation with alpha = beta)
    PermDesc p{};
    p.rank = 2;
    p.out_dims[0] = d.M; p.out_dims[1] = d.N;
    p.out_strides[0] = d.ldc; p.out_strides[1] = 1;
    p.in_strides[0] = d.ldc; p.in_strides[1] = 1;
    p.alpha = d.beta; p.beta = 0.0; p.conj = 0;
    permute_f64(p, d.C, d.C, s);
    return;
  }
  CC_REQUIRE(d.split >= 1, -1, "gemm: split must be >= 1");
  if (tile_id < 0 || tile_id >= kNumTiles) {
    // the library's choice, of the split-K factor too where the caller
    // allowed one (within the workspace it gave)
    const int64_t room = d.split > 1 && d.ws ? (d.ws_elems > 0 ? d.ws_elems : d.split * d.M * d.N) : 0;
    const F64Choice ch = gemm_f64_choose(d.M, d.N, d.K, akc && bkc, room);
    tile_id = ch.tile;
    d.split = ch.split;
  } else if (d.ws && d.split > 1 && d.ws_elems > 0 && d.refine) {
    d.split = gemm_f64_refined_split(d, tile_id, d.ws_elems);
  }
  const TileInfo &ti = kTiles[tile_id];
  const int64_t tm = (d.M + ti.BM - 1) / ti.BM, tn = (d.N + ti.BN - 1) / ti.BN;
  CC_REQUIRE(d.split == 1 || d.ws != nullptr, -1, "gemm: split-K needs a workspace");
  CC_REQUIRE(d.split == 1 || d.ws_elems == 0 || d.ws_elems >= d.split * d.M * d.N, -1,
             "gemm: split-K workspace too small");
  CC_REQUIRE(tm * tn * d.split < (int64_t(1) << 31), -1, "gemm: too many tiles");
  auto one = [&](const GemmDesc &g) {
    const int64_t gm = (g.M + ti.BM - 1) / ti.BM, gn = (g.N + ti.BN - 1) / ti.BN;
    if (g.ladder == 2 && akc && bkc) ti.launch_ladder_tail(g, gm, gn, s);
    else if (g.ladder && akc && bkc) ti.launch_ladder(g, gm, gn, s);
    else ti.launch[(akc ? 2 : 0) + (bkc ? 1 : 0)](g, gm, gn, s);
    CC_HIP_CHECK(hipGetLastError());
    if (g.split > 1) splitk_reduce(false, g.ws, g.split, g.M, g.N, g.C, g.ldc, g.alpha, g.beta, s);
  };
  if (d.ws && d.split == 1) {
    const TailCut tc = f64_cut(d, tile_id);
    if (tc.axis && tc.ws_elems <= d.ws_elems) {
      gemm_run_cut(d, tc, sizeof(double), sizeof(double), one);
      return;
    }
  }
  one(d);
}

}  // namespace ccmi
