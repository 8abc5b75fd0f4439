// Merged launches: the independent steps of one dependency level of a small
// system's iteration, in one grid.
//
// A CCSD iteration at o = 4, v = 20 is 67 kernels of 3 to 8 us each, most of it
// the cost of a launch and the drain of the one before; its dependency chain
// is a dozen levels long.  One launch per level runs the same bodies on the
// same entries, from a table in device memory that is uploaded once per plan (295 ->
// 121 us; a launch takes 4 to 8 us, of which about 3 are its own cost).
// GEMMs run on 32 x 32 tiles (the LDS-direct kernel's where both operands are
// K-contiguous): larger tiles would cost the other bodies their occupancy, and
// steps that need them keep launches of their own.  16 x 16 tiles whose four
// waves share the K chunks, faster by themselves, gained nothing here: what
// counts is how much code a launch of a few microseconds has to fetch.
#include "elementwise_dev.hpp"
#include "gemm_f64_dev.hpp"
#include "kernels.hpp"

namespace ccmi {
namespace {

struct ExtPtr {
  LevelExt x;
  __device__ __forceinline__ uintptr_t at(uintptr_t u) const {
    return u > 3 || u == 0 ? u : reinterpret_cast<uintptr_t>(u == 1 ? x.t1 : u == 2 ? x.t2 : x.t3);
  }
  __device__ __forceinline__ const void *operator()(const void *p) const {
    return reinterpret_cast<const void *>(at(reinterpret_cast<uintptr_t>(p)));
  }
  __device__ __forceinline__ void *operator()(void *p) const {
    return reinterpret_cast<void *>(at(reinterpret_cast<uintptr_t>(p)));
  }
};

template <bool AKC, bool BKC>
using Cfg32 = Cfg<32, 32, 16, 2, 2, AKC, BKC>;
using Direct32 = Dma64<32, 32, 2, 2, 3>;
constexpr int kLdsLevel = Direct32::ELEMS * 8;
static_assert(kLdsLevel >= kLdsTile<double> && kLdsLevel >= kLdsPart<double> && kLdsLevel >= kLdsSum, "LDS");
static_assert(kLdsLevel >= 16 * (Cfg32<true, false>::A_ELEMS + Cfg32<true, false>::B_ELEMS) &&
                  kLdsLevel >= 16 * (Cfg32<false, false>::A_ELEMS + Cfg32<false, false>::B_ELEMS),
              "LDS");

__global__ __launch_bounds__(256) void level_kernel(const LevelItem *__restrict__ items, const int *__restrict__ off, int n,
                                                    LevelExt ext) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kLdsLevel];
  // item of this workgroup: one load of the offsets, one vote
  const int lane = threadIdx.x & 63;
  const int o = lane < n ? off[lane] : 0x7fffffff;
  const int b = __popcll(__ballot(o <= int(blockIdx.x))) - 1;
  const int64_t bid = int(blockIdx.x) - __builtin_amdgcn_readlane(o, b);
  const LevelItem &it = items[b];
  const ExtPtr rs{ext};
  switch (it.kind) {
    case LevelItem::PERM_FLAT:
      perm_flat_body<double>(*reinterpret_cast<const PermEntry *>(it.u), bid, smem, rs);
      break;
    case LevelItem::PERM_TILED:
      perm_tiled_body<double>(*reinterpret_cast<const PermEntry *>(it.u), bid, smem, rs);
      break;
    case LevelItem::OUTER:
      outer_body<double>(*reinterpret_cast<const OuterEntry *>(it.u), bid, smem, rs);
      break;
    case LevelItem::FILL:
      fill_body<double>(*reinterpret_cast<const FillEntry *>(it.u), bid, smem);
      break;
    case LevelItem::SPLITK:
      splitk_body<double>(*reinterpret_cast<const SplitkEntry *>(it.u), bid, smem);
      break;
    case LevelItem::TAU:
      tau_body<double>(*reinterpret_cast<const TauEntry *>(it.u), bid, smem, rs);
      break;
    case LevelItem::PAIR:
      pair_body<double>(*reinterpret_cast<const PairEntry *>(it.u), bid, smem, rs);
      break;
    default: {
      const GemmGroupEntry &g = *reinterpret_cast<const GemmGroupEntry *>(it.u);
      GemmDesc d = g.d;
      d.A = rs(d.A);
      d.B = rs(d.B);
      double *S = reinterpret_cast<double *>(smem);
      if (it.kind == LevelItem::GEMM_KK) {
        gemm_f64_dma_body<32, 32, 2, 2, 3, true>(d, g.tilesM, g.tilesN, bid, S);
      } else if (it.kind == LevelItem::GEMM_KN) {
        gemm_f64_body<32, 32, 16, 2, 2, true, false>(d, g.tilesM, g.tilesN, bid, S);
      } else if (it.kind == LevelItem::GEMM_MK) {
        gemm_f64_body<32, 32, 16, 2, 2, false, true>(d, g.tilesM, g.tilesN, bid, S);
      } else {
        gemm_f64_body<32, 32, 16, 2, 2, false, false>(d, g.tilesM, g.tilesN, bid, S);
      }
    }
  }
}

}  // namespace

void launch_level(const LevelItem *items, const int *off, int n, int blocks, const LevelExt &ext, hipStream_t s) {
  CC_REQUIRE(n > 0 && n <= kLevelItems && blocks > 0, -7, "merged launch: items");
  hipLaunchKernelGGL(level_kernel, dim3(blocks), dim3(256), 0, s, items, off, n, ext);
  CC_HIP_CHECK(hipGetLastError());
}

}  // namespace ccmi
