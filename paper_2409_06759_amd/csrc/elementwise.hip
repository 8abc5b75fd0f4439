// Data-movement and elementwise kernels of the residual path (HBM bound):
//  * LDS-tiled index permutation with scale/accumulate (the two transposes of
//    the transpose-transpose-GEMM-transpose scheme, paper Sec. "Tensor
//    contractions");
//  * outer-product accumulation (tau formation, the t1 t1 pieces);
//  * tau / tau~ formation fused with the energy reduction (Eq. eq:amp, first
//    line: E = sum f_ia t_i^a + 1/4 sum <ij||ab> tau_ij^ab);
//  * the doubles-residual assembly that applies P(ij), P(ab) and P(ij)P(ab)
//    (the permutation operators of the contraction list) fused with the
//    Jacobi update t <- t + R/(D - s) and the residual norm;
//  * deterministic two-stage reductions (fixed order: bitwise reproducible).
#include "elementwise_dev.hpp"
#include "kernels.hpp"

namespace ccmi {
namespace {

// Fock diagonals (real parts) into contiguous arrays.
template <class T>
__global__ void fock_diag_kernel(int o, int v, const T *foo, const T *fvv, double *d_oo, double *d_vv) {
  for (int e = threadIdx.x + blockIdx.x * blockDim.x; e < o + v; e += blockDim.x * gridDim.x) {
    if (e < o) d_oo[e] = re(foo[int64_t(e) * o + e]);
    else d_vv[e - o] = re(fvv[int64_t(e - o) * v + (e - o)]);
  }
}

// ------------------------------------------------------- kernels (both forms)
#define CC_EW_KERNELS(NAME, ENTRY, BODY, LDS)                                                     \
  template <class T>                                                                              \
  __global__ __launch_bounds__(256) void k_##NAME(ENTRY e) {                                     \
    __shared__ __attribute__((aligned(16))) unsigned char smem[LDS];                             \
    BODY<T>(e, blockIdx.x, smem);                                                                 \
  }                                                                                               \
  template <class T>                                                                              \
  __global__ __launch_bounds__(256) void g_##NAME(const ENTRY *__restrict__ es,                  \
                                                  const int64_t *__restrict__ off, int n) {      \
    __shared__ __attribute__((aligned(16))) unsigned char smem[LDS];                             \
    const int b = group_find(off, n, blockIdx.x);                                                 \
    BODY<T>(es[b], int64_t(blockIdx.x) - off[b], smem);                                           \
  }

CC_EW_KERNELS(perm_flat, PermEntry, perm_flat_body, 16)
CC_EW_KERNELS(perm_tiled, PermEntry, perm_tiled_body, kLdsTile<T>)
CC_EW_KERNELS(outer, OuterEntry, outer_body, 16)
CC_EW_KERNELS(fill, FillEntry, fill_body, 16)
CC_EW_KERNELS(splitk, SplitkEntry, splitk_body, kLdsPart<T>)
CC_EW_KERNELS(tau, TauEntry, tau_body, kLdsSum)
CC_EW_KERNELS(asm, AsmEntry, asm_body, kLdsAsm<T>)
CC_EW_KERNELS(t3, T3Entry, t3_body, kLdsT3<T>)
CC_EW_KERNELS(pair, PairEntry, pair_body, 16)

template <class T>
__global__ __launch_bounds__(RED_THREADS) void k_r1(R1Entry e) {
  __shared__ double sh[RED_THREADS];
  r1_body<T>(e, sh);
}
template <class T>
__global__ __launch_bounds__(RED_THREADS) void g_r1(const R1Entry *__restrict__ es) {
  __shared__ double sh[RED_THREADS];
  r1_body<T>(es[blockIdx.x], sh);
}
// Doubles assembly, the singles update in one more workgroup, and, with a
// ticket, the scalars in the workgroup that finishes last (whose sums are in
// the order of k_fin's).  Each workgroup's fence before its ticket writes back
// what its L2 holds: with many of them that costs more than the launch saved
// (about 900 workgroups: 604 us per residual against 584), so the scalars are
// left to a launch of their own above kFinUnits.
constexpr int64_t kFinUnits = 128;
__global__ __launch_bounds__(RED_THREADS) void k_asm_r1_fin(AsmEntry e, R1Entry r, FinEntry f, unsigned *ticket) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[kLdsAsm<double>];
  if (int64_t(blockIdx.x) < e.units) asm_body<double>(e, blockIdx.x, smem);
  else r1_body<double>(r, smem);
  if (ticket == nullptr) return;
  // the partial sums (each written by its workgroup's thread 0) before the ticket
  __shared__ unsigned last;
  if (threadIdx.x == 0) {
    __threadfence();
    last = atomicAdd(ticket, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  fin_body(f, smem);
  if (threadIdx.x == 0) *ticket = 0;
}
__global__ __launch_bounds__(RED_THREADS) void k_fin(FinEntry e) {
  __shared__ double sh[RED_THREADS];
  fin_body(e, sh);
}
__global__ __launch_bounds__(RED_THREADS) void g_fin(const FinEntry *__restrict__ es) {
  __shared__ double sh[RED_THREADS];
  fin_body(es[blockIdx.x], sh);
}

int64_t chunks(int64_t n, int64_t ch) { return std::max<int64_t>(1, (n + ch - 1) / ch); }

}  // namespace

// ============================================================ host: entries ==
PermEntry make_perm_entry(const PermDesc &d, const void *in, void *out) {
  PermEntry e{};
  PermArgs &p = e.p;
  // Drop dims of extent 1 and merge each dim into the one outside it when it
  // continues that one in both tensors (outer stride = inner stride x inner
  // extent): the same element map over fewer, longer dims.
  int64_t total = 1;
  p.rank = 0;
  for (int i = 0; i < d.rank; ++i) {
    const int64_t n = d.out_dims[i];
    total *= n;
    if (n == 1) continue;
    const int r = p.rank;
    if (r > 0 && p.istr[r - 1] == d.in_strides[i] * n && p.ostr[r - 1] == d.out_strides[i] * n) {
      p.dims[r - 1] *= n;
      p.istr[r - 1] = d.in_strides[i];
      p.ostr[r - 1] = d.out_strides[i];
    } else {
      p.dims[r] = n;
      p.istr[r] = d.in_strides[i];
      p.ostr[r] = d.out_strides[i];
      p.rank = r + 1;
    }
  }
  if (p.rank == 0) {  // one element
    p.rank = 1;
    p.dims[0] = 1;
    p.istr[0] = p.ostr[0] = 0;
  }
  p.total = total;
  p.alpha = d.alpha;
  p.beta = d.beta;
  p.conj = d.conj;
  int d_o = -1, d_i = -1;
  for (int i = 0; i < p.rank; ++i) {
    if (p.ostr[i] == 1 && p.dims[i] > 1) d_o = i;
    if (p.istr[i] == 1 && p.dims[i] > 1) d_i = i;
  }
  e.in = in;
  e.out = out;
  if (total == 0) {
    e.units = 0;
    return e;
  }
  if (d_o < 0 || d_i < 0 || d_o == d_i) {
    e.tiled = 0;
    e.units = chunks(total, CH);
  } else {
    e.tiled = 1;
    p.d_o = d_o;
    p.d_i = d_i;
    p.nrest = 0;
    p.n_rest_total = 1;
    for (int i = 0; i < p.rank; ++i) {
      if (i == d_o || i == d_i) continue;
      p.rest_dims[p.nrest] = p.dims[i];
      p.rest_istr[p.nrest] = p.istr[i];
      p.rest_ostr[p.nrest] = p.ostr[i];
      p.n_rest_total *= p.dims[i];
      ++p.nrest;
    }
    // 32 x 32, or a narrow, long tile when one of the two fast dims is short
    // (the occupied index of small systems) instead of a mostly empty one
    auto lg = [](int64_t n) {  // log2 of the smallest power of two >= n, in [2, 8]
      int l = 2;
      while (l < 8 && (int64_t(1) << l) < n) ++l;
      return l;
    };
    const int li = lg(p.dims[d_i]), lo = lg(p.dims[d_o]);
    p.lti = li < 5 ? li : (lo < 5 ? 10 - lo : 5);
    p.tiles_i = (p.dims[d_i] + (1 << p.lti) - 1) >> p.lti;
    p.tiles_o = (p.dims[d_o] + (1 << (10 - p.lti)) - 1) >> (10 - p.lti);
    e.units = p.n_rest_total * p.tiles_o * p.tiles_i;
  }
  return e;
}

OuterEntry make_outer_entry(const OuterArgs &a, const void *A, const void *B, void *C) {
  OuterEntry e{};
  e.a = a;
  e.A = A;
  e.B = B;
  e.C = C;
  e.total = 1;
  for (int i = 0; i < a.rank; ++i) e.total *= a.dims[i];
  e.units = e.total ? chunks(e.total, CH) : 0;
  return e;
}

FillEntry make_fill_entry(void *p, int64_t n) { return FillEntry{p, n, n > 0 ? chunks(n, CH) : 0}; }

SplitkEntry make_splitk_entry(const void *ws, int split, int64_t M, int64_t N, void *C, int64_t ldc, double alpha,
                              double beta) {
  int lanes = 1;
  while (lanes < 16 && 2 * lanes <= split) lanes *= 2;
  return SplitkEntry{ws, split, lanes, M, N, C, ldc, alpha, beta, M * N > 0 ? chunks(M * N, 256 / lanes) : 0};
}

int64_t tau_units(int o, int v) { return chunks(int64_t(o) * o * v * v, CH_TAU); }

TauEntry make_tau_entry(int o, int v, const void *t1, const void *t2, const void *oovv, const void *fov,
                        void *tau, void *taut, double *partials) {
  return TauEntry{o, v, t1, t2, oovv, fov, tau, taut, partials, tau_units(o, v)};
}

int64_t t3_units(int o, int v) {
  const int64_t rep = 3 * int64_t(o) * o - 2 * int64_t(o);  // ordered ijk with a repeated index
  return t3_value_units(o, v) + rep * chunks(int64_t(v) * v * v, CH_T3);
}

PairEntry make_pair_entry(const void *src, void *dst, const int *rows, const int *cols, int64_t nP, int64_t nQ,
                          int64_t ldq, int64_t n1, int64_t n2, int64_t n3, int mode) {
  CC_REQUIRE(ldq >= nQ, -1, "pair: row stride below the row length");
  return PairEntry{src, dst, rows, cols, nP, nQ, ldq, n1, n2, n3, mode, nP * nQ > 0 ? chunks(nP * nQ, CH) : 0};
}

int64_t asm_units(int o, int v) {
  const int64_t tiles = (v + 31) / 32;
  return (int64_t(o) * (o + 1) / 2) * (tiles * (tiles + 1) / 2);
}

AsmEntry make_asm_entry(const R2Args &a, const void *XP, const void *Xij, const void *Xab, const void *Xr, void *R,
                        void *t2, double *partials) {
  return AsmEntry{a, XP, Xij, Xab, Xr, R, t2, partials, asm_units(a.o, a.v)};
}

// ========================================================= host: launches ==
#define CC_LAUNCH1(KER, E, UNITS, CPLX, S)                                                          \
  do {                                                                                            \
    if ((UNITS) <= 0) return;                                                                     \
    CC_REQUIRE((UNITS) < (int64_t(1) << 31), -1, "grid too large");                               \
    if (CPLX) hipLaunchKernelGGL(KER<double2>, dim3(UNITS), dim3(256), 0, S, E);                  \
    else hipLaunchKernelGGL(KER<double>, dim3(UNITS), dim3(256), 0, S, E);                        \
    CC_HIP_CHECK(hipGetLastError());                                                              \
  } while (0)

#define CC_LAUNCHG(KER, E, OFF, N, BLOCKS, CPLX, S)                                                 \
  do {                                                                                            \
    if ((BLOCKS) <= 0) return;                                                                    \
    CC_REQUIRE((BLOCKS) < (int64_t(1) << 31), -1, "grid too large");                              \
    if (CPLX) hipLaunchKernelGGL(KER<double2>, dim3(BLOCKS), dim3(256), 0, S, E, OFF, N);         \
    else hipLaunchKernelGGL(KER<double>, dim3(BLOCKS), dim3(256), 0, S, E, OFF, N);               \
    CC_HIP_CHECK(hipGetLastError());                                                              \
  } while (0)

void launch_perm(const PermEntry &e, bool cplx, hipStream_t s) {
  if (e.tiled) CC_LAUNCH1(k_perm_tiled, e, e.units, cplx, s);
  else CC_LAUNCH1(k_perm_flat, e, e.units, cplx, s);
}
void launch_outer(const OuterEntry &e, bool cplx, hipStream_t s) { CC_LAUNCH1(k_outer, e, e.units, cplx, s); }
void launch_fill(const FillEntry &e, bool cplx, hipStream_t s) { CC_LAUNCH1(k_fill, e, e.units, cplx, s); }
void launch_splitk(const SplitkEntry &e, bool cplx, hipStream_t s) { CC_LAUNCH1(k_splitk, e, e.units, cplx, s); }
void launch_tau(const TauEntry &e, bool cplx, hipStream_t s) { CC_LAUNCH1(k_tau, e, e.units, cplx, s); }
void launch_asm(const AsmEntry &e, bool cplx, hipStream_t s) { CC_LAUNCH1(k_asm, e, e.units, cplx, s); }
void launch_t3(const T3Entry &e, bool cplx, hipStream_t s) { CC_LAUNCH1(k_t3, e, e.units, cplx, s); }
void launch_pair(const PairEntry &e, bool cplx, hipStream_t s) { CC_LAUNCH1(k_pair, e, e.units, cplx, s); }
void launch_r1(const R1Entry &e, bool cplx, hipStream_t s) {
  if (cplx) hipLaunchKernelGGL(k_r1<double2>, dim3(1), dim3(RED_THREADS), 0, s, e);
  else hipLaunchKernelGGL(k_r1<double>, dim3(1), dim3(RED_THREADS), 0, s, e);
  CC_HIP_CHECK(hipGetLastError());
}
void launch_asm_r1_fin(const AsmEntry &e, const R1Entry *r, const FinEntry &f, unsigned *ticket, hipStream_t s) {
  const int64_t blocks = e.units + (r ? 1 : 0);
  CC_REQUIRE(blocks > 0 && blocks < (int64_t(1) << 31), -1, "grid too large");
  const bool fin = blocks <= kFinUnits;
  hipLaunchKernelGGL(k_asm_r1_fin, dim3(blocks), dim3(RED_THREADS), 0, s, e, r ? *r : R1Entry{}, f, fin ? ticket : nullptr);
  CC_HIP_CHECK(hipGetLastError());
  if (!fin) launch_fin(f, s);
}
void launch_fin(const FinEntry &e, hipStream_t s) {
  hipLaunchKernelGGL(k_fin, dim3(1), dim3(RED_THREADS), 0, s, e);
  CC_HIP_CHECK(hipGetLastError());
}

void launch_perm_grouped(const PermEntry *e, const int64_t *off, int n, int64_t blocks, bool tiled, bool cplx,
                         hipStream_t s) {
  if (tiled) CC_LAUNCHG(g_perm_tiled, e, off, n, blocks, cplx, s);
  else CC_LAUNCHG(g_perm_flat, e, off, n, blocks, cplx, s);
}
void launch_outer_grouped(const OuterEntry *e, const int64_t *off, int n, int64_t blocks, bool cplx, hipStream_t s) {
  CC_LAUNCHG(g_outer, e, off, n, blocks, cplx, s);
}
void launch_pair_grouped(const PairEntry *e, const int64_t *off, int n, int64_t blocks, bool cplx, hipStream_t s) {
  CC_LAUNCHG(g_pair, e, off, n, blocks, cplx, s);
}
void launch_fill_grouped(const FillEntry *e, const int64_t *off, int n, int64_t blocks, bool cplx, hipStream_t s) {
  CC_LAUNCHG(g_fill, e, off, n, blocks, cplx, s);
}
void launch_splitk_grouped(const SplitkEntry *e, const int64_t *off, int n, int64_t blocks, bool cplx,
                           hipStream_t s) {
  CC_LAUNCHG(g_splitk, e, off, n, blocks, cplx, s);
}
void launch_tau_grouped(const TauEntry *e, const int64_t *off, int n, int64_t blocks, bool cplx, hipStream_t s) {
  CC_LAUNCHG(g_tau, e, off, n, blocks, cplx, s);
}
void launch_asm_grouped(const AsmEntry *e, const int64_t *off, int n, int64_t blocks, bool cplx, hipStream_t s) {
  CC_LAUNCHG(g_asm, e, off, n, blocks, cplx, s);
}
void launch_r1_grouped(const R1Entry *e, int n, bool cplx, hipStream_t s) {
  if (n <= 0) return;
  if (cplx) hipLaunchKernelGGL(g_r1<double2>, dim3(n), dim3(RED_THREADS), 0, s, e);
  else hipLaunchKernelGGL(g_r1<double>, dim3(n), dim3(RED_THREADS), 0, s, e);
  CC_HIP_CHECK(hipGetLastError());
}
void launch_fin_grouped(const FinEntry *e, int n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(g_fin, dim3(n), dim3(RED_THREADS), 0, s, e);
  CC_HIP_CHECK(hipGetLastError());
}

// ====================================================== host: conveniences ==
void permute_f64(const PermDesc &d, const void *in, void *out, hipStream_t s) {
  launch_perm(make_perm_entry(d, in, out), false, s);
}
void permute_c128(const PermDesc &d, const void *in, void *out, hipStream_t s) {
  launch_perm(make_perm_entry(d, in, out), true, s);
}
void outer_acc(const OuterArgs &a, bool cplx, const void *A, const void *B, void *C, hipStream_t s) {
  launch_outer(make_outer_entry(a, A, B, C), cplx, s);
}
void fill_zero(void *p, int64_t n_elems, bool cplx, hipStream_t s) {
  launch_fill(make_fill_entry(p, n_elems), cplx, s);
}
void splitk_reduce(bool cplx, const void *ws, int split, int64_t M, int64_t N, void *C, int64_t ldc,
                   double alpha, double beta, hipStream_t s) {
  launch_splitk(make_splitk_entry(ws, split, M, N, C, ldc, alpha, beta), cplx, s);
}
void fock_diag(bool cplx, int o, int v, const void *foo, const void *fvv, double *d_oo, double *d_vv,
               hipStream_t s) {
  if (cplx)
    hipLaunchKernelGGL(fock_diag_kernel<double2>, dim3(1), dim3(256), 0, s, o, v, (const double2 *)foo,
                       (const double2 *)fvv, d_oo, d_vv);
  else
    hipLaunchKernelGGL(fock_diag_kernel<double>, dim3(1), dim3(256), 0, s, o, v, (const double *)foo,
                       (const double *)fvv, d_oo, d_vv);
  CC_HIP_CHECK(hipGetLastError());
}

}  // namespace ccmi
