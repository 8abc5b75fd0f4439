// Device bodies of the data-movement and elementwise steps, shared by their
// own kernels (single and grouped) and by the merged launches of small
// systems.  LDS comes from the calling kernel; a body that may read or write
// a tensor supplied per call takes its pointers through a resolver.
#pragma once

#include "kernels.hpp"

namespace ccmi {
namespace {

// ---------------------------------------------------------------- scalars --
__device__ __forceinline__ double cj(double x) { return x; }
__device__ __forceinline__ double2 cj(double2 x) { return make_double2(x.x, -x.y); }
__device__ __forceinline__ double sc(double a, double x) { return a * x; }
__device__ __forceinline__ double2 sc(double a, double2 x) { return make_double2(a * x.x, a * x.y); }
__device__ __forceinline__ double add(double a, double b) { return a + b; }
__device__ __forceinline__ double2 add(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double sub(double a, double b) { return a - b; }
__device__ __forceinline__ double2 sub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double mul(double a, double b) { return a * b; }
__device__ __forceinline__ double2 mul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double abs2(double a) { return a * a; }
__device__ __forceinline__ double abs2(double2 a) { return a.x * a.x + a.y * a.y; }
template <class T> __device__ __forceinline__ T zero();
template <> __device__ __forceinline__ double zero<double>() { return 0.0; }
template <> __device__ __forceinline__ double2 zero<double2>() { return make_double2(0.0, 0.0); }
__device__ __forceinline__ double re(double a) { return a; }
__device__ __forceinline__ double re(double2 a) { return a.x; }
__device__ __forceinline__ double im(double) { return 0.0; }
__device__ __forceinline__ double im(double2 a) { return a.y; }

constexpr int RED_THREADS = 256;

struct SamePtr {  // pointers as the entry holds them
  template <class P> __device__ __forceinline__ P operator()(P p) const { return p; }
};

// Block-wide sum in a fixed order (tree over LDS); result in every thread.
__device__ __forceinline__ double block_sum(double v, double *sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int w = RED_THREADS / 2; w > 0; w >>= 1) {
    if (t < w) sh[t] += sh[t + w];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}


constexpr int64_t CH = 1024;      // elements per workgroup, flat kernels
constexpr int64_t CH_TAU = 2048;  // elements per workgroup, tau + energy

// ------------------------------------------------------------- permutation --
// Flat path: input and output share their unit-stride dimension.
template <class T, class Res = SamePtr>
__device__ __forceinline__ void perm_flat_body(const PermEntry &E, int64_t bid, void *, Res rs = Res{}) {
  const PermArgs &p = E.p;
  const T *__restrict__ in = static_cast<const T *>(rs(E.in));
  T *__restrict__ out = static_cast<T *>(rs(E.out));
  const int64_t e1 = std::min<int64_t>(p.total, (bid + 1) * CH);
  // Real tensors whose shared unit-stride dimension is even, whose other
  // strides are even and whose bases are 16-byte aligned move pairs of
  // elements with 16-byte accesses (every pair starts at an even offset and
  // never straddles a row, so one offset computation serves both).
  if constexpr (sizeof(T) == 8) {
    const int r1 = p.rank - 1;
    bool even = true;
    for (int d = 0; d < r1; ++d) even = even && (p.istr[d] % 2 == 0) && (p.ostr[d] % 2 == 0);
    if (p.rank >= 1 && even && p.dims[r1] % 2 == 0 && p.istr[r1] == 1 && p.ostr[r1] == 1 &&
        p.total < (int64_t(1) << 31) && (reinterpret_cast<uintptr_t>(in) & 15) == 0 &&
        (reinterpret_cast<uintptr_t>(out) & 15) == 0 && !p.conj) {
      typedef double d2v __attribute__((ext_vector_type(2)));
      for (int64_t e = bid * CH + 2 * threadIdx.x; e < e1; e += 512) {
        uint32_t rem = uint32_t(e);
        int64_t io = 0, oo = 0;
        for (int d = r1; d >= 0; --d) {
          const uint32_t n = uint32_t(p.dims[d]), x = rem % n;
          rem /= n;
          io += int64_t(x) * p.istr[d];
          oo += int64_t(x) * p.ostr[d];
        }
        d2v v = *reinterpret_cast<const d2v *>(in + io);
        v = d2v{p.alpha * v.x, p.alpha * v.y};
        d2v *o = reinterpret_cast<d2v *>(out + oo);
        if (p.beta != 0.0) {
          const d2v w = *o;
          v = d2v{v.x + p.beta * w.x, v.y + p.beta * w.y};
        }
        *o = v;
      }
      return;
    }
  }
  // element index -> (input, output) offsets; 32-bit division when the
  // whole tensor indexes in 32 bits (several times cheaper than 64-bit)
  const bool narrow = p.total < (int64_t(1) << 31);
  for (int64_t e = bid * CH + threadIdx.x; e < e1; e += 256) {
    int64_t io = 0, oo = 0;
    if (narrow) {
      uint32_t rem = uint32_t(e);
      for (int d = p.rank - 1; d >= 0; --d) {
        const uint32_t n = uint32_t(p.dims[d]), x = rem % n;
        rem /= n;
        io += int64_t(x) * p.istr[d];
        oo += int64_t(x) * p.ostr[d];
      }
    } else {
      int64_t rem = e;
      for (int d = p.rank - 1; d >= 0; --d) {
        const int64_t x = rem % p.dims[d];
        rem /= p.dims[d];
        io += x * p.istr[d];
        oo += x * p.ostr[d];
      }
    }
    T v = in[io];
    if (p.conj) v = cj(v);
    v = sc(p.alpha, v);
    if (p.beta != 0.0) v = add(v, sc(p.beta, out[oo]));
    out[oo] = v;
  }
}

// Tiled path: a TI x TO tile (TI TO = 1,024; 32 x 32 unless one of the two
// dims is shorter) over (input unit-stride dim, output unit-stride dim),
// read coalesced along the input's fast dim, written coalesced along the
// output's fast dim through a padded LDS tile.
template <class T, class Res = SamePtr>
__device__ __forceinline__ void perm_tiled_body(const PermEntry &E, int64_t bid, void *smem, Res rs = Res{}) {
  const PermArgs &p = E.p;
  const T *__restrict__ in = static_cast<const T *>(rs(E.in));
  T *__restrict__ out = static_cast<T *>(rs(E.out));
  T *tile = static_cast<T *>(smem);  // TO rows of TI + 1 (TO <= 256): 1,280 elements
  // workgroup -> tile (fewer than 2^31 of them, so every count fits 32 bits)
  uint32_t b = uint32_t(bid);
  const uint32_t nti = uint32_t(p.tiles_i), nto = uint32_t(p.tiles_o);
  const int64_t ti = b % nti; b /= nti;
  const int64_t to = b % nto; b /= nto;
  int64_t ib = 0, ob = 0;
  for (int d = p.nrest - 1; d >= 0; --d) {
    const uint32_t n = uint32_t(p.rest_dims[d]), x = b % n;
    b /= n;
    ib += int64_t(x) * p.rest_istr[d];
    ob += int64_t(x) * p.rest_ostr[d];
  }
  const int lti = p.lti, lto = 10 - lti, TI = 1 << lti, TO = 1 << lto;
  const int64_t Do = p.dims[p.d_o], Di = p.dims[p.d_i];
  const int64_t i0 = ti * TI, o0 = to * TO;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int t = threadIdx.x + 256 * k, ri = t & (TI - 1), ro = t >> lti;
    const int64_t xi = i0 + ri, xo = o0 + ro;
    if (xi < Di && xo < Do) tile[ro * (TI + 1) + ri] = in[ib + xi * p.istr[p.d_i] + xo * p.istr[p.d_o]];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int t = threadIdx.x + 256 * k, ro = t & (TO - 1), ri = t >> lto;
    const int64_t xo = o0 + ro, xi = i0 + ri;
    if (xi < Di && xo < Do) {
      T v = tile[ro * (TI + 1) + ri];
      if (p.conj) v = cj(v);
      v = sc(p.alpha, v);
      T *o = out + ob + xo * p.ostr[p.d_o] + xi * p.ostr[p.d_i];
      if (p.beta != 0.0) v = add(v, sc(p.beta, *o));
      *o = v;
    }
  }
}

// ------------------------------------------------------------ outer product --
// C[I] += alpha * A[sum_d I_d sa_d] * B[sum_d I_d sb_d]  (rank <= 4)
template <class T, class Res = SamePtr>
__device__ __forceinline__ void outer_body(const OuterEntry &E, int64_t bid, void *, Res rs = Res{}) {
  const OuterArgs &p = E.a;
  const T *__restrict__ A = static_cast<const T *>(rs(E.A));
  const T *__restrict__ B = static_cast<const T *>(rs(E.B));
  T *__restrict__ C = static_cast<T *>(rs(E.C));
  const int64_t e1 = std::min<int64_t>(E.total, (bid + 1) * CH);
  for (int64_t e = bid * CH + threadIdx.x; e < e1; e += 256) {
    int64_t rem = e, ia = 0, ibb = 0;
    for (int d = p.rank - 1; d >= 0; --d) {
      const int64_t quo = idiv(rem, p.dims[d]), x = rem - quo * p.dims[d];
      rem = quo;
      ia += x * p.sa[d];
      ibb += x * p.sb[d];
    }
    T a = A[ia], bb = B[ibb];
    if (p.conj_a) a = cj(a);
    if (p.conj_b) bb = cj(bb);
    C[e] = add(C[e], sc(p.alpha, mul(a, bb)));
  }
}

// ------------------------------------------------------------------- fill --
template <class T>
__device__ __forceinline__ void fill_body(const FillEntry &E, int64_t bid, void *) {
  T *__restrict__ p = static_cast<T *>(E.p);
  const int64_t e1 = std::min<int64_t>(E.n, (bid + 1) * CH);
  for (int64_t e = bid * CH + threadIdx.x; e < e1; e += 256) p[e] = zero<T>();
}

// ---------------------------------------------------------- split-K sum --
// C = alpha * sum_s W[s] + beta * C.  A workgroup covers 256 / lanes
// outputs; lane l of an output sums the partials s = l, l + lanes, ... in
// increasing order, then lane 0 adds the lanes' sums in lane order.  The
// order depends only on (split, lanes), never on timing.
template <class T>
__device__ __forceinline__ void splitk_body(const SplitkEntry &E, int64_t bid, void *smem) {
  T *part = static_cast<T *>(smem);
  const T *__restrict__ W = static_cast<const T *>(E.ws);
  T *__restrict__ C = static_cast<T *>(E.C);
  const int64_t total = E.M * E.N;
  const int L = E.lanes, nout = 256 / L;
  const int oi = threadIdx.x % nout, lane = threadIdx.x / nout;
  const int64_t e = bid * nout + oi;
  T acc = zero<T>();
  if (e < total)
    for (int k = lane; k < E.split; k += L) acc = add(acc, W[int64_t(k) * total + e]);
  part[threadIdx.x] = acc;
  __syncthreads();
  if (lane == 0 && e < total) {
    T sum = part[oi];
    for (int l = 1; l < L; ++l) sum = add(sum, part[l * nout + oi]);
    const int64_t m = idiv(e, E.N), n = e - m * E.N;
    T v = sc(E.alpha, sum);
    if (E.beta != 0.0) v = add(v, sc(E.beta, C[m * E.ldc + n]));
    C[m * E.ldc + n] = v;
  }
}

// --------------------------------------------------- tau + energy partials --
// tau = t2 + (t_i^a t_j^b - t_i^b t_j^a), taut = t2 + 1/2 (...),
// energy partial: 1/4 sum <ij||ab> tau_ij^ab  (+ sum f_ia t_i^a by unit 0).
template <class T, class Res = SamePtr>
__device__ __forceinline__ void tau_body(const TauEntry &E, int64_t bid, void *smem, Res rs = Res{}) {
  double *sh = static_cast<double *>(smem);
  const T *__restrict__ t1 = static_cast<const T *>(rs(E.t1));
  const T *__restrict__ t2 = static_cast<const T *>(rs(E.t2));
  const T *__restrict__ oovv = static_cast<const T *>(E.oovv);
  const T *__restrict__ fov = static_cast<const T *>(E.fov);
  T *__restrict__ tau = static_cast<T *>(E.tau);
  T *__restrict__ taut = static_cast<T *>(E.taut);
  const int o = E.o, v = E.v;
  const int64_t vv = int64_t(v) * v, total = int64_t(o) * o * vv;
  double er = 0.0, ei = 0.0;
  const int64_t e1 = std::min<int64_t>(total, (bid + 1) * CH_TAU);
  for (int64_t e = bid * CH_TAU + threadIdx.x; e < e1; e += RED_THREADS) {
    T x = t2[e];
    if (t1 != nullptr) {
      const int64_t ija = idiv(e, v);
      const int b = int(e - ija * v);
      const uint32_t ij = uint32_t(idiv(ija, v));
      const int a = int(ija - int64_t(ij) * v), i = ij / uint32_t(o), j = ij - uint32_t(i) * uint32_t(o);
      const T p = sub(mul(t1[i * v + a], t1[j * v + b]), mul(t1[i * v + b], t1[j * v + a]));
      const T full = add(x, p), half = add(x, sc(0.5, p));
      tau[e] = full;
      taut[e] = half;
      x = full;
    }
    const T w = mul(oovv[e], x);
    er += re(w);
    ei += im(w);
  }
  er = 0.25 * er;
  ei = 0.25 * ei;
  if (bid == 0 && t1 != nullptr) {
    for (int e = threadIdx.x; e < o * v; e += RED_THREADS) {
      const T w = mul(fov[e], t1[e]);
      er += re(w);
      ei += im(w);
    }
  }
  const double sr = block_sum(er, sh);
  const double si = block_sum(ei, sh);
  if (threadIdx.x == 0) {
    E.partials[2 * bid] = sr;
    E.partials[2 * bid + 1] = si;
  }
}

// ------------------------------------------- doubles residual + Jacobi ------
// R_ijab = XP + (Xij_ijab - Xij_jiab) + (Xab_ijab - Xab_ijba)
//        + ((Xr_ijab - Xr_jiab) - (Xr_ijba - Xr_jiba))
// evaluated once per canonical element (i < j, a < b) and written to its
// four images R_ijab = -R_jiab = -R_ijba = R_jiba; the diagonals i == j and
// a == b are exact zeros.  The amplitudes are updated the same way, so the
// result is bitwise antisymmetric whatever the rounding of the intermediates.
// One workgroup per (i <= j, 32-tile A <= 32-tile B); the (b,a)-ordered
// operands are read coalesced into padded LDS tiles, and the (b,a)-ordered
// images are written coalesced through an LDS tile.
__device__ __forceinline__ void tri_decode(int64_t k, int n, int &i, int &j) {
  int r = 0;
  while (k >= n - r) {
    k -= n - r;
    ++r;
  }
  i = r;
  j = r + int(k);
}

template <class T>
__device__ __forceinline__ void asm_body(const AsmEntry &E, int64_t bid, void *smem) {
  const R2Args &p = E.a;
  const T *__restrict__ XP = static_cast<const T *>(E.XP);
  const T *__restrict__ Xij = static_cast<const T *>(E.Xij);
  const T *__restrict__ Xab = static_cast<const T *>(E.Xab);
  const T *__restrict__ Xr = static_cast<const T *>(E.Xr);
  T *__restrict__ R = static_cast<T *>(E.R);
  T *__restrict__ t2 = static_cast<T *>(E.t2);
  double *partials = E.partials;
  typedef T Tile[32][33];
  Tile *tiles5 = static_cast<Tile *>(smem);
  Tile &sab = tiles5[0], &sr_ij = tiles5[1], &sr_ji = tiles5[2], &sv = tiles5[3], &st = tiles5[4];
  double *sh = reinterpret_cast<double *>(tiles5 + 5);
  const int o = p.o, v = p.v;
  const int tiles = (v + 31) / 32;
  const int64_t ntp = int64_t(tiles) * (tiles + 1) / 2;
  int ta, tb, i, j;
  const uint32_t pair = uint32_t(bid) / uint32_t(ntp);  // fewer than 2^31 workgroups
  tri_decode(uint32_t(bid) - pair * uint32_t(ntp), tiles, ta, tb);
  tri_decode(pair, o, i, j);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t vv = int64_t(v) * v;
  const int64_t base_ij = (int64_t(i) * o + j) * vv, base_ji = (int64_t(j) * o + i) * vv;
  const int a0 = ta * 32, b0 = tb * 32;
  const bool diag_tile = (ta == tb);
  double nrm = 0.0;
  if (i == j) {
    // the whole (i,i) block is zero: write both tile orientations
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int aa = a0 + ty + 8 * k, bb = b0 + tx;
      if (aa < v && bb < v) {
        if (R != nullptr) {
          R[base_ij + int64_t(aa) * v + bb] = zero<T>();
          R[base_ij + int64_t(bb) * v + aa] = zero<T>();
        }
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int bb = b0 + ty + 8 * k, aa = a0 + tx;
      if (bb < v && aa < v) {
        const int64_t off = int64_t(bb) * v + aa;
        sab[ty + 8 * k][tx] = Xab[base_ij + off];
        sr_ij[ty + 8 * k][tx] = Xr[base_ij + off];
        sr_ji[ty + 8 * k][tx] = Xr[base_ji + off];
      }
    }
    __syncthreads();
    const double *d_oo = p.fdiag_o, *d_vv = p.fdiag_v;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int la = ty + 8 * k, lb = tx;
      const int aa = a0 + la, bb = b0 + lb;
      const bool canon = aa < v && bb < v && (!diag_tile || aa < bb);
      T r = zero<T>(), tn = zero<T>();
      if (canon) {
        const int64_t e = base_ij + int64_t(aa) * v + bb, e_ji = base_ji + int64_t(aa) * v + bb;
        const T g_ij = sub(Xij[e], Xij[e_ji]);
        const T g_ab = sub(Xab[e], sab[lb][la]);
        const T g_r = sub(sub(Xr[e], Xr[e_ji]), sub(sr_ij[lb][la], sr_ji[lb][la]));
        r = add(add(add(XP[e], g_ij), g_ab), g_r);
        nrm += 4.0 * abs2(r);
        if (R != nullptr) {
          R[e] = r;
          R[e_ji] = sc(-1.0, r);
        }
        if (t2 != nullptr) {
          double D;
          if (p.dressed) {
            const T *Fo = static_cast<const T *>(p.Fo), *Fv = static_cast<const T *>(p.Fv);
            D = (re(Fo[int64_t(i) * o + i]) + re(Fo[int64_t(j) * o + j])) -
                (re(Fv[int64_t(aa) * v + aa]) + re(Fv[int64_t(bb) * v + bb]));
          } else {
            D = (d_oo[i] + d_oo[j]) - (d_vv[aa] + d_vv[bb]);
          }
          tn = add(t2[e], sc(1.0 / (D - p.shift), r));
          t2[e] = tn;
          t2[e_ji] = sc(-1.0, tn);
        }
      } else if (diag_tile && aa == bb && aa < v) {
        const int64_t e = base_ij + int64_t(aa) * v + bb, e_ji = base_ji + int64_t(aa) * v + bb;
        if (R != nullptr) {
          R[e] = zero<T>();
          R[e_ji] = zero<T>();
        }
      }
      sv[la][lb] = r;
      st[la][lb] = tn;
    }
    __syncthreads();
    // images with (b, a) order: rows b, columns a (coalesced along a)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int lb = ty + 8 * k, la = tx;
      const int aa = a0 + la, bb = b0 + lb;
      if (aa < v && bb < v && (!diag_tile || aa < bb)) {
        const int64_t e = base_ij + int64_t(bb) * v + aa, e_ji = base_ji + int64_t(bb) * v + aa;
        if (R != nullptr) {
          R[e] = sc(-1.0, sv[la][lb]);
          R[e_ji] = sv[la][lb];
        }
        if (t2 != nullptr) {
          t2[e] = sc(-1.0, st[la][lb]);
          t2[e_ji] = st[la][lb];
        }
      }
    }
  }
  const double s = block_sum(nrm, sh);
  if (threadIdx.x == 0) partials[bid] = s;
}


// ----------------------------------------------------------------- singles --
// R1 already assembled: norm partial and optional update.
template <class T>
__device__ __forceinline__ void r1_body(const R1Entry &E, void *smem) {
  double *sh = static_cast<double *>(smem);
  const T *__restrict__ R1 = static_cast<const T *>(E.R1);
  T *__restrict__ t1 = static_cast<T *>(E.t1);
  T *__restrict__ out = static_cast<T *>(E.out);
  const T *Fo = static_cast<const T *>(E.Fo), *Fv = static_cast<const T *>(E.Fv);
  const int o = E.o, v = E.v;
  double nrm = 0.0;
  for (int e = threadIdx.x; e < o * v; e += RED_THREADS) {
    const int i = e / v, a = e % v;
    const T r = R1[e];
    if (out != nullptr) out[e] = r;
    nrm += abs2(r);
    const double D = E.dressed ? re(Fo[int64_t(i) * o + i]) - re(Fv[int64_t(a) * v + a])
                               : E.d_oo[i] - E.d_vv[a];
    if (t1 != nullptr) t1[e] = add(t1[e], sc(1.0 / (D - E.shift), r));
  }
  const double s = block_sum(nrm, sh);
  if (threadIdx.x == 0) E.partial[0] = s;
}

// Packed index pairs, gathered (mode 0), added back (1) or scattered (2).
template <class T, class Res = SamePtr>
__device__ __forceinline__ void pair_body(const PairEntry &E, int64_t bid, void *, Res rs = Res{}) {
  const T *__restrict__ src = static_cast<const T *>(rs(E.src));
  T *__restrict__ dst = static_cast<T *>(rs(E.dst));
  const int64_t total = E.nP * E.nQ;
  const int64_t e1 = std::min<int64_t>(total, (bid + 1) * CH);
  for (int64_t e = bid * CH + threadIdx.x; e < e1; e += 256) {
    const int64_t P = idiv(e, E.nQ), Q = e - P * E.nQ;
    const int r0 = E.rows[2 * P], r1 = E.rows[2 * P + 1], c0 = E.cols[2 * Q], c1 = E.cols[2 * Q + 1];
    const int64_t q = ((int64_t(r0) * E.n1 + r1) * E.n2 + c0) * E.n3 + c1;
    const int64_t pe = P * E.ldq + Q;  // packed side
    if (E.mode == 0) dst[pe] = src[q];
    else if (E.mode == 1) dst[q] = add(dst[q], src[pe]);
    else dst[q] = src[pe];
  }
}

// Triples: R3 = sum over permutations (s of ijk, r of abc) of
// sign(s) sign(r) Y3[s(ijk)][r(abc)].
//
// Bound by HBM: Y3 read once, R3 written once, t3 read and written once.  One
// workgroup takes one i < j < k and one triple of 8-wide tiles ta <= tb <= tc.
// It sums the six ijk images of each of the six permuted abc tiles while
// loading them (runs of 8 along the last index; neighbouring tiles, which
// hold the other half of a 128-byte line, run on the same XCD), forms the
// antisymmetrised value of every (a, b, c) of the tile from LDS, and writes
// its 36 signed images tile by tile.  Reading all 36 images per element took
// 11.8 ms at o = 10, v = 40 (64e6 elements, 1 GB of compulsory traffic); the
// tiles take 0.22 ms (4.6 TB/s).  Blocks with a repeated occupied index are exact zeros,
// written by workgroups of their own.
constexpr int T3T = 8;                          // tile edge
constexpr int T3X = 93, T3Y = T3T + 1;          // LDS strides: any two of (93, 9, 1) spread over the banks
constexpr int64_t CH_T3 = 4096;                 // zeros per workgroup

__host__ __device__ __forceinline__ int64_t t3_tiles(int v) {
  const int64_t t = (v + T3T - 1) / T3T;
  return t * (t + 1) * (t + 2) / 6;
}
__host__ __device__ __forceinline__ int64_t t3_value_units(int o, int v) {
  return (int64_t(o) * (o - 1) * (o - 2) / 6) * t3_tiles(v);
}

template <class T>
__device__ __forceinline__ void t3_body(const T3Entry &E, int64_t bid, void *smem) {
  typedef T Cube[T3T * T3X];
  Cube *S = static_cast<Cube *>(smem), &V = S[6];
  double *sh = reinterpret_cast<double *>(S + 7);
  const int o = E.o, v = E.v;
  const int64_t vvv = int64_t(v) * v * v;
  const T *__restrict__ Y = static_cast<const T *>(E.Y3);
  T *__restrict__ R = static_cast<T *>(E.R3);
  T *__restrict__ t3 = static_cast<T *>(E.t3);
  // the six permutations of three slots and their signs
  constexpr int P[6][3] = {{0, 1, 2}, {1, 2, 0}, {2, 0, 1}, {1, 0, 2}, {0, 2, 1}, {2, 1, 0}};
  constexpr double sgn[6] = {1, 1, 1, -1, -1, -1};
  const int64_t nval = t3_value_units(o, v);
  if (bid >= nval) {  // (i,i,k), (i,j,i), (i,j,j): zeros
    const int64_t nch = (vvv + CH_T3 - 1) / CH_T3, z = (bid - nval) / nch, c0 = ((bid - nval) % nch) * CH_T3;
    int i, j, k;
    if (z < int64_t(o) * o) {
      i = j = int(z / o);
      k = int(z % o);
    } else {
      const int64_t y = (z - int64_t(o) * o) / 2;
      i = int(y / (o - 1));
      j = int(y % (o - 1));
      if (j >= i) ++j;
      k = (z - int64_t(o) * o) % 2 ? j : i;
    }
    const int64_t base = ((int64_t(i) * o + j) * o + k) * vvv;
    const int64_t e1 = std::min<int64_t>(vvv, c0 + CH_T3);
    for (int64_t e = c0 + threadIdx.x; e < e1; e += RED_THREADS) {
      if (R != nullptr) R[base + e] = zero<T>();
      if (t3 != nullptr) t3[base + e] = zero<T>();
    }
    if (threadIdx.x == 0) E.partials[bid] = 0.0;
    return;
  }
  // neighbouring units (the last tile index fastest) on one XCD
  const int64_t u = xcd_remap(bid, nval);
  const int64_t ntt = t3_tiles(v);
  const int nt = (v + T3T - 1) / T3T;
  int h[3], tl[3];
  {
    int64_t x = u / ntt;  // i < j < k
    int i = 0;
    while (x >= int64_t(o - 1 - i) * (o - 2 - i) / 2) x -= int64_t(o - 1 - i) * (o - 2 - i) / 2, ++i;
    int j = i + 1;
    while (x >= o - 1 - j) x -= o - 1 - j, ++j;
    h[0] = i;
    h[1] = j;
    h[2] = j + 1 + int(x);
    x = u % ntt;  // ta <= tb <= tc
    int a = 0;
    while (x >= int64_t(nt - a) * (nt - a + 1) / 2) x -= int64_t(nt - a) * (nt - a + 1) / 2, ++a;
    int b = a;
    while (x >= nt - b) x -= nt - b, ++b;
    tl[0] = a;
    tl[1] = b;
    tl[2] = b + int(x);
  }
  int64_t hb[6];
#pragma unroll
  for (int s = 0; s < 6; ++s) hb[s] = ((int64_t(h[P[s][0]]) * o + h[P[s][1]]) * o + h[P[s][2]]) * vvv;

  // S[p] over tile (tl[P0], tl[P1], tl[P2]): the sum over the ijk images
#pragma unroll
  for (int p = 0; p < 6; ++p)
    for (int e = threadIdx.x; e < T3T * T3T * T3T; e += RED_THREADS) {
      const int x = e / (T3T * T3T), y = (e / T3T) % T3T, z = e % T3T;
      const int a = tl[P[p][0]] * T3T + x, b = tl[P[p][1]] * T3T + y, c = tl[P[p][2]] * T3T + z;
      T sum = zero<T>();
      if (a < v && b < v && c < v) {
        const int64_t off = (int64_t(a) * v + b) * v + c;
#pragma unroll
        for (int s = 0; s < 6; ++s) sum = add(sum, sc(sgn[s], Y[hb[s] + off]));
      }
      S[p][x * T3X + y * T3Y + z] = sum;
    }
  __syncthreads();
  // V(a, b, c), a in ta, b in tb, c in tc: antisymmetrised over abc
  for (int e = threadIdx.x; e < T3T * T3T * T3T; e += RED_THREADS) {
    const int x[3] = {e / (T3T * T3T), (e / T3T) % T3T, e % T3T};
    const int a = tl[0] * T3T + x[0], b = tl[1] * T3T + x[1], c = tl[2] * T3T + x[2];
    T val = zero<T>();
    if (a != b && b != c && a != c) {
#pragma unroll
      for (int p = 0; p < 6; ++p)
        val = add(val, sc(sgn[p], S[p][x[P[p][0]] * T3X + x[P[p][1]] * T3Y + x[P[p][2]]]));
    }
    V[x[0] * T3X + x[1] * T3Y + x[2]] = val;
  }
  __syncthreads();
  double nrm = 0.0;
#pragma unroll
  for (int p = 0; p < 6; ++p) {
    // tiles that coincide under this permutation were written by an earlier one
    bool dup = false;
#pragma unroll
    for (int r = 0; r < p; ++r)
      dup = dup || (tl[P[r][0]] == tl[P[p][0]] && tl[P[r][1]] == tl[P[p][1]] && tl[P[r][2]] == tl[P[p][2]]);
    if (dup) continue;
    for (int e = threadIdx.x; e < T3T * T3T * T3T; e += RED_THREADS) {
      const int y[3] = {e / (T3T * T3T), (e / T3T) % T3T, e % T3T};
      const int a = tl[P[p][0]] * T3T + y[0], b = tl[P[p][1]] * T3T + y[1], c = tl[P[p][2]] * T3T + y[2];
      if (a >= v || b >= v || c >= v) continue;
      int x[3];  // local indices in (ta, tb, tc) order
#pragma unroll
      for (int q = 0; q < 3; ++q) x[P[p][q]] = y[q];
      const T val = sc(sgn[p], V[x[0] * T3X + x[1] * T3Y + x[2]]);
      nrm += 6.0 * abs2(val);
      const int64_t off = (int64_t(a) * v + b) * v + c;
      const bool rep = a == b || b == c || a == c;
      double inv = 0.0;
      if (t3 != nullptr && !rep)
        inv = 1.0 / (E.d_oo[h[0]] + E.d_oo[h[1]] + E.d_oo[h[2]] - E.d_vv[a] - E.d_vv[b] - E.d_vv[c] - E.shift);
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        const T w = sc(sgn[s], val);
        if (R != nullptr) R[hb[s] + off] = w;
        if (t3 != nullptr) t3[hb[s] + off] = rep ? zero<T>() : add(t3[hb[s] + off], sc(inv, w));
      }
    }
  }
  const double tot = block_sum(nrm, sh);
  if (threadIdx.x == 0) E.partials[bid] = tot;
}

// scalars[0] = ||R||, scalars[1..2] = E (re, im); fixed summation order.
__device__ __forceinline__ void fin_body(const FinEntry &E, void *smem) {
  double *sh = static_cast<double *>(smem);
  double a = 0.0, b = 0.0, c = 0.0;
  for (int k = threadIdx.x; k < E.ne; k += RED_THREADS) {
    a += E.epart[2 * k];
    b += E.epart[2 * k + 1];
  }
  for (int k = threadIdx.x; k < E.nn; k += RED_THREADS) c += E.n2part[k];
  for (int k = threadIdx.x; k < E.nn3; k += RED_THREADS) c += E.n3part[k];
  const double sa = block_sum(a, sh), sb = block_sum(b, sh), scn = block_sum(c, sh);
  if (threadIdx.x == 0) {
    const double n2 = scn + (E.n1part ? E.n1part[0] : 0.0);
    E.scalars[0] = sqrt(n2);
    E.scalars[1] = sa;
    E.scalars[2] = sb;
    if (E.host != nullptr) {
      E.host[0] = sqrt(n2);
      E.host[1] = sa;
      E.host[2] = sb;
    }
  }
}

// LDS bytes of each body
template <class T> constexpr int kLdsTile = 1280 * int(sizeof(T));
template <class T> constexpr int kLdsPart = 256 * int(sizeof(T));
constexpr int kLdsSum = RED_THREADS * 8;
template <class T> constexpr int kLdsAsm = 5 * 32 * 33 * int(sizeof(T)) + kLdsSum;
template <class T> constexpr int kLdsT3 = 7 * T3T * T3X * int(sizeof(T)) + kLdsSum;

}  // namespace
}  // namespace ccmi
