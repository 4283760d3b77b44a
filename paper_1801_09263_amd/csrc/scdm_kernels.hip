// Selected columns of the density matrix (SCDM) on the grid orbitals.
//
// The localization step of Sec. 2 picks N grid points r_k greedily: each
// pick is the point where the column a_r = conj(psi(r)) of Psi^H (one
// entry per orbital) has the largest part outside the span of the columns
// already picked, i.e. column-pivoted QR of Psi^H.  The residual norms
// d(r) = |a_r|^2 - sum_k |q_k^H a_r|^2 are kept on the device and downdated
// with each new orthonormal direction q_k; no step returns to the host.
//
// Small grid sets: every step downdates every point (a matrix-vector
// product over the grids, read once) with the next pick's argmax.
//
// Large grid sets: d only falls, so a point whose last computed d lies
// below an exact current value cannot be the next pick, and it need not be
// downdated until then.  A refresh selects the points with d >= tau, tau
// chosen from a histogram so that at most LZ_MAX of them are taken, copies
// their columns into a compact buffer and applies the directions each has
// missed; steps then downdate only these (those still >= tau), and as long
// as their maximum stays >= tau it is the maximum over the grid, with the
// same index among equals.  When it falls below, the next refresh follows.
// 256 localized orbitals mixed by a rotation at 120^3: 9 refreshes, 4 of them
// over every point.  If that does not pay (more points in the top
// histogram bin than fit, as for orbitals of uniform density, or more than
// LZ_ZERO refreshes without a pick), every point is brought up to date and
// each later step downdates them all as for small sets.
//
// Grids are the workspace's orbital grids in the plan precision: complex
// (orbital-major, n^3 points each) or real (Gamma plans).  Sums and the
// directions q_k are FP64.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "internal.hpp"
#include "mfma.hpp"

namespace lace {

template <typename T> struct GridVal;
template <> struct GridVal<float2> {
  __device__ static double2 get(const float2* g, int64_t i) {
    const float2 v = g[i];
    return make_double2(v.x, v.y);
  }
};
template <> struct GridVal<double2> {
  __device__ static double2 get(const double2* g, int64_t i) { return g[i]; }
};
template <> struct GridVal<float> {
  __device__ static double2 get(const float* g, int64_t i) {
    return make_double2(g[i], 0.0);
  }
};
template <> struct GridVal<double> {
  __device__ static double2 get(const double* g, int64_t i) {
    return make_double2(g[i], 0.0);
  }
};

// The scalar of the directions: real for real grids.
template <typename G> struct Scal;
template <> struct Scal<float> { using S = double; };
template <> struct Scal<double> { using S = double; };
template <> struct Scal<float2> { using S = double2; };
template <> struct Scal<double2> { using S = double2; };

__device__ inline double to_s(float v, double) { return v; }
__device__ inline double to_s(double v, double) { return v; }
__device__ inline double2 to_s(float2 v, double2) { return make_double2(v.x, v.y); }
__device__ inline double2 to_s(double2 v, double2) { return v; }

__device__ inline double zero_s(double) { return 0.0; }
__device__ inline double2 zero_s(double2) { return make_double2(0.0, 0.0); }
__device__ inline double conj_s(double a) { return a; }
__device__ inline double2 conj_s(double2 a) { return make_double2(a.x, -a.y); }
// acc + a b
__device__ inline double mad(double a, double b, double acc) { return fma(a, b, acc); }
__device__ inline double2 mad(double2 a, double2 b, double2 acc) {
  acc.x = fma(a.x, b.x, acc.x);
  acc.x = fma(-a.y, b.y, acc.x);
  acc.y = fma(a.x, b.y, acc.y);
  acc.y = fma(a.y, b.x, acc.y);
  return acc;
}
__device__ inline double add_s(double a, double b) { return a + b; }
__device__ inline double2 add_s(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double sub_s(double a, double b) { return a - b; }
__device__ inline double2 sub_s(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double scl_s(double a, double f) { return a * f; }
__device__ inline double2 scl_s(double2 a, double f) { return make_double2(a.x * f, a.y * f); }
__device__ inline double norm_s(double a) { return a * a; }
__device__ inline double norm_s(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline double2 wave_sum(double2 v) {
  return make_double2(wave_sum(v.x), wave_sum(v.y));
}

struct ArgMax {
  double v;
  int64_t i;
};
// The largest value, the smallest index among equals.  Picked points hold
// -1 and are never chosen again.
__device__ inline ArgMax better(ArgMax a, ArgMax b) {
  if (b.v > a.v || (b.v == a.v && b.i < a.i)) return b;
  return a;
}

template <int NT>
__device__ inline ArgMax block_argmax(ArgMax m) {
  __shared__ double sv[NT / 64];
  __shared__ int64_t si[NT / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ArgMax t;
    t.v = __shfl_xor(m.v, o, 64);
    t.i = __shfl_xor(m.i, o, 64);
    m = better(m, t);
  }
  if (threadIdx.x % 64 == 0) {
    sv[threadIdx.x / 64] = m.v;
    si[threadIdx.x / 64] = m.i;
  }
  __syncthreads();
  m.v = sv[0];
  m.i = si[0];
  for (int w = 1; w < NT / 64; ++w) m = better(m, ArgMax{sv[w], si[w]});
  __syncthreads();
  return m;
}

constexpr int AM_NT = 256;
constexpr int AM_BLOCKS = 1024;   // block-wise maxima: one per thread of the pick

// A vector of VW consecutive points of one grid, 16 bytes where aligned.
template <typename G, int VW> struct GridVec {
  G v[VW];
};
template <typename G, int VW>
__device__ inline GridVec<G, VW> ldgrid(const G* p) {
  GridVec<G, VW> r;
  if constexpr (VW * sizeof(G) == 16) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    __builtin_memcpy(&r, &t, 16);
  } else {
#pragma unroll
    for (int e = 0; e < VW; ++e) r.v[e] = p[e];
  }
  return r;
}

// use(n, ld(n)) for n = n0, n0 + step, ... < n1, in that order, with U loads
// issued before the first of them is used, the rest in rounds of half as
// many.  The order is pinned: left to itself the compiler put each load of an
// unrolled loop right before its use, one in flight at a time.  Whole call, so
// -> pinned: 24^3 with 450 complex FP64 orbitals 121 -> 46 ms, 300 real FP32 14.8
// -> 10.0, 48^3 with 200 complex FP32 19.2 -> 10.3, 64^3 with 64 real FP32 2.05 ->
// 1.77.
template <int U, class Ld, class Use>
__device__ __forceinline__ void in_flight(int n0, int n1, int step, Ld ld, Use use) {
  decltype(ld(0)) v[U];
  int n = n0;
  for (; n + (U - 1) * step < n1; n += U * step) {
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = ld(n + u * step);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) use(n + u * step, v[u]);
  }
  if constexpr (U > 4) {
    in_flight<U / 2>(n, n1, step, ld, use);
  } else {
    if (n >= n1) return;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (n + u * step < n1) v[u] = ld(n + u * step);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (n + u * step < n1) use(n + u * step, v[u]);
  }
}

// Loads in flight per thread: two 16-byte ones on the grids that fill the chip,
// where more only spread the accesses over more grids (16 / 4 / 2, whole call:
// complex FP64 64^3 with 40 orbitals 2.02 / 1.79 / 1.74 ms, 120^3 with 7 557 / 556
// / 546 us; one in flight costs 96^3 with 64 complex FP32 plane waves 8.08 for
// 7.28 ms), sixteen on smaller ones, whose waves do not (16 / 8 / 4: 24^3 with
// 450 complex FP64 46.2 / 49.3 / 55.5 ms, 48^3 with 200 complex FP32 within 3%).
constexpr int VEC_U = 2;
constexpr int SMALL_U = 16;

// d(r) = sum_n |psi_n(r)|^2 (the diagonal of the density matrix), with
// block-wise maxima of it; points <- 0, and missed <- 0 where given.
template <typename G, int VW, int U>
__global__ __launch_bounds__(AM_NT) void k_scdm_density(
    const G* psi, int n_orb, int64_t ng, double* d, uint16_t* missed,
    int32_t* points, double* pv, int64_t* pi) {
  using S = typename Scal<G>::S;
  ArgMax m{-2.0, 0};
  const int64_t stride = int64_t(gridDim.x) * AM_NT * VW;
  for (int64_t r0 = (blockIdx.x * int64_t(AM_NT) + threadIdx.x) * VW; r0 < ng;
       r0 += stride) {
    double s[VW];
#pragma unroll
    for (int e = 0; e < VW; ++e) s[e] = 0.0;
    in_flight<U>(0, n_orb, 1, [&](int n) { return ldgrid<G, VW>(psi + n * ng + r0); },
                 [&](int, const GridVec<G, VW>& g) {
#pragma unroll
                   for (int e = 0; e < VW; ++e) s[e] += norm_s(to_s(g.v[e], S{}));
                 });
#pragma unroll
    for (int e = 0; e < VW; ++e) {
      d[r0 + e] = s[e];
      if (missed) missed[r0 + e] = 0;
      m = better(m, ArgMax{s[e], r0 + e});
    }
  }
  if (blockIdx.x == 0)
    for (int k = threadIdx.x; k < n_orb; k += AM_NT) points[k] = 0;
  m = block_argmax<AM_NT>(m);
  if (threadIdx.x == 0) {
    pv[blockIdx.x] = m.v;
    pi[blockIdx.x] = m.i;
  }
}

// Rows of Q and QT are padded to whole 16-byte vectors.
template <typename S> __host__ __device__ constexpr int q_ld(int n_orb) {
  return sizeof(S) == 8 ? (n_orb + 1) & ~1 : n_orb;
}

// out(y, sum over x < nx of A[x ld + y] v[x]) for every y < ny (conj(A)
// when CJ), by one thread each.  A thread takes the 16-byte vector of VS
// columns at y and, when NT allows, one of ngrp shares of x; the shares'
// sums meet in part (NT VS scalars).  Every load is coalesced over y and
// depends on no other.
template <bool CJ, int NT, class S, class Out>
__device__ __forceinline__ void colsum(const S* A, int ld, int nx, int ny, const S* v,
                              S* part, Out out) {
  constexpr int VS = 16 / (int)sizeof(S);
  const int tid = threadIdx.x;
  const int nv = (ny + VS - 1) / VS;     // vectors
  // at most 8 shares: their sums are added one after the other
  const int ngrp = NT / nv < 1 ? 1 : NT / nv > 8 ? 8 : NT / nv;
  for (int y0 = 0; y0 < nv; y0 += NT) {  // more than one round only for ngrp = 1
    const int yv = y0 + (ngrp > 1 ? tid % nv : tid), g = ngrp > 1 ? tid / nv : 0;
    S sm[VS];
#pragma unroll
    for (int e = 0; e < VS; ++e) sm[e] = zero_s(S{});
    const bool on = yv < nv && g < ngrp;
    if (on) {
      in_flight<NT == 256 ? 8 : 16>(g, nx, ngrp,
                    [&](int x) { return ldgrid<S, VS>(A + (int64_t)x * ld + yv * VS); },
                    [&](int x, const GridVec<S, VS>& a) {
                      const S vx = v[x];
#pragma unroll
                      for (int e = 0; e < VS; ++e)
                        sm[e] = mad(CJ ? conj_s(a.v[e]) : a.v[e], vx, sm[e]);
                    });
    }
    if (ngrp > 1) {
      if (on) {
#pragma unroll
        for (int e = 0; e < VS; ++e) part[(g * nv + yv) * VS + e] = sm[e];
      }
      __syncthreads();
      for (int y = tid; y < ny; y += NT) {
        S t = part[y];
        for (int q = 1; q < ngrp; ++q) t = add_s(t, part[q * nv * VS + y]);
        out(y, t);
      }
    } else if (on) {
#pragma unroll
      for (int e = 0; e < VS; ++e)
        if (yv * VS + e < ny) out(yv * VS + e, sm[e]);
    }
  }
  __syncthreads();
}

// q_k: the picked column a = conj(psi(r)) made orthogonal to q_0..q_{k-1}
// (classical Gram-Schmidt, twice) and normalized; Q row-major, q_m = Q[m][.],
// and QT its transpose.  One workgroup of NT threads; us, hs: n_orb scalars
// of LDS each, part: NT 16-byte vectors more.  h = Q^H u sums over rows of QT, u -= Q h over
// rows of Q, so that lanes walk the result and no cross-lane sum is needed
// (a wave per h_m with a shuffle sum took 55 us at k = 250 of 256 real
// directions).  Bound by the latency of L2 and one CU's
// share of it.
template <typename G, int NT>
__device__ __forceinline__ void scdm_direction(const G* psi, int n_orb, int64_t ng, int64_t r,
                               int k, typename Scal<G>::S* Q,
                               typename Scal<G>::S* QT,
                               typename Scal<G>::S* lds, double* red) {
  using S = typename Scal<G>::S;
  S* us = lds;
  S* hs = lds + n_orb;
  S* part = lds + 2 * n_orb;   // any alignment: scalar accesses
  const int tid = threadIdx.x, lane = tid % 64, wv = tid / 64;
  for (int n = tid; n < n_orb; n += NT) us[n] = conj_s(to_s(psi[n * ng + r], S{}));
  __syncthreads();
  const int ld = q_ld<S>(n_orb);
  for (int pass = 0; k > 0 && pass < 2; ++pass) {
    colsum<true, NT>(QT, ld, n_orb, k, us, part, [&](int m, S v) { hs[m] = v; });
    colsum<false, NT>(Q, ld, k, n_orb, hs, part,
                      [&](int n, S v) { us[n] = sub_s(us[n], v); });
  }
  double t = 0.0;
  for (int n = tid; n < n_orb; n += NT) t += norm_s(us[n]);
  t = wave_sum(t);
  if (lane == 0) red[wv] = t;
  __syncthreads();
  double nrm = 0.0;
  for (int w = 0; w < NT / 64; ++w) nrm += red[w];
  const double inv = nrm > 0.0 ? 1.0 / sqrt(nrm) : 0.0;
  for (int n = tid; n < n_orb; n += NT) {
    const S v = scl_s(us[n], inv);
    Q[(int64_t)k * ld + n] = v;
    QT[(int64_t)n * ld + k] = v;
  }
}

// Pick k from the block-wise maxima, then (unless it is the last) q_k.
template <typename G, int NT>
__global__ __launch_bounds__(NT) void k_scdm_pick(
    const G* psi, int n_orb, int64_t ng, const double* pv, const int64_t* pi,
    int nparts, double* d, int32_t* points, int k, typename Scal<G>::S* Q,
    typename Scal<G>::S* QT) {
  using S = typename Scal<G>::S;
  extern __shared__ double2 lds[];
  __shared__ double red[NT / 64];
  ArgMax m{-2.0, 0};
  for (int b = threadIdx.x; b < nparts; b += NT) m = better(m, ArgMax{pv[b], pi[b]});
  m = block_argmax<NT>(m);
  if (threadIdx.x == 0) {
    points[k] = (int32_t)m.i;
    d[m.i] = -1.0;
  }
  if (k + 1 == n_orb) return;
  scdm_direction<G, NT>(psi, n_orb, ng, m.i, k, Q, QT, reinterpret_cast<S*>(lds),
                            red);
}

// d(r) -= |q_k^H a_r|^2 = |sum_n q_kn psi_n(r)|^2 for every point not yet
// taken, with the next pick's block-wise argmax.  A thread takes VW
// consecutive points, one 16-byte load per orbital.  q: q_k in LDS.
template <typename G, int VW, int U>
__device__ __forceinline__ ArgMax downdate_all(const G* psi, int n_orb, int64_t ng,
                               const typename Scal<G>::S* q, double* d) {
  using S = typename Scal<G>::S;
  ArgMax m{-2.0, 0};
  const int64_t stride = int64_t(gridDim.x) * AM_NT * VW;
  for (int64_t r0 = (blockIdx.x * int64_t(AM_NT) + threadIdx.x) * VW; r0 < ng;
       r0 += stride) {
    S s[VW];
#pragma unroll
    for (int e = 0; e < VW; ++e) s[e] = zero_s(S{});
    in_flight<U>(0, n_orb, 1, [&](int n) { return ldgrid<G, VW>(psi + n * ng + r0); },
                 [&](int n, const GridVec<G, VW>& g) {
                   const S qn = q[n];
#pragma unroll
                   for (int e = 0; e < VW; ++e) s[e] = mad(qn, to_s(g.v[e], S{}), s[e]);
                 });
#pragma unroll
    for (int e = 0; e < VW; ++e) {
      const double old = d[r0 + e];
      double nv = old;
      if (old >= 0.0) {
        nv = fmax(old - norm_s(s[e]), 0.0);
        d[r0 + e] = nv;
      }
      m = better(m, ArgMax{nv, r0 + e});
    }
  }
  return m;
}

template <typename G, int VW, int U>
__global__ __launch_bounds__(AM_NT) void k_scdm_downdate(
    const G* psi, int n_orb, int64_t ng, const typename Scal<G>::S* Q, int k,
    double* d, double* pv, int64_t* pi) {
  using S = typename Scal<G>::S;
  extern __shared__ double2 lds[];
  S* qs = reinterpret_cast<S*>(lds);
  for (int n = threadIdx.x; n < n_orb; n += AM_NT) qs[n] = Q[(int64_t)k * q_ld<S>(n_orb) + n];
  __syncthreads();
  const ArgMax m = block_argmax<AM_NT>(downdate_all<G, VW, U>(psi, n_orb, ng, qs, d));
  if (threadIdx.x == 0) {
    pv[blockIdx.x] = m.v;
    pi[blockIdx.x] = m.i;
  }
}

// --------------------------------------------------- lazy point selection
constexpr int LZ_MAX = 65536;      // selected points at most
constexpr int LZ_PTS = 64;         // selected points per workgroup
constexpr int LZ_BLOCKS = AM_BLOCKS;   // workgroups of the downdates
constexpr int LZ_ZERO = 8;         // refreshes without a pick before all points
constexpr int LZ_FRESH = 24;       // directions after which a refresh updates all
constexpr int LZ_BINS = 2048;      // 64 octaves of 32 bins from 2^-40
constexpr long long LZ_BASE = (1023ll - 40ll) << 5;

struct LazyCtl {
  double tau, tau2;    // current selection bound; the refresh's new one
  int32_t k;           // picks made
  int32_t picked;      // this tick made a pick (and its direction)
  int32_t refreshed;   // this tick refreshed
  int32_t full;        // every point is up to date and downdated
  int32_t want_full;   // the next refresh takes every point
  int32_t zero;        // refreshes without a pick
  int32_t count;       // selected points
  int32_t fresh;       // directions applied to every point
  int32_t hist[LZ_BINS];
};

// Bin of d >= 0: monotone, and d >= lz_edge(b) exactly when lz_key(d) >= b.
__device__ inline int lz_key(double d) {
  const long long b = (__double_as_longlong(d) >> 47) - LZ_BASE;
  return b < 0 ? 0 : b >= LZ_BINS ? LZ_BINS - 1 : (int)b;
}
__device__ inline double lz_edge(int b) {
  return b <= 0 ? 0.0 : __longlong_as_double((b + LZ_BASE) << 47);
}

// Whether this tick starts with a refresh: the selected points' maximum
// fell below tau.  Every workgroup evaluates it from the block-wise maxima.
__device__ inline bool lz_need(const LazyCtl* c, const double* pv, int n_orb) {
  if (c->full || c->k >= n_orb) return false;
  const double tau = c->tau;
  bool any = false;
  for (int b = threadIdx.x; b < LZ_BLOCKS; b += blockDim.x) any |= pv[b] >= tau;
  return !__syncthreads_or(any);
}

__global__ void k_lazy_init(LazyCtl* c, double* pv) {
  for (int b = threadIdx.x; b < LZ_BINS; b += blockDim.x) c->hist[b] = 0;
  for (int b = threadIdx.x; b < LZ_BLOCKS; b += blockDim.x) pv[b] = -2.0;
  if (threadIdx.x == 0) {
    c->tau = 0.0;
    c->tau2 = 0.0;
    c->k = c->picked = c->refreshed = c->full = c->want_full = c->zero = c->count = c->fresh = 0;
  }
}

// The directions [s, k) that 16 MP points have missed, applied to their d by
// one wave on the matrix cores: q_m^T psi for 16 directions m at a time.
// Lane l supplies QT[n + l / 16][m0 + l % 16] and the entry of orbital n +
// l / 16 at point l % 16 of each 16; col + n ld: those entries, the last at
// position `last`.  on, dv, s:
// lane l's point l % 16 of each 16 (the four lanes of a point agree).
// Directions below a point's own s are computed and not applied.
// Blocks of 16 directions start at multiples of 16 and are subtracted one
// by one, so that a point's d depends on its own s and k alone and not on
// the points that share its wave.
template <typename S> constexpr int CU_MP = 2;

// MD blocks from direction kb on.  The entries of the next four orbitals are
// read while the matrix cores work on these four.
template <int MD, typename G>
__device__ __forceinline__ void catch_up_blocks(const G* col, int64_t ld, int last,
                                                int n_orb,
                                                const typename Scal<G>::S* QT,
                                                int kb, int k, double* dv,
                                                const int* s) {
  using S = typename Scal<G>::S;
  constexpr bool CX = sizeof(S) == 16;
  constexpr int MP = CU_MP<S>;
  const int lane = threadIdx.x & 63, l16 = lane & 15, g4 = lane >> 4;
  const int ldq = q_ld<S>(n_orb);
  d4 re[MD][MP], im[CX ? MD : 1][MP];
#pragma unroll
  for (int a = 0; a < MD; ++a)
#pragma unroll
    for (int j = 0; j < MP; ++j) {
      re[a][j] = d4{0, 0, 0, 0};
      if (CX) im[a][j] = d4{0, 0, 0, 0};
    }
  G x[MP];
  S q[MD];
  // every load runs: past the last orbital or direction a valid entry is
  // read and its factor zeroed, past the last point one that is not used
  auto fetch = [&](int n0) {
    const int n = min(n0 + g4, n_orb - 1);
#pragma unroll
    for (int j = 0; j < MP; ++j) x[j] = col[(int64_t)n * ld + min(16 * j + l16, last)];
#pragma unroll
    for (int a = 0; a < MD; ++a)
      q[a] = QT[(int64_t)n * ldq + min(kb + 16 * a + l16, k - 1)];
  };
  fetch(0);
  for (int n0 = 0; n0 < n_orb; n0 += 4) {
    S xc[MP], qc[MD];
#pragma unroll
    for (int j = 0; j < MP; ++j) xc[j] = to_s(x[j], S{});
#pragma unroll
    for (int a = 0; a < MD; ++a)
      qc[a] = n0 + g4 < n_orb && kb + 16 * a + l16 < k ? q[a] : zero_s(S{});
    fetch(n0 + 4);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int a = 0; a < MD; ++a)
#pragma unroll
      for (int j = 0; j < MP; ++j) {
        if constexpr (CX) {
          re[a][j] = mfma(qc[a].x, xc[j].x, re[a][j]);
          im[a][j] = mfma(qc[a].x, xc[j].y, im[a][j]);
          re[a][j] = mfma(-qc[a].y, xc[j].y, re[a][j]);
          im[a][j] = mfma(qc[a].y, xc[j].x, im[a][j]);
        } else {
          re[a][j] = mfma(qc[a], xc[j], re[a][j]);
        }
      }
  }
#pragma unroll
  for (int j = 0; j < MP; ++j)
#pragma unroll
    for (int a = 0; a < MD; ++a) {
      double sum = 0.0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = kb + 16 * a + g4 + 4 * e;
        double v = re[a][j][e] * re[a][j][e];
        if (CX) v += im[a][j][e] * im[a][j][e];
        if (m >= s[j] && m < k) sum += v;
      }
      sum += __shfl_xor(sum, 16, 64);
      sum += __shfl_xor(sum, 32, 64);
      if (dv[j] >= 0.0) dv[j] = fmax(dv[j] - sum, 0.0);
    }
}

template <typename G>
__device__ inline void catch_up(const G* col, int64_t ld, int last, int n_orb,
                                const typename Scal<G>::S* QT, int k,
                                const bool* on, double* dv, const int* s) {
  int smin = k;
#pragma unroll
  for (int j = 0; j < CU_MP<typename Scal<G>::S>; ++j)
    if (on[j] && dv[j] >= 0.0) smin = min(smin, s[j]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) smin = min(smin, __shfl_xor(smin, o, 64));
  if (smin >= k) return;
  int kb = smin & ~15;
  for (; k - kb > 48; kb += 64) catch_up_blocks<4, G>(col, ld, last, n_orb, QT, kb, k, dv, s);
  if (k - kb > 32) catch_up_blocks<3, G>(col, ld, last, n_orb, QT, kb, k, dv, s);
  else if (k - kb > 16) catch_up_blocks<2, G>(col, ld, last, n_orb, QT, kb, k, dv, s);
  else if (k - kb > 0) catch_up_blocks<1, G>(col, ld, last, n_orb, QT, kb, k, dv, s);
}

// A refresh's histogram of d.  When LZ_FRESH directions or more have come
// since every point was last up to date (or every point is wanted), first
// the directions each point missed, read from the grids: d then ranks the
// points as they are, and the selection that follows lasts for many picks
// (256 rotated localized orbitals at 120^3: 9 refreshes, 4 of them over
// every point, where 37 were needed without, each with up to 250 missed
// directions of 65,536 points).
template <typename G>
__global__ __launch_bounds__(AM_NT) void k_lazy_hist(
    const G* psi, int n_orb, int64_t ng, LazyCtl* c, const typename Scal<G>::S* QT,
    double* d, uint16_t* missed, const double* pv) {
  __shared__ int32_t h[LZ_BINS];
  if (!lz_need(c, pv, n_orb)) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int k = c->k;
  const bool all = k > c->fresh && (c->want_full || k - c->fresh >= LZ_FRESH);
  if (blockIdx.x == 0 && tid == 0) c->count = 0;   // the new list's
  for (int b = tid; b < LZ_BINS; b += AM_NT) h[b] = 0;
  __syncthreads();
  constexpr int MP = CU_MP<typename Scal<G>::S>, TP = 16 * MP;
  const int64_t tiles = (ng + TP - 1) / TP;
  const int64_t stride = (int64_t)gridDim.x * (AM_NT / 64);
  for (int64_t t = blockIdx.x * (int64_t)(AM_NT / 64) + wv; t < tiles; t += stride) {
    const int64_t p0 = t * TP;
    if (all) {
      double dv[MP];
      int s[MP];
      bool on[MP];
#pragma unroll
      for (int j = 0; j < MP; ++j) {
        const int64_t p = p0 + 16 * j + (lane & 15);
        on[j] = p < ng;
        dv[j] = on[j] ? d[p] : -1.0;
        s[j] = on[j] ? missed[p] : k;
      }
      catch_up<G>(psi + p0, ng, (int)min((int64_t)TP - 1, ng - 1 - p0), n_orb, QT, k, on, dv, s);
#pragma unroll
      for (int j = 0; j < MP; ++j) {
        const int64_t p = p0 + 16 * j + (lane & 15);
        if (on[j] && lane < 16) {
          d[p] = dv[j];
          missed[p] = (uint16_t)k;
          if (dv[j] >= 0.0) atomicAdd(&h[lz_key(dv[j])], 1);
        }
      }
    } else if (lane < TP && p0 + lane < ng) {
      const double v = d[p0 + lane];
      if (v >= 0.0) atomicAdd(&h[lz_key(v)], 1);
    }
  }
  __syncthreads();
  for (int b = tid; b < LZ_BINS; b += AM_NT)
    if (h[b]) atomicAdd(&c->hist[b], h[b]);
}

// The new bound and the list of points at or above it (any order: only
// values and indices decide).  cap: points that may be selected.
__global__ __launch_bounds__(AM_NT) void k_lazy_select(LazyCtl* c, const double* pv,
                                                       const double* d, int64_t ng,
                                                       int n_orb, int cap,
                                                       int32_t* list) {
  __shared__ int32_t part[AM_NT];
  __shared__ int32_t s_bin, s_over, s_base, s_wave[AM_NT / 64];
  if (!lz_need(c, pv, n_orb)) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  constexpr int PER = LZ_BINS / AM_NT;
  // bins from the top: thread t owns bins LZ_BINS - 1 - t PER, downwards
  int32_t own = 0;
  for (int e = 0; e < PER; ++e) own += c->hist[LZ_BINS - 1 - tid * PER - e];
  part[tid] = own;
  if (tid == 0) { s_bin = LZ_BINS; s_over = 0; }
  __syncthreads();
  if (tid == 0) {
    int64_t sum = 0;   // points in the bins taken
    int bin = LZ_BINS, t = 0;
    while (t < AM_NT && sum + part[t] <= cap) { sum += part[t]; ++t; bin -= PER; }
    if (t < AM_NT)
      for (int e = 0; e < PER; ++e) {
        const int64_t nx = sum + c->hist[bin - 1];
        if (nx > cap) break;
        sum = nx;
        --bin;
      }
    s_bin = bin;
    s_over = (sum == 0 || c->want_full) ? 1 : 0;
  }
  __syncthreads();
  const int bin = s_bin;
  const bool over = s_over;
  if (blockIdx.x == 0 && tid == 0) {
    // every point, from here on, once they are up to date (k_lazy_hist sees
    // to that in the next tick when they are not)
    const bool fresh = c->k == c->fresh || c->want_full || c->k - c->fresh >= LZ_FRESH;
    c->refreshed = over ? (fresh ? 2 : 0) : 1;
    if (over) c->want_full = 1;
    c->tau2 = over ? -1.0 : lz_edge(bin);
  }
  if (over) return;
  // this workgroup's contiguous share: count, reserve once, write
  const int64_t per = (ng + gridDim.x - 1) / gridDim.x;
  const int64_t lo = blockIdx.x * per, hi = min(lo + per, ng);
  int mine = 0;
  for (int64_t r = lo + tid; r < hi; r += AM_NT) {
    const double v = d[r];
    mine += v >= 0.0 && lz_key(v) >= bin;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o, 64);
  if (lane == 0) s_wave[wv] = mine;
  __syncthreads();
  if (tid == 0) {
    int t = 0;
    for (int w = 0; w < AM_NT / 64; ++w) t += s_wave[w];
    s_base = t ? atomicAdd(&c->count, t) : 0;
  }
  __syncthreads();
  // each wave writes its own 64-point pieces, in wave order
  int at = s_base;
  for (int w = 0; w < wv; ++w) at += s_wave[w];
  for (int64_t r0 = lo + 64 * wv; r0 < hi; r0 += AM_NT) {
    const int64_t r = r0 + lane;
    const double v = r < hi ? d[r] : -1.0;
    const bool take = v >= 0.0 && lz_key(v) >= bin;
    const unsigned long long bal = __ballot(take);
    if (take) list[at + __popcll(bal & ((1ull << lane) - 1ull))] = (int32_t)r;
    at += __popcll(bal);
  }
}

// The refresh's last part.  A wave takes TP selected points: their columns
// go to buf (orbital n's entries at buf + n cap), then the directions they
// missed are applied.  With every point taken (up to date then): their
// maxima.
template <typename G>
__global__ __launch_bounds__(AM_NT) void k_lazy_gather(
    const G* psi, int n_orb, int64_t ng, const LazyCtl* c, const int32_t* list,
    int cap, G* buf, const typename Scal<G>::S* QT, double* d, uint16_t* missed,
    double* pv, int64_t* pi) {
  constexpr int MP = CU_MP<typename Scal<G>::S>, TP = 16 * MP;
  if (!c->refreshed) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int k = c->k;
  ArgMax best{-2.0, 0};
  if (c->refreshed == 2) {
    const int64_t stride = int64_t(gridDim.x) * AM_NT;
    for (int64_t r = blockIdx.x * int64_t(AM_NT) + tid; r < ng; r += stride)
      best = better(best, ArgMax{d[r], r});
  } else {
    const int count = c->count, tiles = (count + TP - 1) / TP;
    for (int t = blockIdx.x * (AM_NT / 64) + wv; t < tiles; t += gridDim.x * (AM_NT / 64)) {
      const int p0 = t * TP;
      const int pc = p0 + lane % TP;   // 64 / TP rows of TP points per step
      if (pc < count) {
        const int64_t r = list[pc];
        in_flight<16>(lane / TP, n_orb, 64 / TP, [&](int n) { return psi[n * ng + r]; },
                      [&](int n, const G& g) { buf[(int64_t)n * cap + pc] = g; });
      }
      __threadfence_block();   // read back by other lanes of the wave
      int64_t r[MP];
      double dv[MP];
      int s[MP];
      bool on[MP];
#pragma unroll
      for (int j = 0; j < MP; ++j) {
        const int p = p0 + 16 * j + (lane & 15);
        on[j] = p < count;
        r[j] = on[j] ? list[p] : 0;
        dv[j] = on[j] ? d[r[j]] : -1.0;
        s[j] = on[j] ? missed[r[j]] : k;
      }
      catch_up<G>(buf + p0, cap, min(TP - 1, count - 1 - p0), n_orb, QT, k, on, dv, s);
#pragma unroll
      for (int j = 0; j < MP; ++j)
        if (on[j]) {
          if (lane < 16) {
            d[r[j]] = dv[j];
            missed[r[j]] = (uint16_t)k;
          }
          best = better(best, ArgMax{dv[j], r[j]});
        }
    }
  }
  best = block_argmax<AM_NT>(best);
  if (tid == 0) {
    pv[blockIdx.x] = best.v;
    pi[blockIdx.x] = best.i;
  }
}

// One tick's pick: adopt a refresh, then take the selected points' maximum
// if it is at or above the bound, and form its direction.
template <typename G, int NT>
__global__ __launch_bounds__(NT) void k_lazy_pick(
    const G* psi, int n_orb, int64_t ng, LazyCtl* c, const double* pv,
    const int64_t* pi, double* d, int32_t* points, typename Scal<G>::S* Q,
    typename Scal<G>::S* QT) {
  using S = typename Scal<G>::S;
  extern __shared__ double2 lds[];
  __shared__ double red[NT / 64];
  const int k = c->k, fresh = c->refreshed;
  const double tau = fresh ? c->tau2 : c->tau;
  const bool full = c->full || fresh == 2;
  // as k_lazy_hist decided
  const bool all = fresh && k > c->fresh && (c->want_full || k - c->fresh >= LZ_FRESH);
  __syncthreads();   // every thread has read the control block
  ArgMax m{-2.0, 0};
  for (int b = threadIdx.x; b < LZ_BLOCKS; b += NT) m = better(m, ArgMax{pv[b], pi[b]});
  m = block_argmax<NT>(m);
  const bool pick = k < n_orb && (full || m.v >= tau);
  for (int b = threadIdx.x; b < LZ_BINS; b += NT) c->hist[b] = 0;
  if (threadIdx.x == 0) {
    c->tau = tau;
    c->full = full;
    c->refreshed = 0;
    if (all) c->fresh = k;
    c->picked = pick && k + 1 < n_orb;
    if (!pick) {
      c->zero += 1;
      if (c->zero > LZ_ZERO) c->want_full = 1;
    } else {
      c->k = k + 1;
      points[k] = (int32_t)m.i;
      d[m.i] = -1.0;
    }
  }
  if (!pick || k + 1 == n_orb) return;
  scdm_direction<G, NT>(psi, n_orb, ng, m.i, k, Q, QT, reinterpret_cast<S*>(lds),
                            red);
}

// Downdate with the new direction: the selected points still at or above
// the bound, or every point.
template <typename G, int VW>
__global__ __launch_bounds__(AM_NT) void k_lazy_downdate(
    const G* psi, int n_orb, int64_t ng, const LazyCtl* c, const int32_t* list,
    int cap, const G* buf, const typename Scal<G>::S* Q, double* d,
    uint16_t* missed, double* pv, int64_t* pi) {
  using S = typename Scal<G>::S;
  extern __shared__ double2 lds[];
  if (!c->picked) return;
  const int k = c->k - 1, tid = threadIdx.x;
  S* qs = reinterpret_cast<S*>(lds);
  ArgMax m{-2.0, 0};
  if (c->full) {
    for (int n = tid; n < n_orb; n += AM_NT) qs[n] = Q[(int64_t)k * q_ld<S>(n_orb) + n];
    __syncthreads();
    m = downdate_all<G, VW, VEC_U>(psi, n_orb, ng, qs, d);
  } else if (blockIdx.x * LZ_PTS < (unsigned)c->count) {
    // 64 points a workgroup, a quarter of the orbitals a wave
    __shared__ S part[AM_NT / 64][64];
    const int lane = tid & 63, wv = tid >> 6;
    for (int n = tid; n < n_orb; n += AM_NT) qs[n] = Q[(int64_t)k * q_ld<S>(n_orb) + n];
    __syncthreads();
    const int at = blockIdx.x * LZ_PTS + lane;
    const bool on = at < c->count;
    const int64_t r = on ? list[at] : 0;
    const double old = on ? d[r] : -1.0;
    const bool live = on && old >= c->tau;   // picked points hold -1, tau >= 0
    if (__any(live)) {
      const int nq = (n_orb + 3) / 4, n1 = min(n_orb, (wv + 1) * nq);
      S s = zero_s(S{});
      if (live) {
        in_flight<16>(wv * nq, n1, 1, [&](int n) { return buf[(int64_t)n * cap + at]; },
                      [&](int n, const G& g) { s = mad(qs[n], to_s(g, S{}), s); });
      }
      part[wv][lane] = s;
    }
    __syncthreads();
    if (wv == 0 && live) {
      const S s = add_s(add_s(part[0][lane], part[1][lane]),
                        add_s(part[2][lane], part[3][lane]));
      const double nv = fmax(old - norm_s(s), 0.0);
      d[r] = nv;
      missed[r] = (uint16_t)(k + 1);
      m = ArgMax{nv, r};
    }
  }
  m = block_argmax<AM_NT>(m);
  if (tid == 0) {
    pv[blockIdx.x] = m.v;
    pi[blockIdx.x] = m.i;
  }
}

// Y[k][n] = conj(psi_n(r_k)): the picked columns of Psi^H, transposed.
template <typename G>
__global__ void k_scdm_gather(const G* psi, int n_orb, int64_t ng,
                              const int32_t* points, double2* Y) {
  const int64_t total = (int64_t)n_orb * n_orb;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < total;
       e += stride) {
    const int k = (int)(e / n_orb), n = (int)(e % n_orb);
    const double2 v = GridVal<G>::get(psi, n * ng + points[k]);
    Y[e] = make_double2(v.x, -v.y);
  }
}

// Points selected at most: an eighth of the grid, whole workgroups.
static int lazy_cap(int64_t ng) {
  const int64_t c = ng / 8 / LZ_PTS * LZ_PTS;
  return (int)(c < LZ_MAX ? c : LZ_MAX);
}
static size_t up256(size_t b) { return (b + 255) & ~size_t(255); }

// Bytes of `buf` that the lazy selection takes.
static size_t lazy_bytes(int n_orb, int64_t ng, size_t point) {
  const size_t cap = (size_t)lazy_cap(ng);
  return up256(sizeof(LazyCtl)) + up256(2 * (size_t)ng) + up256(4 * cap) +
         point * cap * (size_t)n_orb;
}

// The lazy selection replaces n_orb passes over the grids by launches (three a
// step that return at once, 15 us) and a few refreshes.  It pays where a
// pass takes more than the launches (at 5.6 TB/s 192 MB take 34 us; complex
// grids, whose catch-ups cost twice the arithmetic per byte, 256 MB) and all
// passes together more than the refreshes (11 GB: 2 ms).  Measured, whole
// call, every point each step -> lazy, localized orbitals mixed by a rotation
// / random ones: 120^3 real FP32 with 200 (1.4 GB) 59.3 -> 16.0 / with 220 72.0
// -> 24.8 ms, 96^3 with 128 (453 MB) 13.6 -> 6.2 / 13.8 -> 7.7, 96^3 with 60
// (212 MB, 12.7 GB in all) 3.2 -> 2.8 / 3.6 -> 2.9, 80^3 with 96 (197 MB) 4.8 ->
// 4.0; complex FP32 96^3 with 40 (283 MB, 11.3 GB in all) 2.6 -> 2.1, 96^3 with
// 64 - / 7.1 -> 6.6, 120^3 with 30 (415 MB, 12.4 GB in all) - / 3.5 -> 3.7;
// complex FP64 120^3 with 30 (829 MB) 6.2 -> 3.1.  Beyond the line: complex FP32
// 64^3 with 100 (210 MB) - / 5.3 -> 5.8, 80^3 with 60 (246 MB) - / 3.6 -> 4.0,
// 120^3 with 16 (221 MB, 3.5 GB in all) - / 1.1 -> 2.2; real FP32 120^3 with 28
// (193 MB, 5.4 GB in all) - / 1.7 -> 2.1.
static bool lazy_pays(bool complex_grids, double n_orb, double bytes) {
  return bytes >= (complex_grids ? 256e6 : 192e6) && n_orb * bytes >= 11e9;
}

template <typename G>
static hipError_t scdm_t(const G* psi, int n_orb, int64_t ng, double* d,
                         double* pv, int64_t* pi, void* Qv, void* QTv,
                         void* buf, int64_t buf_bytes, int32_t* points,
                         double2* Y, hipStream_t st) {
  using S = typename Scal<G>::S;
  S* Q = static_cast<S*>(Qv);
  S* QT = static_cast<S*>(QTv);
  constexpr int VW = 16 / (int)sizeof(G);
  // 16-byte vectors of points where they still make four workgroups per CU
  // (64^3 real FP32, 64 orbitals: 24 us a downdate with vectors, 11 without)
  const bool vec = ng % VW == 0 && ng >= (int64_t)VW * AM_NT * 1024;
  const size_t qlds = sizeof(S) * (size_t)n_orb;
  // one vector of points per thread where the partials allow
  const int64_t per_block = (int64_t)AM_NT * (vec ? VW : 1);
  const int parts = (int)std::min<int64_t>(AM_BLOCKS, (ng + per_block - 1) / per_block);
  const bool lazy = ng % VW == 0 &&
                    lazy_pays(sizeof(S) == 16, n_orb,
                              (double)n_orb * (double)ng * sizeof(G)) &&
                    (int64_t)lazy_bytes(n_orb, ng, sizeof(G)) <= buf_bytes;
  char* b = static_cast<char*>(buf);
  LazyCtl* ctl = reinterpret_cast<LazyCtl*>(b);
  b += up256(sizeof(LazyCtl));
  uint16_t* missed = lazy ? reinterpret_cast<uint16_t*>(b) : nullptr;
  b += up256(2 * (size_t)ng);
  const int cap = lazy_cap(ng);
  int32_t* list = reinterpret_cast<int32_t*>(b);
  b += up256(4 * (size_t)cap);
  G* cols = reinterpret_cast<G*>(b);
  if (vec)
    LACE_LAUNCH((k_scdm_density<G, VW, VEC_U>), dim3(parts), dim3(AM_NT), 0, st, psi,
                n_orb, ng, d, missed, points, pv, pi);
  else
    LACE_LAUNCH((k_scdm_density<G, 1, SMALL_U>), dim3(parts), dim3(AM_NT), 0, st, psi,
                n_orb, ng, d, missed, points, pv, pi);
  hipError_t e = hipGetLastError();
  // Threads of the pick: Gram-Schmidt against many directions is bound by how
  // much one CU has in flight, a few directions by the barriers of many
  // waves.  Measured, whole call, 256 / 512 / 1024 threads: complex FP64 32^3
  // with 64 orbitals 1.33 / 1.43 / 1.66 ms, real FP32 48^3 with 32 526 / 526 /
  // 634 us, complex FP32 48^3 with 200 11.8 / 10.7 / 11.8 ms, complex FP64 24^3
  // with 300 23.5 / 17.8 / 18.9, 450 - / 46.3 / 49.1, 700 - / 155.6 / 152.3.
  const int nt = n_orb <= 64 ? 256 : n_orb <= 512 ? 512 : 1024;
  const size_t dir_lds = 2 * qlds + 16 * (size_t)nt;
  auto eager_pick = [&](int k) -> hipError_t {
    if (nt == 256)
      LACE_LAUNCH((k_scdm_pick<G, 256>), dim3(1), dim3(256), dir_lds, st, psi, n_orb,
                  ng, pv, pi, parts, d, points, k, Q, QT);
    else if (nt == 512)
      LACE_LAUNCH((k_scdm_pick<G, 512>), dim3(1), dim3(512), dir_lds, st, psi, n_orb,
                  ng, pv, pi, parts, d, points, k, Q, QT);
    else
      LACE_LAUNCH((k_scdm_pick<G, 1024>), dim3(1), dim3(1024), dir_lds, st, psi, n_orb,
                  ng, pv, pi, parts, d, points, k, Q, QT);
    return hipGetLastError();
  };
  auto lazy_pick = [&]() -> hipError_t {
    if (nt == 256)
      LACE_LAUNCH((k_lazy_pick<G, 256>), dim3(1), dim3(256), dir_lds, st, psi, n_orb,
                  ng, ctl, pv, pi, d, points, Q, QT);
    else if (nt == 512)
      LACE_LAUNCH((k_lazy_pick<G, 512>), dim3(1), dim3(512), dir_lds, st, psi, n_orb,
                  ng, ctl, pv, pi, d, points, Q, QT);
    else
      LACE_LAUNCH((k_lazy_pick<G, 1024>), dim3(1), dim3(1024), dir_lds, st, psi, n_orb,
                  ng, ctl, pv, pi, d, points, Q, QT);
    return hipGetLastError();
  };
  if (lazy) {
    LACE_LAUNCH(k_lazy_init, dim3(1), dim3(AM_NT), 0, st, ctl, pv);
    // a tick makes a pick, except after a refresh that leaves no point at
    // its bound (at most LZ_ZERO + 1 of them) or that asks for every point
    for (int t = 0; t < n_orb + LZ_ZERO + 2 && e == hipSuccess; ++t) {
      LACE_LAUNCH(k_lazy_hist<G>, dim3(LZ_BLOCKS), dim3(AM_NT), 0, st, psi, n_orb, ng,
                  ctl, QT, d, missed, pv);
      LACE_LAUNCH(k_lazy_select, dim3(256), dim3(AM_NT), 0, st, ctl, pv, d, ng,
                  n_orb, cap, list);
      LACE_LAUNCH(k_lazy_gather<G>, dim3(LZ_BLOCKS), dim3(AM_NT), 0, st, psi, n_orb,
                  ng, ctl, list, cap, cols, QT, d, missed, pv, pi);
      if ((e = lazy_pick()) != hipSuccess) return e;
      LACE_LAUNCH((k_lazy_downdate<G, VW>), dim3(LZ_BLOCKS), dim3(AM_NT), qlds, st,
                  psi, n_orb, ng, ctl, list, cap, cols, Q, d, missed, pv, pi);
      e = hipGetLastError();
    }
  } else {
    for (int k = 0; k < n_orb && e == hipSuccess; ++k) {
      if ((e = eager_pick(k)) != hipSuccess) return e;
      if (k + 1 < n_orb) {
        if (vec)
          LACE_LAUNCH((k_scdm_downdate<G, VW, VEC_U>), dim3(parts), dim3(AM_NT), qlds, st,
                      psi, n_orb, ng, Q, k, d, pv, pi);
        else
          LACE_LAUNCH((k_scdm_downdate<G, 1, SMALL_U>), dim3(parts), dim3(AM_NT), qlds, st,
                      psi, n_orb, ng, Q, k, d, pv, pi);
      }
      e = hipGetLastError();
    }
  }
  if (e == hipSuccess) {
    int64_t b2 = ((int64_t)n_orb * n_orb + AM_NT - 1) / AM_NT;
    if (b2 > 2048) b2 = 2048;
    LACE_LAUNCH(k_scdm_gather<G>, dim3((unsigned)b2), dim3(AM_NT), 0, st, psi, n_orb,
                ng, points, Y);
    e = hipGetLastError();
  }
  return e;
}

int64_t scdm_scratch_bytes(int n_orb) {
  return (int64_t)AM_BLOCKS * (sizeof(double) + sizeof(int64_t)) +
         2 * (int64_t)sizeof(double2) * n_orb * n_orb;
}

hipError_t launch_scdm(bool fp64, bool real, const void* psi, int n_orb,
                       int64_t ng, double* d, void* scratch, void* buf,
                       int64_t buf_bytes, int32_t* points, void* Y,
                       hipStream_t st) {
  if (n_orb > 48 * 1024 / (int)sizeof(double2)) return hipErrorInvalidValue;
  char* p = static_cast<char*>(scratch);
  double* pv = reinterpret_cast<double*>(p);
  p += AM_BLOCKS * sizeof(double);
  int64_t* pi = reinterpret_cast<int64_t*>(p);
  p += AM_BLOCKS * sizeof(int64_t);
  void* Q = p;
  void* QT = p + sizeof(double2) * (size_t)n_orb * n_orb;
  double2* y = static_cast<double2*>(Y);
  if (real)
    return fp64 ? scdm_t(static_cast<const double*>(psi), n_orb, ng, d, pv, pi,
                         Q, QT, buf, buf_bytes, points, y, st)
                : scdm_t(static_cast<const float*>(psi), n_orb, ng, d, pv, pi,
                         Q, QT, buf, buf_bytes, points, y, st);
  return fp64 ? scdm_t(static_cast<const double2*>(psi), n_orb, ng, d, pv, pi,
                       Q, QT, buf, buf_bytes, points, y, st)
              : scdm_t(static_cast<const float2*>(psi), n_orb, ng, d, pv, pi,
                       Q, QT, buf, buf_bytes, points, y, st);
}

}  // namespace lace
