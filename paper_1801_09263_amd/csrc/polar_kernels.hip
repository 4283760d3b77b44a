// polar_kernels.hip - unitary polar factor of a small complex matrix on the
// FP64 matrix cores (the alignment at the end of Sec. 2 and the Loewdin
// step of SCDM).
//
// X_0 = A s with s^2 = 1 / (Gershgorin bound of A^H A), then the
// Newton-Schulz steps X <- X (3 I - X^H X) / 2, at most POLAR_STEPS of
// them.  The matrix is kept transposed, Y = X^T (row-major), so that both
// products read rows: with B = X^H X,
//   B[a][b]  = sum_k conj(Y[a][k]) Y[b][k],
//   Y'[b][a] = sum_k conj(C[b][k]) Y[k][a],  C = (3 I - B) / 2 = C^H.
// A step takes |B - I|_2 = e to 3/4 e^2 or less.  Once n max |B_ab - d_ab|
// (a bound on e) is at most 3e-9, the step that follows leaves 1e-17, below
// the rounding of the products, so later steps change nothing but rounding
// and are not run.  Two consecutive outer steps' orbitals take 6-7 steps.
//
// n <= 64: one workgroup runs every step with Y and C in LDS (at most 133
// KB), one wave per 16 x 16 tile.  The work of a step (two products of
// 8 n^3 flops) is at most 10 us on one CU, about what two launches and
// their gap cost.  Larger n: two launches per step (B, then Y'), each wave
// reading its operands straight from L2 (Y, B and Y' of n = 256 take 3 MB);
// the launches after convergence read one flag and return (2 us).
// Measured, whole alignment of 1,331-coefficient orbitals rotated and
// perturbed by 1e-3 (before: 30 steps of four launches, split-K product,
// reduction, element step and tall product): n = 96 987 -> 189 us, 129
// 1280 -> 195 us, 256 2080 -> 296 us, 400 3385 -> 673 us; of unrelated sets
// (17 steps) n = 256 2011 -> 740 us.  An outer step of the request loop at
// 48^3 with 32 orbitals 2317 -> 1592 us.
#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "mfma.hpp"

namespace lace {

namespace {

constexpr int POLAR_STEPS = 30;
constexpr double POLAR_TOL = 3e-9;

// Device state of a large-n run: word-wise maxima of non-negative doubles
// are taken on their bit patterns (the order of the integers), which a
// maximum makes independent of the order of the updates.
struct PolarState {
  unsigned long long gmax;                 // max row sum of |B_0|
  unsigned long long emax[POLAR_STEPS];    // max |B - I| of each step
  int32_t done[POLAR_STEPS + 1];           // converged before this step
};

__device__ inline unsigned long long bits_of(double v) {
  return (unsigned long long)__double_as_longlong(v);
}
__device__ inline double of_bits(unsigned long long v) {
  return __longlong_as_double((long long)v);
}

// ------------------------------------------------- n <= 64: one workgroup
template <int TL>
__global__ __launch_bounds__(64 * TL * TL) void k_polar_small(
    const double2* Y0, int conj_in, int n, double2* U, double* resid) {
  constexpr int NP = 16 * TL, LS = NP + 1, NT = 64 * TL * TL;
  __shared__ double2 y[NP * LS];
  __shared__ double2 c[NP * LS];
  __shared__ double red[TL * TL];
  __shared__ double s_scale;
  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64;
  const int ti = w / TL, tj = w % TL;       // this wave's tile
  const int l16 = lane % 16, g = lane / 16;
  const int kmax = (n + 3) & ~3;            // whole MFMA steps; the pad is 0
  for (int e = tid; e < NP * NP; e += NT) {
    const int a = e / NP, b = e % NP;
    double2 v = make_double2(0.0, 0.0);
    if (a < n && b < n) {
      v = Y0[(int64_t)a * n + b];
      if (conj_in) v.y = -v.y;
    }
    y[a * LS + b] = v;
  }
  __syncthreads();
  d4 br, bi;
  auto gram = [&]() {   // this wave's tile of B = X^H X
    br = d4{0, 0, 0, 0};
    bi = d4{0, 0, 0, 0};
    for (int k = g; k < kmax; k += 4) {
      const double2 p = y[(ti * 16 + l16) * LS + k];
      const double2 q = y[(tj * 16 + l16) * LS + k];
      br = mfma(p.x, q.x, br);
      bi = mfma(p.x, q.y, bi);
      br = mfma(p.y, q.y, br);
      bi = mfma(-p.y, q.x, bi);
    }
  };
  auto wave_max = [](double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
  };
  const int col = tj * 16 + l16;
  for (int it = 0; it < POLAR_STEPS; ++it) {
    gram();
    double s2 = 1.0, f = 1.0;
    bool last = false;
    if (it == 0) {   // scale: s^2 = 1 / max row sum of |B|
#pragma unroll
      for (int e = 0; e < 4; ++e)
        c[(ti * 16 + g + 4 * e) * LS + col] = make_double2(br[e], bi[e]);
      __syncthreads();
      if (w == 0) {
        double r = 0.0;
        if (lane < NP)
          for (int b = 0; b < n; ++b) {
            const double2 v = c[lane * LS + b];
            r += sqrt(v.x * v.x + v.y * v.y);
          }
        r = wave_max(r);
        if (lane == 0) s_scale = r > 0.0 ? 1.0 / r : 0.0;
      }
      __syncthreads();
      s2 = s_scale;
      f = sqrt(s2);
    } else {
      double m = 0.0;   // keeps a NaN, which fails the comparison below
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double re = br[e] - ((ti * 16 + g + 4 * e) == col && col < n ? 1.0 : 0.0);
        const double v = sqrt(re * re + bi[e] * bi[e]);
        if (v > m || v != v) m = v;
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const double u = __shfl_xor(m, o, 64);
        if (u > m || u != u) m = u;
      }
      if (lane == 0) red[w] = m;
      __syncthreads();
      last = true;
#pragma unroll
      for (int k = 0; k < TL * TL; ++k) last = last && red[k] * n <= POLAR_TOL;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = ti * 16 + g + 4 * e;
      c[row * LS + col] = make_double2((row == col ? 1.5 : 0.0) - 0.5 * s2 * br[e],
                                       -0.5 * s2 * bi[e]);
    }
    __syncthreads();
    d4 yr = d4{0, 0, 0, 0}, yi = d4{0, 0, 0, 0};
    for (int k = g; k < kmax; k += 4) {
      const double2 p = c[(ti * 16 + l16) * LS + k];
      const double2 q = y[k * LS + tj * 16 + l16];
      yr = mfma(p.x, q.x, yr);
      yi = mfma(p.x, q.y, yi);
      yr = mfma(p.y, q.y, yr);
      yi = mfma(-p.y, q.x, yi);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e)
      y[(ti * 16 + g + 4 * e) * LS + col] = make_double2(f * yr[e], f * yi[e]);
    __syncthreads();
    if (last) break;
  }
  for (int e = tid; e < n * n; e += NT) {   // U = Y^T
    const int a = e / n, b = e % n;
    U[e] = y[b * LS + a];
  }
  if (resid) {
    gram();
    double t = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double re = br[e] - ((ti * 16 + g + 4 * e) == col && col < n ? 1.0 : 0.0);
      t += re * re + bi[e] * bi[e];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    __syncthreads();
    if (lane == 0) red[w] = t;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int k = 0; k < TL * TL; ++k) s += red[k];
      *resid = sqrt(s / n);
    }
  }
}

// ------------------------------------------------------ n > 64: launches
// Y <- Y_0 (conjugated when conj_in), and the cleared state.
__global__ void k_polar_init(const double2* in, int conj_in, int n, double2* Y,
                             PolarState* st) {
  const int64_t nn = (int64_t)n * n;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < nn;
       e += stride) {
    const double2 v = in[e];
    Y[e] = make_double2(v.x, conj_in ? -v.y : v.y);
  }
  if (blockIdx.x == 0) {
    int32_t* p = reinterpret_cast<int32_t*>(st);
    for (int e = threadIdx.x; e < (int)(sizeof(PolarState) / 4); e += blockDim.x) p[e] = 0;
  }
}

// The operand rows of one 16-row tile: lane (l16, g) takes the four
// consecutive k of its group, k0 + 4 g + {0, 1, 2, 3}, of row r0 + l16 (64
// contiguous bytes a lane; the sum over k may take any order).
__device__ inline void row_frag(const double2* A, int n, int r0, int k0, int l16,
                                int g, double2 v[4]) {
  const int r = r0 + l16;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = k0 + 4 * g + s;
    v[s] = make_double2(0.0, 0.0);
    if (r < n && k < n) v[s] = A[(int64_t)r * n + k];
  }
}

// A workgroup of four waves takes one 16 x 16 tile: k is dealt to the waves
// in blocks of 16 and the four partial tiles are added in wave order
// through LDS, which gives 256 workgroups at n = 256 and short chains (32 x
// 32 tiles with one 16 x 16 tile per wave measured 1176 against 713 us for
// the whole alignment at n = 257, 2731 against 2215 us at 512, and the same
// from 700 on).  body(k0) accumulates one block of k; on return the wave
// holds element `w` of the tile's accumulators: row g + 4 w.
template <class Body>
__device__ inline double2 polar_tile(int n, int w, Body body) {
  __shared__ double part[4][64][9];
  d4 re = d4{0, 0, 0, 0}, im = d4{0, 0, 0, 0};
  for (int k0 = 16 * w; k0 < n; k0 += 64) body(k0, re, im);
  const int lane = threadIdx.x % 64;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    part[w][lane][e] = re[e];
    part[w][lane][4 + e] = im[e];
  }
  __syncthreads();
  double2 v = make_double2(0.0, 0.0);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v.x += part[q][lane][w];
    v.y += part[q][lane][4 + w];
  }
  return v;
}

// B = X^H X: tiles on and above the diagonal, mirrored.  it >= 0: nothing
// once converged, and the step's max |B - I| (not for it = 0, whose B is
// not scaled yet); it < 0: always (the residual).
__global__ __launch_bounds__(256) void k_polar_gram(const double2* Ya,
                                                    const double2* Yb, int n,
                                                    double2* B, PolarState* st,
                                                    int it) {
  const double2* Y = Ya;
  if (it >= 0) {
    if (st->done[it]) return;
  } else {
    int steps = 0;
    while (steps < POLAR_STEPS && !st->done[steps]) ++steps;
    Y = (steps & 1) ? Yb : Ya;
  }
  int ta = blockIdx.x;   // tile pairs ta <= tb, column by column
  // first guess from the triangular numbers, then exact
  int tb = (int)((sqrt(8.0 * ta + 1.0) - 1.0) * 0.5);
  while (tb * (tb + 1) / 2 > ta) --tb;
  while ((tb + 1) * (tb + 2) / 2 <= ta) ++tb;
  ta -= tb * (tb + 1) / 2;
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int l16 = lane % 16, g = lane / 16;
  const int a0 = ta * 16, b0 = tb * 16;
  const double2 v = polar_tile(n, w, [&](int k0, d4& re, d4& im) {
    double2 p[4], q[4];
    row_frag(Y, n, a0, k0, l16, g, p);
    row_frag(Y, n, b0, k0, l16, g, q);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      re = mfma(p[s].x, q[s].x, re);
      im = mfma(p[s].x, q[s].y, im);
      re = mfma(p[s].y, q[s].y, re);
      im = mfma(-p[s].y, q[s].x, im);
    }
  });
  double m = 0.0;
  const int a = a0 + g + 4 * w, b = b0 + l16;
  if (a < n && b < n) {
    B[(int64_t)a * n + b] = v;
    if (ta != tb) B[(int64_t)b * n + a] = make_double2(v.x, -v.y);
    const double d = v.x - (a == b ? 1.0 : 0.0);
    m = sqrt(d * d + v.y * v.y);
  }
  if (it > 0) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double u = __shfl_xor(m, o, 64);
      if (u > m || u != u) m = u;
    }
    // |.|: a NaN's sign bit must not hide it from the integer maximum
    if (lane == 0) atomicMax(&st->emax[it], bits_of(fabs(m)));
  }
}

// gmax = max_a sum_b |B_ab|, one wave per row.
__global__ __launch_bounds__(256) void k_polar_rowmax(const double2* B, int n,
                                                      PolarState* st) {
  const int a = blockIdx.x * 4 + threadIdx.x / 64, lane = threadIdx.x % 64;
  if (a >= n) return;
  double r = 0.0;
  for (int b = lane; b < n; b += 64) {
    const double2 v = B[(int64_t)a * n + b];
    r += sqrt(v.x * v.x + v.y * v.y);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
  if (lane == 0 && r > 0.0) atomicMax(&st->gmax, bits_of(r));
}

// Y' = f C Y of step `it` (C from B, scaled by s^2 in the first step).
__global__ __launch_bounds__(256) void k_polar_step(const double2* Y,
                                                    const double2* B, int n,
                                                    double2* Yn, PolarState* st,
                                                    int it) {
  const bool done = st->done[it] != 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const bool conv = it > 0 && of_bits(st->emax[it]) * n <= POLAR_TOL;
    st->done[it + 1] = done || conv;
  }
  if (done) return;
  double s2 = 1.0, f = 1.0;
  if (it == 0) {
    const double gm = of_bits(st->gmax);
    s2 = gm > 0.0 ? 1.0 / gm : 0.0;
    f = sqrt(s2);
  }
  const int nt = (n + 15) / 16;
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int l16 = lane % 16, g = lane / 16;
  const int b0 = (int)(blockIdx.x / nt) * 16, a0 = (int)(blockIdx.x % nt) * 16;
  const double2 v = polar_tile(n, w, [&](int k0, d4& re, d4& im) {
    double2 p[4], q[4];
    row_frag(B, n, b0, k0, l16, g, p);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = k0 + 4 * g + s, a = a0 + l16;
      q[s] = make_double2(0.0, 0.0);
      if (k < n && a < n) q[s] = Y[(int64_t)k * n + a];
      p[s].x = (b0 + l16 == k ? 1.5 : 0.0) - 0.5 * s2 * p[s].x;
      p[s].y = -0.5 * s2 * p[s].y;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      re = mfma(p[s].x, q[s].x, re);
      im = mfma(p[s].x, q[s].y, im);
      re = mfma(p[s].y, q[s].y, re);
      im = mfma(-p[s].y, q[s].x, im);
    }
  });
  const int b = b0 + g + 4 * w, a = a0 + l16;
  if (a < n && b < n) Yn[(int64_t)b * n + a] = make_double2(f * v.x, f * v.y);
}

// U = Y^T from the buffer the last step that ran wrote.
__global__ void k_polar_out(const double2* Ya, const double2* Yb, int n,
                            double2* U, const PolarState* st) {
  int steps = 0;
  while (steps < POLAR_STEPS && !st->done[steps]) ++steps;
  const double2* Y = (steps & 1) ? Yb : Ya;
  const int64_t nn = (int64_t)n * n;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < nn;
       e += stride)
    U[e] = Y[(e % n) * n + e / n];
}

// *out = ||B - I||_F / sqrt(n), one workgroup, fixed order.
__global__ __launch_bounds__(1024) void k_polar_resid(const double2* B, int n,
                                                      double* out) {
  __shared__ double red[16];
  double t = 0.0;
  for (int64_t e = threadIdx.x; e < (int64_t)n * n; e += 1024) {
    const double2 x = B[e];
    const double re = x.x - (e / n == e % n ? 1.0 : 0.0);
    t += re * re + x.y * x.y;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
  if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < 16; ++w) s += red[w];
    *out = sqrt(s / n);
  }
}

template <int TL>
hipError_t polar_small(const double2* Y0, bool conj_in, int n, double2* U,
                       double* resid, hipStream_t st) {
  LACE_LAUNCH(k_polar_small<TL>, dim3(1), dim3(64 * TL * TL), 0, st, Y0,
              conj_in ? 1 : 0, n, U, resid);
  return hipGetLastError();
}

hipError_t polar_large(const double2* Y0, bool conj_in, int n, double2* ya,
                       double2* yb, double2* b, double2* U, double* resid,
                       PolarState* ps, hipStream_t st) {
  const int64_t nt = (n + 15) / 16;
  const dim3 gtiles((unsigned)(nt * (nt + 1) / 2)), stiles((unsigned)(nt * nt));
  int64_t eb = ((int64_t)n * n + 255) / 256;
  if (eb > 2048) eb = 2048;
  LACE_LAUNCH(k_polar_init, dim3((unsigned)eb), dim3(256), 0, st, Y0,
              conj_in ? 1 : 0, n, ya, ps);
  double2* cur = ya;
  double2* nxt = yb;
  for (int it = 0; it < POLAR_STEPS; ++it) {
    LACE_LAUNCH(k_polar_gram, gtiles, dim3(256), 0, st, cur, cur, n, b, ps, it);
    if (it == 0)
      LACE_LAUNCH(k_polar_rowmax, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st,
                  b, n, ps);
    LACE_LAUNCH(k_polar_step, stiles, dim3(256), 0, st, cur, b, n, nxt, ps, it);
    double2* t = cur;
    cur = nxt;
    nxt = t;
  }
  if (resid) {
    LACE_LAUNCH(k_polar_gram, gtiles, dim3(256), 0, st, ya, yb, n, b, ps, -1);
    LACE_LAUNCH(k_polar_resid, dim3(1), dim3(1024), 0, st, b, n, resid);
  }
  LACE_LAUNCH(k_polar_out, dim3((unsigned)eb), dim3(256), 0, st, ya, yb, n, U, ps);
  return hipGetLastError();
}

}  // namespace

int64_t polar_state_bytes() { return (int64_t)sizeof(PolarState); }

hipError_t launch_polar(const void* Y0, bool conj_in, int n, void* ya, void* yb,
                        void* b, void* state, void* U, double* resid,
                        hipStream_t st) {
  const double2* y0 = static_cast<const double2*>(Y0);
  double2* u = static_cast<double2*>(U);
  if (n <= 16) return polar_small<1>(y0, conj_in, n, u, resid, st);
  if (n <= 32) return polar_small<2>(y0, conj_in, n, u, resid, st);
  if (n <= 48) return polar_small<3>(y0, conj_in, n, u, resid, st);
  if (n <= 64) return polar_small<4>(y0, conj_in, n, u, resid, st);
  return polar_large(y0, conj_in, n, static_cast<double2*>(ya),
                     static_cast<double2*>(yb), static_cast<double2*>(b), u,
                     resid, static_cast<PolarState*>(state), st);
}

}  // namespace lace
