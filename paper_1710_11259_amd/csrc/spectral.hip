// gfx950 kernels that build the eigenbasis form of the solve at plan time:
// eigenpairs of the symmetric tridiagonal parity blocks of A~ (App. B
// decoupling) and the coefficient maps merged with them.
//
// The vectors and the merged maps are formed in pairs of doubles (error-free sums and
// products: T. J. Dekker, Numer. Math. 18 (1971)) and rounded once.  With vectors and
// maps formed in double the rounding of the solves they enter was up to twice as large
// (adjoint, native, n = 64: rms 8e-16 of the result, 4e-16 from these, 3e-16 from
// half-sweeps).
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace fps {

namespace {

struct EigPair {
  TridiagEig p[2];
};

// Eigenvalue k (ascending) of the positive definite B = -T (diagonal d,
// squared couplings e2) by multisection on Sturm counts: one wavefront per
// eigenvalue, the 64 lanes counting at 64 interior points, so a pass over the
// matrix cuts the bracket by 65 instead of 2 (10 passes, 60 bits; its logarithm starts below
// 43, so it ends below half an ulp; the recurrence is a serial chain of m divisions, so
// passes are what costs, and both parities run in one launch).  The points are
// spaced geometrically until the bracket is within a factor 2: the spectrum
// spans 30 n^4 and every eigenvalue is wanted to relative accuracy.  A zero
// pivot is left to IEEE: e2 / 0 = inf, the next pivot is -inf and counts.
__global__ __launch_bounds__(256) void k_tridiag_values(EigPair both, double lo0, double hi0) {
  const TridiagEig &g = both.p[blockIdx.y];
  const double *__restrict__ d = g.d.p, *__restrict__ e2 = g.e2;
  double *__restrict__ lam = g.lam;
  const int m = g.m;
  const int lane = threadIdx.x & 63;
  const int k = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (k >= m) return;
  double lo = lo0, hi = hi0;
  for (int pass = 0; pass < 10; ++pass) {
    const double f = (lane + 1) * (1.0 / 65.0);
    const double x = hi > 2.0 * lo ? lo * exp2(f * log2(hi / lo)) : lo + (hi - lo) * f;
    double q = d[0] - x;
    int c = q < 0.0 ? 1 : 0;
    for (int i = 1; i < m; ++i) {
      q = (d[i] - x) - e2[i - 1] / q;
      c += q < 0.0 ? 1 : 0;
    }
    // lanes whose point lies at or below the eigenvalue form a prefix
    const unsigned long long above = ~__ballot(c <= k);
    const int below = above ? __builtin_ctzll(above) : 64;
    const double xl = __shfl(x, below > 0 ? below - 1 : 0), xh = __shfl(x, below < 64 ? below : 63);
    if (below > 0) lo = xl;
    if (below < 64) hi = xh;
  }
  if (lane == 0) lam[k] = -(lo + 0.5 * (hi - lo));
}

// Pairs h + l with |l| <= ulp(h) / 2.  (No contraction: a product folded into a sum is
// not the rounded product whose error is wanted.)
struct Pair {
  double h, l;
};
__device__ __forceinline__ Pair quick_sum(double a, double b) {  // |a| >= |b|
#pragma clang fp contract(off)
  const double s = a + b;
  return Pair{s, b - (s - a)};
}
__device__ __forceinline__ Pair two_sum(double a, double b) {
#pragma clang fp contract(off)
  const double s = a + b, t = s - a;
  return Pair{s, (a - (s - t)) + (b - t)};
}
__device__ __forceinline__ Pair add(Pair a, Pair b) {
#pragma clang fp contract(off)
  Pair s = two_sum(a.h, b.h);
  const Pair t = two_sum(a.l, b.l);
  s = quick_sum(s.h, s.l + t.h);
  return quick_sum(s.h, s.l + t.l);
}
__device__ __forceinline__ Pair neg(Pair a) { return Pair{-a.h, -a.l}; }
__device__ __forceinline__ Pair mul(Pair a, Pair b) {
#pragma clang fp contract(off)
  const double p = a.h * b.h;
  return quick_sum(p, __builtin_fma(a.l, b.h, __builtin_fma(a.h, b.l, __builtin_fma(a.h, b.h, -p))));
}
__device__ __forceinline__ Pair div(Pair a, Pair b) {
#pragma clang fp contract(off)
  const double inv = 1.0 / b.h, q = a.h * inv, r = __builtin_fma(-q, b.h, a.h);
  return quick_sum(q, __builtin_fma(-q, b.l, r + a.l) * inv);
}
__device__ __forceinline__ Pair load(const PairArray &a, int64_t i) { return Pair{a.p[i], a.p[a.lo + i]}; }
__device__ __forceinline__ void store(const PairArray &a, int64_t i, Pair v) {
  a.p[i] = v.h;
  a.p[a.lo + i] = v.l;
}

// Eigenvector of every eigenvalue by the twisted factorization of B - x: the ratios
// coupling / pivot of the top-down and bottom-up eliminations, twisted where the
// pivots' combination g is smallest, then one multiplication per entry in each
// direction.  x comes with the error of a double (1e-12 of the smallest); g / |z|^2 is
// the Rayleigh quotient's correction, so the first pass squares that error against the gap
// (neighbours differ by a relative 2 / m) and the second leaves the vector's error at 1e-18
// or less, the few highest modes apart (1e-14 at n = 4096: T's entries have 64 bits): the
// vectors are orthonormal as they are.  One lane per vector; ratios and
// vectors are stored [row][vector], so every access of a wavefront is one
// 512-byte run.  Bound by the serial chain of divisions.
// (The pointers are parameters for their no-alias promise: without it no entry is read
// before the last one is stored.)
__device__ __forceinline__ double tridiag_vector(
    const double *__restrict__ dh, const double *__restrict__ dl, const double *__restrict__ eh,
    const double *__restrict__ el, int m, int64_t a, double lam, double *__restrict__ cph,
    double *__restrict__ cpl, double *__restrict__ cmh, double *__restrict__ cml,
    double *__restrict__ Vh, double *__restrict__ Vl, int64_t ld) {
  const Pair zero{0.0, 0.0};
  auto d = [&](int i) { return Pair{dh[i], dl[i]}; };
  auto e = [&](int i) { return i < 0 ? zero : Pair{eh[i], el[i]}; };
  auto guard = [](Pair q, double c) {
    constexpr double kTiny = 4.9303806576313238e-32;  // 2^-104
    return q.h == 0.0 ? Pair{kTiny * c, 0.0} : q;
  };
  Pair x{-lam, 0.0};
  for (int pass = 0; pass < 2; ++pass) {
    Pair cp = zero, cm = zero;
#pragma unroll 2
    for (int i = 0; i < m; ++i) {
      const int j = m - 1 - i;
      const Pair ei = e(i), em = e(j - 1);
      const Pair qp = add(add(d(i), neg(x)), neg(mul(e(i - 1), cp)));
      const Pair qm = add(add(d(j), neg(x)), neg(mul(e(j), cm)));
      cp = div(ei, guard(qp, i + 1 < m ? ei.h : dh[i]));
      cm = div(em, guard(qm, j > 0 ? em.h : dh[j]));
      cph[i * ld + a] = cp.h;
      cpl[i * ld + a] = cp.l;
      cmh[j * ld + a] = cm.h;
      cml[j * ld + a] = cm.l;
    }
    Pair best = zero;
    int r = 0;
#pragma unroll 4
    for (int i = 0; i < m; ++i) {
      const int64_t up = (int64_t)(i > 0 ? i - 1 : 0) * ld + a, dn = (int64_t)(i + 1 < m ? i + 1 : i) * ld + a;
      Pair t = add(d(i), neg(x));
      t = add(t, neg(mul(e(i - 1), Pair{cph[up], cpl[up]})));
      t = add(t, neg(mul(e(i), Pair{cmh[dn], cml[dn]})));  // e(m - 1) = 0
      if (i == 0 || fabs(t.h) < fabs(best.h)) {
        best = t;
        r = i;
      }
    }
    Pair s{1.0, 0.0}, zu{1.0, 0.0}, zd{1.0, 0.0};  // towards row 0, towards row m - 1
#pragma unroll 4
    for (int i = 0; i < m; ++i) {
      const int j = m - 1 - i;
      if (j < r) {
        zu = mul(zu, Pair{cph[j * ld + a], cpl[j * ld + a]});
        Vh[j * ld + a] = zu.h;
        Vl[j * ld + a] = zu.l;
        s = add(s, mul(zu, zu));
      }
      if (i > r) {
        zd = mul(zd, Pair{cmh[i * ld + a], cml[i * ld + a]});
        Vh[i * ld + a] = zd.h;
        Vl[i * ld + a] = zd.l;
        s = add(s, mul(zd, zd));
      }
      if (i == r) {
        Vh[i * ld + a] = 1.0;
        Vl[i * ld + a] = 0.0;
      }
    }
    x = add(x, div(best, s));
    if (pass == 0) continue;
    // 1 / sqrt(s): a Newton step from the double's
    const double y = 1.0 / sqrt(s.h);
    const Pair f = add(Pair{1.0, 0.0}, neg(mul(s, mul(Pair{y, 0.0}, Pair{y, 0.0}))));
    const Pair inv = quick_sum(y, 0.5 * y * f.h);
#pragma unroll 4
    for (int i = 0; i < m; ++i) {
      const Pair v = mul(Pair{Vh[i * ld + a], Vl[i * ld + a]}, inv);
      Vh[i * ld + a] = v.h;
      Vl[i * ld + a] = v.l;
    }
  }
  return -x.h;
}

__global__ __launch_bounds__(64) void k_tridiag_vectors(EigPair both) {
  const TridiagEig &g = both.p[blockIdx.y];
  const int a = blockIdx.x * 64 + threadIdx.x;
  if (a < g.m)
    g.lam[a] = tridiag_vector(g.d.p, g.d.p + g.d.lo, g.e.p, g.e.p + g.e.lo, g.m, a, g.lam[a], g.cp.p,
                              g.cp.p + g.cp.lo, g.cm.p, g.cm.p + g.cm.lo, g.V.p, g.V.p + g.V.lo, g.ld);
}

struct MapBatch {
  MapEntries m[4];
};

__global__ __launch_bounds__(256) void k_map_entries(MapBatch b) {
  const MapEntries &g = b.m[blockIdx.z];
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x, i = blockIdx.y;
  if (i >= g.prows || j >= g.ld) return;
  Pair v{0.0, 0.0};
  if (i < g.rows && j < g.cols)
    v = mul(mul(load(g.row, i), load(g.col, j)), mul(load(g.t, j - i + g.rows - 1), load(g.u, i + j)));
  store(g.M, i * g.ld + j, v);
}

struct ProductBatch {
  MapProduct p[4];
};

// One 64 x 64 tile of W = V^T M, 16 k at a time through LDS, 4 x 4 entries a thread.  Every
// product enters its sum with its rounding error and the pairs' cross terms, 12 vector
// instructions; n = 4096: 0.4 T of them in all four products, a plan's largest pass.
__global__ __launch_bounds__(256) void k_map_products(ProductBatch b) {
#pragma clang fp contract(off)
  constexpr int BK = 16;
  __shared__ double A[2][BK][64], B[2][BK][64];
  const MapProduct &g = b.p[blockIdx.z];
  const int64_t i0 = (int64_t)blockIdx.y * 64, j0 = (int64_t)blockIdx.x * 64;
  if (i0 >= g.rows || j0 >= g.cols) return;
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  double h[4][4], l[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) h[i][j] = l[i][j] = 0.0;
  for (int k0 = 0; k0 < g.m; k0 += BK) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kk = (tid + 256 * q) >> 6, c = tid & 63, k = k0 + kk;
      // (V beyond its m rows and columns is not written)
      const Pair v = k < g.m && i0 + c < g.m ? load(g.V, k * g.ldv + i0 + c) : Pair{0.0, 0.0};
      const Pair w = k < g.m ? load(g.M, k * g.cols + j0 + c) : Pair{0.0, 0.0};
      A[0][kk][c] = v.h;
      A[1][kk][c] = v.l;
      B[0][kk][c] = w.h;
      B[1][kk][c] = w.l;
    }
    __syncthreads();
#pragma unroll 2
    for (int k = 0; k < BK; ++k) {
      Pair v[4], w[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v[q] = Pair{A[0][k][ty + 16 * q], A[1][k][ty + 16 * q]};
        w[q] = Pair{B[0][k][tx + 16 * q], B[1][k][tx + 16 * q]};
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double p = v[i].h * w[j].h;
          double e = __builtin_fma(v[i].h, w[j].h, -p);
          e = __builtin_fma(v[i].l, w[j].h, __builtin_fma(v[i].h, w[j].l, e));
          const Pair s = two_sum(h[i][j], p);
          h[i][j] = s.h;
          l[i][j] += s.l + e;
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t r = i0 + ty + 16 * i, c = j0 + tx + 16 * j;
      double v = h[i][j] + l[i][j];
      if (g.zlim != nullptr && r >= g.zlim[c / kGemmGroup]) v = 0.0;
      g.W[r * g.cols + c] = v;
      if (g.WT != nullptr) g.WT[c * g.rows + r] = v;
    }
}

// Error factors of slice z along y and x: Algorithm 2 leaves
// prod (a - p)/(a - q) (b - q)/(b - p) of the error for left eigenvalue a and
// right eigenvalue b; FP64: a = -mu^2 / (l + mu), b = -(l + mu); refined:
// a = -(|mu| k + 1/2), k = -1/l, b = -a, q = -p.
__global__ void k_slice_factors(const double *__restrict__ lam, const double *__restrict__ mu,
                                const int *__restrict__ off, const double *__restrict__ p,
                                const double *__restrict__ q, int refined, double *__restrict__ ey,
                                double *__restrict__ ex, int64_t npad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, z = blockIdx.y;
  if (i >= npad) return;
  const double m = mu[z], l = lam[i];
  const double a = refined ? -(-m * (-1.0 / l) + 0.5) : -m * m / (l + m);
  const double b = refined ? -a : -(l + m);
  double e = 1.0, f = 1.0;
  for (int j = off[z]; j < off[z + 1]; ++j) {
    e *= (a - p[j]) / (a - q[j]);
    f *= (b - q[j]) / (b - p[j]);
  }
  ey[z * npad + i] = e;
  ex[z * npad + i] = f;
}

__global__ void k_slice_multiplier(const double *__restrict__ lam, const double *__restrict__ ey,
                                   const double *__restrict__ ex, double *__restrict__ mt,
                                   int64_t npad) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y, z = blockIdx.z;
  if (x >= npad) return;
  const double lx = lam[x], ly = lam[y], lz = lam[z];
  mt[(z * npad + y) * npad + x] =
      fma(ey[z * npad + y], ex[z * npad + x], -1.0) / (lz * ly + lz * lx + ly * lx);
}

// Inner error factors of the nested method, a = -(k + q_i/2), k = -1/l:
// r[i][k] = prod (a - p)/(a + p).
__global__ void k_nested_factors(const double *__restrict__ lam, const double *__restrict__ q,
                                 const int *__restrict__ off, const double *__restrict__ p,
                                 double *__restrict__ r, int64_t npad) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y;
  if (k >= npad) return;
  const double a = 1.0 / lam[k] - 0.5 * q[i];
  double e = 1.0;
  for (int j = off[i]; j < off[i + 1]; ++j) e *= (a - p[j]) / (a + p[j]);
  r[i * npad + k] = e;
}

// Outer error of the nested method in mode (z, y, x), h = k_y + k_x, v = k_z:
// an exact step takes eps to rho eps, rho = (h + p)(v - q) / ((v - p)(h + q)),
// and the inner iteration, started from 0, scales its result by 1 - e.
__global__ void k_nested_multiplier(const double *__restrict__ lam, const double *__restrict__ p,
                                    const double *__restrict__ q, const double *__restrict__ r,
                                    int J, double *__restrict__ mt, int64_t npad) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y, z = blockIdx.z;
  if (x >= npad) return;
  const double lx = lam[x], ly = lam[y], lz = lam[z];
  const double h = -1.0 / lx - 1.0 / ly, v = -1.0 / lz;
  double eps = 1.0;
  for (int i = 0; i < J; ++i) {
    const double e = r[i * npad + y] * r[i * npad + x];
    const double rho = ((h + p[i]) / (h + q[i])) * ((v - q[i]) / (v - p[i]));
    eps = e + (1.0 - e) * rho * eps;
  }
  mt[(z * npad + y) * npad + x] = (eps - 1.0) / (lz * ly + lz * lx + ly * lx);
}

}  // namespace

hipError_t launch_slice_factors(const double *lam, const double *mu, const int *off,
                                const double *p, const double *q, bool refined, double *ey,
                                double *ex, int64_t npad, hipStream_t st) {
  hipLaunchKernelGGL(k_slice_factors, dim3((unsigned)((npad + 63) / 64), (unsigned)npad), dim3(64),
                     0, st, lam, mu, off, p, q, refined ? 1 : 0, ey, ex, npad);
  return hipGetLastError();
}

hipError_t launch_slice_multiplier(const double *lam, const double *ey, const double *ex, double *mt,
                                   int64_t npad, hipStream_t st) {
  hipLaunchKernelGGL(k_slice_multiplier,
                     dim3((unsigned)((npad + 255) / 256), (unsigned)npad, (unsigned)npad), dim3(256),
                     0, st, lam, ey, ex, mt, npad);
  return hipGetLastError();
}

hipError_t launch_nested_factors(const double *lam, const double *q, const int *off,
                                 const double *p_in, double *r, int J, int64_t npad,
                                 hipStream_t st) {
  hipLaunchKernelGGL(k_nested_factors, dim3((unsigned)((npad + 63) / 64), (unsigned)J), dim3(64), 0,
                     st, lam, q, off, p_in, r, npad);
  return hipGetLastError();
}

hipError_t launch_nested_multiplier(const double *lam, const double *p, const double *q,
                                    const double *r, int J, double *mt, int64_t npad,
                                    hipStream_t st) {
  hipLaunchKernelGGL(k_nested_multiplier,
                     dim3((unsigned)((npad + 255) / 256), (unsigned)npad, (unsigned)npad), dim3(256),
                     0, st, lam, p, q, r, J, mt, npad);
  return hipGetLastError();
}

hipError_t launch_tridiag_eig(const TridiagEig *p, double lo, double hi, hipStream_t st) {
  const int m = p[0].m > p[1].m ? p[0].m : p[1].m;
  if (m <= 0) return hipSuccess;
  const EigPair both{{p[0], p[1]}};
  hipLaunchKernelGGL(k_tridiag_values, dim3((unsigned)((m + 3) / 4), 2), dim3(256), 0, st, both, lo, hi);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL(k_tridiag_vectors, dim3((unsigned)((m + 63) / 64), 2), dim3(64), 0, st, both);
  return hipGetLastError();
}

hipError_t launch_map_entries(const MapEntries *m, int count, hipStream_t st) {
  if (count < 1 || count > 4) return hipErrorInvalidValue;
  MapBatch b{};
  int64_t rows = 0, ld = 0;
  for (int i = 0; i < count; ++i) {
    b.m[i] = m[i];
    rows = m[i].prows > rows ? m[i].prows : rows;
    ld = m[i].ld > ld ? m[i].ld : ld;
  }
  hipLaunchKernelGGL(k_map_entries, dim3((unsigned)((ld + 255) / 256), (unsigned)rows, (unsigned)count),
                     dim3(256), 0, st, b);
  return hipGetLastError();
}

hipError_t launch_map_products(const MapProduct *p, int count, hipStream_t st) {
  if (count < 1 || count > 4) return hipErrorInvalidValue;
  ProductBatch b{};
  int64_t rows = 0, cols = 0;
  for (int i = 0; i < count; ++i) {
    if (p[i].rows % 64 || p[i].cols % 64) return hipErrorInvalidValue;
    b.p[i] = p[i];
    rows = p[i].rows > rows ? p[i].rows : rows;
    cols = p[i].cols > cols ? p[i].cols : cols;
  }
  hipLaunchKernelGGL(k_map_products, dim3((unsigned)(cols / 64), (unsigned)(rows / 64), (unsigned)count),
                     dim3(256), 0, st, b);
  return hipGetLastError();
}

}  // namespace fps
