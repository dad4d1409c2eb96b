// gfx950 kernels that build the eigenbasis form of the solve at plan time:
// eigenpairs of the symmetric tridiagonal parity blocks of A~ (App. B
// decoupling) and the small dense passes around them.
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
  const double *__restrict__ d = g.d, *__restrict__ e2 = g.e2;
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
  if (lane == 0) lam[m - 1 - k] = -(lo + 0.5 * (hi - lo));  // most negative first
}

// Eigenvector of every eigenvalue by the twisted factorization of B - x: the
// pivots of the top-down and bottom-up eliminations, twisted where their
// combination is smallest, then one multiplication per entry in each
// direction.  One lane per vector; pivots and vectors are stored [row][vector],
// so every access of a wavefront is one 512-byte run.  Dp and Dm are scratch
// of V's shape (ld columns; V and its padding are zeroed by the caller).
// (The pointers are parameters for their no-alias promise: without it no entry of d
// or e is read before the last pivot is stored.)
__device__ __forceinline__ void tridiag_vector(const double *__restrict__ d,
                                               const double *__restrict__ e, int m, int a, double x,
                                               double *__restrict__ Dp, double *__restrict__ Dm,
                                               double *__restrict__ V, int64_t ld) {
  constexpr double kEps = 2.220446049250313e-16;
  auto pivot = [&](double q, double c) { return q == 0.0 ? kEps * c : q; };
  // both eliminations at once: two independent chains of divisions
  double qp = 0.0, qm = 0.0;
#pragma unroll 4
  for (int i = 0; i < m; ++i) {
    const int j = m - 1 - i;
    qp = i == 0 ? d[0] - x : (d[i] - x) - e[i - 1] * e[i - 1] / qp;
    qm = i == 0 ? d[j] - x : (d[j] - x) - e[j] * e[j] / qm;
    qp = pivot(qp, i + 1 < m ? e[i] : d[i]);
    qm = pivot(qm, j > 0 ? e[j - 1] : d[0]);
    Dp[i * ld + a] = qp;
    Dm[j * ld + a] = qm;
  }
  double best = 0.0;
  int r = m - 1;
#pragma unroll 8
  for (int i = m - 1; i >= 0; --i) {
    const double t = fabs(Dp[i * ld + a] + Dm[i * ld + a] - (d[i] - x));
    if (i == m - 1 || t < best) {
      best = t;
      r = i;
    }
  }
  double s = 0.0, zu = 0.0, zd = 0.0;  // towards row 0, towards row m - 1
#pragma unroll 4
  for (int i = 0; i < m; ++i) {
    const int j = m - 1 - i;
    if (j < r) zu *= e[j] / Dp[j * ld + a];
    if (j == r) zu = 1.0;
    if (j <= r) {
      V[j * ld + a] = zu;
      s += zu * zu;
    }
    if (i > r) {
      zd *= e[i - 1] / Dm[i * ld + a];
      V[i * ld + a] = zd;
      s += zd * zd;
    }
    if (i == r) zd = 1.0;
  }
  const double inv = 1.0 / sqrt(s);
#pragma unroll 8
  for (int i = 0; i < m; ++i) V[i * ld + a] *= inv;
}

__global__ __launch_bounds__(64) void k_tridiag_vectors(EigPair both) {
  const TridiagEig &g = both.p[blockIdx.y];
  const int a = blockIdx.x * 64 + threadIdx.x;
  if (a < g.m) tridiag_vector(g.d, g.e, g.m, a, -g.lam[a], g.Dp, g.Dm, g.V, g.ld);
}

// H = 1.5 I - 0.5 H (n x n): with H = V^T V, V H is the first-order step to
// the nearest orthonormal basis.
__global__ void k_polar_factor(double *__restrict__ H, int64_t n) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y;
  if (j >= n) return;
  H[i * n + j] = (i == j ? 1.5 : 0.0) - 0.5 * H[i * n + j];
}

__global__ void k_zero_below(double *__restrict__ W, const int *__restrict__ klo, int64_t ld) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y;
  if (j < ld && j < klo[i / kGemmGroup]) W[i * ld + j] = 0.0;
}

// out[j][i] = in[i][j] through a 64 x 64 LDS tile (both sides in 512-byte
// runs); rows and cols multiples of 64.
__global__ __launch_bounds__(256) void k_transpose(const double *__restrict__ in, int64_t ldi,
                                                   double *__restrict__ out, int64_t ldo) {
  __shared__ double t[64][65];
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int x = threadIdx.x & 63, y = threadIdx.x >> 6;
  for (int k = y; k < 64; k += 4) t[k][x] = in[(r0 + k) * ldi + c0 + x];
  __syncthreads();
  for (int k = y; k < 64; k += 4) out[(c0 + k) * ldo + r0 + x] = t[x][k];
}

// out[i][j] = sinv[2i + s] in[i][j] for i < m (rows beyond are zeroed).
__global__ void k_scale_rows(const double *__restrict__ in, const double *__restrict__ sinv, int s,
                             int64_t m, int64_t ld, double *__restrict__ out) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, i = blockIdx.y;
  if (j >= ld) return;
  out[i * ld + j] = i < m ? sinv[2 * i + s] * in[i * ld + j] : 0.0;
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

hipError_t launch_zero_below(double *W, const int *klo, int64_t rows, int64_t ld, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_below, dim3((unsigned)((ld + 255) / 256), (unsigned)rows), dim3(256), 0,
                     st, W, klo, ld);
  return hipGetLastError();
}

hipError_t launch_polar_factor(double *H, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_polar_factor, dim3((unsigned)((n + 255) / 256), (unsigned)n), dim3(256), 0,
                     st, H, n);
  return hipGetLastError();
}

hipError_t launch_transpose(const double *in, int64_t ldi, double *out, int64_t ldo, int64_t rows,
                            int64_t cols, hipStream_t st) {
  if (rows % 64 || cols % 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_transpose, dim3((unsigned)(cols / 64), (unsigned)(rows / 64)), dim3(256), 0,
                     st, in, ldi, out, ldo);
  return hipGetLastError();
}

hipError_t launch_scale_rows(const double *in, const double *sinv, int s, int64_t m, int64_t rows,
                             int64_t ld, double *out, hipStream_t st) {
  hipLaunchKernelGGL(k_scale_rows, dim3((unsigned)((ld + 255) / 256), (unsigned)rows), dim3(256), 0,
                     st, in, sinv, s, m, ld, out);
  return hipGetLastError();
}

}  // namespace fps
