// gfx950 element-wise and data-movement kernels of the spectral Poisson
// solver: parity-blocked permutations, the sweeps' final pass, fill.
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace fps {

namespace {

__global__ void k_finalize(const double *__restrict__ x, const double *__restrict__ ab,
                           const double *__restrict__ tab, double *__restrict__ out, int64_t n,
                           int64_t npad, int64_t mp0, int64_t mstride, int64_t ncmax) {
  const int64_t col = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
  if (col >= npad) return;
  const int s = r >= mp0 ? 1 : 0;
  const int64_t k = r - (s ? mp0 : 0);
  const int64_t c = k / kChunk;
  const double *tp = tab + (int64_t)s * kNTab * mstride;
  const double *e = ab + (((int64_t)s * ncmax + c) * npad + col) * 2;
  const double v = x[r * npad + col] + e[0] * tp[T_BF2 * mstride + k] + e[1] * tp[T_BK2 * mstride + k];
  const int t = col >= mp0 ? 1 : 0;
  const int64_t kc = col - (t ? mp0 : 0);
  const int64_t i = 2 * k + s, j = 2 * kc + t;
  if (i >= n || j >= n) return;
  out[i * n + j] = v;
}

__global__ void k_permute_in(const double *__restrict__ src, double *__restrict__ dst, int64_t n,
                             int64_t npad, int64_t mp0) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
  if (q >= npad) return;
  const int s = r >= mp0 ? 1 : 0, t = q >= mp0 ? 1 : 0;
  const int64_t i = 2 * (r - (s ? mp0 : 0)) + s, j = 2 * (q - (t ? mp0 : 0)) + t;
  double v = 0.0;
  if (i < n && j < n) v = src[i * n + j];
  dst[r * npad + q] = v;
}

__global__ void k_fill(double *__restrict__ dst, int64_t count, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = v;
}

__global__ void k_copy(const double *__restrict__ src, double *__restrict__ dst, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = src[i];
}

// --- cube ----------------------------------------------------------------

// natural n^3 -> parity-blocked npad^3 (zero padding)
__global__ void k_permute3_in(const double *__restrict__ src, double *__restrict__ dst, int64_t n,
                              int64_t npad, int64_t mp0) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t ry = blockIdx.y, rz = blockIdx.z;
  if (q >= npad) return;
  auto nat = [&](int64_t r) {
    const int s = r >= mp0 ? 1 : 0;
    return 2 * (r - (s ? mp0 : 0)) + s;
  };
  const int64_t ix = nat(q), iy = nat(ry), iz = nat(rz);
  double v = 0.0;
  if (ix < n && iy < n && iz < n) v = src[(iz * n + iy) * n + ix];
  dst[(rz * npad + ry) * npad + q] = v;
}

}  // namespace

hipError_t launch_permute3_in(const double *src, double *dst, int64_t n, int64_t npad, int64_t mp0,
                              hipStream_t st) {
  dim3 grid((unsigned)((npad + 255) / 256), (unsigned)npad, (unsigned)npad);
  hipLaunchKernelGGL(k_permute3_in, grid, dim3(256), 0, st, src, dst, n, npad, mp0);
  return hipGetLastError();
}

hipError_t launch_finalize(const double *x, const double *ab, const double *tab, double *out,
                           int64_t n, int64_t npad, int64_t mp0, int64_t mstride, int64_t ncmax,
                           hipStream_t st) {
  dim3 grid((unsigned)((npad + 255) / 256), (unsigned)npad);
  hipLaunchKernelGGL(k_finalize, grid, dim3(256), 0, st, x, ab, tab, out, n, npad, mp0, mstride, ncmax);
  return hipGetLastError();
}

hipError_t launch_permute_in(const double *src, double *dst, int64_t n, int64_t npad, int64_t mp0,
                             hipStream_t st) {
  dim3 grid((unsigned)((npad + 255) / 256), (unsigned)npad);
  hipLaunchKernelGGL(k_permute_in, grid, dim3(256), 0, st, src, dst, n, npad, mp0);
  return hipGetLastError();
}

hipError_t launch_copy(const double *src, double *dst, int64_t count, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, src, dst, count);
  return hipGetLastError();
}

hipError_t launch_fill(double *dst, int64_t count, double v, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, dst, count,
                     v);
  return hipGetLastError();
}

}  // namespace fps
