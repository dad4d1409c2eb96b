// gfx950 kernels of the nonhomogeneous Dirichlet lift (Sec. 6.1): the
// solution is u = u0 + u_bc with u_bc the transfinite interpolant of the four
// boundary traces,
//   u_bc = (1-s)/2 L(t) + (1+s)/2 R(t) + (1-t)/2 B(s) + (1+t)/2 T(s)
//          - (bilinear interpolant of the corner values B(-1), B(1), T(-1), T(1)),
// and u0 the zero-data solution for f - Lap u_bc.  Because u_bc is linear in
// s in its L, R terms and linear in t in its B, T terms,
//   Lap u_bc = sx2 [(1-t)/2 B''(s) + (1+t)/2 T''(s)]
//            + sy2 [(1-s)/2 L''(t) + (1+s)/2 R''(t)],
// a sum of four outer products.  In the eigenbasis of A~ its 1-D factors are
// the plan's merged lift map V^T S^-1 C~(T_k'') applied to the traces'
// Chebyshev coefficients (4 matrix-vector products with its parity blocks) and
// V^T of the linear factors (in the plan); the product that forms Y^ subtracts
// the outer products before its multiplier, and all other work is O(n).
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace fps {

namespace {

constexpr int kCornerThreads = 256;

// One workgroup per trace (L, R, B, T): its values at -1 and +1 into
// corner[2 tr], corner[2 tr + 1].
__global__ __launch_bounds__(kCornerThreads) void k_bc_corner(const double *__restrict__ bc,
                                                              double *__restrict__ corner,
                                                              int64_t n) {
  __shared__ double lds[2 * kCornerThreads];
  const int tr = blockIdx.x, t = threadIdx.x;
  const int64_t N = n + 2;
  const double *c = bc + tr * N;
  double vm = 0.0, vp = 0.0;
  for (int64_t k = t; k < N; k += kCornerThreads) {
    vp += c[k];
    vm += (k & 1) ? -c[k] : c[k];
  }
  lds[t] = vm;
  lds[kCornerThreads + t] = vp;
  __syncthreads();
  for (int h = kCornerThreads / 2; h > 0; h >>= 1) {
    if (t < h) {
      lds[t] += lds[t + h];
      lds[kCornerThreads + t] += lds[kCornerThreads + t + h];
    }
    __syncthreads();
  }
  if (t == 0) {
    corner[2 * tr] = lds[0];
    corner[2 * tr + 1] = lds[kCornerThreads];
  }
}

// One wavefront per eigenbasis row: w_X = V^T S^-1 C~(g_X'') of the four
// traces (the sum over k of the lift map's row times g_X), then the row's
// entries of the outer-product factors of
//   sx2 [am (B'')^T + ap (T'')^T] + sy2 [L'' am^T + R'' ap^T],
// am / ap the linear factors (1 - t)/2 and (1 + t)/2 (lina).
__global__ __launch_bounds__(256) void k_bc_cmap(const double *__restrict__ Ml0,
                                                 const double *__restrict__ Ml1, int64_t ld0,
                                                 int64_t ld1, const double *__restrict__ bc,
                                                 const double *__restrict__ lina,
                                                 double *__restrict__ lr, double *__restrict__ lc,
                                                 int64_t n, int64_t mp0, int64_t mo0, int64_t mo1,
                                                 double sx2, double sy2) {
  const int lane = threadIdx.x & 63;
  const int64_t pos = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // npad is a multiple of 4
  const int s = pos < mp0 ? 0 : 1;
  const int64_t a = s ? pos - mp0 : pos;
  double *r = lr + 4 * pos, *c = lc + 4 * pos;
  if (a >= (s ? n / 2 : (n + 1) / 2)) {  // padding (uniform per wavefront): inert
    if (lane < 4) r[lane] = c[lane] = 0.0;
    return;
  }
  const int64_t mo = s ? mo1 : mo0, N = n + 2;
  const double *Mrow = s ? Ml1 + a * ld1 : Ml0 + a * ld0;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  for (int64_t b = lane; b < mo; b += 64) {
    const double m = Mrow[b];
    const int64_t k = 2 * b + s;
    a0 += m * bc[k];
    a1 += m * bc[N + k];
    a2 += m * bc[2 * N + k];
    a3 += m * bc[3 * N + k];
  }
  for (int off = 32; off > 0; off >>= 1) {
    a0 += __shfl_xor(a0, off, 64);
    a1 += __shfl_xor(a1, off, 64);
    a2 += __shfl_xor(a2, off, 64);
    a3 += __shfl_xor(a3, off, 64);
  }
  if (lane == 0) {
    const double am = lina[2 * pos], ap = lina[2 * pos + 1];
    r[0] = sx2 * am;  // B is trace 2, T trace 3
    r[1] = sx2 * ap;
    r[2] = sy2 * a0;  // L is trace 0, R trace 1
    r[3] = sy2 * a1;
    c[0] = a2;
    c[1] = a3;
    c[2] = am;
    c[3] = ap;
  }
}

// U += Chebyshev coefficients of u_bc (natural (n+2) x (n+2), rows <-> t).
// (1 -+ s)/2 has Chebyshev coefficients (1/2, -+1/2).
__global__ void k_bc_out(double *__restrict__ U, const double *__restrict__ bc,
                         const double *__restrict__ corner, int64_t n) {
  const int64_t N = n + 2;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 2 * N + (N - 2) * 2) return;
  int64_t j, k;
  if (e < 2 * N) {
    j = e / N;
    k = e % N;
  } else {
    const int64_t f = e - 2 * N;
    j = 2 + f / 2;
    k = f % 2;
  }
  const double hm[2] = {0.5, -0.5}, hp[2] = {0.5, 0.5};
  const double *L = bc, *R = bc + N, *B = bc + 2 * N, *T = bc + 3 * N;
  double v = 0.0;
  if (k < 2) v += L[j] * hm[k] + R[j] * hp[k];
  if (j < 2) v += hm[j] * B[k] + hp[j] * T[k];
  if (j < 2 && k < 2) {
    const double c00 = corner[4], c10 = corner[5], c01 = corner[6], c11 = corner[7];
    v -= hm[j] * hm[k] * c00 + hm[j] * hp[k] * c10 + hp[j] * hm[k] * c01 + hp[j] * hp[k] * c11;
  }
  U[j * N + k] += v;
}

}  // namespace

hipError_t launch_bc_lift_rhs(const double *bc, const double *Ml0, const double *Ml1, int64_t ld0,
                              int64_t ld1, const double *lina, double *lr, double *lc, double *corner,
                              const Layout &L, double sx2, double sy2, hipStream_t st) {
  const int64_t n = L.n;
  hipLaunchKernelGGL(k_bc_corner, dim3(4), dim3(kCornerThreads), 0, st, bc, corner, n);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bc_cmap, dim3((unsigned)(L.npad / 4)), dim3(256), 0, st, Ml0, Ml1, ld0, ld1,
                     bc, lina, lr, lc, n, L.mp[0], L.mo[0], L.mo[1], sx2, sy2);
  return hipGetLastError();
}

hipError_t launch_bc_lift_out(double *U, const double *bc, const double *corner, int64_t n,
                              hipStream_t st) {
  const int64_t N = n + 2, total = 2 * N + (N - 2) * 2;
  hipLaunchKernelGGL(k_bc_out, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, U, bc,
                     corner, n);
  return hipGetLastError();
}

}  // namespace fps
