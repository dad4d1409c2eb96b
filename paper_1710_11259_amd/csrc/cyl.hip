// gfx950 kernels of the cylinder solve: the input permutation into the
// parity-blocked per-mode layout and the banded solves in r (one thread per
// |k| and z column, applying the LU factors computed by the plan with
// partial pivoting to the modes k and -k, real and imaginary parts).
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace fps {

namespace {

// X0[((slot * 2 + part) * npad + rpos) * npad + zpos] = F[idx][part][i][j]
// (zero at padded positions).  Thread e = ((sp * npad) + rpos) * mp + a
// reads the pair F[..][i][2a], F[..][i][2a + 1] (adjacent lanes read
// adjacent pairs) and writes the even-parity position a and the odd-parity
// position mp + a of row rpos.
__global__ __launch_bounds__(256) void k_cyl_permute_in(const double *__restrict__ F,
                                                        double *__restrict__ X0,
                                                        const int *__restrict__ slot_idx,
                                                        uint32_t n, uint32_t mp, uint32_t total) {
  const uint32_t e = blockIdx.x * 256u + threadIdx.x;
  if (e >= total) return;
  const uint32_t npad = 2 * mp, m = n / 2;
  const uint32_t a = e % mp, row = e / mp;
  const uint32_t rpos = row % npad, sp = row / npad;
  const uint32_t rs = rpos >= mp ? 1u : 0u, ra = rpos - (rs ? mp : 0u);
  double v0 = 0.0, v1 = 0.0;
  if (ra < m && a < m) {
    const int64_t i = 2 * (int64_t)ra + rs;
    const double *src = F + (((int64_t)slot_idx[sp >> 1] * 2 + (sp & 1)) * n + i) * n + 2 * (int64_t)a;
    v0 = src[0];
    v1 = src[1];
  }
  double *dst = X0 + ((int64_t)sp * npad + rpos) * npad;
  dst[a] = v0;
  dst[mp + a] = v1;
}

// One z column of half a |k| group: the banded systems (Q_k + lambda_j P_k)
// yhat = rhs of its kCylRhs / 2 right-hand sides (real and imaginary part), with
// the factors fac[((kabs * 8 + t) * mp + a) * npad + zpos], t: pivot offset,
// two multipliers, 1/u_aa, four superdiagonal entries of U.  rhs: X0 rows
// of parity rp (column zpos, stride npad), overwritten by the forward
// substitution; yhat: X1 rows of parity wp (zeros beyond m and for padded
// columns).
//
// Bound by HBM and by latency: 170 MB of factors and 134 MB a pass over the right-hand
// sides at 256 x 256, in 1032 wavefronts that each walk 256 dependent steps.  The
// factors and right-hand sides of kCylStep steps are loaded while the steps before
// are computed.  The halves of a group (one wavefront each) use the same factors.
// paired: they are one workgroup, so that one of them finds what the other has read
// in the compute unit's cache; else their workgroups are 8 apart, on one die, sharing
// its L2.
//
// Piv: false where none of the wavefront's 64 columns was factored with a row
// exchange (CylSolveGroup::pivots): the pivot offsets and the last two
// superdiagonals are then zero and are not read, 3 of the 8 fields: 101 MB of 806 at
// 256 x 256, the solve of the whole cylinder 523 -> 495 us.  At n = 64 and 256 the
// matrices with |k| != 2 need no exchange, those with |k| = 2 in few columns.
constexpr int kCylStep = 8, kHalf = kCylRhs / 2;

template <bool Piv>
struct CylForward {
  double pv[Piv ? kCylStep : 1], l1[kCylStep], l2[kCylStep], nb[kHalf][kCylStep];
};
template <bool Piv>
struct CylBackward {
  double iu[kCylStep], u[Piv ? 4 : 2][kCylStep], bv[kHalf][kCylStep];
};

template <bool Piv>
__device__ void cyl_columns(double *const (&b)[kHalf], double *const (&x)[kHalf],
                            const double *__restrict__ f0, int m, int mp, int npad) {
  const int64_t fs = (int64_t)mp * npad;  // between factor fields

  auto load_fwd = [&](CylForward<Piv> &q, int a0) {
#pragma unroll
    for (int t = 0; t < kCylStep; ++t) {
      const int a = min(a0 + t, m - 1);
      const double *f = f0 + (int64_t)a * npad;
      if constexpr (Piv) q.pv[t] = f[0];
      q.l1[t] = f[fs];
      q.l2[t] = f[2 * fs];
#pragma unroll
      for (int r = 0; r < kHalf; ++r) q.nb[r][t] = b[r][(int64_t)min(a0 + t + 3, m - 1) * npad];
    }
  };
  double w0[kHalf], w1[kHalf], w2[kHalf];
#pragma unroll
  for (int r = 0; r < kHalf; ++r) {
    w0[r] = b[r][0];
    w1[r] = m > 1 ? b[r][npad] : 0.0;
    w2[r] = m > 2 ? b[r][2 * npad] : 0.0;
  }
  auto run_fwd = [&](const CylForward<Piv> &q, int a0) {
#pragma unroll
    for (int t = 0; t < kCylStep; ++t) {
      const int a = a0 + t;
      if (a >= m) break;
      const int p = Piv ? (int)q.pv[Piv ? t : 0] : 0;
#pragma unroll
      for (int r = 0; r < kHalf; ++r) {
        const double v0 = p == 1 ? w1[r] : p == 2 ? w2[r] : w0[r];
        w1[r] = (p == 1 ? w0[r] : w1[r]) - q.l1[t] * v0;
        w2[r] = (p == 2 ? w0[r] : w2[r]) - q.l2[t] * v0;
        b[r][(int64_t)a * npad] = v0;
        w0[r] = w1[r];
        w1[r] = w2[r];
        w2[r] = a + 3 < m ? q.nb[r][t] : 0.0;
      }
    }
  };
  // (loads run ahead of the stores: those of step a are at rows past a + 2)
  CylForward<Piv> fa, fb;
  load_fwd(fa, 0);
  for (int a0 = 0; a0 < m; a0 += 2 * kCylStep) {
    load_fwd(fb, a0 + kCylStep);
    run_fwd(fa, a0);
    load_fwd(fa, a0 + 2 * kCylStep);
    run_fwd(fb, a0 + kCylStep);
  }

  auto load_bwd = [&](CylBackward<Piv> &q, int a1) {
#pragma unroll
    for (int t = 0; t < kCylStep; ++t) {
      const int a = max(a1 - t, 0);
      const double *f = f0 + (int64_t)a * npad;
      q.iu[t] = f[3 * fs];
#pragma unroll
      for (int i = 0; i < (Piv ? 4 : 2); ++i) q.u[i][t] = f[(4 + i) * fs];
#pragma unroll
      for (int r = 0; r < kHalf; ++r) q.bv[r][t] = b[r][(int64_t)a * npad];
    }
  };
  double x1[kHalf], x2[kHalf], x3[kHalf], x4[kHalf];
#pragma unroll
  for (int r = 0; r < kHalf; ++r) x1[r] = x2[r] = x3[r] = x4[r] = 0.0;
  auto run_bwd = [&](const CylBackward<Piv> &q, int a1) {
#pragma unroll
    for (int t = 0; t < kCylStep; ++t) {
      const int a = a1 - t;
      if (a < 0) break;
#pragma unroll
      for (int r = 0; r < kHalf; ++r) {
        double v = q.bv[r][t] - q.u[0][t] * x1[r] - q.u[1][t] * x2[r];
        if constexpr (Piv) {
          v = v - q.u[2][t] * x3[r] - q.u[3][t] * x4[r];
          x4[r] = x3[r];
          x3[r] = x2[r];
        }
        v *= q.iu[t];
        x[r][(int64_t)a * npad] = v;
        x2[r] = x1[r];
        x1[r] = v;
      }
    }
  };
  CylBackward<Piv> ba, bb;
  load_bwd(ba, m - 1);
  for (int a1 = m - 1; a1 >= 0; a1 -= 2 * kCylStep) {
    load_bwd(bb, a1 - kCylStep);
    run_bwd(ba, a1);
    load_bwd(ba, a1 - 2 * kCylStep);
    run_bwd(bb, a1 - kCylStep);
  }
}

__global__ __launch_bounds__(128, 1) void k_cyl_solve(double *__restrict__ X0,
                                                      double *__restrict__ X1,
                                                      const double *__restrict__ fac,
                                                      const CylSolveGroup *__restrict__ grp, int m,
                                                      int mp, int nzb, int nunits, int paired) {
  const int npad = 2 * mp;
  const int id = blockIdx.x, unit = paired ? id : (id >> 4) * 8 + (id & 7);
  const int half = paired ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : (id >> 3) & 1;
  if (unit >= nunits) return;
  const int zb = unit % nzb, zpos = zb * 64 + (threadIdx.x & 63);
  if (zpos >= npad) return;
  const CylSolveGroup &e = grp[unit / nzb];
  const int *sp = e.sp + half * kHalf;
  if (sp[0] < 0) return;  // the parts of a slot come in pairs
  double *b[kHalf], *x[kHalf];
#pragma unroll
  for (int r = 0; r < kHalf; ++r) {
    b[r] = X0 + ((int64_t)sp[r] * npad + e.rp * mp) * npad + zpos;
    x[r] = X1 + ((int64_t)sp[r] * npad + e.wp * mp) * npad + zpos;
  }
  int a = 0;
  if (zpos - (zpos >= mp ? mp : 0) < m) {
    const double *f0 = fac + ((int64_t)e.kabs * 8 * mp) * npad + zpos;
    if (e.pivots >> zb & 1)
      cyl_columns<true>(b, x, f0, m, mp, npad);
    else
      cyl_columns<false>(b, x, f0, m, mp, npad);
    a = m;
  }
  for (; a < mp; ++a)
#pragma unroll
    for (int r = 0; r < kHalf; ++r) x[r][(int64_t)a * npad] = 0.0;
}

}  // namespace

hipError_t launch_cyl_permute_in(const double *F, double *X0, const int *slot_idx, int64_t n,
                                 int64_t nt, int64_t mp, hipStream_t st) {
  const int64_t total = nt * 2 * (2 * mp) * mp;
  if (total <= 0) return hipSuccess;
  if (total >= ((int64_t)1 << 32) - 256) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cyl_permute_in, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, F,
                     X0, slot_idx, (uint32_t)n, (uint32_t)mp, (uint32_t)total);
  return hipGetLastError();
}

hipError_t launch_cyl_solve(double *X0, double *X1, const double *fac, const CylSolveGroup *grp,
                            int ngroups, int64_t m, int64_t mp, hipStream_t st) {
  if (ngroups <= 0) return hipSuccess;
  const int64_t nzb = (2 * mp + 63) / 64, units = nzb * ngroups;
  // n <= 512, n_theta <= 1024: at most 8 x 513 units
  // Pairs from two units per compute unit on: 496 -> 481 us for the whole solve at
  // 256 x 256 (516 units).  With fewer units the halves are as fast or faster apart, on more
  // compute units (apart / paired): 22.5 / 24.4 us at 64 x 64 (33 units), 118 / 123 at 256 x 64
  // (132), 190 / 193 at 256 x 96 (196), 306 / 318 at 256 x 160 (324), 420 / 421 at 256 x 224 (452),
  // 465.6 / 465.1 at 256 x 254 (512); the one size found the other way is 256 x 128 (260), 244 / 234.
  const int paired = units >= 512;
  const unsigned grid = (unsigned)(paired ? units : (units + 7) / 8 * 16);
  hipLaunchKernelGGL(k_cyl_solve, dim3(grid), dim3(paired ? 128 : 64), 0, st, X0, X1, fac, grp,
                     (int)m, (int)mp, (int)nzb, (int)units, paired);
  return hipGetLastError();
}

}  // namespace fps
