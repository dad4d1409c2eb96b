// Eigenbasis form of the square, rectangle and cube solves.
//
// Every step of Algorithm 2 multiplies by rational functions of A~ from the
// left and from the right, so with A~ = V diag(lambda) V^T (per parity block)
// the J-step iterate is
//   Y_J = V [ (V^T G V) o (1 - e_i f_j) / (sx2 lambda_i + sy2 lambda_j) ] V^T,
//   e_i = prod_j (a_i - p_j) / (a_i - q_j),  a_i = sx2 lambda_i,
//   f_j = prod_j (b_j - q_j) / (b_j - p_j),  b_j = -sy2 lambda_j
// (the error of step j is (A - p)(A - q)^-1 E (B - q)(B - p)^-1; refinement
// rounds multiply their error factors).  The plan merges V with the dense
// coefficient maps on either side, V^T S^-1 R and P S^-1 V, so the whole
// solve is four dense products, whatever J: 4 n^3 operations on the matrix
// cores against 2 n^3 for the coefficient maps alone plus 2J passes of the
// array through HBM.  At n = 4096 (J = 96) the passes took 10.7 ms of 13.3;
// the extra 2 n^3 take 2.3 ms.  The passes grow as n^2 log n, the products as
// n^3, and at the largest size accepted (n = 16384) the products still take
// less.  One orthogonal transform each way also leaves less rounding than 2J
// sweeps (n = 4096: 2e-15 against 3e-14).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "solver.hpp"

namespace fps {
namespace detail {

namespace {

// C = A B for one block of zero-padded, contiguous operands.
hipError_t product(const double *A, int64_t lda, const double *B, int64_t ldb, double *C, int64_t ldc,
                   int64_t M, int64_t N, int64_t K, hipStream_t st) {
  fps::GemmProb g{A, B, C, M, N, K, lda, 1, ldb, 1, ldc, 1};
  return fps::launch_gemm(&g, 1, st);
}

// rows x cols (row-major) zero-padded to rp x cp.
std::vector<double> padded(const std::vector<double> &M, int64_t rows, int64_t cols, int64_t rp,
                           int64_t cp) {
  std::vector<double> out((size_t)(rp * cp), 0.0);
  for (int64_t i = 0; i < rows; ++i)
    std::copy(M.begin() + i * cols, M.begin() + (i + 1) * cols, out.begin() + i * cp);
  return out;
}

// Zeros of Wo.  Mode a of parity s is u = cos or sin of x y, x = (pi / 2)
// (2a + s + 1), as far as it is resolved, so its Chebyshev coefficient of
// index k is ~ J_k(x), which beyond k = x falls like
// exp(-k (acosh(k/x) - sqrt(1 - (x/k)^2))); its C~ coefficients are
// ~ J_{k+3/2}(x).  Entries below exp(-43) = 2e-19 of their column are taken as
// zero: 0.004 of an ulp of what the mode contributes, while the rounding of the
// eigenvectors leaves ~1e-17 there (LAPACK's vectors have at most 1e-30 in this
// region, n = 200 ... 4096).  A mode with coefficients to drop at some k <= n + 1
// is resolved to better than that.  The share of zeros is 17 % at n = 200, 26 %
// at 1000 and 29 % at 4096.
void wo_zeros(int s, int64_t rows, int64_t modes, std::vector<int> &klo, std::vector<int> &khi) {
  constexpr double kPi = 3.14159265358979323846;
  const int64_t ng = (rows + fps::kGemmGroup - 1) / fps::kGemmGroup;
  const int64_t nh = (modes + fps::kGemmGroup - 1) / fps::kGemmGroup;
  klo.assign((size_t)ng, 0);
  khi.assign((size_t)nh, 0);
  for (int64_t g = 0; g < ng; ++g) {
    const double k = (double)(2 * g * fps::kGemmGroup + s);
    double lo = 0.0, hi = k;  // the largest x with k (...) >= 43
    for (int it = 0; it < 60 && k > 0.0; ++it) {
      const double x = 0.5 * (lo + hi), t = x / k;
      if (k * (std::acosh(1.0 / t) - std::sqrt(1.0 - t * t)) >= 43.0) lo = x; else hi = x;
    }
    const double a = std::floor(lo / kPi - 0.5 * (s + 1));
    klo[(size_t)g] = (int)std::min((double)modes, std::max(0.0, a));
  }
  for (int64_t h = 0; h < nh; ++h)
    for (int64_t g = 0; g < ng; ++g)
      if (klo[(size_t)g] < (h + 1) * fps::kGemmGroup)
        khi[(size_t)h] = (int)std::min(rows, (g + 1) * fps::kGemmGroup);
}

fps_status alloc(DeviceBuf &b, int64_t doubles) {
  if (hipMalloc(&b.p, (size_t)doubles * 8) != hipSuccess)
    return fail(FPS_E_NOMEM, "hipMalloc of a plan table failed");
  return FPS_OK;
}

}  // namespace

// Eigenpairs of the parity blocks of A~ and the merged maps, in both
// orientations (d_Wi / d_WiT, d_Wo / d_WoT); pl->lam gets the eigenvalues by
// storage position.  The plan's L, Rs, P, mop and sinv are set; lift (or null)
// holds the Dirichlet lift map S^-1 C~(T_k''), merged the same way.
fps_status spectral_build(fps_plan *pl, const std::vector<double> *lift) {
  const fps::Layout &L = pl->L;
  const bool native = pl->out_basis == FPS_OUT_NATIVE;
  const double n = (double)pl->n;
  hipStream_t st = nullptr;
  fps_status s;
  pl->lam.assign((size_t)L.npad, -1.0);
  std::vector<double> v0((size_t)L.npad, 0.0);  // first row of each V_s
  for (int sp = 0; sp < 2; ++sp) {
    const int64_t m = L.m[sp], mp = L.mp[sp], mop = native ? mp : pl->mop[sp];
    if (m == 0) continue;
    std::vector<double> d((size_t)m), e((size_t)m, 0.0), e2((size_t)m, 0.0);
    for (int64_t k = 0; k < m; ++k) {
      d[(size_t)k] = -fps::atilde_diag(2 * k + sp);
      if (k + 1 < m) e[(size_t)k] = fps::atilde_off(2 * k + sp);
      e2[(size_t)k] = e[(size_t)k] * e[(size_t)k];
    }
    DeviceBuf dd, de, de2, dl, map, tmp;
    if ((s = upload(dd, d)) != FPS_OK || (s = upload(de, e)) != FPS_OK ||
        (s = upload(de2, e2)) != FPS_OK || (s = alloc(dl, m)) != FPS_OK ||
        (s = alloc(tmp, 4 * mp * mp)) != FPS_OK)
      return s;
    double *T0 = (double *)tmp.p, *T1 = T0 + mp * mp, *V = T1 + mp * mp, *VT = V + mp * mp;
    const double *lam = (const double *)dl.p;
    // Lemma B.1: sigma(-A~) lies in [1 / (30 n^4), 1]
    FPS_HIP(fps::launch_fill(V, mp * mp, 0.0, st));
    FPS_HIP(fps::launch_tridiag_eig((const double *)dd.p, (const double *)de.p, (const double *)de2.p,
                                    m, 0.5 / (30.0 * n * n * n * n), 1.01, (double *)dl.p, T0, T1, V,
                                    mp, st));
    // The vectors are orthogonal to about m eps (neighbouring eigenvalues
    // differ by a relative 2 / m); one polar step V <- V (3 I - V^T V) / 2
    // squares that.
    FPS_HIP(fps::launch_transpose(V, mp, VT, mp, mp, mp, st));
    FPS_HIP(product(VT, mp, V, mp, T0, mp, mp, mp, mp, st));
    FPS_HIP(fps::launch_polar_factor(T0, mp, st));
    FPS_HIP(product(V, mp, T0, mp, T1, mp, mp, mp, mp, st));
    std::swap(V, T1);
    FPS_HIP(fps::launch_transpose(V, mp, VT, mp, mp, mp, st));
    // input map V^T (S^-1 R)
    if ((s = upload(map, padded(pl->Rs[sp], m, m, mp, mp))) != FPS_OK ||
        (s = alloc(pl->d_Wi[sp], mp * mp)) != FPS_OK || (s = alloc(pl->d_WiT[sp], mp * mp)) != FPS_OK ||
        (s = alloc(pl->d_Wo[sp], mop * mp)) != FPS_OK || (s = alloc(pl->d_WoT[sp], mop * mp)) != FPS_OK)
      return s;
    double *Wi = (double *)pl->d_Wi[sp].p, *Wo = (double *)pl->d_Wo[sp].p;
    FPS_HIP(product(VT, mp, (const double *)map.p, mp, Wi, mp, mp, mp, mp, st));
    FPS_HIP(fps::launch_transpose(Wi, mp, (double *)pl->d_WiT[sp].p, mp, mp, mp, st));
    // output map (P S^-1) V, or S^-1 V for the native coefficients
    DeviceBuf pmap;
    if (native) {
      FPS_HIP(fps::launch_scale_rows(V, (const double *)pl->d_sinv.p, sp, m, mp, mp, Wo, st));
    } else {
      if ((s = upload(pmap, padded(pl->P[sp], L.mo[sp], m, mop, mp))) != FPS_OK) return s;
      FPS_HIP(product((const double *)pmap.p, mp, V, mp, Wo, mp, mop, mp, mp, st));
    }
    wo_zeros(sp, native ? m : L.mo[sp], m, pl->klo[sp], pl->khi[sp]);
    if ((s = upload(pl->d_klo[sp], pl->klo[sp])) != FPS_OK ||
        (s = upload(pl->d_khi[sp], pl->khi[sp])) != FPS_OK)
      return s;
    FPS_HIP(fps::launch_zero_below(Wo, (const int *)pl->d_klo[sp].p, native ? m : L.mo[sp], mp, st));
    FPS_HIP(fps::launch_transpose(Wo, mp, (double *)pl->d_WoT[sp].p, mop, mop, mp, st));
    // Dirichlet lift map V^T S^-1 C~(T_k''), m x mop
    DeviceBuf lmap;
    if (lift) {
      const int64_t lp = pl->mop[sp];
      if ((s = upload(lmap, padded(lift[sp], m, L.mo[sp], mp, lp))) != FPS_OK ||
          (s = alloc(pl->d_lift[sp], mp * lp)) != FPS_OK)
        return s;
      FPS_HIP(product(VT, mp, (const double *)lmap.p, lp, (double *)pl->d_lift[sp].p, lp, mp, lp, mp,
                      st));
    }
    FPS_HIP(hipMemcpy(pl->lam.data() + sp * L.mp[0], lam, (size_t)m * 8, hipMemcpyDeviceToHost));
    FPS_HIP(hipMemcpy(v0.data() + sp * L.mp[0], V, (size_t)m * 8, hipMemcpyDeviceToHost));
  }
  if (lift) {
    // V^T of the scaled C~ coefficients of (1 - t)/2 and (1 + t)/2, which are
    // nonzero at degrees 0 and 1 only
    const BcLiftConst k = bc_lift_const();
    std::vector<double> a((size_t)(2 * L.npad), 0.0);
    for (int sp = 0; sp < 2; ++sp)
      for (int64_t i = 0; i < L.m[sp]; ++i) {
        const size_t r = (size_t)(sp * L.mp[0] + i);
        a[2 * r] = k.sinv[sp] * k.am[sp] * v0[r];
        a[2 * r + 1] = k.sinv[sp] * k.ap[sp] * v0[r];
      }
    if ((s = upload(pl->d_lina, a)) != FPS_OK) return s;
  }
  return FPS_OK;
}

// Row and column factors of the 2-D multiplier (see the top of the file) by
// storage position: (sx2 lambda_i, e_i) and (sy2 lambda_j, f_j).
fps_status spectral_factors_2d(fps_plan *pl) {
  const fps::Layout &L = pl->L;
  std::vector<double> r((size_t)(2 * L.npad)), c((size_t)(2 * L.npad));
  for (int64_t i = 0; i < L.npad; ++i) {
    const double a = pl->sx2 * pl->lam[(size_t)i], b = -pl->sy2 * pl->lam[(size_t)i];
    double e = 1.0, f = 1.0;
    for (const fps::ShiftSet &sh : pl->rsh)
      for (int j = 0; j < sh.J; ++j) {
        e *= (a - sh.p[(size_t)j]) / (a - sh.q[(size_t)j]);
        f *= (b - sh.q[(size_t)j]) / (b - sh.p[(size_t)j]);
      }
    r[2 * i] = a;
    r[2 * i + 1] = e;
    c[2 * i] = -b;
    c[2 * i + 1] = f;
  }
  fps_status s;
  if ((s = upload(pl->d_mr, r)) != FPS_OK) return s;
  return upload(pl->d_mc, c);
}

}  // namespace detail
}  // namespace fps
