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
fps::GemmProb product(const double *A, int64_t lda, const double *B, int64_t ldb, double *C, int64_t ldc,
                      int64_t M, int64_t N, int64_t K) {
  return fps::GemmProb{A, B, C, M, N, K, lda, 1, ldb, 1, ldc, 1};
}

// rows x cols (row-major) into zeros with row stride cp.
void padded(const std::vector<double> &M, int64_t rows, int64_t cols, int64_t cp, double *out) {
  for (int64_t i = 0; i < rows; ++i) std::copy(M.begin() + i * cols, M.begin() + (i + 1) * cols, out + i * cp);
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

// Consecutive pieces of one allocation, in doubles, each 256-byte aligned.
struct Pieces {
  int64_t size = 0;
  int64_t take(int64_t doubles) {
    const int64_t at = size;
    size += (doubles + 31) / 32 * 32;
    return at;
  }
};

// Row and column factors of the 2-D multiplier (see the top of the file) by
// storage position: (sx2 lambda_i, e_i) and (sy2 lambda_j, f_j).
void factors_2d(const fps_plan *pl, double *r, double *c) {
  for (int64_t i = 0; i < pl->L.npad; ++i) {
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
}

}  // namespace

// Eigenpairs of the parity blocks of A~ and the merged maps, in both
// orientations (d_Wi / d_WiT, d_Wo / d_WoT); pl->lam gets the eigenvalues by
// storage position; 2-D plans also get the multiplier's factors.  The plan's L, Rs, P,
// mop, sinv (and shifts) are set; lift (or null) holds the Dirichlet lift map
// S^-1 C~(T_k''), merged the same way.  One allocation for the plan's tables, one
// for the temporaries, an upload per parity, one read-back and one more upload: at
// n = 64 the calls took longer than the kernels (plan creation 1.32 -> 0.95 ms).
fps_status spectral_build(fps_plan *pl, const std::vector<double> *lift) {
  const fps::Layout &L = pl->L;
  const bool native = pl->out_basis == FPS_OUT_NATIVE;
  const double n = (double)pl->n;
  hipStream_t st = nullptr;
  const int64_t *mp = L.mp;
  int64_t mop[2];
  Pieces keep, tmp;
  int64_t wi[2], wit[2], wo[2], wot[2], li[2], small[2], v[2];  // offsets in the two allocations
  struct Input {
    int64_t d, e, e2, klo, map, pmap, lmap, size;  // of one parity's upload
  } in[2];
  const int64_t lam_at = tmp.take(L.npad);
  int64_t up[2];
  for (int sp = 0; sp < 2; ++sp) {
    const int64_t m = L.m[sp];
    mop[sp] = native ? mp[sp] : pl->mop[sp];
    if (m == 0) continue;
    wo_zeros(sp, native ? m : L.mo[sp], m, pl->klo[sp], pl->khi[sp]);
    wi[sp] = keep.take(mp[sp] * mp[sp]);
    wit[sp] = keep.take(mp[sp] * mp[sp]);
    wo[sp] = keep.take(mop[sp] * mp[sp]);
    wot[sp] = keep.take(mop[sp] * mp[sp]);
    li[sp] = lift ? keep.take(mp[sp] * pl->mop[sp]) : 0;
    Pieces q;
    in[sp].d = q.take(m);
    in[sp].e = q.take(m);
    in[sp].e2 = q.take(m);
    in[sp].klo = q.take((int64_t)pl->klo[sp].size());  // ints
    in[sp].map = q.take(mp[sp] * mp[sp]);
    in[sp].pmap = native ? 0 : q.take(mop[sp] * mp[sp]);
    in[sp].lmap = lift ? q.take(mp[sp] * pl->mop[sp]) : 0;
    in[sp].size = q.size;
    up[sp] = tmp.take(q.size);
    v[sp] = tmp.take(4 * mp[sp] * mp[sp]);
  }
  const int64_t nf = pl->dim == 2 ? 2 * L.npad : 0;
  Pieces fin;  // the last upload
  const int64_t mr = fin.take(nf), mc = fin.take(nf), lina = fin.take(lift ? 2 * L.npad : 0);
  for (int sp = 0; sp < 2; ++sp)
    small[sp] = fin.take((int64_t)(pl->klo[sp].size() + pl->khi[sp].size()));  // ints
  const int64_t fin_at = keep.take(fin.size);
  DeviceBuf work;
  if (hipMalloc(&pl->d_maps.p, (size_t)keep.size * 8) != hipSuccess ||
      hipMalloc(&work.p, (size_t)tmp.size * 8) != hipSuccess)
    return fail(FPS_E_NOMEM, "hipMalloc of a plan table failed");
  double *K = (double *)pl->d_maps.p, *W = (double *)work.p;

  fps::TridiagEig eig[2] = {};
  for (int sp = 0; sp < 2; ++sp) {
    const int64_t m = L.m[sp], mm = mp[sp];
    if (m == 0) continue;
    const Input &q = in[sp];
    std::vector<double> h((size_t)q.size, 0.0);
    for (int64_t k = 0; k < m; ++k) {
      const double off = k + 1 < m ? fps::atilde_off(2 * k + sp) : 0.0;
      h[(size_t)(q.d + k)] = -fps::atilde_diag(2 * k + sp);
      h[(size_t)(q.e + k)] = off;
      h[(size_t)(q.e2 + k)] = off * off;
    }
    std::copy(pl->klo[sp].begin(), pl->klo[sp].end(), (int *)(h.data() + q.klo));
    padded(pl->Rs[sp], m, m, mm, h.data() + q.map);
    if (!native) padded(pl->P[sp], L.mo[sp], m, mm, h.data() + q.pmap);
    if (lift) padded(lift[sp], m, L.mo[sp], pl->mop[sp], h.data() + q.lmap);
    const double *D = W + up[sp];
    FPS_HIP(hipMemcpy(W + up[sp], h.data(), h.size() * 8, hipMemcpyHostToDevice));
    double *T0 = W + v[sp];
    eig[sp] = fps::TridiagEig{D + q.d, D + q.e, D + q.e2, W + lam_at + sp * mp[0],
                              T0, T0 + mm * mm, T0 + 2 * mm * mm, mm, (int)m};
    FPS_HIP(fps::launch_fill(eig[sp].V, mm * mm, 0.0, st));
  }
  // Lemma B.1: sigma(-A~) lies in [1 / (30 n^4), 1]
  FPS_HIP(fps::launch_tridiag_eig(eig, 0.5 / (30.0 * n * n * n * n), 1.01, st));
  // Stage by stage, the products of both parities in one launch.
  const int np = L.m[1] > 0 ? 2 : 1;
  double *Vs[2] = {}, *VTs[2] = {};
  fps::GemmProb g[4];
  // The vectors are orthogonal to about m eps (neighbouring eigenvalues
  // differ by a relative 2 / m); one polar step V <- V (3 I - V^T V) / 2
  // squares that.
  for (int sp = 0; sp < np; ++sp) {
    const int64_t mm = mp[sp];
    const fps::TridiagEig &x = eig[sp];
    VTs[sp] = x.V + mm * mm;
    FPS_HIP(fps::launch_transpose(x.V, mm, VTs[sp], mm, mm, mm, st));
    g[sp] = product(VTs[sp], mm, x.V, mm, x.Dp, mm, mm, mm, mm);
  }
  FPS_HIP(fps::launch_gemm(g, np, st));
  for (int sp = 0; sp < np; ++sp) {
    const int64_t mm = mp[sp];
    const fps::TridiagEig &x = eig[sp];
    FPS_HIP(fps::launch_polar_factor(x.Dp, mm, st));
    g[sp] = product(x.V, mm, x.Dp, mm, x.Dm, mm, mm, mm, mm);
    Vs[sp] = x.Dm;
  }
  FPS_HIP(fps::launch_gemm(g, np, st));
  // input maps V^T (S^-1 R); output maps (P S^-1) V, or S^-1 V for the native
  // coefficients; Dirichlet lift maps V^T S^-1 C~(T_k''), m x mop
  int cnt = 0;
  for (int sp = 0; sp < np; ++sp) {
    const int64_t mm = mp[sp];
    const double *D = W + up[sp];
    pl->d_Wi[sp].p = K + wi[sp];
    pl->d_WiT[sp].p = K + wit[sp];
    pl->d_Wo[sp].p = K + wo[sp];
    pl->d_WoT[sp].p = K + wot[sp];
    FPS_HIP(fps::launch_transpose(Vs[sp], mm, VTs[sp], mm, mm, mm, st));
    g[cnt++] = product(VTs[sp], mm, D + in[sp].map, mm, K + wi[sp], mm, mm, mm, mm);
    if (native)
      FPS_HIP(fps::launch_scale_rows(Vs[sp], (const double *)pl->d_sinv.p, sp, L.m[sp], mm, mm,
                                     K + wo[sp], st));
    else
      g[cnt++] = product(D + in[sp].pmap, mm, Vs[sp], mm, K + wo[sp], mm, mop[sp], mm, mm);
  }
  FPS_HIP(fps::launch_gemm(g, cnt, st));
  for (int sp = 0; sp < np; ++sp) {
    const int64_t mm = mp[sp], lp = pl->mop[sp];
    const double *D = W + up[sp];
    FPS_HIP(fps::launch_transpose(K + wi[sp], mm, K + wit[sp], mm, mm, mm, st));
    FPS_HIP(fps::launch_zero_below(K + wo[sp], (const int *)(D + in[sp].klo),
                                   native ? L.m[sp] : L.mo[sp], mm, st));
    FPS_HIP(fps::launch_transpose(K + wo[sp], mm, K + wot[sp], mop[sp], mop[sp], mm, st));
    if (lift) {
      pl->d_lift[sp].p = K + li[sp];
      g[sp] = product(VTs[sp], mm, D + in[sp].lmap, lp, K + li[sp], lp, mm, lp, mm);
    }
  }
  if (lift) FPS_HIP(fps::launch_gemm(g, np, st));
  std::vector<double> lam((size_t)L.npad);
  FPS_HIP(hipMemcpy(lam.data(), W + lam_at, lam.size() * 8, hipMemcpyDeviceToHost));
  pl->lam.assign((size_t)L.npad, -1.0);
  for (int sp = 0; sp < 2; ++sp)
    std::copy_n(lam.begin() + sp * mp[0], L.m[sp], pl->lam.begin() + sp * mp[0]);
  std::vector<double> h((size_t)fin.size, 0.0);
  if (nf > 0) factors_2d(pl, h.data() + mr, h.data() + mc);
  if (lift) {
    // V^T of the scaled C~ coefficients of (1 - t)/2 and (1 + t)/2, which are
    // nonzero at degrees 0 and 1 only: the first row of each V
    const BcLiftConst k = bc_lift_const();
    for (int sp = 0; sp < 2; ++sp) {
      if (L.m[sp] == 0) continue;
      std::vector<double> v0((size_t)L.m[sp]);
      FPS_HIP(hipMemcpy(v0.data(), Vs[sp], v0.size() * 8, hipMemcpyDeviceToHost));
      for (int64_t i = 0; i < L.m[sp]; ++i) {
        const int64_t r = lina + 2 * (sp * mp[0] + i);
        h[(size_t)r] = k.sinv[sp] * k.am[sp] * v0[(size_t)i];
        h[(size_t)(r + 1)] = k.sinv[sp] * k.ap[sp] * v0[(size_t)i];
      }
    }
  }
  for (int sp = 0; sp < 2; ++sp) {
    int *z = (int *)(h.data() + small[sp]);
    std::copy(pl->klo[sp].begin(), pl->klo[sp].end(), z);
    std::copy(pl->khi[sp].begin(), pl->khi[sp].end(), z + pl->klo[sp].size());
    pl->d_klo[sp].p = (int *)(K + fin_at + small[sp]);
    pl->d_khi[sp].p = (int *)(K + fin_at + small[sp]) + pl->klo[sp].size();
  }
  pl->d_mr.p = K + fin_at + mr;
  pl->d_mc.p = K + fin_at + mc;
  if (lift) pl->d_lina.p = K + fin_at + lina;
  FPS_HIP(hipMemcpy(K + fin_at, h.data(), h.size() * 8, hipMemcpyHostToDevice));
  return FPS_OK;
}

}  // namespace detail
}  // namespace fps
