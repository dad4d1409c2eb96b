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
// less at tolerances below 1e-6.  With few steps at n > 5000 they take more (n = 10000, J =
// 13: 55 ms against 44), but the half-sweeps of so loose a tolerance round by up to
// 7e-11, the products by 2.5e-15.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "solver.hpp"

namespace fps {
namespace detail {

namespace {

// Zeros of Wo.  Mode a of parity s is u = cos or sin of x y, x = (pi / 2)
// (2a + s + 1), as far as it is resolved, so its Chebyshev coefficient of
// index k is ~ J_k(x), which beyond k = x falls like
// exp(-k (acosh(k/x) - sqrt(1 - (x/k)^2))); its C~ coefficients are
// ~ J_{k+3/2}(x).  Entries below exp(-43) = 2e-19 of their column are taken as
// zero: 0.004 of an ulp of what the mode contributes (LAPACK's vectors have at most
// 1e-30 in this region, n = 200 ... 4096).  A mode with coefficients to drop at some k <= n + 1
// is resolved to better than that.  The share of zeros is 17 % at n = 200, 26 %
// at 1000 and 29 % at 4096.  Modes are stored the highest first: mode a at modes - 1 - a.
void wo_zeros(int s, int64_t rows, int64_t modes, std::vector<int> &mlim, std::vector<int> &clim) {
  constexpr double kPi = 3.14159265358979323846;
  const int64_t ng = (rows + fps::kGemmGroup - 1) / fps::kGemmGroup;
  const int64_t nh = (modes + fps::kGemmGroup - 1) / fps::kGemmGroup;
  mlim.assign((size_t)ng, 0);
  clim.assign((size_t)nh, 0);
  for (int64_t g = 0; g < ng; ++g) {
    const double k = (double)(2 * g * fps::kGemmGroup + s);
    double lo = 0.0, hi = k;  // the largest x with k (...) >= 43
    for (int it = 0; it < 60 && k > 0.0; ++it) {
      const double x = 0.5 * (lo + hi), t = x / k;
      if (k * (std::acosh(1.0 / t) - std::sqrt(1.0 - t * t)) >= 43.0) lo = x; else hi = x;
    }
    const double a = std::floor(lo / kPi - 0.5 * (s + 1));
    mlim[(size_t)g] = (int)(modes - (int64_t)std::min((double)modes, std::max(0.0, a)));
  }
  for (int64_t h = 0; h < nh; ++h)
    for (int64_t g = 0; g < ng; ++g)
      if (mlim[(size_t)g] > h * fps::kGemmGroup)
        clim[(size_t)h] = (int)std::min(rows, (g + 1) * fps::kGemmGroup);
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

// Sweep tables of the stage entry point fps_adi_native: one per step (a rectangle has
// two).
struct SweepTables {
  std::vector<double> pos, chunk, l1;
  explicit SweepTables(const fps_plan *pl) {
    std::vector<double> alpha, beta;
    for (int j = 0; j < pl->shifts.J; ++j) {
      alpha.push_back(pl->rect ? pl->sy2 : 1.0);  // rectangle: table 2j: sy2 A~ + p_j,
      beta.push_back(pl->shifts.p[j]);
      if (pl->rect) {  // 2j + 1: sx2 A~ - q_j
        alpha.push_back(pl->sx2);
        beta.push_back(-pl->shifts.q[j]);
      }
    }
    fps::build_sweep_tables_ab(pl->L, alpha, beta, pos, chunk, nullptr, l1);
  }
};

// Extended-precision values as pairs in a host image of doubles: h at `at`, l
// v.size() further on.
void put_pairs(std::vector<double> &h, int64_t at, const std::vector<long double> &v) {
  for (size_t i = 0; i < v.size(); ++i) {
    h[(size_t)at + i] = (double)v[i];
    h[(size_t)at + v.size() + i] = (double)(v[i] - (long double)(double)v[i]);
  }
}

// A map's tables in the upload image, its entries' place among the temporaries.
struct MapAt {
  fps::MapTables tab;
  int64_t row, col, t, u;
  void place(Pieces &q) {
    row = q.take(2 * (int64_t)tab.row.size());
    col = q.take(2 * (int64_t)tab.col.size());
    t = q.take(2 * (int64_t)tab.t.size());
    u = q.take(2 * (int64_t)tab.u.size());
  }
  void put(std::vector<double> &h) const {
    put_pairs(h, row, tab.row);
    put_pairs(h, col, tab.col);
    put_pairs(h, t, tab.t);
    put_pairs(h, u, tab.u);
  }
  // entries M, zero-padded to prows x ld
  fps::MapEntries entries(double *W, double *M, int64_t prows, int64_t ld) const {
    auto pair = [&](int64_t at, const std::vector<long double> &v) {
      return fps::PairArray{W + at, (int64_t)v.size()};
    };
    return fps::MapEntries{pair(row, tab.row), pair(col, tab.col), pair(t, tab.t), pair(u, tab.u),
                           fps::PairArray{M, prows * ld}, tab.rows, tab.cols, prows, ld};
  }
};

}  // namespace

// Eigenpairs of the parity blocks of A~ and the merged maps, in both
// orientations (d_Wi / d_WiT, d_Wo / d_WoT); pl->lam gets the eigenvalues by
// storage position, in each parity the one next to zero (the highest mode) first, so that
// sums over modes end with the largest terms (lowest mode first: rms error of adjoints
// against an extended-precision reference 1.5e-15 of the result at n = 1024, 3e-15 at 2048;
// this way 2e-16 and 1e-16, half-sweeps 2e-16 and 5e-16); 2-D plans also get the multiplier's factors.  The plan's L, mop
// (and shifts) are set; lift: also the Dirichlet lift map, merged the same way.  The maps'
// closed forms (MapTables) are tables of O(n), so the uploads are short and everything of
// O(n^2) or more is formed on the device, in pairs of doubles until its one
// rounding.  One allocation for the plan's tables, one for the temporaries, and FP64 2-D
// plans build their sweep tables on the host while the kernels run (plan creation at n = 64
// 766 -> 495 us, at 515 5.5 -> 2.6 ms, the bisection for the computed spectrum without its
// square roots and idle steps included).
fps_status spectral_build(fps_plan *pl, bool lift) {
  const fps::Layout &L = pl->L;
  const bool native = pl->out_basis == FPS_OUT_NATIVE;
  const double n = (double)pl->n;
  hipStream_t st = nullptr;
  const int64_t *mp = L.mp;
  const int np = L.m[1] > 0 ? 2 : 1;
  int64_t mop[2];
  Pieces keep, tmp;
  int64_t wi[2], wit[2], wo[2], wot[2], li[2], small[2];  // offsets in the two allocations
  int64_t d[2], e[2], e2[2], lim[2], v[2], s0[2], s1[2];
  MapAt in[2], out[2], lm[2];
  for (int sp = 0; sp < np; ++sp) {
    const int64_t m = L.m[sp];
    mop[sp] = native ? mp[sp] : pl->mop[sp];
    wo_zeros(sp, native ? m : L.mo[sp], m, pl->mlim[sp], pl->clim[sp]);
    wi[sp] = keep.take(mp[sp] * mp[sp]);
    wit[sp] = keep.take(mp[sp] * mp[sp]);
    wo[sp] = keep.take(mop[sp] * mp[sp]);
    wot[sp] = keep.take(mop[sp] * mp[sp]);
    li[sp] = lift ? keep.take(mp[sp] * pl->mop[sp]) : 0;
    // the upload, at the front of the temporaries
    d[sp] = tmp.take(2 * m);
    e[sp] = tmp.take(2 * m);
    e2[sp] = tmp.take(m);
    lim[sp] = tmp.take((int64_t)pl->mlim[sp].size());  // ints
    in[sp].tab = fps::input_map(L, sp);
    in[sp].place(tmp);
    out[sp].tab = native ? fps::native_map(L, sp) : fps::output_map(L, sp);
    out[sp].place(tmp);
    if (!lift) continue;
    lm[sp].tab = fps::lift_map(L, sp);
    lm[sp].place(tmp);
  }
  const int64_t up = tmp.size;
  const int64_t lam_at = tmp.take(L.npad);
  for (int sp = 0; sp < np; ++sp) {
    // vectors; the eliminations' ratios, then the maps' entries
    const int64_t wide = std::max(mp[sp], pl->mop[sp]);
    v[sp] = tmp.take(2 * mp[sp] * mp[sp]);
    s0[sp] = tmp.take(2 * mp[sp] * wide);
    s1[sp] = tmp.take(2 * mp[sp] * wide);
  }
  const bool sweeps = pl->dim == 2 && pl->prec == FPS_FP64;
  const int64_t steps = sweeps ? (pl->rect ? 2 : 1) * (int64_t)pl->shifts.J : 0;
  const int64_t tab = keep.take(steps * 2 * fps::kNTab * L.mstride);
  const int64_t ctab = keep.take(steps * 2 * fps::kNCTab * L.ncmax);
  const int64_t l1 = keep.take(steps * 2 * L.ncmax * fps::kL1);
  const int64_t nf = pl->dim == 2 ? 2 * L.npad : 0;
  Pieces fin;  // the last upload
  const int64_t mr = fin.take(nf), mc = fin.take(nf), lina = fin.take(lift ? 2 * L.npad : 0);
  for (int sp = 0; sp < 2; ++sp)
    small[sp] = fin.take((int64_t)(pl->mlim[sp].size() + pl->clim[sp].size()));  // ints
  const int64_t fin_at = keep.take(fin.size);
  DeviceBuf work;
  if (hipMalloc(&pl->d_maps.p, (size_t)keep.size * 8) != hipSuccess ||
      hipMalloc(&work.p, (size_t)tmp.size * 8) != hipSuccess)
    return fail(FPS_E_NOMEM, "hipMalloc of a plan table failed");
  double *K = (double *)pl->d_maps.p, *W = (double *)work.p;

  std::vector<double> h((size_t)up, 0.0);
  fps::TridiagEig eig[2] = {};
  fps::MapEntries me[4];
  int cnt = 0;
  for (int sp = 0; sp < np; ++sp) {
    const int64_t m = L.m[sp], mm = mp[sp];
    std::vector<long double> diag((size_t)m), off((size_t)m);
    for (int64_t k = 0; k < m; ++k) {
      diag[(size_t)k] = -fps::atilde_diag_ld(2 * k + sp);
      off[(size_t)k] = k + 1 < m ? fps::atilde_off_ld(2 * k + sp) : 0.0L;
      h[(size_t)(e2[sp] + k)] = (double)(off[(size_t)k] * off[(size_t)k]);
    }
    put_pairs(h, d[sp], diag);
    put_pairs(h, e[sp], off);
    std::copy(pl->mlim[sp].begin(), pl->mlim[sp].end(), (int *)(h.data() + lim[sp]));
    in[sp].put(h);
    out[sp].put(h);
    if (lift) lm[sp].put(h);
    const int64_t sq = mm * mm;
    eig[sp] = fps::TridiagEig{{W + d[sp], m}, {W + e[sp], m}, W + e2[sp], W + lam_at + sp * mp[0],
                              {W + s0[sp], sq}, {W + s1[sp], sq}, {W + v[sp], sq}, mm, (int)m};
    me[cnt++] = in[sp].entries(W, W + s0[sp], mm, mm);
    me[cnt++] = out[sp].entries(W, W + s1[sp], mm, mop[sp]);
  }
  FPS_HIP(hipMemcpy(W, h.data(), h.size() * 8, hipMemcpyHostToDevice));
  // Lemma B.1: sigma(-A~) lies in [1 / (30 n^4), 1]
  FPS_HIP(fps::launch_tridiag_eig(eig, 0.5 / (30.0 * n * n * n * n), 1.01, st));
  // Wi = V^T (S^-1 R); Wo^T = V^T (P S^-1)^T, or V^T S^-1 for the native coefficients
  FPS_HIP(fps::launch_map_entries(me, cnt, st));
  fps::MapProduct mq[4];
  for (int i = 0; i < cnt; ++i) {
    const int sp = i / 2;
    double *w[4] = {K + wi[sp], K + wit[sp], K + wot[sp], K + wo[sp]};
    mq[i] = fps::MapProduct{eig[sp].V, me[i].M, mp[sp], mp[sp], me[i].ld, eig[sp].m,
                            i % 2 ? (const int *)(W + lim[sp]) : nullptr, w[i % 2 * 2], w[i % 2 * 2 + 1]};
    if (i % 2) continue;
    pl->d_Wi[sp].p = K + wi[sp];
    pl->d_WiT[sp].p = K + wit[sp];
    pl->d_Wo[sp].p = K + wo[sp];
    pl->d_WoT[sp].p = K + wot[sp];
  }
  FPS_HIP(fps::launch_map_products(mq, cnt, st));
  if (lift) {  // V^T S^-1 C~(T_k''), m x mop
    for (int sp = 0; sp < np; ++sp) {
      pl->d_lift[sp].p = K + li[sp];
      me[sp] = lm[sp].entries(W, W + s0[sp], mp[sp], pl->mop[sp]);
      mq[sp] = fps::MapProduct{eig[sp].V, me[sp].M, mp[sp], mp[sp], pl->mop[sp], eig[sp].m, nullptr,
                               K + li[sp], nullptr};
    }
    FPS_HIP(fps::launch_map_entries(me, np, st));
    FPS_HIP(fps::launch_map_products(mq, np, st));
  }
  if (sweeps) {
    const SweepTables t(pl);
    pl->d_tab.p = K + tab;
    pl->d_ctab.p = K + ctab;
    pl->d_l1.p = K + l1;
    FPS_HIP(hipMemcpy(K + tab, t.pos.data(), t.pos.size() * 8, hipMemcpyHostToDevice));
    FPS_HIP(hipMemcpy(K + ctab, t.chunk.data(), t.chunk.size() * 8, hipMemcpyHostToDevice));
    FPS_HIP(hipMemcpy(K + l1, t.l1.data(), t.l1.size() * 8, hipMemcpyHostToDevice));
  }
  std::vector<double> lam((size_t)L.npad);
  FPS_HIP(hipMemcpy(lam.data(), W + lam_at, lam.size() * 8, hipMemcpyDeviceToHost));
  pl->lam.assign((size_t)L.npad, -1.0);
  for (int sp = 0; sp < 2; ++sp)
    std::copy_n(lam.begin() + sp * mp[0], L.m[sp], pl->lam.begin() + sp * mp[0]);
  h.assign((size_t)fin.size, 0.0);
  if (nf > 0) factors_2d(pl, h.data() + mr, h.data() + mc);
  if (lift) {
    // V^T of the scaled C~ coefficients of (1 - t)/2 and (1 + t)/2, which are
    // nonzero at degrees 0 and 1 only: the first row of each V
    const BcLiftConst k = bc_lift_const();
    for (int sp = 0; sp < np; ++sp) {
      std::vector<double> v0((size_t)L.m[sp]);
      FPS_HIP(hipMemcpy(v0.data(), eig[sp].V.p, v0.size() * 8, hipMemcpyDeviceToHost));
      for (int64_t i = 0; i < L.m[sp]; ++i) {
        const int64_t r = lina + 2 * (sp * mp[0] + i);
        h[(size_t)r] = k.sinv[sp] * k.am[sp] * v0[(size_t)i];
        h[(size_t)(r + 1)] = k.sinv[sp] * k.ap[sp] * v0[(size_t)i];
      }
    }
  }
  for (int sp = 0; sp < 2; ++sp) {
    int *z = (int *)(h.data() + small[sp]);
    std::copy(pl->mlim[sp].begin(), pl->mlim[sp].end(), z);
    std::copy(pl->clim[sp].begin(), pl->clim[sp].end(), z + pl->mlim[sp].size());
    pl->d_mlim[sp].p = (int *)(K + fin_at + small[sp]);
    pl->d_clim[sp].p = (int *)(K + fin_at + small[sp]) + pl->mlim[sp].size();
  }
  pl->d_mr.p = K + fin_at + mr;
  pl->d_mc.p = K + fin_at + mc;
  if (lift) pl->d_lina.p = K + fin_at + lina;
  FPS_HIP(hipMemcpy(K + fin_at, h.data(), h.size() * 8, hipMemcpyHostToDevice));
  return FPS_OK;
}

}  // namespace detail
}  // namespace fps
