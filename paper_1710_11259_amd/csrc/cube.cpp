// Poisson on the cube [-1,1]^3 (Sec. 5).
//
// In symmetric variables the cube system (5.2) reads
//   (A~ x A~ x I + A~ x I x A~ + I x A~ x A~) Y = -G,  G = (S^-1)^{x3} F_C,
// and with K = -A~^-1 (symmetric positive definite, spectrum in
// [1, 1/delta], Lemma B.1) it becomes (K_x + K_y + K_z) Y = B with
// B = (A~^-1)^{x3} G.  Two iterations solve it (the plan's method):
//   nested (the paper's (5.3)-(5.9) with its innermost level replaced by
//   banded solves): an outer Algorithm 2 for (-H) Y - Y V = -B, H = K_x + K_y,
//   V = K_z, whose (x, y) half-step (H + q) Y = R is, on every z-slice, an
//   inner Algorithm 2 for (K + q/2) Y + Y (K + q/2) = R from Y = 0;
//   z-eigenbasis (FPS_PLAN_CUBE_ZEIG): A~ diagonalized along z, and on every
//   z-slice (eigenvalue mu, P = A~ + mu) an Algorithm 2 for
//   (-mu^2 P^-1) Z - Z (-P) = -G^, Z = P Y; refined plans run rounds of the
//   K-form (|mu| K + 1/2) dY + dY (|mu| K + 1/2) = K q K instead.
// Every operator in them is a function of A~ along one axis, so the iterate
// they reach is diagonal in the tensor eigenbasis of A~: mode (z, y, x) of Y is
// that of G times -(1 - eps) / (lz ly + lz lx + ly lx), eps the iteration's
// error factor in that mode.  The plan tabulates this multiplier
// (spectral.hip), and a solve is one dense product per axis on the way in, the
// multiplier in the epilogue of the last, and one per axis on the way out.
// The iterations themselves took 1.4 of 2.2 ms (z-eigenbasis, n = 256, every
// slice's steps in LDS) and 105 of 107 ms (nested).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "solver.hpp"

namespace fps {
namespace detail {

namespace {

// Sizes [z][y][x] of one stage of the coefficient maps and the offset of
// the parity-1 block on every axis.
struct Dims {
  int64_t d[3];
  int64_t b0[3];
};

// GEMM problems of out = M along axis `mode` (0: z, 1: y, 2: x) of `in`,
// one per parity s (and per z-slice for mode 1).  MA[s] is M_s row-major
// (N[s] rows, row stride lda[s]); MB[s] is M_s^T row-major (K[s] rows, row
// stride ldb[s]).
void mode_probs(const double *in, const Dims &di, double *out, const Dims &dout, int mode,
                const double *const MA[2], const int64_t lda[2], const double *const MB[2],
                const int64_t ldb[2], const int64_t N[2], const int64_t K[2],
                std::vector<fps::GemmProb> &probs) {
  for (int s = 0; s < 2; ++s) {
    if (N[s] == 0 || K[s] == 0) continue;
    if (mode == 2) {
      probs.push_back(fps::GemmProb{in + s * di.b0[2], MB[s], out + s * dout.b0[2],
                                    di.d[0] * di.d[1], N[s], K[s], di.d[2], 1, ldb[s], 1,
                                    dout.d[2], 1});
    } else if (mode == 0) {
      const int64_t pin = di.d[1] * di.d[2], pout = dout.d[1] * dout.d[2];
      probs.push_back(fps::GemmProb{MA[s], in + s * di.b0[0] * pin, out + s * dout.b0[0] * pout,
                                    N[s], pin, K[s], lda[s], 1, pin, 1, pout, 1});
    } else {
      for (int64_t z = 0; z < di.d[0]; ++z)
        probs.push_back(fps::GemmProb{
            MA[s], in + z * di.d[1] * di.d[2] + s * di.b0[1] * di.d[2],
            out + z * dout.d[1] * dout.d[2] + s * dout.b0[1] * dout.d[2], N[s], di.d[2], K[s],
            lda[s], 1, di.d[2], 1, dout.d[2], 1});
    }
  }
}

fps_status launch_probs(fps_plan *pl, const std::vector<fps::GemmProb> &probs, hipStream_t st) {
  for (size_t i = 0; i < probs.size(); i += 4) {
    const fps_status s = run_products(pl, probs.data() + i,
                                      (int)std::min<size_t>(4, probs.size() - i), st);
    if (s != FPS_OK) return s;
  }
  return FPS_OK;
}

// One table launch, timed like run_products.
fps_status run_table(fps_plan *pl, const fps::GemmTable &g, const DeviceBuf &d, const DeviceBuf &map,
                     char *w, char *out, hipStream_t st) {
  hipEvent_t e0 = next_event(pl, 0), e1 = next_event(pl, 1);
  FPS_HIP(fps::launch_gemm_table(g, (const fps::GemmDesc *)d.p, (const int *)map.p, nullptr, w, out, st,
                                 e0, e1));
  if (e0) ++pl->ev_used;
  return FPS_OK;
}

// Device GEMM table of per-slice problems (A absolute, B workspace-relative, C
// of base id `cbase`).
fps_status upload_table(const std::vector<fps::GemmProb> &probs, int cbase, DeviceBuf &d,
                        DeviceBuf &map, fps::GemmTable &t) {
  std::vector<fps::GemmDesc> tab;
  for (const fps::GemmProb &q : probs) tab.push_back(fps::GemmDesc{q, 0, 1, cbase});
  std::vector<int> m;
  if (!fps::gemm_table(tab, t, m)) return fail(FPS_E_STATE, "internal: cube GEMM operand layout");
  fps_status s;
  if ((s = upload(d, tab)) != FPS_OK || (s = upload(map, m)) != FPS_OK) return s;
  return FPS_OK;
}

// Enclosure [ea, eb] of sigma(A~): Lemma B.1, or the computed one.
void enclosure(const fps_plan *pl, double *ea, double *eb) {
  const double n = (double)pl->n;
  *ea = -1.0;
  *eb = -1.0 / (30.0 * n * n * n * n);
  if (pl->flags & FPS_PLAN_TIGHT_SPECTRUM) spectrum_tight(pl->n, ea, eb);
}

// Shifts of the nested method: outer, and one inner set per outer step.
fps_status nested_shifts(fps_plan *pl, double ea, double eb) {
  const double klo = -1.0 / ea, khi = -1.0 / eb;  // sigma(K)
  std::string err;
  if (!fps::zolotarev_shifts(-2.0 * khi, -2.0 * klo, klo, khi, pl->tol, pl->shifts, err))
    return fail(FPS_E_ARG, err);
  // The outer iteration needs its (x, y) half-steps solved well below its
  // own tolerance.
  const double inner_tol = pl->tol * 0.1;
  const int J1 = pl->shifts.J;
  pl->inner_J.assign(J1, 0);
  pl->inner_off.assign(J1, 0);
  pl->inner_p.clear();
  for (int i = 0; i < J1; ++i) {
    const double c = 0.5 * pl->shifts.q[i];
    fps::ShiftSet in;
    if (!fps::zolotarev_shifts(-(khi + c), -(klo + c), klo + c, khi + c, inner_tol, in, err))
      return fail(FPS_E_ARG, err);
    pl->inner_J[i] = in.J;
    pl->inner_off[i] = (int)pl->inner_p.size();
    pl->inner_p.insert(pl->inner_p.end(), in.p.begin(), in.p.end());
  }
  return FPS_OK;
}

// Shifts of the z-eigenbasis method, per storage slice c in zoff[c] ..
// zoff[c + 1] - 1 of zp / zq (rounds one after another), and the slice counts.
//
// FP64: sigma(-mu^2 P^-1) lies in [mu^2 / (|ea| + |mu|), mu^2 / (|eb| + |mu|)],
// sigma(-P) in [|eb| + |mu|, |ea| + |mu|].  Refined rounds: sigma(|mu| K + 1/2)
// lies in [|mu| / |ea| + 1/2, |mu| / |eb| + 1/2], symmetric shifts.
fps_status zeig_shifts(fps_plan *pl, double ea, double eb) {
  const fps::Layout &L = pl->L;
  const bool refined = pl->prec == FPS_FP32_REFINED;
  std::vector<double> rtol{pl->tol};
  if (refined) {
    rtol.clear();
    for (const RefineRound &r : refine_schedule(pl->tol, false)) rtol.push_back(r.tol);
    pl->rtol = rtol;
    pl->rounds = (int)rtol.size();
    pl->zrJmax.assign(rtol.size(), 0);
  }
  struct Slice {
    double mu;
    int J;
    fps::ShiftSet sh;
  };
  std::vector<Slice> sl;
  std::string err;
  pl->zoff.assign((size_t)pl->cnp + 1, 0);
  pl->zp.clear();
  pl->zq.clear();
  for (int64_t c = 0; c < pl->cnp; ++c) {
    pl->zoff[(size_t)c] = (int)pl->zp.size();
    const int sp = c < pl->cmp[0] ? 0 : 1;
    const int64_t k = c - sp * pl->cmp[0];
    if (k == 0) fps::atilde_eigenvalues(pl->n, sp, pl->zlam[sp]);
    if (k >= L.m[sp]) continue;
    Slice x;
    x.mu = pl->zlam[sp][(size_t)k];
    const double am = std::fabs(x.mu), ra = std::fabs(ea), rb = std::fabs(eb);
    for (size_t r = 0; r < rtol.size(); ++r) {
      fps::ShiftSet sh;
      const double a = am / ra + 0.5, b = am / rb + 0.5;
      const bool ok = refined ? fps::zolotarev_shifts(-b, -a, a, b, rtol[r], sh, err)
                              : fps::zolotarev_shifts(am * am / (ra + am), am * am / (rb + am),
                                                      rb + am, ra + am, rtol[r], sh, err);
      if (!ok) return fail(FPS_E_ARG, err);
      if (refined) {
        std::reverse(sh.p.begin(), sh.p.end());  // increasing |p|
        std::reverse(sh.q.begin(), sh.q.end());
        pl->zrJmax[r] = std::max(pl->zrJmax[r], sh.J);
      }
      pl->zp.insert(pl->zp.end(), sh.p.begin(), sh.p.end());
      pl->zq.insert(pl->zq.end(), sh.q.begin(), sh.q.end());
      if (r == 0) {
        x.J = sh.J;
        x.sh = sh;
      }
    }
    sl.push_back(x);
  }
  pl->zoff[(size_t)pl->cnp] = (int)pl->zp.size();
  pl->n_f32 = 0;
  for (int J : pl->zrJmax) pl->n_f32 += J;
  // the queries report the slices by decreasing steps (of equal ones the lowest mode
  // first), and the longest slice's shifts as the plan's
  std::reverse(sl.begin(), sl.begin() + L.m[0]);
  std::reverse(sl.begin() + L.m[0], sl.end());
  std::stable_sort(sl.begin(), sl.end(), [&](const Slice &u, const Slice &v) {
    return refined ? std::fabs(u.mu) > std::fabs(v.mu) : u.J > v.J;
  });
  pl->zJ.clear();
  for (const Slice &x : sl) pl->zJ.push_back(x.J);
  pl->shifts = sl[0].sh;
  return FPS_OK;
}

// Tables of the chains that replace the per-axis products of a cube with blocks of
// at most 128 entries (n <= 256), three launches: every z-slice of F to its x and
// y maps in G, every strip of columns of G along z through the input map, the
// multiplier and the output map to O0, every z-slice of O0 to its x and y
// output maps in U.
constexpr int kChainMode[3] = {0, 2, 3};
fps_status upload_chains(fps_plan *pl) {
  const fps::Layout &L = pl->L;
  const bool native = pl->out_basis == FPS_OUT_NATIVE;
  const int64_t n = L.n, N = out_extent(pl), npad = pl->cnp, *mp = pl->cmp, plane = npad * npad;
  const int64_t *mo = native ? L.m : L.mo, *mop = native ? L.mp : pl->mop;
  const int nb = pl->cnb;
  auto at = [](int64_t off, int64_t elem) { return (double *)(intptr_t)(off + 8 * elem); };
  auto map = [&](fps::ChainDesc &e, int i, bool out, int s) {
    e.m[i] = (const double *)(out ? pl->d_WoT[s].p : pl->d_WiT[s].p);
    e.ld[i] = (int)(out ? mop[s] : L.mp[s]);
    e.k[i] = (int)((mp[s] + 31) / 32 * 32);
    e.n[i] = (int)(out ? mo[s] : mp[s]);
  };
  std::vector<fps::ChainDesc> d[3];
  // slices, in and out: natural position zn is row zn / 2 of parity zn % 2.  The
  // units of one slice and row parity read the same rows.
  int group[2] = {1, 1};
  for (int io = 0; io < 2; ++io)
    for (int64_t zn = 0; zn < (io ? N : n); ++zn) {
      const int sz = zn & 1;
      if (L.m[sz] == 0) continue;
      for (int sy = 0; sy < 2; ++sy) {
        const size_t first = d[2 * io].size();
        for (int sx = 0; sx < 2; ++sx) {
          if (L.m[sy] == 0 || L.m[sx] == 0) continue;
          fps::ChainDesc e{};
          map(e, 0, io, sx);
          map(e, 1, io, sy);
          e.in_r = (int)L.m[sy];
          e.in_c = (int)L.m[sx];
          const int64_t slice = sz * (io ? pl->mqc[0] : mp[0]) + zn / 2;
          const int64_t blk = (slice * npad + sy * mp[0]) * npad + sx * mp[0];
          if (io) {
            e.in = at(pl->off_O0, blk);
            e.ibase = 1;
            e.in_rs = npad;
            e.in_cs = 1;
            e.out = at(0, (zn * N + sy) * N + sx);
            e.obase = 3;
            e.out_rs = 2 * N;
            e.out_cs = 2;
            e.out_r = (int)mo[sy];
            e.out_c = (int)mo[sx];
          } else {
            e.in = at(0, (zn * n + sy) * n + sx);
            e.ibase = 2;
            e.in_rs = 2 * n;
            e.in_cs = 2;
            e.out = at(pl->off_G, blk);
            e.obase = 1;
            e.out_rs = npad;
            e.out_cs = 1;
            e.out_r = (int)mp[sy];
            e.out_c = (int)mp[sx];
          }
          for (e.r0 = 0; e.r0 < std::min(e.n[1], 32 * nb); e.r0 += fps::chain_part(nb))
            d[2 * io].push_back(e);
        }
        group[io] = std::max(group[io], (int)(d[2 * io].size() - first));
      }
    }
  // strips along z
  const int64_t S = fps::chain_part(nb);
  for (int sz = 0; sz < 2; ++sz)
    for (int64_t c = 0; c < plane && L.m[sz] > 0; c += S) {
      fps::ChainDesc e{};
      map(e, 1, false, sz);
      map(e, 3, true, sz);
      e.in = at(pl->off_G, sz * mp[0] * plane + c);
      e.out = at(pl->off_O0, sz * pl->mqc[0] * plane + c);
      e.ibase = e.obase = 1;
      e.in_rs = e.out_rs = e.mt_rs = plane;
      e.in_cs = e.out_cs = 1;
      e.in_r = (int)L.m[sz];
      e.out_r = (int)mo[sz];
      e.in_c = e.out_c = (int)std::min(S, plane - c);
      e.mt = (const double *)pl->d_mt.p + sz * mp[0] * plane + c;
      d[1].push_back(e);
    }
  for (int t = 0; t < 3; ++t) {
    for (const fps::ChainDesc &e : d[t])
      if (!fps::chain_ok(e, nb, kChainMode[t])) return fail(FPS_E_STATE, "internal: cube chain");
    if (t != 1) fps::chain_order(d[t], group[t / 2]);
    const fps_status s = upload(pl->d_cchain[t], d[t]);
    if (s != FPS_OK) return s;
    pl->cchain_count[t] = (int)d[t].size();
  }
  return FPS_OK;
}

}  // namespace

fps_status cube_plan_build(fps_plan *pl) {
  const int64_t n = pl->n;
  pl->zeig = (pl->flags & FPS_PLAN_CUBE_ZEIG) != 0;
  pl->L = fps::make_layout(n);
  const fps::Layout &L = pl->L;
  for (int sp = 0; sp < 2; ++sp) pl->cmp[sp] = k_round(L.m[sp]);
  pl->cnp = pl->cmp[0] + pl->cmp[1];
  double ea, eb;
  enclosure(pl, &ea, &eb);
  const fps_status s = pl->zeig ? zeig_shifts(pl, ea, eb) : nested_shifts(pl, ea, eb);
  if (s != FPS_OK) return s;
  const bool native = pl->out_basis == FPS_OUT_NATIVE;
  for (int sp = 0; sp < 2; ++sp) {
    pl->mop[sp] = (L.mo[sp] + fps::kPad - 1) / fps::kPad * fps::kPad;
    pl->mqc[sp] = ((native ? L.m[sp] : L.mo[sp]) + 1) / 2 * 2;
  }
  // Workspace: six arrays of (up to) npad^3 (input stages in G / O0 / O1, Y^ in ZR,
  // output stages in O0..O1 and RX..RX + 1), then room for the chunk carries of npad^2
  // chains, which nothing uses: the size is what callers have allocated.
  const int64_t vol = align256(L.npad * L.npad * L.npad * 8);
  const int64_t ch = L.npad * L.npad;
  pl->off_G = 0;
  pl->off_ZR = vol;
  pl->off_RX = 2 * vol;
  pl->off_O0 = 4 * vol;
  pl->off_O1 = 5 * vol;
  pl->ws_bytes = 6 * vol + align256(L.ncmax * 4 * ch * 8) +
                 (pl->zeig && L.ncmax <= 2 ? align256(L.ncmax * 4 * ch * 8) : 0) +
                 align256(2 * L.ncmax * ch * 2 * 8);
  // output stages: [mq][npad][npad] in O0..O1, [mq][npad][mq] in RX..
  const int64_t mq = pl->mqc[0] + pl->mqc[1];
  if (L.npad * L.npad * mq * 8 > 2 * vol || L.npad * mq * mq * 8 > 2 * vol)
    return fail(FPS_E_STATE, "internal: cube output temporaries exceed the workspace");
  return FPS_OK;
}

fps_status cube_plan_upload(fps_plan *pl) {
  const fps::Layout &L = pl->L;
  const int64_t npad = pl->cnp, *mp = pl->cmp;
  fps_status s;
  if ((s = spectral_build(pl, false)) != FPS_OK) return s;
  // the multiplier of every mode
  hipStream_t st = nullptr;
  DeviceBuf lam, ey, ex, p, q, off, mu;
  if (hipMalloc(&pl->d_mt.p, (size_t)(npad * npad * npad) * 8) != hipSuccess)
    return fail(FPS_E_NOMEM, "hipMalloc of a plan table failed");
  std::vector<double> lc((size_t)npad, -1.0);  // eigenvalues by cube position
  for (int sp = 0; sp < 2; ++sp)
    std::copy_n(pl->lam.begin() + sp * L.mp[0], L.m[sp], lc.begin() + sp * mp[0]);
  if ((s = upload(lam, lc)) != FPS_OK) return s;
  const double *dl = (const double *)lam.p;
  if (pl->zeig) {
    std::vector<double> t((size_t)(npad * npad), 0.0), m((size_t)npad, -1.0);
    for (int sp = 0; sp < 2; ++sp)
      for (int64_t k = 0; k < L.m[sp]; ++k) m[(size_t)(sp * mp[0] + k)] = pl->zlam[sp][(size_t)k];
    if ((s = upload(ey, t)) != FPS_OK || (s = upload(ex, t)) != FPS_OK ||
        (s = upload(p, pl->zp)) != FPS_OK || (s = upload(q, pl->zq)) != FPS_OK ||
        (s = upload(off, pl->zoff)) != FPS_OK || (s = upload(mu, m)) != FPS_OK)
      return s;
    FPS_HIP(fps::launch_slice_factors(dl, (const double *)mu.p, (const int *)off.p,
                                      (const double *)p.p, (const double *)q.p,
                                      pl->prec == FPS_FP32_REFINED, (double *)ey.p, (double *)ex.p,
                                      npad, st));
    FPS_HIP(fps::launch_slice_multiplier(dl, (const double *)ey.p, (const double *)ex.p,
                                         (double *)pl->d_mt.p, npad, st));
  } else {
    const int J1 = pl->shifts.J;
    std::vector<int> io(pl->inner_off);
    io.push_back((int)pl->inner_p.size());
    std::vector<double> t((size_t)(J1 * npad), 0.0);
    if ((s = upload(ey, t)) != FPS_OK || (s = upload(p, pl->shifts.p)) != FPS_OK ||
        (s = upload(q, pl->shifts.q)) != FPS_OK || (s = upload(off, io)) != FPS_OK ||
        (s = upload(ex, pl->inner_p)) != FPS_OK)
      return s;
    FPS_HIP(fps::launch_nested_factors(dl, (const double *)q.p, (const int *)off.p,
                                       (const double *)ex.p, (double *)ey.p, J1, npad, st));
    FPS_HIP(fps::launch_nested_multiplier(dl, (const double *)p.p, (const double *)q.p,
                                          (const double *)ey.p, J1, (double *)pl->d_mt.p, npad, st));
  }
  FPS_HIP(hipStreamSynchronize(st));
  pl->cnb = fps::chain_size(mp[0]);
  if (pl->cnb > 0) return upload_chains(pl);
  // per-slice products: y on the way in, y (the last, into U) on the way out
  const Dims full{{npad, npad, npad}, {mp[0], mp[0], mp[0]}};
  const double *Wi[2] = {(const double *)pl->d_Wi[0].p, (const double *)pl->d_Wi[1].p};
  const int64_t ld[2] = {L.mp[0], L.mp[1]};
  std::vector<fps::GemmProb> probs;
  mode_probs((const double *)(intptr_t)pl->off_O1, full, (double *)(intptr_t)pl->off_O0, full, 1, Wi,
             ld, nullptr, ld, mp, mp, probs);
  if ((s = upload_table(probs, 1, pl->d_gy_in, pl->d_gy_map_in, pl->t_gy[0])) != FPS_OK)
    return s;
  const bool native = pl->out_basis == FPS_OUT_NATIVE;
  const int64_t *mo = native ? L.m : L.mo;
  const int64_t N = out_extent(pl), mq = pl->mqc[0] + pl->mqc[1];
  probs.clear();
  for (int sz = 0; sz < 2; ++sz)
    for (int64_t z = 0; z < mo[sz]; ++z)
      for (int sy = 0; sy < 2; ++sy)
        for (int sx = 0; sx < 2; ++sx) {
          if (L.m[sz] == 0 || L.m[sy] == 0 || L.m[sx] == 0) continue;
          const int64_t zs = sz * pl->mqc[0] + z, zn = 2 * z + sz;
          const int64_t in = (zs * npad + sy * mp[0]) * mq + sx * pl->mqc[0];
          const int64_t out = (zn * N + sy) * N + sx;
          probs.push_back(fps::GemmProb{(const double *)pl->d_Wo[sy].p,
                                        (const double *)(intptr_t)(pl->off_RX + 8 * in),
                                        (double *)(intptr_t)(8 * out), mo[sy], mo[sx], mp[sy],
                                        L.mp[sy], 1, mq, 1, 2 * N, 2});
        }
  return upload_table(probs, 2, pl->d_gy_out, pl->d_gy_map_out, pl->t_gy[1]);
}

fps_status cube_solve(fps_plan *pl, const double *F, double *U, char *w, hipStream_t st) {
  const fps::Layout &L = pl->L;
  const int64_t npad = pl->cnp, mp0 = pl->cmp[0], *K = pl->cmp;
  double *G = (double *)(w + pl->off_G), *Y = (double *)(w + pl->off_ZR);
  double *RX = (double *)(w + pl->off_RX);
  double *O0 = (double *)(w + pl->off_O0), *O1 = (double *)(w + pl->off_O1);
  const bool native = pl->out_basis == FPS_OUT_NATIVE;
  const int64_t *mo = native ? L.m : L.mo, *mop = native ? L.mp : pl->mop;
  const double *Wi[2], *WiT[2], *Wo[2], *WoT[2];
  for (int s = 0; s < 2; ++s) {
    Wi[s] = (const double *)pl->d_Wi[s].p;
    WiT[s] = (const double *)pl->d_WiT[s].p;
    Wo[s] = (const double *)pl->d_Wo[s].p;
    WoT[s] = (const double *)pl->d_WoT[s].p;
  }
  const int64_t ldi[2] = {L.mp[0], L.mp[1]};
  const int64_t No[2] = {L.m[0] > 0 ? mo[0] : 0, L.m[1] > 0 ? mo[1] : 0};
  const int64_t ldo[2] = {mop[0], mop[1]};
  const Dims full{{npad, npad, npad}, {mp0, mp0, mp0}};
  fps_status s;
  if (pl->cnb > 0) {
    const int64_t N = out_extent(pl);
    for (int t = 0; t < 3; ++t) {
      // no odd modes (n = 1): parts of U that no chain writes (F is read by now)
      if (t == 1 && L.m[1] == 0) FPS_HIP(fps::launch_fill(U, N * N * N, 0.0, st));
      hipEvent_t e0 = next_event(pl, 0), e1 = next_event(pl, 1);
      FPS_HIP(fps::launch_chain_table((const fps::ChainDesc *)pl->d_cchain[t].p, pl->cchain_count[t],
                                      pl->cnb, kChainMode[t], F, w, U, st, e0, e1));
      if (e0) ++pl->ev_used;
    }
    return FPS_OK;
  }
  // in: x, y, z (the multiplier in the last product's epilogue)
  FPS_HIP(fps::launch_permute3_in(F, G, L.n, npad, mp0, st));
  std::vector<fps::GemmProb> px, pz, qz, qx;
  mode_probs(G, full, O1, full, 2, Wi, ldi, WiT, ldi, K, K, px);
  if ((s = launch_probs(pl, px, st)) != FPS_OK) return s;
  if ((s = run_table(pl, pl->t_gy[0], pl->d_gy_in, pl->d_gy_map_in, w, nullptr, st)) != FPS_OK)
    return s;
  mode_probs(O0, full, Y, full, 0, Wi, ldi, WiT, ldi, K, K, pz);
  for (fps::GemmProb &g : pz) g.mt = (const double *)pl->d_mt.p + (g.C - Y);
  if ((s = launch_probs(pl, pz, st)) != FPS_OK) return s;
  // out: z, x, y
  const int64_t mq = pl->mqc[0] + pl->mqc[1], mb0 = pl->mqc[0];
  const Dims d1{{mq, npad, npad}, {mb0, mp0, mp0}};
  const Dims d2{{mq, npad, mq}, {mb0, mp0, mb0}};
  mode_probs(Y, full, O0, d1, 0, Wo, ldi, WoT, ldo, No, K, qz);
  if ((s = launch_probs(pl, qz, st)) != FPS_OK) return s;
  mode_probs(O0, d1, RX, d2, 2, Wo, ldi, WoT, ldo, No, K, qx);
  if ((s = launch_probs(pl, qx, st)) != FPS_OK) return s;
  return run_table(pl, pl->t_gy[1], pl->d_gy_out, pl->d_gy_map_out, w, (char *)U, st);
}

// The plan's default-priority side stream and its fork / join events
// (2-D plans, whose fps_adi_native splits the ADI by row parity).
fps_status create_side_stream(fps_plan *pl) {
  if (pl->zside != nullptr) return FPS_OK;
  if (hipStreamCreateWithFlags(&pl->zside, hipStreamNonBlocking) != hipSuccess ||
      hipEventCreateWithFlags(&pl->zfork, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&pl->zjoin, hipEventDisableTiming) != hipSuccess) {
    if (pl->zside) (void)hipStreamDestroy(pl->zside);
    if (pl->zfork) (void)hipEventDestroy(pl->zfork);
    if (pl->zjoin) (void)hipEventDestroy(pl->zjoin);
    pl->zside = nullptr;
    pl->zfork = pl->zjoin = nullptr;
    return fail(FPS_E_HIP, "creating the side stream failed");
  }
  return FPS_OK;
}

}  // namespace detail
}  // namespace fps
