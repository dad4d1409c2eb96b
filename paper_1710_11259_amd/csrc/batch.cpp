// Batched square solves (fps_batch_* in include/fps.h): many independent
// problems, possibly of different sizes, each stage of the eigenbasis solve
// (spectral.cpp) as one launch for all of them.  Every problem keeps the maps,
// workspace layout and kernels of its own single-problem plan.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <new>
#include <vector>

#include "solver.hpp"

using namespace fps::detail;

namespace {

constexpr uint64_t kBatchMagic = 0x66707362'61746331ull;  // "fpsbatc1"

}  // namespace

struct fps_batch {
  uint64_t magic = kBatchMagic;
  int count = 0, prec = FPS_FP64, out_basis = FPS_OUT_CHEB;
  bool on_device = false;
  std::vector<int64_t> n;            // per problem, caller's order
  std::vector<fps_plan *> sub;       // one plan per distinct n (owned)
  std::vector<int> which;            // problem -> index into sub
  std::vector<int64_t> f_off, u_off, ws_off;  // per problem: F / U entries, workspace bytes
  int64_t in_entries = 0, out_entries = 0, ws_bytes = 0;
  int J_max = 0;                     // steps of the longest ADI (over all rounds)
  bool has_n1 = false;               // a problem of size 1 (parts of its U no product writes)
  // products of all problems: input map g1, g2; output map g1, g2; (FP64
  // batches) the adjoint's input map g1, g2 and output map g1, g2
  DeviceBuf d_gd[8], d_gmap[8];
  fps::GemmTable gt[8];
  // the problems small enough for chains (forward 0, adjoint 1): one
  // launch each; the products hold the others
  DeviceBuf d_chain[2];
  int nchain[2] = {0, 0}, chain_nb[2] = {3, 3};
  ~fps_batch() {
    for (fps_plan *p : sub) fps_plan_destroy(p);
  }
  const fps_plan *plan_of(int problem) const { return sub[which[problem]]; }
};

namespace {

bool valid_batch(const fps_batch *b) { return b != nullptr && b->magic == kBatchMagic; }

fps_status run_chains(const fps_batch *bt, int t, const double *in, double *out, hipStream_t st) {
  FPS_HIP(fps::launch_chain_table((const fps::ChainDesc *)bt->d_chain[t].p, bt->nchain[t],
                                  bt->chain_nb[t], 1, in, nullptr, out, st));
  return FPS_OK;
}

// GEMM tables of the coefficient maps: the single-problem builders run on
// synthetic base pointers (the problem's workspace offset, its U offset in
// bytes), so every workspace or output operand comes out as an offset.
fps_status build_gemm_tables(fps_batch *bt) {
  std::vector<fps::GemmDesc> tab[8];
  std::vector<fps::ChainDesc> chain[2];
  const bool refined = bt->prec == FPS_FP32_REFINED;
  for (int b = 0; b < bt->count; ++b) {
    const fps_plan *pl = bt->plan_of(b);
    char *wsyn = (char *)(intptr_t)bt->ws_off[b];
    fps::GemmProb g[8][4];
    double *Usyn = (double *)(intptr_t)(bt->u_off[b] * (int64_t)sizeof(double));
    double *Fsyn = (double *)(intptr_t)(bt->f_off[b] * (int64_t)sizeof(double));
    fps::ChainDesc cd[4];
    for (int t = 0; t < (refined ? 1 : 2); ++t) {
      int nb = 0;
      const int c = t ? adjoint_chain(pl, Usyn, Fsyn, cd, &nb)
                      : solve_chain(pl, Fsyn, Usyn, nullptr, nullptr, cd, &nb);
      for (int i = 0; i < c; ++i) {
        cd[i].ibase = 2;
        cd[i].obase = 3;
        chain[t].push_back(cd[i]);
      }
      if (c > 0) bt->chain_nb[t] = std::max(bt->chain_nb[t], nb);
    }
    int counts[8] = {};
    if (!forward_chained(pl)) {
      counts[1] = rhs_gemms(pl, Fsyn, wsyn, g[0], &counts[0], g[1]);
      counts[2] = counts[3] = out_gemms(pl, Usyn, wsyn, g[2], g[3]);
    }
    if (!refined && !adjoint_chained(pl)) {
      counts[5] = adj_in_gemms(pl, Usyn, wsyn, g[4], &counts[4], g[5]);
      counts[6] = counts[7] = adj_out_gemms(pl, Fsyn, wsyn, g[6], g[7]);
    }
    // base ids (A, B, C): absolute 0, relative to ws 1, to the output 2, to the input 3
    static const int ids[8][3] = {{0, 3, 1}, {1, 0, 1}, {1, 0, 1}, {0, 1, 2},
                                  {0, 3, 1}, {1, 0, 1}, {1, 0, 1}, {0, 1, 2}};
    for (int t = 0; t < 8; ++t)
      for (int i = 0; i < counts[t]; ++i)
        tab[t].push_back(fps::GemmDesc{g[t][i], ids[t][0], ids[t][1], ids[t][2]});
  }
  for (int t = 0; t < 2; ++t) {
    for (const fps::ChainDesc &e : chain[t])
      if (!fps::chain_ok(e, bt->chain_nb[t], 1)) return fail(FPS_E_STATE, "internal: batched chain");
    const fps_status s = upload(bt->d_chain[t], chain[t]);
    if (s != FPS_OK) return s;
    bt->nchain[t] = (int)chain[t].size();
  }
  for (int t = 0; t < 8; ++t) {
    if (tab[t].empty()) continue;
    std::vector<int> map;
    if (!fps::gemm_table(tab[t], bt->gt[t], map))
      return fail(FPS_E_STATE, "internal: batched GEMM operand layout");
    fps_status s;
    if ((s = upload(bt->d_gd[t], tab[t])) != FPS_OK || (s = upload(bt->d_gmap[t], map)) != FPS_OK)
      return s;
  }
  return FPS_OK;
}

// All stages (t 0: of the solve, 1: of the adjoint) in place of the tables where `in`
// and `out` overlap: every problem's input is consumed before any output is
// written, one launch per problem and stage.
fps_status run_overlapping(const fps_batch *bt, int t, const double *in, double *out, char *w,
                           hipStream_t st) {
  for (int stage = 0; stage < 4; ++stage)
    for (int b = 0; b < bt->count; ++b) {
      const fps_plan *pl = bt->plan_of(b);
      char *wb = w + bt->ws_off[b];
      const double *x = in + (t ? bt->u_off[b] : bt->f_off[b]);
      double *y = out + (t ? bt->f_off[b] : bt->u_off[b]);
      fps::GemmProb g[4][4];
      int cnt[4] = {};
      if (pl->n == 1) {  // its one block: the input kept in the workspace until the end
        const int64_t n = t ? out_extent(pl) : 1;
        double *keep = (double *)(wb + pl->off_GT);
        if (stage == 0) FPS_HIP(fps::launch_copy(x, keep, n * n, st));
        if (stage < 3) continue;
        fps::ChainDesc d[4];
        int nb = 0;
        const int c = t ? adjoint_chain(pl, keep, y, d, &nb)
                        : solve_chain(pl, keep, y, nullptr, nullptr, d, &nb);
        FPS_HIP(fps::launch_chain(d, c, nb, st));
        const fps_status s = t ? FPS_OK : clear_n1(pl, y, st);
        if (s != FPS_OK) return s;
        continue;
      }
      if (t == 0) {
        cnt[1] = rhs_gemms(pl, x, wb, g[0], &cnt[0], g[1]);
        cnt[2] = cnt[3] = out_gemms(pl, y, wb, g[2], g[3]);
      } else {
        cnt[1] = adj_in_gemms(pl, x, wb, g[0], &cnt[0], g[1]);
        cnt[2] = cnt[3] = adj_out_gemms(pl, y, wb, g[2], g[3]);
      }
      FPS_HIP(fps::launch_gemm(g[stage], cnt[stage], st));
    }
  return FPS_OK;
}

// Enqueues the solve's (t 0) or the adjoint's (1) launches.
fps_status run_batch(const fps_batch *bt, int t, const double *in, double *out, char *w,
                     hipStream_t st) {
  const int64_t n_in = t ? bt->out_entries : bt->in_entries;
  const int64_t n_out = t ? bt->in_entries : bt->out_entries;
  if (!chain_in_out(in, n_in, out, n_out)) return run_overlapping(bt, t, in, out, w, st);
  if (t == 0 && bt->has_n1 && n_in != n_out) FPS_HIP(fps::launch_fill(out, n_out, 0.0, st));
  const fps_status s = run_chains(bt, t, in, out, st);
  if (s != FPS_OK) return s;
  for (int i = 4 * t; i < 4 * t + 4; ++i)
    FPS_HIP(fps::launch_gemm_table(bt->gt[i], (const fps::GemmDesc *)bt->d_gd[i].p,
                                   (const int *)bt->d_gmap[i].p, in, w, (char *)out, st));
  return FPS_OK;
}

}  // namespace

extern "C" {

fps_status fps_batch_create(fps_batch **out, int dim, int count, const int64_t *n, double tol,
                            int prec, int out_basis, unsigned flags) {
  if (!out) return fail(FPS_E_ARG, "out must not be null");
  *out = nullptr;
  if (dim == 3) return fail(FPS_E_UNSUPPORTED, "batched solves are square only");
  if (dim != 2) return fail(FPS_E_ARG, "dim must be 2 or 3");
  if (count < 1 || count > 65536) return fail(FPS_E_ARG, "count must lie in [1, 65536]");
  if (!n) return fail(FPS_E_ARG, "n must not be null");
  for (int b = 0; b < count; ++b)
    if (n[b] < 1 || n[b] > 16384) return fail(FPS_E_ARG, "every n must lie in [1, 16384]");
  fps_batch *bt = new (std::nothrow) fps_batch();
  if (!bt) return fail(FPS_E_NOMEM, "batch allocation failed");
  bt->count = count;
  bt->prec = prec;
  bt->out_basis = out_basis;
  bt->n.assign(n, n + count);
  std::map<int64_t, int> idx;
  bt->which.resize(count);
  for (int b = 0; b < count; ++b) {
    auto it = idx.find(n[b]);
    if (it == idx.end()) {
      fps_plan *pl = nullptr;
      fps_status s = fps_plan_create(&pl, 2, n[b], FPS_BC_DIRICHLET_ZERO, tol, prec, out_basis, flags);
      if (s != FPS_OK) {
        delete bt;
        return s;
      }
      it = idx.emplace(n[b], (int)bt->sub.size()).first;
      bt->sub.push_back(pl);
    }
    bt->which[b] = it->second;
  }
  bt->f_off.resize(count);
  bt->u_off.resize(count);
  bt->ws_off.resize(count);
  for (int b = 0; b < count; ++b) {
    const fps_plan *pl = bt->plan_of(b);
    bt->f_off[b] = bt->in_entries;
    bt->u_off[b] = bt->out_entries;
    bt->ws_off[b] = bt->ws_bytes;
    const int64_t e = out_basis == FPS_OUT_NATIVE ? n[b] : n[b] + 2;
    bt->in_entries += n[b] * n[b];
    bt->out_entries += e * e;
    bt->ws_bytes += align256(pl->ws_bytes);
  }
  // the limit on a batch: 64 x 64 tiles of all problems' padded arrays (the products' units
  // are at most 4 per tile, but a batch whose memory exists has far fewer)
  int64_t tiles = 0;
  for (int b = 0; b < count; ++b) {
    const fps::Layout &L = bt->plan_of(b)->L;
    tiles += (L.npad / fps::kCols) * (L.nc[0] + L.nc[1]);
    if (tiles > (int64_t)1 << 30) {
      delete bt;
      return fail(FPS_E_UNSUPPORTED, "batch too large for one launch");
    }
  }
  for (const fps_plan *pl : bt->sub) {
    for (const fps::ShiftSet &sh : pl->rsh) bt->J_max = std::max(bt->J_max, sh.J);
    bt->has_n1 = bt->has_n1 || pl->n == 1;
  }
  if (!(flags & FPS_PLAN_HOST_ONLY)) {
    const fps_status s = build_gemm_tables(bt);
    if (s != FPS_OK) {
      delete bt;
      return s;
    }
    bt->on_device = true;
  }
  *out = bt;
  return FPS_OK;
}

fps_status fps_batch_info(const fps_batch *bt, int64_t *ws_bytes, int64_t *in_entries,
                          int64_t *out_entries, int *max_J) {
  if (!valid_batch(bt)) return fail(FPS_E_STATE, "invalid or destroyed batch");
  if (ws_bytes) *ws_bytes = bt->ws_bytes;
  if (in_entries) *in_entries = bt->in_entries;
  if (out_entries) *out_entries = bt->out_entries;
  if (max_J) *max_J = bt->J_max;
  return FPS_OK;
}

fps_status fps_batch_solve(fps_batch *bt, const double *F, double *U, void *ws, void *stream) {
  if (!valid_batch(bt)) return fail(FPS_E_STATE, "invalid or destroyed batch");
  if (!bt->on_device) return fail(FPS_E_STATE, "batch was created host-only");
  if (!F || !U || !ws) return fail(FPS_E_ARG, "null pointer argument");
  if (((uintptr_t)ws) % 256 != 0) return fail(FPS_E_ARG, "workspace must be 256-byte aligned");
  hipStream_t st = (hipStream_t)stream;
  return run_batch(bt, 0, F, U, (char *)ws, st);
}

fps_status fps_batch_solve_adjoint(fps_batch *bt, const double *Ubar, double *Fbar, void *ws,
                                   void *stream) {
  if (!valid_batch(bt)) return fail(FPS_E_STATE, "invalid or destroyed batch");
  if (!bt->on_device) return fail(FPS_E_STATE, "batch was created host-only");
  if (!Ubar || !Fbar || !ws) return fail(FPS_E_ARG, "null pointer argument");
  if (((uintptr_t)ws) % 256 != 0) return fail(FPS_E_ARG, "workspace must be 256-byte aligned");
  if (bt->prec != FPS_FP64) return fail(FPS_E_UNSUPPORTED, "batched adjoint: FP64 batches only");
  hipStream_t st = (hipStream_t)stream;
  return run_batch(bt, 1, Ubar, Fbar, (char *)ws, st);
}

void fps_batch_destroy(fps_batch *bt) {
  if (!valid_batch(bt)) return;
  bt->magic = 0;
  delete bt;
}

}  // extern "C"
