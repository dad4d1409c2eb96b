// Batched square solves (fps_batch_* in include/fps.h): many independent
// problems, possibly of different sizes, each stage of the eigenbasis solve
// (spectral.cpp) as one launch for all of them.  Every problem keeps the maps,
// workspace layout and kernels of its own single-problem plan.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <new>
#include <numeric>
#include <vector>

#include "launch_limits.hpp"
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
  std::vector<int> order;            // sorted position -> problem (n descending)
  std::vector<int64_t> f_off, u_off, ws_off;  // per problem: F / U entries, workspace bytes
  int64_t in_entries = 0, out_entries = 0, ws_bytes = 0;
  int J_max = 0;                     // steps of the longest ADI (over all rounds)
  bool has_n1 = false;               // a problem of size 1 (parts of its U no product writes)
  // products of all problems: input map g1, g2; output map g1, g2; (FP64
  // batches) the adjoint's input map g1, g2 and output map g1, g2
  DeviceBuf d_gd[8], d_gmap[8];
  fps::GemmTable gt[8];
  // the problems small enough for chains (forward 0, adjoint 1): one
  // launch each; the products and permutations below hold the others
  DeviceBuf d_chain[2];
  int nchain[2] = {0, 0}, chain_nb[2] = {3, 3};
  // the permutations of F (0) and of the adjoint's cotangent (1) as one
  // launch each (elem_ok; else, for very large batches, one per problem)
  bool elem_ok = false;
  DeviceBuf d_ed[2], d_emap[2];
  int ewg[2] = {0, 0};

  ~fps_batch() {
    for (fps_plan *p : sub) fps_plan_destroy(p);
  }
  const fps_plan *plan_of(int problem) const { return sub[which[problem]]; }
};

namespace {

bool valid_batch(const fps_batch *b) { return b != nullptr && b->magic == kBatchMagic; }

// Whether the plan's solves (t 0) or adjoints (1) run as chains.
bool chained(const fps_plan *pl, int t) { return t ? adjoint_chained(pl) : forward_chained(pl); }

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
    const bool fwd = !chained(pl, 0), adj = !refined && !chained(pl, 1);
    const int c_in = fwd ? rhs_gemms(pl, wsyn, g[0], g[1]) : 0;
    const int c_out = fwd ? out_gemms(pl, Usyn, wsyn, g[2], g[3]) : 0;
    const int c_ain = adj ? adj_in_gemms(pl, wsyn, g[4], g[5]) : 0;
    const int c_aout = adj ? adj_out_gemms(pl, Fsyn, wsyn, g[6], g[7]) : 0;
    // base ids (A, B, C): ws-relative 1, absolute 0, output-relative 2
    static const int ids[8][3] = {{1, 0, 1}, {0, 1, 1}, {1, 0, 1}, {0, 1, 2},
                                  {1, 0, 1}, {0, 1, 1}, {1, 0, 1}, {0, 1, 2}};
    const int counts[8] = {c_in, c_in, c_out, c_out, c_ain, c_ain, c_aout, c_aout};
    for (int t = 0; t < 8; ++t) {
      const int cnt = counts[t];
      for (int i = 0; i < cnt; ++i) {
        tab[t].push_back(fps::GemmDesc{g[t][i], ids[t][0], ids[t][1], ids[t][2]});
      }
    }
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

// Tables of the batched permutations (sorted order, largest problems first).
// Left unbuilt (elem_ok false) when a launch would not fit one 1-D grid of
// 256-thread workgroups (elem_launch_fits); such batches keep the per-problem
// launches.
fps_status build_elem_tables(fps_batch *bt) {
  std::vector<fps::ElemDesc> ed[2];
  std::vector<int> map[2];
  for (int k = 0; k < bt->count; ++k) {
    const int b = bt->order[k];
    const fps_plan *pl = bt->plan_of(b);
    const fps::Layout &L = pl->L;
    const bool native = bt->out_basis == FPS_OUT_NATIVE;
    const int64_t *mop = native ? L.mp : pl->mop;
    for (int t = 0; t < 2; ++t) {
      if (chained(pl, t)) continue;
      fps::ElemDesc e{};
      e.n = t ? out_extent(pl) : L.n;
      e.npad = t ? mop[0] + mop[1] : L.npad;
      e.mp0 = t ? mop[0] : L.mp[0];
      e.src = (t ? bt->u_off[b] : bt->f_off[b]) * (int64_t)sizeof(double);
      e.sbase = 2;
      e.dst = bt->ws_off[b] + (t ? pl->off_X : pl->off_GT);
      e.dbase = 1;
      e.nbx = (int)((e.npad + 255) / 256);
      const int64_t nwg = (int64_t)e.nbx * e.npad;
      if (!fps::elem_launch_fits((int64_t)map[t].size() + nwg)) return FPS_OK;
      e.wg_start = (int)map[t].size();
      map[t].insert(map[t].end(), (size_t)nwg, (int)ed[t].size());
      ed[t].push_back(e);
    }
  }
  fps_status s;
  for (int t = 0; t < 2; ++t) {
    bt->ewg[t] = (int)map[t].size();
    if ((s = upload(bt->d_ed[t], ed[t])) != FPS_OK || (s = upload(bt->d_emap[t], map[t])) != FPS_OK)
      return s;
  }
  bt->elem_ok = true;
  return FPS_OK;
}

// The permutation of every problem's F (t = 0, into its GT region) or output
// cotangent (t = 1, into its X region).
fps_status permute_all(const fps_batch *bt, int t, const double *in, char *w, hipStream_t st) {
  if (bt->elem_ok) {
    FPS_HIP(fps::launch_permute_in_batch((const fps::ElemDesc *)bt->d_ed[t].p,
                                         (const int *)bt->d_emap[t].p, bt->ewg[t], in, w, st));
    return FPS_OK;
  }
  for (int b = 0; b < bt->count; ++b) {
    const fps_plan *pl = bt->plan_of(b);
    if (chained(pl, t)) continue;
    const fps::Layout &L = pl->L;
    const int64_t *mop = bt->out_basis == FPS_OUT_NATIVE ? L.mp : pl->mop;
    char *wb = w + bt->ws_off[b];
    if (t == 0)
      FPS_HIP(fps::launch_permute_in(in + bt->f_off[b], (double *)(wb + pl->off_GT), L.n, L.npad,
                                     L.mp[0], st));
    else
      FPS_HIP(fps::launch_permute_in(in + bt->u_off[b], (double *)(wb + pl->off_X), out_extent(pl),
                                     mop[0] + mop[1], mop[0], st));
  }
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
  bt->order.resize(count);
  std::iota(bt->order.begin(), bt->order.end(), 0);
  std::stable_sort(bt->order.begin(), bt->order.end(), [&](int a, int c) { return n[a] > n[c]; });
  // every problem's 64 x 64 tiles must be countable by one launch
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
    fps_status s = build_gemm_tables(bt);
    if (s == FPS_OK) s = build_elem_tables(bt);
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
  char *w = (char *)ws;
  fps_status s;
  if ((s = permute_all(bt, 0, F, w, st)) != FPS_OK) return s;
  if (bt->has_n1) FPS_HIP(fps::launch_fill(U, bt->out_entries, 0.0, st));
  if ((s = run_chains(bt, 0, F, U, st)) != FPS_OK) return s;
  for (int t = 0; t < 4; ++t)
    FPS_HIP(fps::launch_gemm_table(bt->gt[t], (const fps::GemmDesc *)bt->d_gd[t].p,
                                   (const int *)bt->d_gmap[t].p, w, (char *)U, st));
  return FPS_OK;
}

fps_status fps_batch_solve_adjoint(fps_batch *bt, const double *Ubar, double *Fbar, void *ws,
                                   void *stream) {
  if (!valid_batch(bt)) return fail(FPS_E_STATE, "invalid or destroyed batch");
  if (!bt->on_device) return fail(FPS_E_STATE, "batch was created host-only");
  if (!Ubar || !Fbar || !ws) return fail(FPS_E_ARG, "null pointer argument");
  if (((uintptr_t)ws) % 256 != 0) return fail(FPS_E_ARG, "workspace must be 256-byte aligned");
  if (bt->prec != FPS_FP64) return fail(FPS_E_UNSUPPORTED, "batched adjoint: FP64 batches only");
  hipStream_t st = (hipStream_t)stream;
  char *w = (char *)ws;
  fps_status s;
  if ((s = permute_all(bt, 1, Ubar, w, st)) != FPS_OK) return s;
  if ((s = run_chains(bt, 1, Ubar, Fbar, st)) != FPS_OK) return s;
  for (int t = 4; t < 8; ++t)
    FPS_HIP(fps::launch_gemm_table(bt->gt[t], (const fps::GemmDesc *)bt->d_gd[t].p,
                                   (const int *)bt->d_gmap[t].p, w, (char *)Fbar, st));
  return FPS_OK;
}

void fps_batch_destroy(fps_batch *bt) {
  if (!valid_batch(bt)) return;
  bt->magic = 0;
  delete bt;
}

}  // extern "C"
