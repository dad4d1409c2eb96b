// Internal interfaces shared by the C ABI translation units (not part of
// the public ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/fps.h"
#include "kernels.hpp"
#include "planner.hpp"

namespace fps {
namespace detail {

// Records `msg` as the calling thread's last error and returns `s`.
fps_status fail(fps_status s, const std::string &msg);
const char *last_error();

#define FPS_HIP(call)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess)                                                               \
      return ::fps::detail::fail(FPS_E_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

constexpr uint64_t kMagic = 0x66707370'6c616e31ull;  // "fpsplan1"

struct DeviceBuf {
  void *p = nullptr;
  DeviceBuf() = default;
  DeviceBuf(const DeviceBuf &) = delete;
  DeviceBuf &operator=(const DeviceBuf &) = delete;
  ~DeviceBuf() {
    if (p) (void)hipFree(p);
  }
};

// A table within another allocation.
struct DeviceView {
  void *p = nullptr;
};

}  // namespace detail
}  // namespace fps

struct CylPlan;  // cylinder plans (cylinder.cpp)

struct fps_plan {
  uint64_t magic = fps::detail::kMagic;
  CylPlan *cyl = nullptr;  // non-null for cylinder plans
  fps_plan() = default;
  fps_plan(const fps_plan &) = delete;
  fps_plan &operator=(const fps_plan &) = delete;
  ~fps_plan();
  int dim = 2;
  int64_t n = 0;
  double tol = 0;
  int prec = FPS_FP64;
  int out_basis = FPS_OUT_CHEB;
  unsigned flags = 0;
  bool on_device = false;

  fps::ShiftSet shifts;     // shifts of the ADI (FP32_REFINED: of round 0)
  // Refinement rounds (FP32_REFINED; FP64 plans have one round, the plain
  // ADI): round k is an ADI to rtol[k] with the shifts rsh[k], which enters the
  // solve through its error factors; rf32[k]: a round of the schedule that is derived for
  // float storage (nothing is stored in float).  n_f32 counts those rounds' steps.
  int rounds = 1;
  std::vector<fps::ShiftSet> rsh;
  std::vector<double> rtol;
  std::vector<char> rf32;
  int n_f32 = 0;

  // Rectangle [a, b] x [c, d] (rect plans): the symmetric form reads
  // sx2 A~ Y + sy2 Y A~ = G with sx2 = (2/(b-a))^2, sy2 = (2/(d-c))^2, i.e.
  // A Y - Y B = G for A = sx2 A~ (rows), B = -sy2 A~ (columns).  ADI step j
  // then solves with two matrices: table 2j holds sy2 A~ + p_j (first
  // half-step), table 2j + 1 holds sx2 A~ - q_j (second half-step).  The
  // square uses one table per step (A~ + p_j, q_j = -p_j) and sx2 = sy2 = 1.
  bool rect = false;
  double box[4] = {-1.0, 1.0, -1.0, 1.0};
  double sx2 = 1.0, sy2 = 1.0;
  int tab1(int j) const { return rect ? 2 * j : j; }
  int tab2(int j) const { return rect ? 2 * j + 1 : j; }
  fps::Layout L;
  int64_t mop[2] = {0, 0};          // output parity lengths padded to 64

  // device copies
  // Sweep tables of fps_adi_native (FP64 2-D plans), in d_maps.
  fps::detail::DeviceView d_tab, d_ctab, d_l1;
  // Coefficient maps merged with the eigenvectors V of A~ (spectral.cpp), by
  // parity, zero-padded to multiples of 64, in both orientations: Wi =
  // V^T S^-1 R (mp x mp) and Wo = P S^-1 V (mop x mp; native output S^-1 V,
  // mp x mp).  lam: eigenvalues by storage position (-1 on padding); d_mr /
  // d_mc: the multiplier's row and column factors, [npad][2].
  fps::detail::DeviceBuf d_maps;  // holds them and the tables below
  fps::detail::DeviceView d_Wi[2], d_WiT[2], d_Wo[2], d_WoT[2];
  fps::detail::DeviceView d_mr, d_mc;
  // Where Wo is zero (spectral.cpp): row group g of 64 output coefficients has
  // no entries from mode mlim[g] on, and mode group h none from row clim[h] on.
  std::vector<int> mlim[2], clim[2];
  fps::detail::DeviceView d_mlim[2], d_clim[2];
  std::vector<double> lam;
  // Lift map V^T S^-1 C~(T_k'') by parity (mp x mop) and V^T of the lift's
  // linear factors ([npad][2]), only with FPS_PLAN_DIRICHLET.
  fps::detail::DeviceView d_lift[2], d_lina;

  // sweep timing diagnostics
  std::vector<hipEvent_t> ev;  // pairs
  int64_t ev_used = 0;

  // workspace layout (byte offsets)
  int64_t off_G = 0, off_GT = 0, off_O0 = 0, off_O1 = 0, off_lv = 0, off_ab = 0;
  // fps_adi_native: second half-steps write their chunk boundary values to lv2
  // and first ones to lv; the carries of first half-steps go to ab2, those of
  // second ones (and the final pass's) to ab, so that the two row-parity halves of
  // the ADI can run on two streams without sharing a buffer element.
  int64_t off_lv2 = 0, off_ab2 = 0;
  // Dirichlet lift (2-D plans with FPS_PLAN_DIRICHLET): the traces' values at -1
  // and +1 [8].
  int64_t off_bc = 0;

  // Cube (dim 3), nested method: `shifts` holds the outer shifts (p in
  // [-2/delta, -2], q in [1, 1/delta]); inner step (i, j) has shift
  // inner_p[inner_off[i] + j].
  std::vector<int> inner_J, inner_off;
  std::vector<double> inner_p;
  // Cube, z-eigenbasis method (FPS_PLAN_CUBE_ZEIG): the shifts of storage slice
  // c (all rounds) are zp / zq[zoff[c] .. zoff[c + 1] - 1]; zJ the steps per
  // slice (round 0), most first, zrJmax the most steps per refinement round.
  bool zeig = false;
  std::vector<double> zlam[2], zp, zq;
  std::vector<int> zoff, zJ, zrJmax;
  // Cube layout: parity blocks of cmp[s] (rounded up to 16), cnp per axis; output
  // parity sizes rounded up to even.
  int64_t cmp[2] = {0, 0}, cnp = 0, mqc[2] = {0, 0};
  fps::detail::DeviceBuf d_mt;                // multiplier of every mode [cnp]^3
  fps::detail::DeviceBuf d_gy_in, d_gy_out;   // mode-y GEMM tables (input / output map)
  fps::GemmTable t_gy[2];
  fps::detail::DeviceBuf d_gy_map_in, d_gy_map_out;
  int64_t off_ZR = 0, off_RX = 0;
  // Cube plans whose blocks fit one workgroup's LDS (n <= 256): block size of the
  // chains (0: per-axis products) and their tables (slices in, strips along z,
  // slices out).
  int cnb = 0, cchain_count[3] = {0, 0, 0};
  fps::detail::DeviceBuf d_cchain[3];
  // 2-D plans whose chains have more than two chunks: fps_adi_native runs one
  // row-parity block's sweeps on the plan's own stream zside, the other's on
  // the caller's, joined by the events zfork / zjoin.  zlock is held while one
  // call enqueues its fork, both blocks and its join, so concurrent host
  // threads' calls do not interleave on zside.
  hipStream_t zside = nullptr;
  hipEvent_t zfork = nullptr, zjoin = nullptr;
  std::mutex zlock;
  int64_t ws_bytes = 0;

  const double *tab_dev(int j) const {
    return (const double *)d_tab.p + (size_t)j * 2 * fps::kNTab * L.mstride;
  }
  const double *ctab_dev(int j) const {
    return (const double *)d_ctab.p + (size_t)j * 2 * fps::kNCTab * L.ncmax;
  }
  const double *l1_dev(int j) const {
    return (const double *)d_l1.p + (size_t)j * 2 * L.ncmax * fps::kL1;
  }
};

namespace fps {
namespace detail {

bool valid_plan(const fps_plan *p);
// Enclosure [a, b] of sigma(A~) (both negative) from the computed extreme
// eigenvalues, widened by a relative 1e-6.
void spectrum_tight(int64_t n, double *a, double *b);
int64_t align256(int64_t x);
template <typename T>
fps_status upload(DeviceBuf &b, const std::vector<T> &h) {
  if (h.empty()) return FPS_OK;
  if (hipMalloc(&b.p, h.size() * sizeof(T)) != hipSuccess)
    return fail(FPS_E_NOMEM, "hipMalloc of a plan table failed");
  FPS_HIP(hipMemcpy(b.p, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice));
  return FPS_OK;
}
// The refinement rounds of an FP32_REFINED plan with target tolerance tol:
// each round's inner ADI tolerance and whether the schedule derives it for float
// storage (Dirichlet plans end with one for float64).
struct RefineRound {
  double tol;
  bool f32;
};
std::vector<RefineRound> refine_schedule(double tol, bool dirichlet);
// Eigenbasis maps (spectral.cpp).
fps_status spectral_build(fps_plan *pl, bool lift);
fps::BcLiftConst bc_lift_const();
// The products of one square or rectangle solve, per stage up to 4
// parity-block problems (returns their count), operands formed from the
// workspace base `ws` (and U / Fbar).  rhs: g1 then g2 from F, leaving Y^ (the multiplier applied; with lr / lc the
// Dirichlet lift subtracted first) in G; out: g1 then g2 to U (whose entries of
// empty parity blocks the caller clears).  adj_in / adj_out: the same four
// steps of the adjoint, transposed, from the cotangent to Fbar.  The input stages' g1
// is by row parity (cnt1 products).
int rhs_gemms(const fps_plan *pl, const double *F, char *ws, fps::GemmProb *g1, int *cnt1,
              fps::GemmProb *g2, const double *lr = nullptr, const double *lc = nullptr);
int out_gemms(const fps_plan *pl, double *U, char *ws, fps::GemmProb *g1, fps::GemmProb *g2);
int adj_in_gemms(const fps_plan *pl, const double *Ubar, char *w, fps::GemmProb *g1, int *cnt1,
                 fps::GemmProb *g2);
int adj_out_gemms(const fps_plan *pl, double *Fbar, char *w, fps::GemmProb *g1, fps::GemmProb *g2);
// A stage of products on st, timed like a sweep when the plan's timing is on.
fps_status run_products(fps_plan *pl, const fps::GemmProb *g, int cnt, hipStream_t st);
// Start / stop events of the next timed launch (null when timing is off or its
// pairs are used up); the launch then counts one in ev_used.
inline hipEvent_t next_event(const fps_plan *pl, int i) {
  return pl->ev_used * 2 + 1 < (int64_t)pl->ev.size() ? pl->ev[2 * pl->ev_used + i] : nullptr;
}
// Lengths along which products run: rounded up to the k-tile (the arrays are
// padded with zeros beyond).
inline int64_t k_round(int64_t x) { return (x + 15) / 16 * 16; }
// Squares and rectangles solved in one launch of chains: blocks, and inner lengths of
// the products, of at most 64 (n <= 128; an adjoint's first products run over the
// output's coefficients, so n <= 126 unless they are native).
inline bool forward_chained(const fps_plan *pl) { return pl->L.m[0] <= 64; }
inline bool adjoint_chained(const fps_plan *pl) {
  return (pl->out_basis == FPS_OUT_NATIVE ? pl->L.m[0] : pl->L.mo[0]) <= 64;
}
// Their blocks: up to 4 (returns the count, 0 for other plans) from F (or the adjoint's
// cotangent) to U (Fbar); nb for launch_chain.
bool chain_in_out(const double *in, int64_t n_in, const double *out, int64_t n_out);
fps_status clear_n1(const fps_plan *pl, double *U, hipStream_t st);
int solve_chain(const fps_plan *pl, const double *F, double *U, const double *lr, const double *lc,
                fps::ChainDesc *d, int *nb);
int adjoint_chain(const fps_plan *pl, const double *Ubar, double *Fbar, fps::ChainDesc *d, int *nb);
// Entries per axis of the solve's output.
inline int64_t out_extent(const fps_plan *pl) {
  return pl->out_basis == FPS_OUT_NATIVE ? pl->n : pl->n + 2;
}
// Cube: host tables and workspace layout (after the common fields are set),
// their upload, and the solve.
fps_status cube_plan_build(fps_plan *pl);
fps_status cube_plan_upload(fps_plan *pl);
fps_status cube_solve(fps_plan *pl, const double *F, double *U, char *ws, hipStream_t st);
hipError_t timed_sweep(fps_plan *pl, const fps::SweepArgs &a, hipStream_t st, bool rows = false);
// The plan's default-priority side stream and its fork / join events
// (zside / zfork / zjoin), created once.
fps_status create_side_stream(fps_plan *pl);
// Cylinder (Sec. 4.1): host tables and workspace layout, their upload, the
// solve, and the band of one mode's r-operators (inspection).
fps_status cyl_plan_build(fps_plan *pl, int64_t nt);
fps_status cyl_plan_upload(fps_plan *pl);
fps_status cyl_solve(fps_plan *pl, const double *F, double *U, char *ws, hipStream_t st);
int64_t cyl_ws_bytes(const fps_plan *pl);
int64_t cyl_out_entries(const fps_plan *pl);
void cyl_mode_bands(int64_t n, int64_t kabs, std::vector<double> &Pb, std::vector<double> &Qb);

}  // namespace detail
}  // namespace fps
