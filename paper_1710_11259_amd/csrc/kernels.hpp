// Launch interfaces of the gfx950 kernels of the spectral Poisson solver.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "planner.hpp"

namespace fps {

// One FP64 half-sweep of Algorithm 2 (fps_adi_native).  Chains run down the storage
// rows of a parity-blocked array (npad rows = chain positions of both parities, row
// stride ld), one chain per storage column (ncols of them).
//   input  v = in_scale * in + (carry correction of the producing pass)
//   rhs    r = v + sg * g
//   solve  x = T^-1 r along each chain (per parity), T the pass's
//          tridiagonal (tables)
//   output out_mode 1: x; 2: v - sigma x.  Chunk-level carries are not applied by the
//          producer: it leaves its chunk boundary values in `lv`;
//          launch_reduce turns them into carries, which the consumer (the
//          next sweep, or k_finalize) folds in.
struct SweepArgs {
  const double *in;        // [npad rows][ld]
  double in_scale;
  const double *ab_prev;   // producer's chunk carries [2][ncmax][npad][2] (producer chains = npad), or null
  const double *tab_prev;  // producer's per-position tables (its shift) [2][kNTab][mstride]
  // Carries formed in the sweep itself (ctab_prev non-null; chains of at
  // most two chunks per parity, ncmax <= 2): from the producer's chunk
  // boundary values lv_prev (its lv, [ncmax][2][2][npad]) and chunk tables
  // ctab_prev ([2][kNCTab][ncmax]), times carry_scale (the scale launch_reduce
  // would apply); ab_prev is then unused.
  const double *lv_prev;
  const double *ctab_prev;
  double carry_scale;
  const double *g;         // G term, same layout as `in`
  double sg;
  const double *tab;       // this pass's tables [2][kNTab][mstride]
  const double *l1;        // this pass's segment-carry combinations [2][ncmax][kL1]
  double sigma;
  double *out;
  double *lv;              // chunk boundary values [ncmax][2][2][ncols]
  int out_mode;
  int64_t npad, mp0, mp1, mstride, ncmax;
  int64_t ncols, ld;       // chains, row stride (elements)
  int nc0, nc1;
  // The chain blocks (64 chains) blk0 .. blk1-1 and chunk
  // rows (parity-0 chunks first) chk0 .. chk1-1 only; blk1 = 0 / chk1 = 0
  // take all of them.
  int blk0, blk1, chk0, chk1;
};

// With ev0 / ev1 non-null the launch records the dispatch's own start and
// end timestamps in them (no separate event packets).
hipError_t launch_sweep(const SweepArgs &a, hipStream_t st, hipEvent_t ev0 = nullptr,
                        hipEvent_t ev1 = nullptr);

// Row-chain half-sweep: the same pass along the storage rows of `in`
// (chains = rows, positions = columns, ncols = npad chains), stored in the
// same layout; no g term (g null, r = v).  The producer's carries fold in
// as in launch_sweep with the producer's chains along the columns; its
// chunk boundary values go to lv ([ncmax][2][2][npad], chains = rows).
// Equals launch_sweep on the transposed arrays bit for bit.
hipError_t launch_sweep_rows(const SweepArgs &a, hipStream_t st, hipEvent_t ev0 = nullptr,
                             hipEvent_t ev1 = nullptr);

// Chunk carries: for every chain, the forward and backward carry into each
// chunk, scaled by `scale`, into ab [2][ncmax][nchains][2] (ctab: the
// per-chunk coefficients [2][kNCTab][ncmax] of the producing pass's shift).
// Only the chains r_lo .. r_hi-1 (r_hi < 0: all) of the parities s_lo ..
// s_hi-1 are resolved.
hipError_t launch_reduce(const double *lv, const double *ctab, double *ab, double scale,
                         int64_t nchains, int nc0, int nc1, int64_t ncmax, hipStream_t st,
                         int64_t r_lo = 0, int64_t r_hi = -1, int s_lo = 0, int s_hi = 2);

// Shape of the chunk-carry kernels for chains of up to ncmax chunks: each
// chain on a segment of 2 to 16 lanes (the least power of two that holds
// min(ncmax, 16) lanes), and 256 / lanes chains per workgroup (256 threads).
constexpr int kReduceThreads = 256;
constexpr int kReduceMaxLanes = 16;
inline int reduce_lanes(int64_t ncmax) {
  int l = 2;
  while (l < kReduceMaxLanes && l < ncmax) l <<= 1;
  return l;
}
inline int reduce_chains(int64_t ncmax) { return kReduceThreads / reduce_lanes(ncmax); }

// Y = x[r][col] + carries (final pass, non-transposed): the natural-order n x n array
// `out`.
hipError_t launch_finalize(const double *x, const double *ab, const double *tab, double *out,
                           int64_t n, int64_t npad, int64_t mp0, int64_t mstride, int64_t ncmax,
                           hipStream_t st);

// natural n x n (ld n) -> parity-blocked npad x npad (zero padding).
hipError_t launch_permute_in(const double *src, double *dst, int64_t n, int64_t npad, int64_t mp0,
                             hipStream_t st);

// Cube (npad^3 arrays [z][y][x], every axis parity-blocked):
// natural n^3 -> parity-blocked npad^3 (zero padding).
hipError_t launch_permute3_in(const double *src, double *dst, int64_t n, int64_t npad, int64_t mp0,
                              hipStream_t st);
hipError_t launch_fill(double *dst, int64_t count, double v, hipStream_t st);
// A kernel, where a copy would put a memcpy node into a captured graph.
hipError_t launch_copy(const double *src, double *dst, int64_t count, hipStream_t st);

// Nonhomogeneous Dirichlet data (Sec. 6.1), traces bc = [L; R; B; T], each
// n + 2 Chebyshev coefficients in the mapped variable (L, R in t; B, T in s).
// Constants of the lift: sinv[i] = 1/sqrt((i+1)(i+2)) and the C~
// coefficients am / ap of (1 - t)/2 and (1 + t)/2 at degrees 0 and 1.
struct BcLiftConst {
  double sinv[2], am[2], ap[2];
};
// The lift's right-hand side V^T S^-1 C~(Lap u_bc) S^-1 V as a sum of four
// outer products lr[i][q] lc[j][q] by storage position (lr and lc [npad][4]),
// and the traces' values at -1 and +1 (corner [8], for launch_bc_lift_out).  Ml0 / Ml1: the lift map V^T S^-1 C~(T_k'') by parity
// (row length ld0 / ld1); lina [npad][2]: V^T of the lift's linear factors.
hipError_t launch_bc_lift_rhs(const double *bc, const double *Ml0, const double *Ml1, int64_t ld0,
                              int64_t ld1, const double *lina, double *lr, double *lc,
                              double *corner, const Layout &L, double sx2, double sy2,
                              hipStream_t st);
// Cylinder: F [mode][part][n][n] -> X0 [slot][part][r][z] parity-blocked
// (slot -> mode through slot_idx), zero padded to npad = 2 mp per axis.
hipError_t launch_cyl_permute_in(const double *F, double *X0, const int *slot_idx, int64_t n,
                                 int64_t nt, int64_t mp, hipStream_t st);
// Cylinder: the right-hand sides that share one |k| (modes k and -k, real
// and imaginary parts): up to kCylRhs (slot * 2 + part) rows of X0 / X1,
// unused entries -1; rp / wp the row parities of the right-hand side and of
// the solution.
constexpr int kCylRhs = 4;
struct CylSolveGroup {
  int sp[kCylRhs];
  int kabs, rp, wp;
  unsigned pivots;  // bit b: a row exchange in some z column of 64 b .. 64 b + 63
};
// Cylinder: the banded r-solves of every (|k| group, z column) with the
// plan's LU factors (see cylinder.cpp), one thread applying them to half of
// the group's right-hand sides (one mode's two parts); X0 holds the right-hand sides (rows of parity
// rp, overwritten), X1 receives yhat (rows of parity wp).
hipError_t launch_cyl_solve(double *X0, double *X1, const double *fac, const CylSolveGroup *grp,
                            int ngroups, int64_t m, int64_t mp, hipStream_t st);
// U ((n+2) x (n+2) Chebyshev, natural order) += coefficients of u_bc.
hipError_t launch_bc_lift_out(double *U, const double *bc, const double *corner, int64_t n,
                              hipStream_t st);

// FP64 GEMM on MFMA, up to 4 independent problems per launch:
//   C(i,j) = sum_k A(i,k) B(k,j),  A(i,k) = A[i*sai + k], B(k,j) = B[k*sbk + j],
//   C(i,j) at C[i*sci + j*scj]  (sak and sbj must be 1; K a multiple of 16;
//   A, B 16-byte aligned with even row strides).
constexpr int kGemmGroup = 64;  // rows or columns that share one k limit
struct GemmProb {
  const double *A;
  const double *B;
  double *C;
  int64_t M, N, K;
  int64_t sai, sak, sbk, sbj, sci, scj;
  // Limited k-range: kside 1: A(i,k) = 0, kside 2: B(k,j) = 0 from
  // k = klim[x / kGemmGroup] on, x = i or j; klim
  // nonincreasing, a device table (klim_host: the same values on the host).
  int kside;
  const int *klim, *klim_host;
  // Multiplier of the eigenbasis solve, when mr is non-null: C(i,j) becomes
  //   (acc - sum_q lr[4i+q] lc[4j+q]) (1 - mr[2i+1] mc[2j+1]) / (mr[2i] + mc[2j]),
  // the lr / lc term (the Dirichlet lift) only when lr is non-null.
  // Every problem of one launch has it or none does.
  const double *mr, *mc, *lr, *lc;
  // Cube: a tabulated multiplier instead, mt indexed like C (mr null).
  const double *mt;
  // split > 0: B is an array in natural order, of `cols` columns and krows rows (A is
  // zero from k = krows on), 8-byte aligned.  Column j of the product goes to column
  // j / 2 (even j) or split + j / 2 (odd) of C, zeros from j = cols to N - 1.  Every
  // problem of one launch or none.
  int64_t split, cols, krows;
};
hipError_t launch_gemm(const GemmProb *probs, int count, hipStream_t st, hipEvent_t ev0 = nullptr,
                       hipEvent_t ev1 = nullptr);

// Plan-time passes of the eigenbasis form (spectral.hip).  Values of about 2^-100
// relative accuracy, the unevaluated sums p[i] + p[lo + i].
struct PairArray {
  double *p;
  int64_t lo;
};
// Eigenpairs of two negative definite tridiagonals T (m 0: none) whose negated diagonal is d
// and coupling e (e[m - 1] = 0; e2 = e^2 in double; device arrays of m): lam[a] descending
// from the one next to zero, V the orthonormal vectors as columns (row length ld, rows and
// columns from m on unwritten); [lo, hi] encloses sigma(-T); cp, cm scratch of V's shape.
struct TridiagEig {
  PairArray d, e;
  const double *e2;
  double *lam;
  PairArray cp, cm, V;
  int64_t ld;
  int m;
};
hipError_t launch_tridiag_eig(const TridiagEig *p, double lo, double hi, hipStream_t st);
// M[a][b] = row[a] col[b] t[b - a + rows - 1] u[a + b] (planner's MapTables) for a < rows, b <
// cols, zeros up to prows x ld; up to 4 of them.
struct MapEntries {
  PairArray row, col, t, u, M;
  int64_t rows, cols, prows, ld;
};
hipError_t launch_map_entries(const MapEntries *m, int count, hipStream_t st);
// W = V^T M (rows x cols, contiguous) and, if WT is not null, its transpose, rounded once
// from the pairs; V as above, M with row length cols, rows and cols multiples of 64.
// zlim (or null): W[a][j] = 0 from a = zlim[j / kGemmGroup] on.  Up to 4 of them.
struct MapProduct {
  PairArray V, M;
  int64_t ldv, rows, cols;
  int m;
  const int *zlim;
  double *W, *WT;
};
hipError_t launch_map_products(const MapProduct *p, int count, hipStream_t st);
// Cube multipliers -(1 - eps) / (lz ly + lz lx + ly lx) by storage position
// [npad]^3 (cube.cpp states the iterations).  z-eigenbasis: eps = ey[z][y]
// ex[z][x], the error factors of slice z's shifts p / q[off[z] .. off[z+1] - 1]
// (refined: symmetric shifts of the K-form).  Nested: r[i][k] the inner error
// factor of outer step i along one axis, eps by the outer recurrence.
hipError_t launch_slice_factors(const double *lam, const double *mu, const int *off,
                                const double *p, const double *q, bool refined, double *ey,
                                double *ex, int64_t npad, hipStream_t st);
hipError_t launch_slice_multiplier(const double *lam, const double *ey, const double *ex, double *mt,
                                   int64_t npad, hipStream_t st);
hipError_t launch_nested_factors(const double *lam, const double *q, const int *off,
                                 const double *p_in, double *r, int J, int64_t npad,
                                 hipStream_t st);
hipError_t launch_nested_multiplier(const double *lam, const double *p, const double *q,
                                    const double *r, int J, double *mt, int64_t npad,
                                    hipStream_t st);
// Whether an extent has edge rows or columns: 1 to 4 past a multiple of 32.
__host__ __device__ inline bool gemm_has_edge(int64_t x) {
  return x > 32 && x % 32 >= 1 && x % 32 <= 4;
}
// The launcher's operand requirements (also for table-driven problems, with
// offsets in place of pointers).
bool gemm_operands_ok(const GemmProb &q);

// Table-driven GEMM over many problems in one launch.  Each pointer of a
// descriptor's GemmProb is absolute (base id 0), a byte offset from `ws`
// (1), from `out` (2) or from `in` (3).  gemm_table (host) picks the tile and fills the
// workgroup map, (problem, unit) pairs; false
// if a problem does not meet the launcher's requirements.
struct GemmDesc {
  GemmProb p;
  int abase, bbase, cbase;
};
struct GemmTable {
  int T = 0, units = 0, kind = 0;
};
bool gemm_table(std::vector<GemmDesc> &tab, GemmTable &t, std::vector<int> &map);
hipError_t launch_gemm_table(const GemmTable &t, const GemmDesc *d, const int *tile_map,
                             const double *in, char *ws, char *out, hipStream_t st, hipEvent_t ev0 = nullptr,
                             hipEvent_t ev1 = nullptr);
// Chains of products on one LDS-resident block (chain.hip).  The block X is in[r *
// in_rs + c * in_cs] for r < in_r, c < in_c, zero beyond.  Matrix i is m[i][k * ld +
// output index], k[i] its inner length (padded), n[i] its output length; ld covers n
// rounded up to the tiles that read it.
//   mode 1: m3^T (multiplier of m1^T X m0) m2; blocks of up to 64, outputs of up to
//           16 nb (nb = 3, 4, 5); k multiples of 16, ld of n's next one.
//   Modes 0, 2 and 3 with blocks of up to S = 32 nb (nb = 2, 3, 4), k multiples of 32,
//   n of the last matrices up to S + 2 but in mode 0, ld at least n rounded up to 32,
//   or S + 16 past S:
//   mode 0: rows r0 .. r0 + chain_part(nb) of m1^T X m0, in_cs 2 and out_cs 1.
//   mode 3: the same, in_cs 1 and out_cs 2; the last rows below S bring those past it.
//   mode 2: m3^T (multiplier of m1^T X), up to chain_part(nb) columns.
// The multiplier is that of GemmProb (mode 1: mr, mc, lr, lc; mode 2: mt with row
// stride mt_rs), applied to rows < n[1], columns < n[0] (in_c).  The result goes to
// out[r * out_rs + c * out_cs] for r < out_r, c < out_c (mode 3: and a zero zoff
// elements from it, if zoff is not 0; out is column zcol of its row, and the table
// holds the same block for column 1 - zcol, which shares the writing of the zeros).
// in / out are absolute (base 0) or byte offsets from the workspace (1), the solve's
// input (2) or output (3).
struct ChainDesc {
  const double *in;
  double *out;
  const double *m[4];
  const double *mr, *mc, *lr, *lc, *mt;
  int64_t in_rs, out_rs, mt_rs;
  int in_cs, out_cs, in_r, in_c, out_r, out_c, r0;
  int ld[4], k[4], n[4];
  int ibase, obase, zoff, zcol;
};
// Slabs and strips of blocks of up to `len` per side need nb = chain_size(len) (0: too
// large).
inline int chain_size(int64_t len) { return len <= 64 ? 2 : len <= 96 ? 3 : len <= 128 ? 4 : 0; }
constexpr int chain_part(int nb) { return nb >= 3 ? 32 : 64; }
bool chain_ok(const ChainDesc &d, int nb, int mode);
// Table order: runs of `group` descriptors that share operands, of which d holds
// one after another, 8 apart: on one die at the same time.
void chain_order(std::vector<ChainDesc> &d, int group);
hipError_t launch_chain_table(const ChainDesc *d, int count, int nb, int mode, const double *in,
                              char *ws, double *out, hipStream_t st, hipEvent_t ev0 = nullptr,
                              hipEvent_t ev1 = nullptr);
// Mode 1 on up to 4 blocks given by value.
hipError_t launch_chain(const ChainDesc *d, int count, int nb, hipStream_t st,
                        hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);

}  // namespace fps
