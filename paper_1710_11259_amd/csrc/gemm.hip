// gfx950 FP64 MFMA GEMM for the dense coefficient maps of the spectral
// Poisson solver (Chebyshev <-> C~^(3/2) maps of Sec. 3.4 and Table 1).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "device.hpp"
#include "kernels.hpp"

namespace fps {

namespace {

// ---------------------------------------------------------------------------
// FP64 GEMM on v_mfma_f64_16x16x4f64: C = A B with A row-major (k
// contiguous, sai), B row-major (n contiguous, sbk), C(i, j) at
// C[i*sci + j*scj].  Tile T x T x 16, four wavefronts in a 2 x 2 grid, each
// computing a quarter as (T/32)^2 MFMA blocks; k-tiles are loaded into
// registers two ahead and stashed into the second of two LDS stages (one
// barrier per k-tile).
// Operand layout of the 16x16x4 f64 instruction: lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator register r of lane l
// holds C[4r + l / 16][l % 16].
// Every output entry is accumulated over k in the same order whatever the
// tile, so launches with different tiles agree bit for bit; k ascends, so a sum over
// modes starts with the highest and ends with the lowest, which hold most of it.
//
// Requirements (checked by the launcher): K a multiple of 16, sai and sbk
// even, A and B 16-byte aligned; loads are clamped to M and N, so only K needs
// padding.
typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef double dbl2 __attribute__((ext_vector_type(2)));

// order: tile dispatch order (0: natural; 1: row tile slowest; 2: column tile
// slowest), so that with a limited k-range the longest tiles start first and the short ones
// fill the tail.  Workgroups 0 .. nedge-1 take edge units (equal counts per
// problem), mt x nt tiles per problem follow.
struct GemmBatch {
  GemmProb p[4];
  int order, count, mt, nt, nedge;
};

constexpr int kGroup = kGemmGroup, kBK = 16;

// Kinds of products, one per launch: plain; with the eigenbasis multiplier in the
// epilogue; of an array in natural order (GemmProb's split), whose rows past the
// last and whose parity-blocked result cost the plain ones registers.
enum { kPlain = 0, kMul = 1, kNatural = 2 };

// Extent covered by MFMA tiles: the 1 to 4 rows or columns past a multiple of 32
// (the output maps have n/2 + 1) would cost a row of almost empty tiles, so
// they are left to edge units, workgroups of the same launch.  (Carrying them
// along in the last tiles, in FMAs from the staged operands, was slower from
// K = 256 on, 1309 against 1050 us per launch at n = 4096: the border column's
// strided loads arrive late in every k-tile.)
__host__ __device__ inline int64_t main_extent(int64_t x) {
  return gemm_has_edge(x) ? x - x % 32 : x;
}

// Edge units of a problem: first those of its edge columns, then those of its
// edge rows.  A unit covers more rows or columns where k is short, so that its
// loads still fill a memory round trip.
__host__ __device__ inline int edge_rows_per_unit(const GemmProb &g) {
  return g.K <= 128 ? 32 : g.K <= 256 ? 16 : 8;
}
__host__ __device__ inline int edge_column_units(const GemmProb &g) {
  const int64_t mm = main_extent(g.M), r = edge_rows_per_unit(g);
  return main_extent(g.N) < g.N ? (int)((mm + r - 1) / r) : 0;
}
__host__ __device__ inline int edge_units(const GemmProb &g) {
  const int64_t c = g.K <= 256 ? 64 : 16;
  return edge_column_units(g) + (main_extent(g.M) < g.M ? (int)((g.N + c - 1) / c) : 0);
}

// End of the k-range of the tile at (i0, j0): the limit of its 64-row (or column) group,
// rounded up to two k-tiles.
__host__ __device__ inline int64_t tile_kend(const GemmProb &g, const int *lim, int64_t i0, int64_t j0) {
  if (g.kside == 0) return g.K;
  const int64_t h = (lim[(g.kside == 1 ? i0 : j0) / kGroup] + 31) / 32 * 32;
  return h < g.K ? h : g.K;
}

// The output entry (i, j) from its accumulated product v: the eigenbasis
// multiplier
// (compiled in only for launches that hold such problems: the maps without
// it would pay registers and a test per entry).
__device__ __forceinline__ double multiply(const GemmProb &g, int64_t i, int64_t j, double v) {
  if (g.mt != nullptr) return v * g.mt[i * g.sci + j * g.scj];
  if (g.lr != nullptr) {
    const double *r = g.lr + 4 * i, *c = g.lc + 4 * j;
    v -= fma(r[3], c[3], fma(r[2], c[2], fma(r[1], c[1], r[0] * c[0])));
  }
  const dbl2 r = *(const dbl2 *)(g.mr + 2 * i), c = *(const dbl2 *)(g.mc + 2 * j);
  return v * (fma(-r.y, c.y, 1.0) / (r.x + c.x));
}

// LDS of one workgroup: two stages of A [T][BK + 1] and B [BK][T + 2].  A is
// kept row-major with one double of padding: the stash writes each thread's
// k-run in place and the fragment reads (16 rows at one k per quarter-wave) hit
// distinct banks.
template <int T>
struct Tile {
  static constexpr int kA = T * (kBK + 1), kB = kBK * (T + 2), kStage = kA + kB;
  static constexpr int kLds = 2 * kStage;
};

// One T x T output tile at (i0, j0) of problem g.
template <int T, int kKind>
__device__ __forceinline__ void gemm_tile(const GemmProb &g, const int64_t i0, const int64_t j0,
                                          double *lds) {
  constexpr int BK = kBK;
  constexpr int W = T / 2, NB = T / 32;            // quarter of a wavefront, its MFMA blocks
  constexpr int RA = T * BK / 256, TA = BK / RA;   // A: doubles per thread, threads per row
  constexpr int TB = 256 / BK, QB = T / (2 * TB);  // B: threads per k-row, column pairs per thread
  using L = Tile<T>;
  const int64_t Mm = main_extent(g.M), Nm = main_extent(g.N);
  if (i0 >= Mm || j0 >= Nm) return;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wy = wid >> 1, wx = wid & 1;

  // Loaders.  A: thread t reads row t / TA, k-run (t % TA) RA ..; B: thread t
  // reads k-row t / TB, the column pairs bc + 2 TB q, so the threads of a row
  // read and stash one contiguous run per q (no LDS bank conflicts).  Rows and
  // columns past M and N are clamped to the last one: what they add to lands
  // in output entries that are not stored, so the loop has no branches (with
  // one per k-step the compiler waited for every LDS read before its products:
  // 34 against 21 us per 64 x 64 stage at n = 1024).
  const int ar = tid / TA, ak = (tid % TA) * RA;
  const int bk = tid / TB, bc = (tid % TB) * 2;
  const int64_t arow = i0 + ar < g.M ? i0 + ar : g.M - 1;
  const double *Ab = g.A + i0 * g.sai, *Bb = g.B;
  const uint32_t ao = 8 * ((uint32_t)(arow - i0) * (uint32_t)g.sai + ak);
  const int nk = (int)((tile_kend(g, g.klim, i0, j0) + BK - 1) / BK);
  // Columns past N are clamped to the last pair (row strides are even: it exists).
  // Of a natural array the rows past the last are clamped (A is zero there), and the
  // columns past it only in the last k-tile, as before that they lie in the rows that
  // follow; the row may end within a pair, then the pair before holds its first column.
  const int64_t jlast = kKind == kNatural ? g.cols - 2 : (g.N - 1) & ~(int64_t)1;
  const int lrow = kKind == kNatural ? (int)g.krows - (nk - 1) * BK - 1 : 0;
  uint32_t bo[QB], bl[QB];
  bool late[QB];
#pragma unroll
  for (int q = 0; q < QB; ++q) {
    const int64_t j = j0 + bc + 2 * TB * q, jc = j < jlast ? j : jlast;
    bo[q] = 8 * ((uint32_t)bk * (uint32_t)g.sbk + (uint32_t)(kKind == kNatural ? j : jc));
    bl[q] = 8 * ((uint32_t)(bk < lrow ? bk : lrow) * (uint32_t)g.sbk + (uint32_t)jc);
    late[q] = kKind == kNatural && j > jlast;
  }

  dbl2 ra[2][RA / 2], rb[2][QB];
  int tile = 0;
  auto fetch = [&](int r) {
    const Buffer A(Ab), B(Bb);
#pragma unroll
    for (int q = 0; q < RA / 2; ++q) ra[r][q] = A.load2(ao + 16 * q, 0);
    const bool last = kKind == kNatural && tile == nk - 1;
#pragma unroll
    for (int q = 0; q < QB; ++q) rb[r][q] = B.load2(last ? bl[q] : bo[q], 0);
    Ab += BK;
    Bb += BK * g.sbk;
    ++tile;
  };
  auto stash = [&](double *st, int r, bool last) {
    double *Ad = st + ar * (BK + 1) + ak;
    double *Bd = st + L::kA + bk * (T + 2) + bc;
#pragma unroll
    for (int q = 0; q < RA / 2; ++q) {
      Ad[2 * q] = ra[r][q].x;
      Ad[2 * q + 1] = ra[r][q].y;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      if (kKind == kNatural && last && late[q]) rb[r][q].x = rb[r][q].y;
      *(dbl2 *)(Bd + 2 * TB * q) = rb[r][q];
    }
  };

  dbl4 acc[NB][NB];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
  const double *Ar = lds + (wy * W + (lane & 15)) * (BK + 1) + (lane >> 4);
  const double *Br = lds + L::kA + (lane >> 4) * (T + 2) + wx * W + (lane & 15);
  // The products of one k-tile from the stage at offset so; the fragments of
  // the next k-step are read under the products of the current one.
  auto mma = [&](int so) {
    double av[2][NB], bv[2][NB];
    auto frag = [&](int ks) {
      const int f = (ks >> 2) & 1;
#pragma unroll
      for (int a = 0; a < NB; ++a) av[f][a] = Ar[so + a * 16 * (BK + 1) + ks];
#pragma unroll
      for (int b = 0; b < NB; ++b) bv[f][b] = Br[so + ks * (T + 2) + b * 16];
    };
    frag(0);
#pragma unroll
    for (int ks = 0; ks < BK; ks += 4) {
      const int f = (ks >> 2) & 1;
      if (ks + 4 < BK) frag(ks + 4);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[f][a], bv[f][b], acc[a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Stage s is read in k-tile t while stage 1 - s receives tile t + 1; the
  // barrier after the stash orders both the stash before the next tile's
  // reads and this tile's reads before the stash that follows.  The loads of
  // tile t + 2 are issued before the products of tile t, so a load has two
  // k-tiles to arrive.
  if (nk > 0) {
    fetch(0);
    stash(lds, 0, nk == 1);
    if (nk > 1) fetch(1);
    __syncthreads();
    int t = 0;
#pragma unroll 1
    for (; t + 3 < nk; t += 2) {
      fetch(0);
      mma(0);
      stash(lds + L::kStage, 1, false);
      __syncthreads();
      fetch(1);
      mma(L::kStage);
      stash(lds, 0, false);
      __syncthreads();
    }
    // 1, 2 or 3 k-tiles are left, the last of all among them
    const int rest = nk - t;
    if (rest == 3) fetch(0);
    mma(0);
    if (rest > 1) {
      stash(lds + L::kStage, 1, rest == 2);
      __syncthreads();
      mma(L::kStage);
    }
    if (rest == 3) {
      stash(lds, 0, true);
      __syncthreads();
      mma(0);
    }
  }
  const int64_t ri = i0 + wy * W, cj = j0 + wx * W;
  if (kKind != kMul && ri + W <= Mm && cj + W <= (kKind == kNatural && g.cols < Nm ? g.cols : Nm)) {
    // whole tiles: columns 16 b + l15, natural ones by parity
    const int l15 = lane & 15, l4 = lane >> 4;
    const uint32_t rs = 8 * (uint32_t)g.sci, cs = 8 * (uint32_t)g.scj;
    const Buffer C(g.C + ri * g.sci + (kKind == kNatural ? cj / 2 : cj * g.scj));
    const uint32_t co = l4 * rs + (kKind == kNatural ? 8 * ((l15 & 1) * (uint32_t)g.split + (l15 >> 1))
                                                      : l15 * cs);
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          C.store(acc[a][b][r], co, (16 * a + 4 * r) * rs + (kKind == kNatural ? 64 * b : 16 * b * cs));
    return;
  }
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gi = i0 + wy * W + a * 16 + 4 * r + (lane >> 4);
        const int64_t gj = j0 + wx * W + b * 16 + (lane & 15);
        if (gi >= Mm || gj >= Nm) continue;
        const double v = acc[a][b][r];
        if constexpr (kKind == kNatural)
          g.C[gi * g.sci + (gj & 1) * g.split + (gj >> 1)] = gj < g.cols ? v : 0.0;
        else
          g.C[gi * g.sci + gj * g.scj] = kKind == kMul ? multiply(g, gi, gj, v) : v;
      }
}

// One edge unit in plain FP64 FMAs: latency bound, so a unit is small and issues
// its loads together; the units start first and run beside the MFMA tiles.
// (8 loads of A in flight per lane: with 16 the kernel needs more registers
// than its MFMA tiles, which costs those a wavefront per SIMD.)
// Column units: a wavefront takes R rows, lanes along k (U chunks of 128 at a
// time, R U = 8), and sums across lanes by a butterfly.  The last wavefront
// overlaps its neighbour's rows (Mm >= 32) instead of passing the end.
template <int U>
__device__ __forceinline__ void edge_columns(const GemmProb &g, int64_t i, int64_t Mm, int64_t Nm,
                                             int lane) {
  constexpr int R = 8 / U;
  const int K = (int)g.K;
  const int64_t i0 = i + R <= Mm ? i : Mm - R;
  const double *A = g.A + i0 * g.sai;
  for (int64_t j = Nm; j < g.N; ++j) {
    const double *B = g.B + j;
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
    for (int k0 = 2 * lane; k0 < K; k0 += 128 * U) {
      dbl2 a[U][R], b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + 128 * u < K ? k0 + 128 * u : k0;
        b[u].x = B[k * g.sbk];
        b[u].y = B[(k + 1) * g.sbk];
#pragma unroll
        for (int r = 0; r < R; ++r) a[u][r] = *(const dbl2 *)(A + r * g.sai + k);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + 128 * u < K) {
#pragma unroll
          for (int r = 0; r < R; ++r)
            acc[r] = fma(a[u][r].y, b[u].y, fma(a[u][r].x, b[u].x, acc[r]));
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double v = acc[r];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
      if (lane == 0) g.C[(i0 + r) * g.sci + j * g.scj] = v;
    }
  }
}

// Row units: kCols columns x (256 / kCols) parts of k, the parts' sums added in
// order.
template <int kCols>
__device__ __forceinline__ void edge_rows(const GemmProb &g, int64_t j0, int64_t Mm, double *lds) {
  constexpr int kParts = 256 / kCols;
  const int tid = threadIdx.x, part = tid / kCols;
  const int64_t j = j0 + tid % kCols, kp = g.K / kParts;  // K is a multiple of 16
  const int ne = (int)(g.M - Mm);
  const double *bp = g.B + part * kp * g.sbk + (j < g.N ? j : g.N - 1);
  const double *ap = g.A + Mm * g.sai + part * kp;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t k0 = 0; k0 < kp; k0 += 16) {
    double b[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) b[u] = bp[(k0 + u < kp ? k0 + u : k0) * g.sbk];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < ne) {
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (k0 + u < kp) acc[e] = fma(ap[e * g.sai + k0 + u], b[u], acc[e]);
      }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) lds[e * 256 + tid] = acc[e];
  __syncthreads();
  if (j >= g.N) return;
  for (int e = part; e < ne; e += kParts) {
    double v = 0.0;
#pragma unroll
    for (int u = 0; u < kParts; ++u) v += lds[e * 256 + u * kCols + tid % kCols];
    g.C[(Mm + e) * g.sci + j * g.scj] = v;
  }
}

__device__ __forceinline__ void gemm_edge(const GemmProb &g, int unit, double *lds) {
  const int64_t Mm = main_extent(g.M), Nm = main_extent(g.N);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int rows = edge_rows_per_unit(g), ncu = edge_column_units(g);
  if (unit < ncu) {
    const int64_t i0 = (int64_t)unit * rows + wid * (rows / 4);
    if (rows == 32)
      edge_columns<1>(g, i0, Mm, Nm, lane);
    else if (rows == 16)
      edge_columns<2>(g, i0, Mm, Nm, lane);
    else
      edge_columns<4>(g, i0, Mm, Nm, lane);
    return;
  }
  if (g.K > 256)
    edge_rows<16>(g, (int64_t)(unit - ncu) * 16, Mm, lds);
  else
    edge_rows<64>(g, (int64_t)(unit - ncu) * 64, Mm, lds);
}

template <int T, int kKind>
__global__ __launch_bounds__(256, 2) void k_gemm(GemmBatch batch) {
  __shared__ __align__(16) double lds[Tile<T>::kLds];
  int L = blockIdx.x;
  if (kKind == kPlain && L < batch.nedge) {
    const int per = batch.nedge / batch.count;
    const GemmProb &g = batch.p[L / per];
    if (L % per < edge_units(g)) gemm_edge(g, L % per, lds);
    return;
  }
  if (kKind == kPlain) L -= batch.nedge;
  const int nt = batch.nt, mt = batch.mt, nz = batch.count;
  int bx, by, z;
  if (batch.order == 0) {
    bx = L % nt;
    by = L / nt % mt;
    z = L / (nt * mt);
  } else if (batch.order == 2) {
    const int rem = L % (mt * nz);
    bx = L / (mt * nz);
    z = rem / mt;
    by = rem % mt;
  } else {
    const int rem = L % (nt * nz);
    by = L / (nt * nz);
    z = rem / nt;
    bx = rem % nt;
  }
  gemm_tile<T, kKind>(batch.p[z], (int64_t)by * T, (int64_t)bx * T, lds);
}

// Table-driven GEMM: workgroup g computes unit tile_map[2g + 1] of problem
// tile_map[2g]: the tile at rows 32 (u >> 16), columns 32 (u >> 1 & 0x7fff), a 32 x 32 one
// if u is odd, or edge unit -1 - u.
// Operand pointers are rebased per GemmDesc base ids.
__device__ __forceinline__ const double *rebase(const double *p, int id, char *ws, char *out,
                                                const char *in) {
  const char *at = id == 1 ? ws : id == 2 ? out : in;
  return id == 0 ? p : (const double *)(at + (intptr_t)p);
}

template <int T, int kKind>
__global__ __launch_bounds__(256, 2) void k_gemm_table(const GemmDesc *__restrict__ d,
                                                       const int *__restrict__ tile_map, char *ws,
                                                       char *out, const char *in) {
  __shared__ __align__(16) double lds[Tile<T>::kLds];
  const int k = __builtin_amdgcn_readfirstlane(tile_map[2 * blockIdx.x]);
  const int local = __builtin_amdgcn_readfirstlane(tile_map[2 * blockIdx.x + 1]);
  const GemmDesc &e = d[k];
  GemmProb g = e.p;
  g.A = as_global(rebase(g.A, e.abase, ws, out, in));
  g.B = as_global(rebase(g.B, e.bbase, ws, out, in));
  g.C = as_global((double *)rebase(g.C, e.cbase, ws, out, in));
  g.klim = as_global(g.klim);
  g.mr = as_global(g.mr);
  g.mc = as_global(g.mc);
  g.lr = as_global(g.lr);
  g.lc = as_global(g.lc);
  g.mt = as_global(g.mt);
  if (kKind == kPlain && local < 0) {
    gemm_edge(g, -1 - local, lds);
    return;
  }
  const int64_t i0 = (local >> 16) * 32, j0 = ((local >> 1) & 0x7fff) * 32;
  if (T == 32 || (local & 1))
    gemm_tile<32, kKind>(g, i0, j0, lds);
  else
    gemm_tile<64, kKind>(g, i0, j0, lds);
}

}  // namespace

namespace {

int kind_of(const GemmProb &q) {
  return q.split > 0 ? kNatural : q.mr != nullptr || q.mt != nullptr ? kMul : kPlain;
}

// Tile of a set of problems.  32 x 32 where 64 x 64 tiles would be too few for
// the 256 compute units to hide a workgroup's serial chain of k-tiles (measured
// per stage of a square solve, 64 / 32: n = 200 9 / 6 us, 515 17 / 11, 1024 30 /
// 27, 1700 125 / 110; n = 2048, 1024 tiles, 157 / 160; n = 3000 437 / 533), or
// where they would cover much more than the outputs (blocks of 96: the n = 185
// cube's per-slice products 70 / 52 us); a 32 x 32 tile reads its operands
// twice as often, about 15 % of its time.
template <typename Get>
int pick_tile(int64_t count, Get get) {
  double t64 = 0.0, t32 = 0.0;
  for (int64_t i = 0; i < count; ++i) {
    const GemmProb &q = get(i);
    const int64_t m = main_extent(q.M), n = main_extent(q.N);
    t64 += (double)((m + 63) / 64) * (double)((n + 63) / 64);
    t32 += (double)((m + 31) / 32) * (double)((n + 31) / 32);
  }
  return t64 <= 800.0 || 1.15 * t32 < 4.0 * t64 ? 32 : 64;
}

}  // namespace

bool gemm_operands_ok(const GemmProb &q) {
  const int kind = kind_of(q);
  // 32-bit byte offsets within a tile
  if (64 * q.sai >= (int64_t)1 << 28 || 64 * q.sbk + q.N >= (int64_t)1 << 28 ||
      64 * (q.sci + q.scj) >= (int64_t)1 << 28)
    return false;
  if (q.sak != 1 || q.sbj != 1 || q.K % 16 != 0 || (q.sai & 1) || ((uintptr_t)q.A & 15) || q.M < 1 ||
      q.N < 1)
    return false;
  if (kind != kPlain && (main_extent(q.M) != q.M || main_extent(q.N) != q.N)) return false;
  if (kind == kNatural)
    return q.mr == nullptr && q.mt == nullptr && q.cols >= 2 && q.cols <= q.N && q.N % 2 == 0 &&
           q.krows >= 1 && q.krows <= q.K && !((uintptr_t)q.B & 7);
  return !(q.sbk & 1) && !((uintptr_t)q.B & 15);
}

hipError_t launch_gemm_table(const GemmTable &t, const GemmDesc *d, const int *tile_map,
                             const double *in, char *ws, char *out, hipStream_t st, hipEvent_t ev0,
                             hipEvent_t ev1) {
  if (t.units <= 0) return hipSuccess;
  auto kern = t.kind == kMul ? k_gemm_table<64, kMul>
                             : t.kind == kNatural ? k_gemm_table<64, kNatural> : k_gemm_table<64, kPlain>;
  if (t.T == 32)
    kern = t.kind == kMul ? k_gemm_table<32, kMul>
                          : t.kind == kNatural ? k_gemm_table<32, kNatural> : k_gemm_table<32, kPlain>;
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL(kern, dim3((unsigned)t.units), dim3(256), 0, st, ev0, ev1, 0, d, tile_map,
                          ws, out, (const char *)in);
  else
    hipLaunchKernelGGL(kern, dim3((unsigned)t.units), dim3(256), 0, st, d, tile_map, ws, out,
                       (const char *)in);
  return hipGetLastError();
}

bool gemm_table(std::vector<GemmDesc> &tab, GemmTable &t, std::vector<int> &map) {
  map.clear();
  t = GemmTable{};
  if (tab.empty()) return true;
  t.kind = kind_of(tab[0].p);
  t.T = pick_tile((int64_t)tab.size(), [&](int64_t i) -> const GemmProb & { return tab[(size_t)i].p; });
  // Problem by problem, the one with the longest tiles first (workgroups start in
  // id order, so the short tiles fill the tail, and the tiles in flight share
  // their problem's operands in the caches: ordered by k-range across the 64
  // blocks of 16 solves at n = 2048, every column of tiles read them anew);
  // within a problem its edge units, then its tiles, longest k-range first.
  // Tables of 64 x 64 tiles cover the last 32 rows or columns of a problem (past a
  // multiple of 64) by 32 x 32 ones: a batch's blocks have any multiple of 16 (256
  // problems of n = 32 .. 1024: 5.27 -> 5.14 ms).
  struct Unit {
    int64_t work;
    int local;
  };
  std::vector<std::vector<Unit>> units(tab.size());
  std::vector<int> by((size_t)tab.size());
  for (size_t k = 0; k < tab.size(); ++k) {
    const GemmProb &q = tab[k].p;
    by[k] = (int)k;
    if (!gemm_operands_ok(q) || kind_of(q) != t.kind) return false;
    const int64_t M = main_extent(q.M), N = main_extent(q.N);
    if (M >= (int64_t)32 << 15 || N >= (int64_t)32 << 15) return false;
    std::vector<Unit> &u = units[k];
    auto add = [&](int64_t i0, int64_t j0, int T) {
      if (i0 >= M || j0 >= N) return;
      u.push_back(Unit{tile_kend(q, q.klim_host, i0, j0) * T * T, (int)((i0 / 32) << 16 | (j0 / 32) << 1 | (T < t.T ? 1 : 0))});
    };
    for (int64_t i0 = 0; i0 < M; i0 += t.T)
      for (int64_t j0 = 0; j0 < N; j0 += t.T) {
        if (t.T == 32 || (M - i0 > 32 && N - j0 > 32)) {
          add(i0, j0, t.T);
        } else {
          for (int c = 0; c < 4; ++c) add(i0 + (c >> 1) * 32, j0 + (c & 1) * 32, 32);
        }
      }
    std::stable_sort(u.begin(), u.end(), [](const Unit &a, const Unit &b) { return a.work > b.work; });
    for (int i = 0; t.kind == kPlain && i < edge_units(q); ++i) u.insert(u.begin(), Unit{0, -1 - i});
    t.units += (int)u.size();
  }
  std::stable_sort(by.begin(), by.end(), [&](int a, int b) { return tab[a].p.K > tab[b].p.K; });
  map.reserve(2 * (size_t)t.units);
  for (int k : by)
    for (const Unit &u : units[(size_t)k]) {
      map.push_back(k);
      map.push_back(u.local);
    }
  return true;
}

hipError_t launch_gemm(const GemmProb *probs, int count, hipStream_t st, hipEvent_t ev0,
                       hipEvent_t ev1) {
  if (count <= 0) return hipSuccess;
  if (count > 4) return hipErrorInvalidValue;
  const int T = pick_tile(count, [&](int64_t i) -> const GemmProb & { return probs[i]; });
  GemmBatch b{};
  int64_t mt = 1, nt = 1, edge = 0;
  const GemmProb &f = probs[0];
  const int kind = kind_of(f);
  bool same = true;
  for (int i = 0; i < count; ++i) {
    const GemmProb &q = probs[i];
    // contiguous operands, 16-byte aligned, K padded to the k-tile
    if (!gemm_operands_ok(q)) return hipErrorInvalidValue;
    if (kind_of(q) != kind) return hipErrorInvalidValue;
    b.p[i] = q;
    mt = std::max(mt, (main_extent(q.M) + T - 1) / T);
    nt = std::max(nt, (main_extent(q.N) + T - 1) / T);
    if (kind == kPlain) edge = std::max(edge, (int64_t)edge_units(q));
    same = same && q.kside == f.kside;
  }
  // longest k-range first: the limits fall
  if (same) b.order = f.kside;
  b.count = count;
  b.mt = (int)mt;
  b.nt = (int)nt;
  b.nedge = (int)(edge * count);
  const int64_t wgs = (edge + mt * nt) * count;
  if (wgs > (int64_t)1 << 30) return hipErrorInvalidValue;
  auto kern = kind == kMul ? k_gemm<64, kMul> : kind == kNatural ? k_gemm<64, kNatural> : k_gemm<64, kPlain>;
  if (T == 32)
    kern = kind == kMul ? k_gemm<32, kMul> : kind == kNatural ? k_gemm<32, kNatural> : k_gemm<32, kPlain>;
  const dim3 grid((unsigned)wgs);
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL(kern, grid, dim3(256), 0, st, ev0, ev1, 0, b);
  else
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, b);
  return hipGetLastError();
}

}  // namespace fps
