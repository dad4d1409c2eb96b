// gfx950 chains of FP64 products on one LDS-resident block.
//
// The eigenbasis solves multiply each parity block by a matrix on its right
// and one on its left, twice.  For blocks of at most 128 x 128 the block between
// two products fits a workgroup's LDS, so a chain of products goes through HBM
// once: cube slices (x and y maps), cube strips (both z maps with the multiplier in
// between), cylinder modes (z and r maps) and whole square solves up to n = 128.
// Against one product launch per axis: cube n = 256 775 -> 490 us, n = 185 297 ->
// 180 us, n = 128 111 -> 53 us, cylinder 256 x 256 1031 -> 562 us (its z map then
// also ran over the r parity that a mode has not), square n = 64 22.6 -> 14.2 us.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device.hpp"
#include "kernels.hpp"

namespace fps {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef double dbl2 __attribute__((ext_vector_type(2)));
typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));

// Square solves: block of up to S x S (S = 32 NB), NB^2 wavefronts, each 32 x 32 of the output
// as 2 x 2 MFMA blocks (v_mfma_f64_16x16x4f64: lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16], accumulator register r holds C[4r + l / 16][l % 16]).
// X lives in LDS with two columns of padding: 16 rows at one k then fall on
// distinct banks.  The other operand is read from global memory in its
// transposed form [k][row or column], 128 contiguous bytes per k.
// 1 or 2 output rows or columns past S (the output maps have m + 1 or m + 2) are
// 16-wide extra tiles, a tenth of the products more: wavefront w takes the
// extra tiles w, w + NB^2, ...
template <int NB>
struct Chain {
  static constexpr int S = 32 * NB, P = S + 2, kThreads = 64 * NB * NB, kLds = S * P + 16;
  static constexpr int kWaves = NB * NB, kSlots = NB == 2 ? 3 : 2;  // extra tiles per wavefront
};

struct Lane {
  int l15, l4, wave, wy, wx;
};

// acc += X[r0 .. r0 + 16 RB)[0 .. K) W[0 .. K)[c0 .. c0 + 16 CB): X from LDS as the
// left operand, W [k][column] from global memory, loaded 4 k-steps ahead.
template <int P, int RB, int CB>
__device__ __forceinline__ void mul_right(const double *X, const double *__restrict__ W, int ldw,
                                          int K, int r0, int c0, const Lane &l, dbl4 (&acc)[RB][CB]) {
  const double *xa = X + (r0 + l.l15) * P + l.l4;
  const uint32_t wo = l.l4 * ldw + l.l15;  // the lane's part of the address
  const double *wu = W + c0;               // the wavefront's
  double b[4][CB];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int c = 0; c < CB; ++c) b[u][c] = (wu + (4 * u) * ldw + 16 * c)[wo];
#pragma unroll 1
  for (int ks = 0; ks < K; ks += 16) {
    const int nx = ks + 16 < K ? ks + 16 : ks;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double a[RB], bv[CB];
#pragma unroll
      for (int r = 0; r < RB; ++r) a[r] = xa[r * 16 * P + ks + 4 * u];
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        bv[c] = b[u][c];
        b[u][c] = (wu + (nx + 4 * u) * ldw + 16 * c)[wo];
      }
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CB; ++c)
          acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], bv[c], acc[r][c], 0, 0, 0);
    }
  }
}

// acc += W^T[r0 ..)[0 .. K) X[0 .. K)[c0 ..): W [k][row] from global memory as the left
// operand, X from LDS.
template <int P, int RB, int CB>
__device__ __forceinline__ void mul_left(const double *X, const double *__restrict__ W, int ldw,
                                         int K, int r0, int c0, const Lane &l, dbl4 (&acc)[RB][CB]) {
  const uint32_t wo = l.l4 * ldw + l.l15;
  const double *wu = W + r0;
  const double *xb = X + l.l4 * P + c0 + l.l15;
  double a[4][RB];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int r = 0; r < RB; ++r) a[u][r] = (wu + (4 * u) * ldw + 16 * r)[wo];
#pragma unroll 1
  for (int ks = 0; ks < K; ks += 16) {
    const int nx = ks + 16 < K ? ks + 16 : ks;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double av[RB], b[CB];
#pragma unroll
      for (int c = 0; c < CB; ++c) b[c] = xb[(ks + 4 * u) * P + 16 * c];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        av[r] = a[u][r];
        a[u][r] = (wu + (nx + 4 * u) * ldw + 16 * r)[wo];
      }
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < CB; ++c)
          acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[r], b[c], acc[r][c], 0, 0, 0);
    }
  }
}

// The eigenbasis multiplier of entry (i, j), as in the product kernels.
__device__ __forceinline__ double multiplier(const ChainDesc &d, int i, int j, double v) {
  if (d.lr != nullptr) {
    const double *r = d.lr + 4 * i, *c = d.lc + 4 * j;
    v -= fma(r[3], c[3], fma(r[2], c[2], fma(r[1], c[1], r[0] * c[0])));
  }
  const dbl2 r = *(const dbl2 *)(d.mr + 2 * i), c = *(const dbl2 *)(d.mc + 2 * j);
  return v * (fma(-r.y, c.y, 1.0) / (r.x + c.x));
}

// One product step of the chain on X: right (X W) or left (W^T X), with rows x
// cols outputs; the result goes to `put(r, c, value)`, for this lane's row r + l4
// and column c + l15, after every wavefront has read X.
template <int NB, bool kLeft, typename Put>
__device__ __forceinline__ void step(double *X, const double *W, int ldw, int K, int rows, int cols,
                                     const Lane &l, Put put) {
  using C = Chain<NB>;
  dbl4 acc[2][2], ext[C::kSlots];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = dbl4{0.0, 0.0, 0.0, 0.0};
  const int r0 = l.wy * 32, c0 = l.wx * 32;
  const bool mine = r0 < rows && c0 < cols;  // uniform per wavefront
  if (mine) {
    if constexpr (kLeft)
      mul_left<C::P, 2, 2>(X, W, ldw, K, r0, c0, l, acc);
    else
      mul_right<C::P, 2, 2>(X, W, ldw, K, r0, c0, l, acc);
  }
  // extra tiles: columns past S (one per 16 rows), rows past S (one per 16
  // columns; left products only), and the corner
  const int nec = cols > C::S ? 2 * NB : 0, ner = rows > C::S ? 2 * NB : 0;
  const int next = nec + ner + (nec && ner ? 1 : 0);
  auto extra = [&](int t, int *r, int *c) {
    *r = t < nec ? 16 * t : C::S;
    *c = t < nec ? C::S : t < nec + ner ? 16 * (t - nec) : C::S;
  };
#pragma unroll
  for (int s = 0; s < C::kSlots; ++s) {
    const int t = l.wave + s * C::kWaves;
    ext[s] = dbl4{0.0, 0.0, 0.0, 0.0};
    if (t < next) {
      int r, c;
      extra(t, &r, &c);
      dbl4 e[1][1] = {{dbl4{0.0, 0.0, 0.0, 0.0}}};
      if constexpr (kLeft)
        mul_left<C::P, 1, 1>(X, W, ldw, K, r, c, l, e);
      else
        mul_right<C::P, 1, 1>(X, W, ldw, K, r, c, l, e);
      ext[s] = e[0][0];
    }
  }
  __syncthreads();
  if (mine) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          put(r0 + a * 16 + 4 * r, c0 + b * 16, acc[a][b][r]);
  }
#pragma unroll
  for (int s = 0; s < C::kSlots; ++s) {
    const int t = l.wave + s * C::kWaves;
    if (t < next) {
      int er, ec;
      extra(t, &er, &ec);
#pragma unroll
      for (int r = 0; r < 4; ++r) put(er + 4 * r, ec, ext[s][r]);
    }
  }
}

// Where the offsets of a table's blocks start (unused for blocks given by value).
struct Bases {
  const char *in;
  char *ws, *out;
};

template <bool kTable>
__device__ __forceinline__ const double *rebase(const double *p, int id, const Bases &u) {
  if constexpr (!kTable) return p;
  const char *at = id == 1 ? u.ws : id == 2 ? u.in : u.out;
  return as_global(id == 0 ? p : (const double *)(at + (intptr_t)p));
}

// A table's descriptor with its pointers marked global.
__device__ __forceinline__ ChainDesc table_entry(const ChainDesc &d) {
  ChainDesc e = d;
#pragma unroll
  for (int i = 0; i < 4; ++i) e.m[i] = as_global(e.m[i]);
  e.mr = as_global(e.mr);
  e.mc = as_global(e.mc);
  e.lr = as_global(e.lr);
  e.lc = as_global(e.lc);
  e.mt = as_global(e.mt);
  return e;
}

// p[off] with the lanes' part of the address in bytes, 32 bits beside a uniform base.
__device__ __forceinline__ double at(const double *p, uint32_t bytes) {
  return *(const double *)((const char *)p + bytes);
}
__device__ __forceinline__ dbl2 at2(const double *p, uint32_t bytes) {
  return *(const dbl2 *)((const char *)p + bytes);
}

// A whole square solve: right, left, multiplier, right, left.
template <int NB, bool kTable>
__device__ __forceinline__ void solve_block(const ChainDesc &e, const Bases &u) {
  using C = Chain<NB>;
  __shared__ __align__(16) double X[C::kLds];
  const int tid = threadIdx.x;
  Lane l;
  l.l15 = tid & 15;
  l.l4 = (tid & 63) >> 4;
  l.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  l.wy = l.wave / NB;
  l.wx = l.wave % NB;
  static_assert(C::S * C::S == 16 * C::kThreads, "one block is 16 elements per thread");
  // thread t holds column t % S of rows t / S + 2 NB i
  const int tr = tid / C::S, tc = tid % C::S;
  const double *in = rebase<kTable>(e.in, e.ibase, u);
  const uint32_t off = (uint32_t)(tr * (int)e.in_rs + tc * e.in_cs);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int r = i * 2 * NB;
    X[(r + tr) * C::P + tc] = tr + r < e.in_r && tc < e.in_c ? (in + r * e.in_rs)[off] : 0.0;
  }
  __syncthreads();
  double *Xl = X + l.l4 * C::P + l.l15;  // this lane's entry of a 4 x 16 patch
  auto keep = [&](int r, int c, double x) {
    if (r + 4 <= C::S && c + l.l15 < C::P) Xl[r * C::P + c] = x;
  };
  auto keep_mul = [&](int r, int c, double x) {
    const int i = r + l.l4, j = c + l.l15;
    if (r + 4 <= C::S && j < C::S)
      Xl[r * C::P + c] = i < e.n[1] && j < e.n[0] ? multiplier(e, i, j, x) : 0.0;
  };
  double *out = (double *)rebase<kTable>(e.out, e.obase, u);
  const uint32_t oo = (uint32_t)(l.l4 * (int)e.out_rs + l.l15 * e.out_cs);
  auto store = [&](int r, int c, double x) {
    if (r + l.l4 < e.out_r && c + l.l15 < e.out_c)
      (out + r * e.out_rs + (int64_t)c * e.out_cs)[oo] = x;
  };
  step<NB, false>(X, e.m[0], e.ld[0], e.k[0], e.k[1], e.n[0], l, keep);
  __syncthreads();
  step<NB, true>(X, e.m[1], e.ld[1], e.k[1], e.n[1], e.n[0], l, keep_mul);
  __syncthreads();
  step<NB, false>(X, e.m[2], e.ld[2], e.k[2], e.k[3], e.n[2], l, keep);
  __syncthreads();
  step<NB, true>(X, e.m[3], e.ld[3], e.k[3], e.n[3], e.n[2], l, store);
}

template <int NB>
__global__ __launch_bounds__(Chain<NB>::kThreads, NB == 3 ? 5 : 4) void k_chain_table(
    const ChainDesc *__restrict__ d, Bases u) {
  solve_block<NB, true>(table_entry(d[blockIdx.x]), u);
}

struct ChainBatch {
  ChainDesc d[4];
};

template <int NB>
__global__ __launch_bounds__(Chain<NB>::kThreads, NB == 3 ? 5 : 4) void k_chain(ChainBatch b) {
  solve_block<NB, false>(b.d[blockIdx.x], Bases{});
}

// Slabs and strips: two products of one block of up to S x S, S = 32 NB, split so
// that four or five workgroups share a compute unit and one's loads and stores
// run under another's products.  The first product takes both operands straight
// from global memory (X in rows of 16 columns, W transposed), so X needs no LDS;
// its result is the only thing kept there.
//   slab:  rows r0 .. r0 + R of W1^T X, then times W0: R = 32 W rows, all columns
//   strip: C = 32 W columns of W1^T X, multiplier, then W3^T times it: all rows
// Wavefronts of 32 x 32 (2 x 2 MFMA blocks).  The 1 or 2 rows and columns past S ride
// along in some of them: a fused multiply-add of the operands that the matrix
// instructions have just read, summed over the lanes at the end.
// Bound by the matrix unit: 70 % busy at S = 128 (cube n = 256, three launches of 8.6
// GFLOP: 53 TFLOP/s).  W = 1 at S = 128 and 96: 64 rows or columns (two workgroups a
// unit) 523 us, 32 (four) 490, though W is read twice as often from L2; whole
// blocks (one, its input staged in LDS) 678; S = 96: 32 180 us, 96 225.  S = 64: two
// rows of wavefronts 53 us, one 54.
template <int NB, int W>
struct Unit {
  static constexpr int S = 32 * NB, E = 32 * W;  // S and R (C)
  static constexpr int kThreads = 64 * NB * W;
  static constexpr int P = S + 2;  // slab: row stride of the E x S intermediate
};

// Sum over the four lanes (l4) that share a row or column.
__device__ __forceinline__ dbl2 sum_l4(dbl2 v) {
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    v.x += __shfl_xor(v.x, o);
    v.y += __shfl_xor(v.y, o);
  }
  return v;
}

// Where the MFMA rows / columns 16 i + j of a wavefront's 32 lie: interleaved, at
// 2 j + i, so that a lane's two are one 16-byte load (W; X if its columns are
// contiguous).  The L1 serves 32 bytes a cycle whatever the width asked for, and
// the products need 24 .. 48 of its cycles in every 64 of the matrix unit's (strips
// 246 -> 208 us a launch).

// acc = W^T[r0 .. r0 + 32)[0 .. K) X[0 .. K)[c0 .. c0 + 32), W [k][row], X [k][column],
// zero beyond in_r, in_c; K a multiple of 32.  Rows interleaved, columns too if kPair.
// X comes from HBM: 8 k-steps (2048 MFMA cycles of the SIMD's wavefronts) ahead, W
// from the caches: 4.  kExt: ext[c] = the rows S, S + 1 of W^T X in this lane's two
// columns (all four lanes of a column hold them).
template <bool kPair, bool kExt>
__device__ __forceinline__ void mul_stream(const double *__restrict__ W, int ldw, int S,
                                           const double *__restrict__ X, const ChainDesc &e, int K,
                                           int r0, int c0, const Lane &l, dbl4 (&acc)[2][2],
                                           dbl2 (&ext)[2]) {
  const uint32_t wo = 8 * (l.l4 * ldw + 2 * l.l15);
  const double *wu = W + r0;
  const int rs = (int)e.in_rs, cs = e.in_cs;
  // the last k-step with data, and its rows: later ones read it again (masked)
  const int last = (e.in_r - 1) & ~3;
  bool cok[2];
  uint32_t xo[2], xl[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int col = c0 + (kPair ? 2 * l.l15 + c : 16 * c + l.l15);
    cok[c] = col < e.in_c;
    // (a pair may end one past in_c, in the padding)
    const int cc = (cok[c] ? col : kPair ? (e.in_c - 1) & ~1 : e.in_c - 1) * cs;
    xo[c] = 8 * (l.l4 * rs + cc);
    xl[c] = 8 * (min(l.l4, e.in_r - 1 - last) * rs + cc);
  }
  dbl2 a[4], b[8], x[4];
  const uint32_t xwo = 8 * (l.l4 * ldw);
  ext[0] = ext[1] = dbl2{0.0, 0.0};
  auto load_a = [&](int u, int k) {
    const int kk = (k < K ? k : K - 4) * ldw;
    a[u] = at2(wu + kk, wo);
    if constexpr (kExt) x[u] = at2(W + S + kk, xwo);
  };
  auto load_b = [&](int u, int k) {
    const bool z = k >= last;
    const double *p = X + (z ? last : k) * rs;
    if constexpr (kPair)
      b[u] = *(const dbl2u *)((const char *)p + (z ? xl[0] : xo[0]));
    else
      b[u] = dbl2{at(p, z ? xl[0] : xo[0]), at(p, z ? xl[1] : xo[1])};
  };
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    if (u < 4) load_a(u, 4 * u);
    load_b(u, 4 * u);
    __builtin_amdgcn_sched_barrier(0);  // in the order of their use, for the waits
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[r][c] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int ks = 0; ks < K; ks += 32) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = ks + 4 * u;
      const bool rok = k + l.l4 < e.in_r;
      const double bv[2] = {rok && cok[0] ? b[u].x : 0.0, rok && cok[1] ? b[u].y : 0.0};
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u & 3][r], bv[c], acc[r][c], 0, 0, 0);
      if constexpr (kExt) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          ext[c].x = fma(x[u & 3].x, bv[c], ext[c].x);
          ext[c].y = fma(x[u & 3].y, bv[c], ext[c].y);
        }
      }
      // the next loads go into the registers just read; the barrier keeps them
      // from moving next to their use
      __builtin_amdgcn_sched_barrier(0);
      load_a(u & 3, k + 16);
      load_b(u, k + 32);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (kExt)
    for (int c = 0; c < 2; ++c) ext[c] = sum_l4(ext[c]);
}

// The second product's results of one wavefront: 2 x 2 MFMA blocks, and of its
// lanes the extra ones: w[i] = entries S, S + 1 on W's side of T's row or column 16 i
// + l15, t[i] = T's two extra rows times W's column i, tw[i] = the corner, row i.
struct Kept {
  dbl4 acc[2][2];
  dbl2 w[2], t[2], tw[2];
};

// The product of the intermediate T in LDS and W [k][..] from global memory, 4
// k-steps ahead: kLeft W^T T, else T W.  t[.]: this lane's entries of T at k = 0, ts
// their stride per k; w0 the first row (kLeft) or column of W, interleaved if kPair.
// kExtW: also with W's entries S, S + 1.  kExtT (T W only): also T's extra rows, from
// te on (P apart).
template <bool kLeft, bool kPair, bool kExtW, bool kExtT>
__device__ __forceinline__ void mul_kept(const double *T, const int (&t)[2], int ts,
                                         const double *__restrict__ W, int ldw, int S, int K, int w0,
                                         const double *te, int P, const Lane &l, Kept &o) {
  const uint32_t wo = 8 * (l.l4 * ldw + (kPair ? 2 : 1) * l.l15), xwo = 8 * (l.l4 * ldw);
  dbl2 w[4], x[4];
  auto load = [&](int u, int k) {
    const double *p = W + w0 + k * ldw;
    if constexpr (kPair)
      w[u] = at2(p, wo);
    else
      w[u] = dbl2{at(p, wo), at(p + 16, wo)};
    if constexpr (kExtW) x[u] = at2(W + S + k * ldw, xwo);
  };
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    load(u, 4 * u);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();  // T is complete
#pragma unroll
  for (int r = 0; r < 2; ++r) {
#pragma unroll
    for (int c = 0; c < 2; ++c) o.acc[r][c] = dbl4{0.0, 0.0, 0.0, 0.0};
    o.w[r] = o.t[r] = o.tw[r] = dbl2{0.0, 0.0};
  }
#pragma unroll 1
  for (int ks = 0; ks < K; ks += 16) {
    const int nx = ks + 16 < K ? ks + 16 : ks;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double tv[2], ev[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        tv[r] = T[t[r] + (ks + 4 * u) * ts];
        if constexpr (kExtT) ev[r] = te[r * P + l.l4 + ks + 4 * u];
      }
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          o.acc[r][c] = kLeft ? __builtin_amdgcn_mfma_f64_16x16x4f64(w[u][r], tv[c], o.acc[r][c], 0, 0, 0)
                              : __builtin_amdgcn_mfma_f64_16x16x4f64(tv[r], w[u][c], o.acc[r][c], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if constexpr (kExtW) o.w[r] = dbl2{fma(tv[r], x[u].x, o.w[r].x), fma(tv[r], x[u].y, o.w[r].y)};
        if constexpr (kExtT) o.t[r] = dbl2{fma(ev[0], w[u][r], o.t[r].x), fma(ev[1], w[u][r], o.t[r].y)};
        if constexpr (kExtW && kExtT)
          o.tw[r] = dbl2{fma(ev[r], x[u].x, o.tw[r].x), fma(ev[r], x[u].y, o.tw[r].y)};
      }
      __builtin_amdgcn_sched_barrier(0);
      load(u, nx + 4 * u);
    }
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    if constexpr (kExtW) o.w[r] = sum_l4(o.w[r]);
    if constexpr (kExtT) o.t[r] = sum_l4(o.t[r]);
    if constexpr (kExtW && kExtT) o.tw[r] = sum_l4(o.tw[r]);
  }
}

// One result element; zoff: the zero that goes with it (slabs).
__device__ __forceinline__ void store_one(const ChainDesc &e, double *out, int r, int c, double x) {
  if (r < e.out_r && c < e.out_c) {
    double *o = out + r * e.out_rs + (int64_t)c * e.out_cs;
    *o = x;
    if (e.zoff != 0) o[e.zoff] = 0.0;
  }
}

// kOut: the input's columns are contiguous and the output's 2 apart, with 1 or 2 rows
// and columns past S (else the other way round, and none).
template <int NB, int W, bool kOut>
__global__ __launch_bounds__((Unit<NB, W>::kThreads), 4) void k_slab(const ChainDesc *__restrict__ d,
                                                                     Bases u) {
  using C = Unit<NB, W>;
  __shared__ __align__(16) double T[(C::E + (kOut ? 2 : 0)) * C::P];
  const ChainDesc e = table_entry(d[blockIdx.x]);
  const int tid = threadIdx.x;
  Lane l;
  l.l15 = tid & 15;
  l.l4 = (tid & 63) >> 4;
  l.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  l.wy = l.wave / NB;
  l.wx = l.wave % NB;
  const double *X = rebase<true>(e.in, e.ibase, u);
  double *out = (double *)rebase<true>(e.out, e.obase, u);
  const int r0 = e.r0 + 32 * l.wy, c0 = 32 * l.wx;
  // extra rows: the block's last unit, its first wavefronts
  const bool rows = kOut && e.n[1] > C::S && e.r0 + C::E == C::S && l.wy == 0;
  Kept o;
  if (r0 < e.n[1] && c0 < e.k[0]) {
    dbl2 ext[2];
    double *t = T + c0 + (kOut ? 2 : 1) * l.l15;
    if (rows) {
      mul_stream<kOut, kOut>(e.m[1], e.ld[1], C::S, X, e, e.k[1], r0, c0, l, o.acc, ext);
      if (l.l4 == 0)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          t[C::E * C::P + (kOut ? 1 : 16) * b] = ext[b].x;
          t[(C::E + 1) * C::P + (kOut ? 1 : 16) * b] = ext[b].y;
        }
    } else {
      mul_stream<kOut, false>(e.m[1], e.ld[1], C::S, X, e, e.k[1], r0, c0, l, o.acc, ext);
    }
    t += (32 * l.wy + 2 * l.l4) * C::P;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) t[(8 * r + a) * C::P + (kOut ? 1 : 16) * b] = o.acc[a][b][r];
  }
  // every wavefront meets one barrier: here, or behind its first loads of W
  if (r0 >= e.n[1] || c0 >= e.n[0]) {
    __syncthreads();
    return;
  }
  const int t[2] = {(32 * l.wy + l.l15) * C::P + l.l4, (32 * l.wy + 16 + l.l15) * C::P + l.l4};
  const bool cols = kOut && e.n[0] > C::S && l.wx == 0;
  auto second = [&](auto w, auto t2) {
    mul_kept<false, !kOut, decltype(w)::value, decltype(t2)::value>(
        T, t, 1, e.m[0], e.ld[0], C::S, e.k[0], c0, T + C::E * C::P, C::P, l, o);
  };
  using No = std::false_type;
  using Ext = std::integral_constant<bool, kOut>;
  if (cols)
    rows ? second(Ext{}, Ext{}) : second(Ext{}, No{});
  else
    rows ? second(No{}, Ext{}) : second(No{}, No{});
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = r0 + 16 * a + 4 * r + l.l4;
      if constexpr (kOut) {
        store_one(e, out, i, c0 + l.l15, o.acc[a][0][r]);
        store_one(e, out, i, c0 + 16 + l.l15, o.acc[a][1][r]);
      } else {  // out_c is even, out_cs 1
        const int j = c0 + 2 * l.l15;
        if (i < e.out_r && j < e.out_c)
          *(dbl2u *)(out + i * e.out_rs + j) = dbl2{o.acc[a][0][r], o.acc[a][1][r]};
      }
    }
  if constexpr (kOut) {
    // lanes l4 = 0, 1 hold the two extra rows or columns each
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      if (l.l4 < 2 && cols)
        store_one(e, out, r0 + 16 * a + l.l15, C::S + l.l4, l.l4 ? o.w[a].y : o.w[a].x);
      if (l.l4 < 2 && rows)
        store_one(e, out, C::S + l.l4, c0 + 16 * a + l.l15, l.l4 ? o.t[a].y : o.t[a].x);
      if (l.l4 < 2 && l.l15 == 0 && cols && rows)
        store_one(e, out, C::S + a, C::S + l.l4, l.l4 ? o.tw[a].y : o.tw[a].x);
    }
  }
}

template <int NB, int W>
__global__ __launch_bounds__((Unit<NB, W>::kThreads), 4) void k_strip(const ChainDesc *__restrict__ d,
                                                                      Bases u) {
  using C = Unit<NB, W>;
  // rows of C::E columns; in odd rows the two halves of every 32 columns trade
  // places, so that two rows of 16 read at once fall on distinct banks
  __shared__ __align__(16) double T[C::S * C::E];
  const ChainDesc e = table_entry(d[blockIdx.x]);
  const int tid = threadIdx.x;
  Lane l;
  l.l15 = tid & 15;
  l.l4 = (tid & 63) >> 4;
  l.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  l.wy = l.wave / W;
  l.wx = l.wave % W;
  const double *X = rebase<true>(e.in, e.ibase, u);
  double *out = (double *)rebase<true>(e.out, e.obase, u);
  const int r0 = 32 * l.wy, c0 = 32 * l.wx, odd = l.l4 & 1;
  Kept o;
  if (r0 < e.k[3]) {
    dbl2 ext[2];
    mul_stream<true, false>(e.m[1], e.ld[1], C::S, X, e, e.k[1], r0, c0, l, o.acc, ext);
    const int j = c0 + 2 * l.l15;  // columns j, j + 1 (in_c is even)
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 8 * r + 2 * l.l4 + a;
        const dbl2 f = i < e.n[1] && j < e.in_c ? *(const dbl2 *)(e.mt + i * e.mt_rs + j) : dbl2{0.0, 0.0};
        *(dbl2 *)(T + i * C::E + (j ^ (a << 4))) = dbl2{o.acc[a][0][r] * f.x, o.acc[a][1][r] * f.y};
      }
  }
  if (r0 >= e.n[3]) {
    __syncthreads();
    return;
  }
  const int t[2] = {l.l4 * C::E + c0 + 16 * odd + l.l15, l.l4 * C::E + c0 + 16 * (1 - odd) + l.l15};
  const bool rows = e.n[3] > C::S && l.wy == 0;
  if (rows)
    mul_kept<true, true, true, false>(T, t, C::E, e.m[3], e.ld[3], C::S, e.k[3], r0, T, 0, l, o);
  else
    mul_kept<true, true, false, false>(T, t, C::E, e.m[3], e.ld[3], C::S, e.k[3], r0, T, 0, l, o);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        store_one(e, out, r0 + 8 * r + 2 * l.l4 + a, c0 + 16 * b + l.l15, o.acc[a][b][r]);
  if (rows && l.l4 < 2)
#pragma unroll
    for (int a = 0; a < 2; ++a)
      store_one(e, out, C::S + l.l4, c0 + 16 * a + l.l15, l.l4 ? o.w[a].y : o.w[a].x);
}

template <typename K, typename... A>
hipError_t run(K kern, unsigned grid, unsigned block, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1,
               A... args) {
  if (ev0 != nullptr)
    hipExtLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, st, ev0, ev1, 0, args...);
  else
    hipLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, st, args...);
  return hipGetLastError();
}

}  // namespace

bool chain_ok(const ChainDesc &d, int nb, int mode) {
  const int S = 32 * nb;
  const int step = mode == 1 ? 16 : 32;
  auto mat = [&](int i, int most) {
    return d.m[i] != nullptr && d.k[i] >= step && d.k[i] <= S && d.k[i] % step == 0 && d.n[i] >= 1 &&
           d.n[i] <= most && d.ld[i] >= (d.n[i] > S ? S + 16 : (d.n[i] + 31) / 32 * 32);
  };
  // the lanes' address parts are 32-bit
  if (S * d.in_rs >= (int64_t)1 << 31 || 16 * d.out_rs >= (int64_t)1 << 31) return false;
  if (nb < 2 || nb > 4 || d.in_r > S || d.in_c > S || d.in_r < 1 || d.in_c < 1) return false;
  if (mode == 0 ? d.in_cs != 2 || d.out_cs != 1 || d.out_c % 2 || d.out_rs % 2 || d.zoff != 0
                : mode == 3 ? d.in_cs != 1 || d.out_cs != 2
                            : mode == 2 && (d.in_cs != 1 || d.out_cs != 1 || d.in_c % 2 || d.mt_rs % 2))
    return false;
  if (mode == 0 || mode == 3)
    return mat(0, S + 2) && mat(1, S + 2) && d.in_r <= d.k[1] && d.in_c <= d.k[0] && d.r0 >= 0 &&
           d.r0 % chain_part(nb) == 0 && d.r0 < d.n[1] && d.r0 < S &&
           (mode == 3 || (d.n[0] <= S && d.n[1] <= S));
  if (mode == 1)
    return d.mr != nullptr && d.mc != nullptr && mat(0, S) && mat(1, S) && mat(2, S + 2) &&
           mat(3, S + 2) && d.in_r <= d.k[1] && d.in_c <= d.k[0] && d.zoff == 0;
  return mode == 2 && d.mt != nullptr && mat(1, S) && mat(3, S + 2) && d.in_r <= d.k[1] &&
         d.k[3] <= d.ld[1] && d.in_c <= chain_part(nb) && d.out_c <= d.in_c && d.zoff == 0;
}

void chain_order(std::vector<ChainDesc> &d, int group) {
  std::vector<ChainDesc> t(d);
  const size_t step = 8 * (size_t)group;
  for (size_t i = 0; i + step <= d.size(); i += step)
    for (size_t q = 0; q < 8; ++q)
      for (size_t j = 0; j < (size_t)group; ++j) d[i + 8 * j + q] = t[i + q * group + j];
}

hipError_t launch_chain_table(const ChainDesc *d, int count, int nb, int mode, const double *in,
                              char *ws, double *out, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (count <= 0) return hipSuccess;
  const Bases u{(const char *)in, ws, (char *)out};
#define FPS_CHAIN(N, M, KERNEL, THREADS) \
  if (nb == N && mode == M) return run(KERNEL, (unsigned)count, THREADS, st, ev0, ev1, d, u)
#define FPS_UNITS(N, W)                                            \
  static_assert(32 * W == chain_part(N), "rows or columns a unit"); \
  FPS_CHAIN(N, 0, (k_slab<N, W, false>), (Unit<N, W>::kThreads));  \
  FPS_CHAIN(N, 2, (k_strip<N, W>), (Unit<N, W>::kThreads));        \
  FPS_CHAIN(N, 3, (k_slab<N, W, true>), (Unit<N, W>::kThreads))
  FPS_UNITS(2, 2);
  FPS_UNITS(3, 1);
  FPS_UNITS(4, 1);
  FPS_CHAIN(2, 1, k_chain_table<2>, Chain<2>::kThreads);
  FPS_CHAIN(3, 1, k_chain_table<3>, Chain<3>::kThreads);
#undef FPS_UNITS
#undef FPS_CHAIN
  return hipErrorInvalidValue;
}

hipError_t launch_chain(const ChainDesc *d, int count, int nb, hipStream_t st, hipEvent_t ev0,
                        hipEvent_t ev1) {
  if (count < 1 || count > 4 || (nb != 2 && nb != 3)) return hipErrorInvalidValue;
  ChainBatch b{};
  for (int i = 0; i < count; ++i) {
    if (!chain_ok(d[i], nb, 1)) return hipErrorInvalidValue;
    b.d[i] = d[i];
  }
  return nb == 2 ? run(k_chain<2>, (unsigned)count, Chain<2>::kThreads, st, ev0, ev1, b)
                 : run(k_chain<3>, (unsigned)count, Chain<3>::kThreads, st, ev0, ev1, b);
}

}  // namespace fps
