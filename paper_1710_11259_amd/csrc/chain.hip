// gfx950 chains of FP64 products on one LDS-resident block.
//
// The eigenbasis solves multiply each parity block by a matrix on its right
// and one on its left, twice.  For blocks of at most 128 x 128 the block between
// two products fits a workgroup's LDS, so a chain of products goes through HBM
// once: cube slices (x and y maps), cube strips (both z maps with the multiplier in
// between), cylinder modes (z and r maps) and whole square solves up to n = 128.
// Against one product launch per axis: cube n = 256 775 -> 490 us, n = 185 297 ->
// 180 us, n = 128 111 -> 53 us, cylinder 256 x 256 1031 -> 562 us (its z map then
// also ran over the r parity that a mode has not), square n = 64 22.6 -> 8.6 us.
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

struct Lane {
  int l15, l4, wave, wy, wx;
};

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

// A whole square solve, m3^T (multiplier of m1^T X m0) m2, of blocks of up to 64 with
// outputs of up to 16 TT: a wavefront per 16 x 16 tile (v_mfma_f64_16x16x4f64: lane l
// supplies A[l % 16][l / 16] and B[l / 16][l % 16], accumulator register r holds
// C[4r + l / 16][l % 16]), 16 of them at most; the first wavefronts also take the
// tiles left over at TT = 5.  Bound by latency: the four products of n = 64 are 0.25 us
// each, a load from another die's cache or HBM takes 1 to 2.  So the first product
// reads F straight into the matrix unit's layout, the other operand of the next
// product is loaded into registers while the current one runs, and the results go
// to two LDS buffers in turn, one barrier each.  n = 64: 14.2 us with 32 x 32 tiles that
// waited for every operand -> 8.6.
template <int TT>
struct Chain {
  static constexpr int P = 16 * TT + 2;  // 16 rows at one k on distinct banks
  static constexpr int kWaves = TT * TT < 16 ? TT * TT : 16, kThreads = 64 * kWaves;
  static constexpr int kSlots = (TT * TT + kWaves - 1) / kWaves;
};
constexpr int kChainK = 64, kSteps = kChainK / 4;

// Row / column of the wavefront's tile in a product with rows x cols outputs; false
// if there is none.
__device__ __forceinline__ bool chain_tile(int i, int rows, int cols, int *r, int *c) {
  const int nx = (cols + 15) >> 4;
  *r = i / nx * 16;
  *c = i % nx * 16;
  return *r < rows;
}

// w = W[k][w0 + l15] of k = 4u + l4, for k < K (a multiple of 16).
__device__ __forceinline__ void chain_load(const double *W, int ldw, int K, int w0, const Lane &l,
                                           double (&w)[kSteps]) {
  const uint32_t o = 8 * (l.l4 * ldw + l.l15);
#pragma unroll
  for (int u = 0; u < kSteps; ++u)
    if ((u & ~3) * 4 < K) w[u] = at(W + w0 + 4 * u * ldw, o);
}

// The tile X W (kLeft W^T X) with X from LDS.
template <int P, bool kLeft>
__device__ __forceinline__ dbl4 chain_mul(const double *X, const double (&w)[kSteps], int K, int r,
                                          int c, const Lane &l) {
  const double *x = kLeft ? X + l.l4 * P + c + l.l15 : X + (r + l.l15) * P + l.l4;
  dbl4 acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int v = 0; v < kSteps; v += 4)
    if (4 * v < K) {
#pragma unroll
      for (int u = v; u < v + 4; ++u) {
        const double t = x[4 * u * (kLeft ? P : 1)];
        acc = kLeft ? __builtin_amdgcn_mfma_f64_16x16x4f64(w[u], t, acc, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f64_16x16x4f64(t, w[u], acc, 0, 0, 0);
      }
    }
  return acc;
}

template <int TT, bool kTable>
__device__ __forceinline__ void solve_block(const ChainDesc &e, const Bases &u) {
  using C = Chain<TT>;
  constexpr int P = C::P;
  __shared__ __align__(16) double X[2][16 * TT * P];
  const int tid = threadIdx.x;
  Lane l;
  l.l15 = tid & 15;
  l.l4 = (tid & 63) >> 4;
  l.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double *in = rebase<kTable>(e.in, e.ibase, u);
  double *out = (double *)rebase<kTable>(e.out, e.obase, u);
  double wa[kSteps], wb[kSteps];
  int r, c;
  auto keep = [&](double *Y, const dbl4 &acc) {
#pragma unroll
    for (int q = 0; q < 4; ++q) Y[(r + 4 * q + l.l4) * P + c + l.l15] = acc[q];
  };
  // slots past the first (TT = 5) load their W when they come to it
  // 1: X m0, X straight from the input (zero beyond in_r, in_c)
#pragma unroll
  for (int s = 0; s < C::kSlots; ++s)
    if (chain_tile(l.wave + s * C::kWaves, e.k[1], e.n[0], &r, &c)) {
      double x[kSteps];
      const int row = r + l.l15;
      const double *p = in + (int64_t)min(row, e.in_r - 1) * e.in_rs;
#pragma unroll
      for (int v = 0; v < kSteps; ++v)
        if ((v & ~3) * 4 < e.k[0]) x[v] = p[min(4 * v + l.l4, e.in_c - 1) * e.in_cs];
      chain_load(e.m[0], e.ld[0], e.k[0], c, l, wa);
      if (s == 0) {
        int r1, c1;
        if (chain_tile(l.wave, e.n[1], e.n[0], &r1, &c1)) chain_load(e.m[1], e.ld[1], e.k[1], r1, l, wb);
      }
      dbl4 acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int v = 0; v < kSteps; ++v)
        if ((v & ~3) * 4 < e.k[0])
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(
              row < e.in_r && 4 * v + l.l4 < e.in_c ? x[v] : 0.0, wa[v], acc, 0, 0, 0);
      keep(X[0], acc);
    }
  // 2: m1^T X and the multiplier (as in the product kernels)
  if (chain_tile(l.wave, e.k[3], e.n[2], &r, &c)) chain_load(e.m[2], e.ld[2], e.k[2], c, l, wa);
  dbl2 fr[4], fc;
  if (chain_tile(l.wave, e.n[1], e.n[0], &r, &c)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) fr[q] = *(const dbl2 *)(e.mr + 2 * (r + 4 * q + l.l4));
    fc = *(const dbl2 *)(e.mc + 2 * (c + l.l15));
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < C::kSlots; ++s)
    if (chain_tile(l.wave + s * C::kWaves, e.n[1], e.n[0], &r, &c)) {
      if (s > 0) {
        chain_load(e.m[1], e.ld[1], e.k[1], r, l, wb);
#pragma unroll
        for (int q = 0; q < 4; ++q) fr[q] = *(const dbl2 *)(e.mr + 2 * (r + 4 * q + l.l4));
        fc = *(const dbl2 *)(e.mc + 2 * (c + l.l15));
      }
      dbl4 acc = chain_mul<P, true>(X[0], wb, e.k[1], r, c, l);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double v = acc[q];
        if (e.lr != nullptr) {
          const double *a = e.lr + 4 * (r + 4 * q + l.l4), *b = e.lc + 4 * (c + l.l15);
          v -= fma(a[3], b[3], fma(a[2], b[2], fma(a[1], b[1], a[0] * b[0])));
        }
        acc[q] = v * (fma(-fr[q].y, fc.y, 1.0) / (fr[q].x + fc.x));
      }
      keep(X[1], acc);
    }
  // 3: X m2
  if (chain_tile(l.wave, e.n[3], e.n[2], &r, &c)) chain_load(e.m[3], e.ld[3], e.k[3], r, l, wb);
  __syncthreads();
#pragma unroll
  for (int s = 0; s < C::kSlots; ++s)
    if (chain_tile(l.wave + s * C::kWaves, e.k[3], e.n[2], &r, &c)) {
      if (s > 0) chain_load(e.m[2], e.ld[2], e.k[2], c, l, wa);
      keep(X[0], chain_mul<P, false>(X[1], wa, e.k[2], r, c, l));
    }
  __syncthreads();
  // 4: m3^T X
#pragma unroll
  for (int s = 0; s < C::kSlots; ++s)
    if (chain_tile(l.wave + s * C::kWaves, e.n[3], e.n[2], &r, &c)) {
      if (s > 0) chain_load(e.m[3], e.ld[3], e.k[3], r, l, wb);
      const dbl4 acc = chain_mul<P, true>(X[0], wb, e.k[3], r, c, l);
      const int j = c + l.l15;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = r + 4 * q + l.l4;
        if (i < e.out_r && j < e.out_c) out[i * e.out_rs + (int64_t)j * e.out_cs] = acc[q];
      }
    }
}

template <int TT>
__global__ __launch_bounds__(Chain<TT>::kThreads) void k_chain_table(const ChainDesc *__restrict__ d,
                                                                     Bases u) {
  solve_block<TT, true>(table_entry(d[blockIdx.x]), u);
}

struct ChainBatch {
  ChainDesc d[4];
};

template <int TT>
__global__ __launch_bounds__(Chain<TT>::kThreads) void k_chain(ChainBatch b) {
  solve_block<TT, false>(b.d[blockIdx.x], Bases{});
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

// acc = W^T[r0 .. r0 + 32)[0 .. K) X[0 .. K)[c0 .. c0 + 32), W [k][row] (zeros from k =
// in_r on), X [k][column], zero beyond in_c; K a multiple of 32.  Rows interleaved, columns too if kPair.
// X comes from HBM: 8 k-steps (2048 MFMA cycles of the SIMD's wavefronts) ahead, W
// from the caches: 4.  kExt: ext[c] = the rows S, S + 1 of W^T X in this lane's two
// columns (all four lanes of a column hold them).
// kDown: k from K - 1 down to 0, for sums over degrees, whose first terms are the
// largest: with those added last the small ones are not rounded against them.  The
// cylinder's banded solves magnify the rounding of their right-hand sides: three solves
// that must cancel left 9.9e-15 of the result at n = 64 and 1.5e-14 at 130, both input
// products downwards 2.1e-15 and 2.3e-15, at the same speed.
template <bool kPair, bool kExt, bool kDown>
__device__ __forceinline__ void mul_stream(const double *__restrict__ W, int ldw, int S,
                                           const double *__restrict__ X, const ChainDesc &e, int K,
                                           int r0, int c0, const Lane &l, dbl4 (&acc)[2][2],
                                           dbl2 (&ext)[2]) {
  const int l4 = kDown ? 3 - l.l4 : l.l4;  // the lane's row in a k-step
  const uint32_t wo = 8 * (l4 * ldw + 2 * l.l15), xwo = 8 * (l4 * ldw);
  const Buffer wb(W), xb(X);
  const int rs = (int)e.in_rs, cs = e.in_cs;
  auto first_row = [&](int k) { return kDown ? K - 4 - k : k; };  // of the k-step at k
  // the last k-step with data, and its rows
  const int last = (e.in_r - 1) & ~3;
  uint32_t xo[2], xl[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int col = c0 + (kPair ? 2 * l.l15 + c : 16 * c + l.l15);
    // (a pair may end one past in_c, in the padding)
    const int cc = (col < e.in_c ? col : kPair ? (e.in_c - 1) & ~1 : e.in_c - 1) * cs;
    xo[c] = 8 * (l4 * rs + cc);
    xl[c] = 8 * (min(l4, e.in_r - 1 - last) * rs + cc);
  }
  dbl2 a[4], b[8], x[4];
  ext[0] = ext[1] = dbl2{0.0, 0.0};
  auto load_a = [&](int u, int k) {
    a[u] = wb.load2(wo, 8 * (r0 + first_row(k) * ldw));
    if constexpr (kExt) x[u] = wb.load2(xwo, 8 * (S + first_row(k) * ldw));
  };
  // kEnd: the k-steps may end or pass the data (K - in_r < 32); those past it read the
  // last row again, times zeros of W
  auto load_b = [&](int u, int k, auto end) {
    const bool z = decltype(end)::value && first_row(k) >= last;
    const uint32_t row = 8 * (z ? last : first_row(k)) * rs;
    const uint32_t o0 = z ? xl[0] : xo[0], o1 = z ? xl[1] : xo[1];
    if constexpr (kPair)
      b[u] = xb.load2(o0, row);
    else
      b[u] = dbl2{xb.load(o0, row), xb.load(o1, row)};
  };
  using Inner = std::false_type;
  using End = std::true_type;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    if (u < 4) load_a(u, 4 * u);
    load_b(u, 4 * u, End{});
    __builtin_amdgcn_sched_barrier(0);  // in the order of their use, for the waits
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[r][c] = dbl4{0.0, 0.0, 0.0, 0.0};
  // 8 k-steps, and the loads of the 8 (W: of 4 of them) that follow (kNext)
  auto chunk = [&](int ks, auto next, auto end) {
    constexpr bool kNext = decltype(next)::value;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = ks + 4 * u;
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u & 3][r], b[u][c], acc[r][c], 0, 0, 0);
      if constexpr (kExt) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          ext[c].x = fma(x[u & 3].x, b[u][c], ext[c].x);
          ext[c].y = fma(x[u & 3].y, b[u][c], ext[c].y);
        }
      }
      // the next loads go into the registers just read; the barrier keeps them
      // from moving next to their use
      __builtin_amdgcn_sched_barrier(0);
      if (kNext || u < 4) load_a(u & 3, k + 16);
      if constexpr (kNext) load_b(u, k + 32, end);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int ks = 0;
#pragma unroll 1
  for (; ks + (kDown ? 32 : 64) <= (kDown ? K - 1 : e.in_r); ks += 32) chunk(ks, End{}, Inner{});
  if constexpr (!kDown)
#pragma unroll 1
    for (; ks + 32 < K; ks += 32) chunk(ks, End{}, End{});
  chunk(ks, Inner{}, Inner{});
  // columns past in_c took others' data
#pragma unroll
  for (int c = 0; c < 2; ++c)
    if (c0 + (kPair ? 2 * l.l15 + c : 16 * c + l.l15) >= e.in_c) {
      ext[c] = dbl2{0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 2; ++r) acc[r][c] = dbl4{0.0, 0.0, 0.0, 0.0};
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
// kDown (T W without extra rows or columns): k from K - 1 down, as above; t[.] are then those
// of the lane's k within the lowest k-step.
template <bool kLeft, bool kPair, bool kExtW, bool kExtT, bool kDown>
__device__ __forceinline__ void mul_kept(const double *T, const int (&t)[2], int ts,
                                         const double *__restrict__ W, int ldw, int S, int K, int w0,
                                         const double *te, int P, const Lane &l, Kept &o) {
  static_assert(!kDown || !(kExtW || kExtT), "downwards without extra rows or columns");
  const int l4 = kDown ? 3 - l.l4 : l.l4;
  const uint32_t wo = 8 * (l4 * ldw + (kPair ? 2 : 1) * l.l15), xwo = 8 * (l4 * ldw);
  const Buffer wb(W);
  dbl2 w[4], x[4];
  auto first_row = [&](int k) { return kDown ? K - 4 - k : k; };
  auto load = [&](int u, int k) {
    const uint32_t row = 8 * (w0 + first_row(k) * ldw);
    if constexpr (kPair)
      w[u] = wb.load2(wo, row);
    else
      w[u] = dbl2{wb.load(wo, row), wb.load(wo + 128, row)};
    if constexpr (kExtW) x[u] = wb.load2(xwo, 8 * (S + k * ldw));
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
  auto chunk = [&](int ks, auto next) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double tv[2], ev[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        tv[r] = T[t[r] + first_row(ks + 4 * u) * ts];
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
      if constexpr (decltype(next)::value) load(u, ks + 16 + 4 * u);
    }
  };
  int ks = 0;
#pragma unroll 1
  for (; ks + 16 < K; ks += 16) chunk(ks, std::true_type{});
  chunk(ks, std::false_type{});
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
      mul_stream<kOut, kOut, !kOut>(e.m[1], e.ld[1], C::S, X, e, e.k[1], r0, c0, l, o.acc, ext);
      if (l.l4 == 0)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          t[C::E * C::P + (kOut ? 1 : 16) * b] = ext[b].x;
          t[(C::E + 1) * C::P + (kOut ? 1 : 16) * b] = ext[b].y;
        }
    } else {
      mul_stream<kOut, false, !kOut>(e.m[1], e.ld[1], C::S, X, e, e.k[1], r0, c0, l, o.acc, ext);
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
  const int tk = kOut ? l.l4 : 3 - l.l4;
  const int t[2] = {(32 * l.wy + l.l15) * C::P + tk, (32 * l.wy + 16 + l.l15) * C::P + tk};
  const bool cols = kOut && e.n[0] > C::S && l.wx == 0;
  auto second = [&](auto w, auto t2) {
    mul_kept<false, !kOut, decltype(w)::value, decltype(t2)::value, !kOut>(
        T, t, 1, e.m[0], e.ld[0], C::S, e.k[0], c0, T + C::E * C::P, C::P, l, o);
  };
  using No = std::false_type;
  using Ext = std::integral_constant<bool, kOut>;
  if (cols)
    rows ? second(Ext{}, Ext{}) : second(Ext{}, No{});
  else
    rows ? second(No{}, Ext{}) : second(No{}, No{});
  const Buffer ob(out);
  const uint32_t rs = 8 * (uint32_t)e.out_rs, lane = l.l4 * rs + 16 * l.l15;
  if (r0 + 32 <= e.out_r && c0 + 32 <= e.out_c) {
    // the zeros of a unit and its partner of the other column parity: each writes
    // every other row of both (cylinder 256 x 256: 413 -> 341 MB written, 481 -> 475 us)
    const Buffer zb(out + e.zoff - e.zcol);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t row = (r0 + 16 * a + 4 * r) * rs + (kOut ? 16 : 8) * c0;
        if constexpr (kOut) {
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            ob.store(o.acc[a][c][r], lane, row + 256 * c);
            if (e.zoff != 0 && e.zcol == (r & 1)) zb.store2(dbl2{0.0, 0.0}, lane, row + 256 * c);
          }
        } else {
          ob.store2(dbl2{o.acc[a][0][r], o.acc[a][1][r]}, lane, row);
        }
      }
  } else {
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
    mul_stream<true, false, false>(e.m[1], e.ld[1], C::S, X, e, e.k[1], r0, c0, l, o.acc, ext);
    const int j = c0 + 2 * l.l15;  // columns j, j + 1 (in_c is even)
    const Buffer mb(e.mt);
    const uint32_t mrs = 8 * (uint32_t)e.mt_rs, mlane = 2 * l.l4 * mrs + 8 * j;
    const bool inner = r0 + 32 <= e.n[1] && c0 + 32 <= e.in_c;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 8 * r + 2 * l.l4 + a;
        dbl2 f{0.0, 0.0};
        if (inner)
          f = mb.load2(mlane, (r0 + 8 * r + a) * mrs);
        else if (i < e.n[1] && j < e.in_c)
          f = *(const dbl2 *)(e.mt + i * e.mt_rs + j);
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
    mul_kept<true, true, true, false, false>(T, t, C::E, e.m[3], e.ld[3], C::S, e.k[3], r0, T, 0, l, o);
  else
    mul_kept<true, true, false, false, false>(T, t, C::E, e.m[3], e.ld[3], C::S, e.k[3], r0, T, 0, l, o);
  if (r0 + 32 <= e.out_r && c0 + 32 <= e.out_c) {
    const Buffer ob(out);
    const uint32_t rs = 8 * (uint32_t)e.out_rs, lane = 2 * l.l4 * rs + 8 * l.l15;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          ob.store(o.acc[a][b][r], lane, (r0 + 8 * r + a) * rs + 8 * (c0 + 16 * b));
  } else {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          store_one(e, out, r0 + 8 * r + 2 * l.l4 + a, c0 + 16 * b + l.l15, o.acc[a][b][r]);
  }
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
  const int S = mode == 1 ? 16 * nb : 32 * nb, step = mode == 1 ? 16 : 32;
  const int K = mode == 1 && S > kChainK ? kChainK : S;
  auto mat = [&](int i, int most) {
    const int cover = mode == 1 ? (d.n[i] + 15) / 16 * 16 : d.n[i] > S ? S + 16 : (d.n[i] + 31) / 32 * 32;
    return d.m[i] != nullptr && d.k[i] >= step && d.k[i] <= K && d.k[i] % step == 0 && d.n[i] >= 1 &&
           d.n[i] <= most && d.ld[i] >= cover;
  };
  // the lanes' address parts are 32-bit
  if (8 * S * d.in_rs >= (int64_t)1 << 31 || 8 * (S + 2) * d.out_rs >= (int64_t)1 << 31 ||
      8 * S * d.mt_rs >= (int64_t)1 << 31)
    return false;
  if (d.in_r > S || d.in_c > S || d.in_r < 1 || d.in_c < 1) return false;
  if (mode == 1)
    return (nb == 3 || nb == 4 || nb == 5) && d.mr != nullptr && d.mc != nullptr && mat(0, K) &&
           mat(1, K) && mat(2, S) && mat(3, S) && d.in_r <= d.k[1] && d.in_c <= d.k[0] &&
           d.k[2] == (d.n[0] + 15) / 16 * 16 && d.k[3] == (d.n[1] + 15) / 16 * 16;
  if (nb < 2 || nb > 4) return false;
  if (mode == 2)
    return d.mt != nullptr && mat(1, S) && mat(3, S + 2) && d.in_r <= d.k[1] && d.k[3] <= d.ld[1] &&
           d.in_c <= chain_part(nb) && d.out_c <= d.in_c && d.in_cs == 1 && d.out_cs == 1 &&
           d.in_c % 2 == 0 && d.mt_rs % 2 == 0 && d.zoff == 0;
  if (mode == 0 ? d.in_cs != 2 || d.out_cs != 1 || d.out_c % 2 || d.zoff != 0 || d.n[0] > S || d.n[1] > S
                : mode != 3 || d.in_cs != 1 || d.out_cs != 2 || (d.zcol & ~1) != 0)
    return false;
  return mat(0, S + 2) && mat(1, S + 2) && d.in_r <= d.k[1] && d.k[1] - d.in_r < 32 && d.in_c <= d.k[0] && d.r0 >= 0 &&
         d.r0 % chain_part(nb) == 0 && d.r0 < d.n[1] && d.r0 < S;
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
  FPS_CHAIN(3, 1, k_chain_table<3>, Chain<3>::kThreads);
  FPS_CHAIN(4, 1, k_chain_table<4>, Chain<4>::kThreads);
  FPS_CHAIN(5, 1, k_chain_table<5>, Chain<5>::kThreads);
#undef FPS_UNITS
#undef FPS_CHAIN
  return hipErrorInvalidValue;
}

hipError_t launch_chain(const ChainDesc *d, int count, int nb, hipStream_t st, hipEvent_t ev0,
                        hipEvent_t ev1) {
  if (count < 1 || count > 4) return hipErrorInvalidValue;
  ChainBatch b{};
  for (int i = 0; i < count; ++i) {
    if (!chain_ok(d[i], nb, 1)) return hipErrorInvalidValue;
    b.d[i] = d[i];
  }
  if (nb == 3) return run(k_chain<3>, (unsigned)count, Chain<3>::kThreads, st, ev0, ev1, b);
  if (nb == 4) return run(k_chain<4>, (unsigned)count, Chain<4>::kThreads, st, ev0, ev1, b);
  return run(k_chain<5>, (unsigned)count, Chain<5>::kThreads, st, ev0, ev1, b);
}

}  // namespace fps
