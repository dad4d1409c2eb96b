// gfx950 chains of FP64 products on one block held in LDS.
//
// The eigenbasis solves multiply each parity block by a matrix on its right
// and one on its left, twice.  Blocks of at most 128 x 128 fit one workgroup's
// LDS, so a chain of products reads its block from HBM once and writes it once:
// cube slices (x and y maps of one slice block, or both z maps of a strip of
// columns), cylinder modes (z and r maps) and whole square solves up to n = 128.
// Against one product launch per axis: cube n = 256 775 -> 678 us, n = 128 111 ->
// 74 us, cylinder 256 x 256 1031 -> 652 us (its z map then also runs over the r
// parity that a mode has only), square n = 64 22.6 -> 14.4 us.  At 128 x 128 the
// products run at 43 TFLOP/s: a workgroup has its compute unit alone, so
// nothing runs under its fills, first loads and stores.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"

namespace fps {

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef double dbl2 __attribute__((ext_vector_type(2)));

// Block of up to S x S (S = 32 NB), NB^2 wavefronts, each 32 x 32 of the output
// as 2 x 2 MFMA blocks (v_mfma_f64_16x16x4f64: lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16], accumulator register r holds C[4r + l / 16][l % 16]).
// X lives in LDS with two columns of padding: 16 rows at one k then fall on
// distinct banks.  The other operand is read from global memory in its
// transposed form [k][row or column], 128 contiguous bytes per k, a few KB that
// all workgroups share in the caches.  One workgroup per compute unit at NB =
// 4 (133 KB, 4 wavefronts per SIMD), two at 3, four at 2.
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
template <bool kTab>
__device__ __forceinline__ double multiplier(const ChainDesc &d, int i, int j, double v) {
  if constexpr (kTab) return v * d.mt[i * d.mt_rs + j];
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
  return id == 0 ? p : (const double *)(at + (intptr_t)p);
}

// mode 0: right, left.  1: right, left, multiplier, right, left.  2: left,
// multiplier, left.
template <int NB, int kMode, bool kTable>
__device__ __forceinline__ void chain_blocks(const ChainDesc *__restrict__ d, int count,
                                             const Bases &u) {
  using C = Chain<NB>;
  __shared__ __align__(16) double X[C::kLds];
  const int tid = threadIdx.x;
  Lane l;
  l.l15 = tid & 15;
  l.l4 = (tid & 63) >> 4;
  l.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  l.wy = l.wave / NB;
  l.wx = l.wave % NB;
  // 16 elements per thread, in two rounds (one at NB = 4: there a workgroup has
  // its compute unit alone and takes block after block, so the next block's
  // elements are loaded under this block's products; the smaller ones overlap
  // with their neighbours).
  constexpr bool kNext = NB == 4;
  constexpr int kPer = kNext ? 16 : 8;
  static_assert(C::S * C::S == 16 * C::kThreads, "one block is 16 elements per thread");
  double v[kPer];
  // thread t holds column t % S of rows t / S + 2 NB i
  const int tr = tid / C::S, tc = tid % C::S;
  auto load = [&](const ChainDesc &e, int i0) {
    const double *in = rebase<kTable>(e.in, e.ibase, u);
    const uint32_t off = (uint32_t)(tr * (int)e.in_rs + tc * e.in_cs);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int r = (i0 + i) * 2 * NB;
      v[i] = tr + r < e.in_r && tc < e.in_c ? (in + r * e.in_rs)[off] : 0.0;
    }
  };
  double *Xt = X + tr * C::P + tc;
  auto fill = [&](int i0) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) Xt[(i0 + i) * 2 * NB * C::P] = v[i];
  };
  int b = blockIdx.x;
  if (kNext && b < count) load(d[b], 0);
  for (; b < count; b += gridDim.x) {
    const ChainDesc &e = d[b];
    if constexpr (kNext) {
      fill(0);
    } else {
      load(e, 0);
      fill(0);
      load(e, 8);
      fill(8);
    }
    __syncthreads();
    if (kNext && b + (int)gridDim.x < count) load(d[b + gridDim.x], 0);
    double *Xl = X + l.l4 * C::P + l.l15;  // this lane's entry of a 4 x 16 patch
    auto keep = [&](int r, int c, double x) {
      if (r + 4 <= C::S && c + l.l15 < C::P) Xl[r * C::P + c] = x;
    };
    auto keep_mul = [&](int r, int c, double x) {
      const int i = r + l.l4, j = c + l.l15;
      if (r + 4 <= C::S && j < C::S)
        Xl[r * C::P + c] = i < e.n[1] && j < e.mcols ? multiplier<kMode == 2>(e, i, j, x) : 0.0;
    };
    double *out = (double *)rebase<kTable>(e.out, e.obase, u);
    const uint32_t oo = (uint32_t)(l.l4 * (int)e.out_rs + l.l15 * e.out_cs);
    auto store = [&](int r, int c, double x) {
      if (r + l.l4 < e.out_r && c + l.l15 < e.out_c) {
        double *o = out + r * e.out_rs + (int64_t)c * e.out_cs;
        o[oo] = x;
        if (kMode == 0 && e.zoff != 0) (o + e.zoff)[oo] = 0.0;
      }
    };
    if constexpr (kMode != 2) {
      step<NB, false>(X, e.m[0], e.ld[0], e.k[0], e.k[1], e.n[0], l, keep);
      __syncthreads();
    }
    if constexpr (kMode == 0) {
      step<NB, true>(X, e.m[1], e.ld[1], e.k[1], e.n[1], e.n[0], l, store);
    } else {
      step<NB, true>(X, e.m[1], e.ld[1], e.k[1], e.n[1], e.mcols, l, keep_mul);
      __syncthreads();
      if constexpr (kMode == 1) {
        step<NB, false>(X, e.m[2], e.ld[2], e.k[2], e.k[3], e.n[2], l, keep);
        __syncthreads();
      }
      step<NB, true>(X, e.m[3], e.ld[3], e.k[3], e.n[3], kMode == 1 ? e.n[2] : e.mcols, l, store);
    }
    // step() has a barrier between its last read of X and the stores, so the
    // next block may overwrite X here
  }
}

template <int NB, int kMode>
__global__ __launch_bounds__(Chain<NB>::kThreads, NB == 3 ? 5 : 4) void k_chain_table(
    const ChainDesc *__restrict__ d, int count, Bases u) {
  chain_blocks<NB, kMode, true>(d, count, u);
}

struct ChainBatch {
  ChainDesc d[4];
};

template <int NB>
__global__ __launch_bounds__(Chain<NB>::kThreads, NB == 3 ? 5 : 4) void k_chain(ChainBatch b, int count) {
  chain_blocks<NB, 1, false>(b.d, count, Bases{});
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
  auto mat = [&](int i, int most) {
    return d.m[i] != nullptr && d.k[i] >= 16 && d.k[i] <= S && d.k[i] % 16 == 0 && d.n[i] >= 1 &&
           d.n[i] <= most && d.ld[i] >= (d.n[i] > S ? S + 16 : (d.n[i] + 31) / 32 * 32);
  };
  // the lanes' address parts are 32-bit
  if (S * d.in_rs >= (int64_t)1 << 31 || 16 * d.out_rs >= (int64_t)1 << 31) return false;
  if (nb < 2 || nb > 4 || d.in_r > S || d.in_c > S || d.in_r < 1 || d.in_c < 1) return false;
  if (mode == 0) return mat(0, S + 2) && mat(1, S + 2) && d.in_r <= d.k[1] && d.in_c <= d.k[0];
  const bool mul = mode == 2 ? d.mt != nullptr : d.mr != nullptr && d.mc != nullptr;
  if (mode == 1)
    return mul && mat(0, S) && mat(1, S) && mat(2, S + 2) && mat(3, S + 2) && d.in_r <= d.k[1] &&
           d.in_c <= d.k[0] && d.mcols <= S && d.mcols >= d.n[0] && d.k[2] <= S;
  return mode == 2 && mul && mat(1, S) && mat(3, S + 2) && d.in_r <= d.k[1] && d.mcols <= S;
}

void chain_order(std::vector<ChainDesc> &d) {
  for (size_t i = 0; i + 16 <= d.size(); i += 16) {
    ChainDesc t[16];
    for (int q = 0; q < 8; ++q) {
      t[q] = d[i + 2 * q];
      t[8 + q] = d[i + 2 * q + 1];
    }
    std::copy(t, t + 16, d.begin() + i);
  }
}

hipError_t launch_chain_table(const ChainDesc *d, int count, int nb, int mode, const double *in,
                              char *ws, double *out, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (count <= 0) return hipSuccess;
  const unsigned grid = nb == 4 && count > 256 ? 256u : (unsigned)count;
#define FPS_CHAIN(N, M) \
  if (nb == N && mode == M) \
  return run(k_chain_table<N, M>, grid, Chain<N>::kThreads, st, ev0, ev1, d, count, \
             Bases{(const char *)in, ws, (char *)out})
  FPS_CHAIN(2, 0);
  FPS_CHAIN(3, 0);
  FPS_CHAIN(4, 0);
  FPS_CHAIN(2, 2);
  FPS_CHAIN(3, 2);
  FPS_CHAIN(4, 2);
  FPS_CHAIN(2, 1);
  FPS_CHAIN(3, 1);
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
  return nb == 2 ? run(k_chain<2>, (unsigned)count, Chain<2>::kThreads, st, ev0, ev1, b, count)
                 : run(k_chain<3>, (unsigned)count, Chain<3>::kThreads, st, ev0, ev1, b, count);
}

}  // namespace fps
