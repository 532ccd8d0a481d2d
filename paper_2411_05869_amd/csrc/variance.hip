// Posterior variance of the latent process at test points (Sec. 3.2): the
// diagonal of C_{y|z} = C_y - C_{y,z} C_z^{-1} C_{z,y},
//   v(x*) = C_y(x*, x*) - c^T K^{-1} c,   c = C_{z,y}(., x*),
// for up to 32 test points at a time:
//   1. the cross-covariance columns c_s are written into an n x C block X (C = 32,
//      fewer for the last few of a request; rows in binned order): the local
//      (Wendland) entries of each point's cell window, then the bump-group
//      entries over the masked training points are added;
//   2. K W = X is solved by as many conjugate-gradient recurrences in lockstep
//      (one SpMM per step; block-Jacobi or Jacobi preconditioner; per-column
//      scalars; a column stops changing once |r_s| <= rtol |c_s|), with a float64 true residual
//      X - K W at the end (the recurrences restart from it if it is not small
//      enough);
//   3. v_s = C_y(x*_s, x*_s) - sum_q X[q, s] W[q, s].
// Every reduction adds partial sums in a fixed order, so results are
// reproducible.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "device.hpp"

namespace gps {
namespace {

constexpr int kThreads = 256;
constexpr int kC = 32;                 // right-hand sides per batch at most
// The reductions end in one block that adds every block's partials: few, large
// blocks leave it little to add (1024 blocks of 256 threads took it 12 - 18 us
// an iteration, longer than the pass it closed at n = 50,021).
// A block of C right-hand sides (32, or 16, 8 or 1 for the last of a request)
// takes 32 rows at a time, one column at least 256.
template <int C>
constexpr int rows() { return C >= 8 ? 32 : 256 / C; }  // rows handled together by a block of the reducing passes
template <int C>
constexpr int threads() { return rows<C>() * C; }
constexpr unsigned kVBlocks = 512;     // their blocks at most
constexpr int kRowBatch = 4;           // strided rows a thread loads at once in the column reductions
template <int C>
constexpr int tile() { return rows<C>() > 64 ? rows<C>() : 64; }  // rows of a tile of the update, before whole Jacobi blocks
template <int C>
constexpr int tile_max() { return tile<C>() + kMaxBlock - 1; }
constexpr int kCheckEvery = 8;
constexpr int kMaxRefresh = 3;

struct CrossArgs {
  KernelTheta kt;
  int64_t n;
  const double* xb;
  const int32_t* cell_start;
  double lo[3], cell[3];
  int32_t g[3], R[3];
  int64_t nm;
  const int32_t* mlist;
  const uint64_t* mmask;
  const double* F;  // nm x n1
};

struct BcgScalars {
  double rz[kC], pq[kC], alpha[kC], beta[kC], rr[kC], cc[kC];
  int32_t active[kC];
  int32_t status;
};

template <int D>
__device__ __forceinline__ void load_train(const CrossArgs& a, int64_t q, double* x) {
  x[0] = a.xb[q];
  if constexpr (D >= 2) x[1] = a.xb[a.n + q];
  if constexpr (D >= 3) x[2] = a.xb[2 * a.n + q];
}

// X[., s] = 0 for the block
__global__ void __launch_bounds__(kThreads) k_zero(int64_t len, double* __restrict__ X) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x; i < len;
       i += static_cast<int64_t>(gridDim.x) * kThreads)
    X[i] = 0.0;
}

// local part of c_s: C_core(x*, x_q) s0 f0(u) for the training points of the
// cell window with u0^2 < 1 (each q once).  A block per test point, kXl lanes per
// pencil (cell row along x) of its window: walked by one thread the window is a
// chain of as many dependent loads (32 points, n = 109,500: 109 us, now 5.4).
constexpr int kXl = 16;

template <int D, int CK>
__global__ void __launch_bounds__(kThreads) k_cross_local(CrossArgs a, CoreBasis cb, int nb, int ld,
                                                          const double* __restrict__ xs, double* __restrict__ X) {
  const int s = blockIdx.x;
  if (s >= nb) return;
  double xp[3];
  int c[3] = {0, 0, 0};
  for (int k = 0; k < D; ++k) {
    xp[k] = xs[static_cast<int64_t>(s) * D + k];
    c[k] = cell_coord(xp[k], a.lo[k], a.cell[k]);
  }
  int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
  for (int k = 0; k < D; ++k) {
    lo[k] = max(c[k] - a.R[k], 0);
    hi[k] = min(c[k] + a.R[k], a.g[k] - 1);
    if (lo[k] > hi[k]) return;
  }
  double sp = 0.0, Sp = 0.0;
  if constexpr (CK == 2) core_point_fields<D>(cb, xp, &sp, &Sp);
  const int ny = hi[1] - lo[1] + 1;
  const int64_t npen = static_cast<int64_t>(ny) * (hi[2] - lo[2] + 1);
  for (int64_t k = threadIdx.x / kXl; k < npen; k += kThreads / kXl) {
    const int y = lo[1] + static_cast<int>(k % ny), z = lo[2] + static_cast<int>(k / ny);
    const int64_t base = (static_cast<int64_t>(z) * a.g[1] + y) * a.g[0];
    const int32_t e = a.cell_start[base + hi[0] + 1];
    for (int32_t q = a.cell_start[base + lo[0]] + threadIdx.x % kXl; q < e; q += kXl) {
      double xq[3];
      load_train<D>(a, q, xq);
      const double u2 = scaled_sq<D>(xp, xq, a.kt.inv0);
      if (u2 < 1.0) {
        double v = a.kt.s0 * wendland(u2, a.kt.variant);
        if constexpr (CK == 1) v = core_value<D, 1>(a.kt.core, xp, xq, 0.0, 0.0, 0.0, 0.0) * v;
        if constexpr (CK == 2)
          v = core_value<D, 2>(a.kt.core, xp, xq, sp, Sp, a.kt.core.sig[q], a.kt.core.Sig[q]) * v;
        X[static_cast<int64_t>(q) * ld + s] = v;
      }
    }
  }
}

// bump-group part of c_s and the prior variance C_y(x*, x*): gridDim.y blocks of
// waves per test point, each forming the f_i(x*) for itself (lane i < n1, bumps of
// group i in j order) and taking its share of the masked training points.  (One
// wave per test point went through all of them: 32 points, n = 109,500, nearly all
// masked, 202 us, now 8.3.)
constexpr int kGroupShare = 256;  // masked points per wave, about
constexpr int kGroupBlocks = 64;  // blocks per test point at most

template <int D, int CK>
__global__ void __launch_bounds__(kThreads) k_cross_groups(CrossArgs a, CoreBasis cb, int nb, int ld,
                                                           const double* __restrict__ xs, double* __restrict__ X,
                                                           double* __restrict__ prior) {
  __shared__ double fs[kThreads / kWave][kWave];
  const int s = blockIdx.x;
  if (s >= nb) return;
  const int lane = lane_id();
  const int64_t wave = blockIdx.y * (kThreads / kWave) + threadIdx.x / kWave;
  double* f = fs[threadIdx.x / kWave];
  double xp[3];
  for (int k = 0; k < D; ++k) xp[k] = xs[static_cast<int64_t>(s) * D + k];
  bool in_group = false;
  double fi = 0.0;
  if (lane < a.kt.n1) {
#pragma clang fp contract(off)
    for (int j = 0; j < a.kt.n2; ++j) {
      const Bump& bp = a.kt.bumps[lane * a.kt.n2 + j];
      const double ub2 = scaled_sq<D>(xp, bp.h, bp.inv);
      if (bp.a > 0.0 && ub2 < 1.0) {
        in_group = true;
        fi = fi + bp.a * exp(bp.b * (1.0 - 1.0 / (1.0 - ub2)));
      }
    }
  }
  const uint64_t mask = __ballot(in_group);
  f[lane] = fi;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  double sp = 0.0, Sp = 0.0;
  if constexpr (CK == 2) core_point_fields<D>(cb, xp, &sp, &Sp);
  if (wave == 0 && lane == 0) {
#pragma clang fp contract(off)
    double v = a.kt.s0 * wendland(0.0, a.kt.variant);
    uint64_t mm = mask;
    while (mm) {
      const int i = __builtin_ctzll(mm);
      mm &= mm - 1;
      v = v + f[i] * f[i];
    }
    if constexpr (CK == 1) v = core_value<D, 1>(a.kt.core, xp, xp, 0.0, 0.0, 0.0, 0.0) * v;
    if constexpr (CK == 2) v = core_value<D, 2>(a.kt.core, xp, xp, sp, Sp, sp, Sp) * v;
    prior[s] = v;
  }
  if (mask == 0) return;  // uniform
  for (int64_t j = wave * kWave + lane; j < a.nm; j += static_cast<int64_t>(gridDim.y) * kThreads) {
    uint64_t sh = a.mmask[j] & mask;
    if (!sh) continue;
    double bsum = 0.0;
    while (sh) {
      const int i = __builtin_ctzll(sh);
      sh &= sh - 1;
      bsum += f[i] * a.F[j * a.kt.n1 + i];
    }
    const int32_t q = a.mlist[j];
    if constexpr (CK != 0) {
      double xq[3];
      load_train<D>(a, q, xq);
      if constexpr (CK == 1)
        bsum = core_value<D, 1>(a.kt.core, xp, xq, 0.0, 0.0, 0.0, 0.0) * bsum;
      else
        bsum = core_value<D, 2>(a.kt.core, xp, xq, sp, Sp, a.kt.core.sig[q], a.kt.core.Sig[q]) * bsum;
    }
    // row q is listed once, so these read-modify-writes do not race
    X[static_cast<int64_t>(q) * ld + s] += bsum;
  }
}

// ------------------------------------------------------- column reductions
// Thread (r, col) = (threadIdx.x / C, threadIdx.x % C) takes rows
// r, r + rows<C>(), ... of the block's share; per block and column the NV partial sums
// go to part[(blockIdx.x * NV + v) * C + col].  A wave first adds its rows, then
// thread (v, col) the waves in order.
template <int C>
__device__ __forceinline__ double add_wave_rows(double v) {
#pragma unroll
  for (int off = kWave / 2; off >= C; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

template <int NV, int C>
__device__ __forceinline__ void col_partials(const double (&v)[NV], double* __restrict__ part) {
  constexpr int kW = threads<C>() / kWave;
  __shared__ double sh[NV][kW][C];
  const int col = threadIdx.x % C, w = threadIdx.x / kWave;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const double t = add_wave_rows<C>(v[i]);
    if (lane_id() < C) sh[i][w][col] = t;
  }
  __syncthreads();
  if (threadIdx.x < NV * C) {
    const int i = threadIdx.x / C;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kW; ++k) s += sh[i][k][col];
    part[(static_cast<int64_t>(blockIdx.x) * NV + i) * C + col] = s;
  }
}

// Column totals of the partials of nb blocks, in a fixed order: thread
// (chunk, col) adds the partials of blocks chunk, chunk + rows<C>(), ...
// (eight loaded at once), a wave its chunks, then thread
// (v, col) the waves in order.  The result is the total of value threadIdx.x / C,
// valid in threads 0 .. C NV - 1 (column threadIdx.x % C); every thread of the
// block must call it.
template <int NV, int C>
__device__ __forceinline__ double col_total(const double* __restrict__ part, int nb) {
  constexpr int kW = threads<C>() / kWave, kChunks = rows<C>(), kB = 8;
  __shared__ double sh[NV][kW][C];
  const int col = threadIdx.x % C, ch = threadIdx.x / C;
  double s[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) s[v] = 0.0;
  for (int b0 = ch; b0 < nb; b0 += kB * kChunks) {
    double t[kB][NV];
#pragma unroll
    for (int u = 0; u < kB; ++u)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int b = b0 + u * kChunks;
        t[u][v] = b < nb ? part[(static_cast<int64_t>(b) * NV + v) * C + col] : 0.0;
      }
#pragma unroll
    for (int u = 0; u < kB; ++u)
#pragma unroll
      for (int v = 0; v < NV; ++v) s[v] += t[u][v];
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double t = add_wave_rows<C>(s[v]);
    if (lane_id() < C) sh[v][threadIdx.x / kWave][col] = t;
  }
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x < NV * C)
#pragma unroll
    for (int k = 0; k < kW; ++k) r += sh[threadIdx.x / C][k][col];
  return r;
}

// The totals of two values: both valid in threads 0 .. C - 1 (the second handed
// over from threads C .. 2 C - 1 of the same wave).
template <int C>
__device__ __forceinline__ void col_totals2(const double* __restrict__ part, int nb, double (&tot)[2]) {
  const double t = col_total<2, C>(part, nb);
  tot[0] = t;
  tot[1] = __shfl_xor(t, C, kWave);
}

// Preconditioner of the recurrences: the matrix diagonal, or (binv set) the
// block-Jacobi inverses over the binning cells (by columns per block).  Row i of
// z = M^-1 r needs r on the rows of its block; the caller passes a function
// that forms r for any row, so every thread sees the same values without
// waiting for the others.
struct VarPrecond {
  const double* diag;
  const uint64_t* brow;
  const double* binv;
};

// Rows of tile k: from the first Jacobi block that starts at or after row
// tile<C>() k to the one that starts at or after the next tile's, so that a tile
// holds whole blocks (at most tile_max<C>() rows) and the tiles hold every row once.
template <int C>
__device__ __forceinline__ int64_t tile_start(const VarPrecond& M, int64_t n, int64_t k) {
  const int64_t i = k * tile<C>();
  if (i >= n) return n;
  if (!M.binv) return i;
  const BlockRow br(M.brow[i]);
  return br.k == 0 ? i : i - br.k + br.sz;
}

// z = M^-1 r for the rows of a tile (rows lo .. hi - 1, the thread's column):
// rt holds the tile's r; put(i, r, z) takes each of the thread's rows.
// The block product is rt's rows times the block's inverse: r is read once
// from memory for the whole block instead of once per row of it, and a row's
// inverse entries (stored by columns) are loaded eight at a time.
template <int C, typename F>
__device__ __forceinline__ void tile_precond(const VarPrecond& M, int64_t lo, int64_t hi, double (*rt)[C], F&& put) {
  const int col = threadIdx.x % C;
  for (int64_t i = lo + threadIdx.x / C; i < hi; i += rows<C>()) {
    const double r = rt[i - lo][col];
    double z = 0.0;
    if (M.binv) {
      const BlockRow br(M.brow[i]);
      const int sz = br.sz;
      const double* w = M.binv + br.pos;
      const double(*rb)[C] = rt + (i - br.k - lo);
      constexpr int kB = 8;
      for (int j0 = 0; j0 < sz; j0 += kB) {
        double v[kB];
#pragma unroll
        for (int j = 0; j < kB; ++j) v[j] = w[min(j0 + j, sz - 1) * sz];
#pragma unroll
        for (int j = 0; j < kB; ++j)
          if (j0 + j < sz) z += v[j] * rb[j0 + j][col];
      }
    } else {
      z = r / M.diag[i];
    }
    put(i, r, z);
  }
}

#define ROW_LOOP(n)                                                                               \
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * rows<C>() + threadIdx.x / C; i < (n);       \
       i += static_cast<int64_t>(gridDim.x) * rows<C>())

// R = X - KW (KW given, or W = 0 when kw is null); Z = M^-1 R; P = Z;
// partials of r.z and r.r
template <int C>
__global__ void __launch_bounds__(threads<C>()) k_bcg_start(int64_t n, const double* __restrict__ X,
                                                         const double* __restrict__ kw, VarPrecond M,
                                                         double* __restrict__ R, double* __restrict__ Z,
                                                         double* __restrict__ P, double* __restrict__ part) {
  __shared__ double rt[tile_max<C>()][C];
  const int col = threadIdx.x % C;
  double v[2] = {0.0, 0.0};
  for (int64_t k = blockIdx.x; k * tile<C>() < n; k += gridDim.x) {
    const int64_t lo = tile_start<C>(M, n, k), hi = tile_start<C>(M, n, k + 1);
    __syncthreads();  // the previous tile has been read
    for (int64_t i = lo + threadIdx.x / C; i < hi; i += rows<C>()) {
      const int64_t e = i * C + col;
      const double r = kw ? X[e] - kw[e] : X[e];
      R[e] = r;
      rt[i - lo][col] = r;
    }
    __syncthreads();
    tile_precond<C>(M, lo, hi, rt, [&](int64_t i, double r, double z) {
      const int64_t e = i * C + col;
      Z[e] = z;
      P[e] = z;
      v[0] += r * z;
      v[1] += r * r;
    });
  }
  col_partials<2, C>(v, part);
}

// mode 0: first start (|c|^2 = r.r, a column with c = 0 is never active);
// mode 1: restart from the true residual (active columns stay active)
template <int C>
__global__ void __launch_bounds__(threads<C>()) k_bcg_start_fin(const double* __restrict__ part, int nb,
                                                               BcgScalars* __restrict__ S, double tol2, int mode) {
  double t[2];
  col_totals2<C>(part, nb, t);
  if (threadIdx.x >= C) return;
  const int col = threadIdx.x;
  const double rz = t[0], rr = t[1];
  S->rz[col] = rz;
  S->rr[col] = rr;
  if (mode == 0) {
    S->cc[col] = rr;
    S->active[col] = rr > 0.0 ? 1 : 0;
    if (col == 0) S->status = 0;
  } else {
    S->active[col] = rr > tol2 * S->cc[col] ? 1 : 0;
  }
}

template <int C>
__global__ void __launch_bounds__(threads<C>()) k_bcg_pq(int64_t n, const double* __restrict__ P,
                                                      const double* __restrict__ Q, double* __restrict__ part) {
  // four strided rows loaded at once, added in the order of the plain row loop
  const int col = threadIdx.x % C;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * rows<C>();
  double v[1] = {0.0};
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * rows<C>() + threadIdx.x / C; i < n; i += kRowBatch * stride) {
    double pv[kRowBatch], qv[kRowBatch];
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      const int64_t k = i + u * stride;
      pv[u] = k < n ? P[k * C + col] : 0.0;
      qv[u] = k < n ? Q[k * C + col] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u)
      if (i + u * stride < n) v[0] += pv[u] * qv[u];
  }
  col_partials<1, C>(v, part);
}

template <int C>
__global__ void __launch_bounds__(threads<C>()) k_bcg_alpha(const double* __restrict__ part, int nb,
                                                           BcgScalars* __restrict__ S) {
  const double t[1] = {col_total<1, C>(part, nb)};
  if (threadIdx.x >= C) return;
  const int col = threadIdx.x;
  const double pq = t[0];
  S->pq[col] = pq;
  double a = 0.0;
  if (S->active[col]) {
    if (pq > 0.0 && isfinite(pq)) {
      a = S->rz[col] / pq;
    } else {
      S->status = 1;  // non-positive curvature
      S->active[col] = 0;
    }
  }
  S->alpha[col] = a;
}

// R -= alpha Q; Z = M^-1 R; partials of r.z and r.r.  A block takes whole tiles
// of Jacobi blocks, so R is updated in place.  W += alpha P waits for the
// direction's pass, which reads P anyway: the iteration's vector passes move 11
// blocks of n x 32 instead of 12 (n = 1,095,000: 886 -> 776 us with block Jacobi,
// 646 -> 556 with Jacobi, whose 3.1 GB take 598 us at the rate of a large copy).
template <int C>
__global__ void __launch_bounds__(threads<C>()) k_bcg_update(int64_t n, const BcgScalars* __restrict__ S,
                                                          const double* __restrict__ Q, VarPrecond M,
                                                          double* __restrict__ R, double* __restrict__ Z,
                                                          double* __restrict__ part) {
  __shared__ double rt[tile_max<C>()][C];
  const int col = threadIdx.x % C;
  const double a = S->alpha[col];
  constexpr int kPer = (tile_max<C>() + rows<C>() - 1) / rows<C>();  // rows of a tile per thread
  double v[2] = {0.0, 0.0};
  for (int64_t k = blockIdx.x; k * tile<C>() < n; k += gridDim.x) {
    const int64_t lo = tile_start<C>(M, n, k), hi = tile_start<C>(M, n, k + 1);
    double rv[kPer], qv[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int64_t i = lo + threadIdx.x / C + u * rows<C>();
      rv[u] = i < hi ? R[i * C + col] : 0.0;
      qv[u] = i < hi ? Q[i * C + col] : 0.0;
    }
    __syncthreads();  // the previous tile has been read
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int64_t i = lo + threadIdx.x / C + u * rows<C>();
      if (i < hi) {
        const double r = rv[u] - a * qv[u];
        R[i * C + col] = r;
        rt[i - lo][col] = r;
      }
    }
    __syncthreads();
    tile_precond<C>(M, lo, hi, rt, [&](int64_t i, double r, double z) {
      Z[i * C + col] = z;
      v[0] += r * z;
      v[1] += r * r;
    });
  }
  col_partials<2, C>(v, part);
}

// The same pass with the block product on the matrix cores, for larger blocks
// (kBigBlock): Z[block, 0:C] = Binv R[block, 0:C], b x b times b x C, is a
// dense contraction, and with 16 x 16 x 4 FP64 MFMAs a wave loads each inverse
// entry once for C columns instead of once per row and half-wave (broadcast
// loads, which the address unit serves no faster than scattered ones).  A wave
// takes the tile's blocks in turn; lane (i, kk) = (lane % 16, lane / 16) holds
// A[i][kk] = Binv(16 rb + i, 4 s + kk), B[kk][i] = R(4 s + kk, i) from LDS, and
// of the result the rows 16 rb + kk + 4 v, v = 0..3, of columns i and (C = 32)
// i + 16.  Entries past the block have weight 0; with C = 8 the lanes i >= 8 repeat
// a column and keep nothing.
// Vector work of an iteration, n = 50,021 (mixture, blocks up to 32): 104.3 us with
// each row reading its block's R and Q from memory, 65.4 with k_bcg_update, 54.1
// with this; small blocks only pay the padding (space-time n = 109,500, 2.8 points a
// block: 97.4 with k_bcg_update, 108.9 with this), so it takes mean blocks of more
// than kBigBlock rows (uniform n = 8000, mean 7.6: 26.2 and 25.3).
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int kMThreads = 256;
constexpr int kMWaves = kMThreads / kWave;
constexpr int kMSteps = kMaxBlock / 4;  // k-steps of a block at most
constexpr int kBigBlock = 8;

template <int C>
__global__ void __launch_bounds__(kMThreads) k_bcg_update_mfma(int64_t n, const BcgScalars* __restrict__ S,
                                                               const double* __restrict__ Q, VarPrecond M,
                                                               double* __restrict__ R, double* __restrict__ Z,
                                                               double* __restrict__ part) {
  __shared__ double rt[tile_max<C>()][C];
  __shared__ double red[2][kMWaves][C];
  constexpr int kTRows = kMThreads / C;
  constexpr int kPer = (tile_max<C>() + kTRows - 1) / kTRows;
  const int col = threadIdx.x % C, w = threadIdx.x / kWave, lane = lane_id();
  const int i = lane & 15, kk = lane >> 4;
  const double a = S->alpha[col];
  constexpr int kNB = (C + 15) / 16;
  const bool mine = C >= 16 || i < C;
  double rz[kNB] = {}, rr[kNB] = {};  // of columns i and i + 16
  for (int64_t k = blockIdx.x; k * tile<C>() < n; k += gridDim.x) {
    const int64_t lo = tile_start<C>(M, n, k), hi = tile_start<C>(M, n, k + 1);
    double rv[kPer], qv[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int64_t r = lo + threadIdx.x / C + u * kTRows;
      rv[u] = r < hi ? R[r * C + col] : 0.0;
      qv[u] = r < hi ? Q[r * C + col] : 0.0;
    }
    // the tile's rows lane and lane + 64: where a Jacobi block starts, and its place
    static_assert(tile_max<C>() <= 2 * kWave, "two rows per lane");
    uint64_t place[2], starts[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t r = lo + lane + h * kWave;
      place[h] = r < hi ? M.brow[r] : 0;
      starts[h] = __ballot(r < hi && BlockRow(place[h]).k == 0);
    }
    __syncthreads();  // the previous tile has been read
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int64_t r = lo + threadIdx.x / C + u * kTRows;
      if (r < hi) {
        const double x = rv[u] - a * qv[u];
        R[r * C + col] = x;
        rt[r - lo][col] = x;
      }
    }
    __syncthreads();
    const int nlow = __popcll(starts[0]), nb = nlow + __popcll(starts[1]);
    uint64_t todo = starts[0];
    for (int j = 0, h = 0; j < nb; ++j, todo &= todo - 1) {  // uniform over the wave
      if (j == nlow) {
        todo = starts[1];
        h = 1;
      }
      if (j % kMWaves != w) continue;
      const int src = __builtin_ctzll(todo);
      const BlockRow br(__shfl(place[h], src, kWave));
      const int64_t bs = lo + src + h * kWave;
      const int sz = br.sz;
      const double* binv = M.binv + br.pos;
      const double(*rb)[C] = rt + (bs - lo);
      d4 acc[2][kNB];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int c = 0; c < kNB; ++c) acc[t][c] = d4{0.0, 0.0, 0.0, 0.0};
      double av[2][kMSteps];
#pragma unroll
      for (int s = 0; s < kMSteps; ++s) {
        if (4 * s >= sz) break;  // uniform
        const int q = 4 * s + kk;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int r = 16 * t + i;
          av[t][s] = (q < sz && r < sz) ? binv[q * sz + r] : 0.0;
        }
      }
#pragma unroll
      for (int s = 0; s < kMSteps; ++s) {
        if (4 * s >= sz) break;
        const int q = min(4 * s + kk, sz - 1);
        double b[kNB];
#pragma unroll
        for (int c = 0; c < kNB; ++c) b[c] = rb[q][(i + 16 * c) % C];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          if (16 * t >= sz) break;
#pragma unroll
          for (int c = 0; c < kNB; ++c)
            acc[t][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[t][s], b[c], acc[t][c], 0, 0, 0);
        }
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * t + kk + 4 * v;
          if (r >= sz || !mine) continue;
          double* zr = Z + (bs + r) * C;
#pragma unroll
          for (int c = 0; c < kNB; ++c) {
            const double x = rb[r][i + 16 * c], z = acc[t][c][v];
            zr[i + 16 * c] = z;
            rz[c] += x * z;
            rr[c] += x * x;
          }
        }
    }
  }
  // the four lanes of a column, then the waves in order
#pragma unroll
  for (int c = 0; c < kNB; ++c) {
#pragma unroll
    for (int off = 16; off < kWave; off <<= 1) {
      rz[c] += __shfl_xor(rz[c], off, kWave);
      rr[c] += __shfl_xor(rr[c], off, kWave);
    }
    if (kk == 0 && mine) {
      red[0][w][i + 16 * c] = rz[c];
      red[1][w][i + 16 * c] = rr[c];
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 * C) {
    const int v = threadIdx.x / C;
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < kMWaves; ++q) s += red[v][q][col];
    part[(static_cast<int64_t>(blockIdx.x) * 2 + v) * C + col] = s;
  }
}

template <int C>
__global__ void __launch_bounds__(threads<C>()) k_bcg_beta(const double* __restrict__ part, int nb,
                                                          BcgScalars* __restrict__ S, double tol2) {
  double t[2];
  col_totals2<C>(part, nb, t);
  if (threadIdx.x >= C) return;
  const int col = threadIdx.x;
  const double rz = t[0], rr = t[1];
  const bool act = S->active[col] != 0;
  S->beta[col] = act ? rz / S->rz[col] : 0.0;
  S->rz[col] = rz;
  S->rr[col] = rr;
  S->active[col] = (act && rr > tol2 * S->cc[col]) ? 1 : 0;
}

// W += alpha P, and P = Z + beta P for the active columns (a row per thread)
template <int C>
__global__ void __launch_bounds__(kThreads) k_bcg_dir(int64_t n, const BcgScalars* __restrict__ S,
                                                      const double* __restrict__ Z, double* __restrict__ P,
                                                      double* __restrict__ W) {
  const int col = threadIdx.x % C;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * (kThreads / C) + threadIdx.x / C;
  if (i >= n) return;
  const double a = S->alpha[col], b = S->beta[col];
  const bool act = S->active[col] != 0;
  if (a == 0.0 && !act) return;  // a column that ended earlier
  const int64_t e = i * C + col;
  const double p = P[e], w = W[e], z = act ? Z[e] : 0.0;
  W[e] = w + a * p;
  if (act) P[e] = z + b * p;
}

// partials of the true residual |X - KW|^2 and of X.W per column
template <int C>
__global__ void __launch_bounds__(threads<C>()) k_bcg_final(int64_t n, const double* __restrict__ X,
                                                        const double* __restrict__ kw, const double* __restrict__ W,
                                                        double* __restrict__ part) {
  const int col = threadIdx.x % C;
  double v[2] = {0.0, 0.0};
  ROW_LOOP(n) {
    const int64_t e = i * C + col;
    const double r = X[e] - kw[e];
    v[0] += r * r;
    v[1] += X[e] * W[e];
  }
  col_partials<2, C>(v, part);
}

// true residual per column into S->rr; v_s = prior_s - c_s . w_s for s < nbatch
template <int C>
__global__ void __launch_bounds__(threads<C>()) k_bcg_var(const double* __restrict__ part, int nb,
                                                         BcgScalars* __restrict__ S, const double* __restrict__ prior,
                                                         int nbatch, double* __restrict__ var) {
  double t[2];
  col_totals2<C>(part, nb, t);
  if (threadIdx.x >= C) return;
  const int col = threadIdx.x;
  const double rr = t[0], cw = t[1];
  S->rr[col] = rr;
  if (col < nbatch) var[col] = prior[col] - cw;
}

#undef ROW_LOOP

template <typename F3>
void dispatch_dk(int d, int kind, F3&& f) {
  auto with_d = [&](auto DD) {
    if (kind == GP_CORE_MATERN)
      f(DD, std::integral_constant<int, 1>{});
    else if (kind == GP_CORE_PACIOREK)
      f(DD, std::integral_constant<int, 2>{});
    else
      f(DD, std::integral_constant<int, 0>{});
  };
  if (d == 1)
    with_d(std::integral_constant<int, 1>{});
  else if (d == 2)
    with_d(std::integral_constant<int, 2>{});
  else
    with_d(std::integral_constant<int, 3>{});
}

// Columns of the block that takes nb right-hand sides: the narrowest there is.  An
// iteration in blocks of 1 / 8 / 16 / 32: n = 50,021 (mixture, mixed, block Jacobi)
// 30 / 65 / 80 / 107 us, n = 20,021 (FP64, Jacobi) 27 / 43 / 50 / 73, n = 109,500 (space-time)
// 67 / 135 / 174 / 243; every request took blocks of 32 before.  Two narrow blocks
// cost more than one that holds both, so only the last block of a request is
// narrow.  Widths of 2 and 4 would save little on 8: its small kernels are at
// their latency.
int width(int nb) { return nb <= 1 ? 1 : nb <= 8 ? 8 : nb <= 16 ? 16 : kC; }

}  // namespace

VarResult predict_variance(gp_ctx* c, const gp_matrix* m, const gp_theta* th, int64_t ntest, const double* xs,
                           double rtol, int max_iter, int precond, double* var) {
  VarResult res;
  if (ntest == 0) return res;
  VarPrecond M{m->diag, nullptr, nullptr};
  if (precond == GP_PRECOND_BLOCK_JACOBI) {
    // the inverses are cached in the matrix object on first use
    gp_matrix* mm = const_cast<gp_matrix*>(m);
    build_block_jacobi(c, mm);
    M.brow = mm->brow;
    M.binv = mm->binv;
  }
  const gp_dataset* ds = m->ds;
  const int64_t n = m->n;
  const int d = ds->d;
  Bump* bumps = nullptr;
  KernelTheta kt{};
  upload_theta(c, th, &bumps, &kt);
  CoreBasis cb{};
  core_params(th, &kt.core, &cb);
  if (kt.core.kind == GP_CORE_PACIOREK) {
    double* sig = static_cast<double*>(workspace(c, 92, sizeof(double) * n));
    double* Sig = static_cast<double*>(workspace(c, 93, sizeof(double) * n));
    core_fields(c, ds, cb, sig, Sig);
    kt.core.sig = sig;
    kt.core.Sig = Sig;
  }
  Features f;
  if (th->n1 > 0) compute_features(c, ds, kt, &f, 100);
  const Grid grid = make_grid(ds, th);
  CrossArgs a{};
  a.kt = kt;
  a.n = n;
  a.xb = ds->xb;
  a.cell_start = ds->cell_start;
  for (int k = 0; k < 3; ++k) {
    a.lo[k] = ds->lo[k];
    a.cell[k] = ds->cell[k];
    a.g[k] = ds->g[k];
    a.R[k] = grid.Rt[k];
  }
  a.nm = f.nm;
  a.mlist = f.mlist;
  a.mmask = f.mmask;
  a.F = f.F;

  // the widest block of right-hand sides of the request (see width)
  const int cmax = width(static_cast<int>(std::min<int64_t>(kC, ntest)));
  const size_t blk = sizeof(double) * n * cmax;
  double* X = static_cast<double*>(workspace(c, 110, blk));
  double* R = static_cast<double*>(workspace(c, 111, blk));
  double* Z = static_cast<double*>(workspace(c, 112, blk));
  double* P = static_cast<double*>(workspace(c, 113, blk));
  double* Q = static_cast<double*>(workspace(c, 114, blk));
  double* W = static_cast<double*>(workspace(c, 115, blk));
  double* part = static_cast<double*>(workspace(c, 116, sizeof(double) * 2 * kVBlocks * 2 * kC));
  BcgScalars* S = static_cast<BcgScalars*>(workspace(c, 117, sizeof(BcgScalars)));
  double* prior = static_cast<double*>(workspace(c, 118, sizeof(double) * kC));
  BcgScalars* hs = static_cast<BcgScalars*>(pinned(c, sizeof(BcgScalars)));
  // the matrix-core update pays for padding to 16 rows: see kBigBlock
  const bool mfma = M.binv && m->binv_len > kBigBlock * n;  // sum of b^2 over sum of b: the block a row sees on average
  const double tol2 = rtol * rtol;
  auto read = [&]() {
    GPS_HIP(hipMemcpyAsync(hs, S, sizeof(BcgScalars), hipMemcpyDeviceToHost, c->stream));
    sync(c);
    return *hs;
  };
  // test points m0 .. m0 + nb - 1 in a block of C >= nb columns
  auto batch = [&](auto CC, int64_t m0, int nb) {
    constexpr int C = decltype(CC)::value;
    const double* xb = xs + m0 * d;
    const int64_t ntiles = (n + tile<C>() - 1) / tile<C>();
    const unsigned nbv = static_cast<unsigned>(std::min<int64_t>(kVBlocks, ntiles));
    const unsigned nbm = static_cast<unsigned>(std::min<int64_t>(2 * kVBlocks, ntiles));
    const dim3 B(kThreads), RB(threads<C>()), G(nbv), FB(threads<C>());
    auto product = [&](const double* V, double* out) {
      if constexpr (C == 1)
        spmv_f64(c, m, V, out);
      else
        spmm<double>(c, m, C, C, V, out, nullptr);
    };
    // element-wise kernels without a reduction take a row per thread
    const dim3 Gfull(static_cast<unsigned>(grid_for(n * C, kThreads)));
    {
      ProfScope ps(c, "var_cross");
      hipLaunchKernelGGL(k_zero, dim3(grid_for(n * C, kThreads)), B, 0, c->stream, n * C, X);
      dispatch_dk(d, kt.core.kind, [&](auto DD, auto CC) {
        constexpr int D = decltype(DD)::value;
        constexpr int CK = decltype(CC)::value;
        hipLaunchKernelGGL((k_cross_local<D, CK>), dim3(nb), B, 0, c->stream, a, cb, nb, C, xb, X);
        const unsigned share = std::min<unsigned>(kGroupBlocks, grid_for(a.nm, kGroupShare * (kThreads / kWave)));
        hipLaunchKernelGGL((k_cross_groups<D, CK>), dim3(nb, share), B, 0, c->stream, a, cb, nb, C, xb, X, prior);
      });
      check_launch("variance cross-covariance");
    }
    hipLaunchKernelGGL(k_zero, dim3(grid_for(n * C, kThreads)), B, 0, c->stream, n * C, W);
    hipLaunchKernelGGL(k_bcg_start<C>, G, RB, 0, c->stream, n, X, nullptr, M, R, Z, P, part);
    hipLaunchKernelGGL(k_bcg_start_fin<C>, dim3(1), FB, 0, c->stream, part, static_cast<int>(nbv), S, tol2, 0);
    check_launch("variance start");
    BcgScalars hsc = read();
    int it = 0, refresh = 0;
    auto any_active = [](const BcgScalars& s) {
      for (int j = 0; j < C; ++j)
        if (s.active[j]) return true;
      return false;
    };
    while (hsc.status == 0 && it < max_iter) {
      if (!any_active(hsc)) {
        // recurrences done: check the float64 true residual, restart once it is not small enough
        if (refresh >= kMaxRefresh) break;
        product(W, Q);
        hipLaunchKernelGGL(k_bcg_start<C>, G, RB, 0, c->stream, n, X, Q, M, R, Z, P, part);
        hipLaunchKernelGGL(k_bcg_start_fin<C>, dim3(1), FB, 0, c->stream, part, static_cast<int>(nbv), S, tol2, 1);
        check_launch("variance restart");
        ++refresh;
        hsc = read();
        if (!any_active(hsc)) break;
        continue;
      }
      const int steps = std::min(kCheckEvery, max_iter - it);
      for (int t = 0; t < steps; ++t) {
        product(P, Q);
        ProfScope ps(c, "var_vector_ops");
        hipLaunchKernelGGL(k_bcg_pq<C>, G, RB, 0, c->stream, n, P, Q, part);
        hipLaunchKernelGGL(k_bcg_alpha<C>, dim3(1), FB, 0, c->stream, part, static_cast<int>(nbv), S);
        unsigned np = nbv;
        if constexpr (C >= 8) {
          if (mfma) {
            np = nbm;
            hipLaunchKernelGGL(k_bcg_update_mfma<C>, dim3(nbm), B, 0, c->stream, n, S, Q, M, R, Z, part);
          }
        }
        if (C < 8 || !mfma) hipLaunchKernelGGL(k_bcg_update<C>, G, RB, 0, c->stream, n, S, Q, M, R, Z, part);
        hipLaunchKernelGGL(k_bcg_beta<C>, dim3(1), FB, 0, c->stream, part, static_cast<int>(np), S, tol2);
        hipLaunchKernelGGL(k_bcg_dir<C>, Gfull, B, 0, c->stream, n, S, Z, P, W);
        check_launch("variance step");
      }
      it += steps;
      hsc = read();
    }
    // true residual and the variances of this batch
    product(W, Q);
    hipLaunchKernelGGL(k_bcg_final<C>, G, RB, 0, c->stream, n, X, Q, W, part);
    hipLaunchKernelGGL(k_bcg_var<C>, dim3(1), FB, 0, c->stream, part, static_cast<int>(nbv), S, prior, nb, var + m0);
    check_launch("variance final");
    hsc = read();
    res.iters += it;
    res.max_batch_iters = std::max(res.max_batch_iters, it);
    bool ok = hsc.status == 0;
    for (int j = 0; j < nb; ++j) {
      const double rel = hsc.cc[j] > 0.0 ? std::sqrt(hsc.rr[j] / hsc.cc[j]) : 0.0;
      res.relres = std::max(res.relres, rel);
      if (!(rel <= rtol)) ok = false;
    }
    if (hsc.status != 0)
      res.st = GP_ENOTPD;
    else if (!ok && res.st == GP_OK)
      res.st = GP_ENOTCONV;
  };
  for (int64_t m0 = 0; m0 < ntest; m0 += kC) {
    const int nb = static_cast<int>(std::min<int64_t>(kC, ntest - m0));
    switch (width(nb)) {
      case 1:
        batch(std::integral_constant<int, 1>{}, m0, nb);
        break;
      case 8:
        batch(std::integral_constant<int, 8>{}, m0, nb);
        break;
      case 16:
        batch(std::integral_constant<int, 16>{}, m0, nb);
        break;
      default:
        batch(std::integral_constant<int, 32>{}, m0, nb);
    }
  }
  return res;
}

}  // namespace gps
