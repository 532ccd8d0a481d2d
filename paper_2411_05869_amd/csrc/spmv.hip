// CSR products with the assembled matrix (binned order).
//
// SpMV: rows with at most kLongRow entries are handled by groups of G lanes
// (G consecutive lanes stride over the row, then a fixed shuffle tree sums
// the partials), longer rows by one wave each (listed at assembly).  Every
// row's sum is formed in the same order on every call, so results are
// bitwise reproducible; no floating-point atomics are used.
//
// SpMM: k <= 32 right-hand sides, X and Y row-major n x ld, optional
// symmetric diagonal scaling Y = S K S X (32 columns: k_spmm_quad, k_spmm_long; fewer: k_spmm_rows).
#include <algorithm>
#include <type_traits>

#include "device.hpp"

namespace gps {
namespace {

constexpr int kThreads = 256;
constexpr int kG = 8;


inline unsigned round_up8(unsigned v) { return (v + 7u) & ~7u; }

// Partial row sum over entries [s, e) for lane `sub` of a group of G lanes: each
// lane takes 4 consecutive entries at a time (column ids and values by one
// 16-byte load each; a load may run up to 3 entries past the row, which stays
// inside the padded arrays) and gathers their 4 x values together.  Entries past
// the row end read x[self] with weight 0.
template <typename VT, typename XT, typename AT, int G>
__device__ __forceinline__ AT spmv_part(int64_t s, int64_t e, int sub, int32_t self, const int32_t* __restrict__ col,
                                        const VT* __restrict__ val, const XT* __restrict__ x) {
  AT acc = 0;
  for (int64_t j0 = s + 4 * sub; j0 < e; j0 += 4 * G) {
    int32_t c[4];
    VT v[4];
    __builtin_memcpy(c, col + j0, sizeof(c));
    __builtin_memcpy(v, val + j0, sizeof(v));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = j0 + u < e;
      c[u] = in ? c[u] : self;
      v[u] = in ? v[u] : VT(0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc += static_cast<AT>(v[u]) * static_cast<AT>(x[c[u]]);
  }
  return acc;
}

// The same sum with the column ids stored as int16 offsets from the row.
template <typename VT, typename XT, typename AT, int G>
__device__ __forceinline__ AT spmv_part16(int64_t s, int64_t e, int sub, int32_t self, const int16_t* __restrict__ off,
                                          const VT* __restrict__ val, const XT* __restrict__ x) {
  AT acc = 0;
  for (int64_t j0 = s + 4 * sub; j0 < e; j0 += 4 * G) {
    int16_t o[4];
    VT v[4];
    __builtin_memcpy(o, off + j0, sizeof(o));
    __builtin_memcpy(v, val + j0, sizeof(v));
    int32_t c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = j0 + u < e;
      c[u] = in ? self + static_cast<int32_t>(o[u]) : self;
      v[u] = in ? v[u] : VT(0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc += static_cast<AT>(v[u]) * static_cast<AT>(x[c[u]]);
  }
  return acc;
}

// CSR part of the product (entries after each row's leading group entries).
// With off16 (int16 offsets col - row, two bytes per entry instead of four)
// the short rows read the offsets; the long rows always read col.
// One launch: blocks [0, nb_long) take the listed long rows, one wave per row
// (dispatched first, they set the tail); the remaining blocks take rows of at
// most kLongRow entries with kG lanes per row.  Rows with group entries add
// the group-block part that k_group_spmv wrote to y before.
template <typename VT, typename XT, typename AT, typename YT, bool PERM>
__global__ void __launch_bounds__(kThreads) k_spmv(int64_t n, unsigned nb_long, int64_t nlong,
                                                   const int32_t* __restrict__ rows, const int64_t* __restrict__ rp,
                                                   const int32_t* __restrict__ gskip,
                                                   const int32_t* __restrict__ col, const VT* __restrict__ val,
                                                   const XT* __restrict__ x, const YT* y, RowDest<YT> out,
                                                   const int16_t* __restrict__ off16, const int* __restrict__ skip) {
  if (skip && *skip) return;  // a device-side decision cancelled this product
  solve_wave_priority();
  if (blockIdx.x >= nb_long) {
    const unsigned b = xcd_remap(blockIdx.x - nb_long, gridDim.x - nb_long);
    const int64_t row = (b * static_cast<int64_t>(kThreads) + threadIdx.x) / kG;
    const int sub = threadIdx.x & (kG - 1);
    if (row < n) {
      const int32_t gs = gskip[row];
      const int64_t s = rp[row] + gs, e = rp[row + 1];
      if (e - s <= kLongRow) {  // uniform within the group
        AT acc = off16 ? spmv_part16<VT, XT, AT, kG>(s, e, sub, static_cast<int32_t>(row), off16, val, x)
                       : spmv_part<VT, XT, AT, kG>(s, e, sub, static_cast<int32_t>(row), col, val, x);
#pragma unroll
        for (int off = kG / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kG);
        if (sub == 0) *out.template row<PERM>(row, 1) = static_cast<YT>(gs ? static_cast<AT>(y[row]) + acc : acc);
      }
    }
  } else {
    const unsigned b = xcd_remap(blockIdx.x, nb_long);
    const int64_t w = (b * static_cast<int64_t>(kThreads) + threadIdx.x) / kWave;
    if (w < nlong) {
      const int lane = lane_id();
      const int32_t row = rows[w];
      const int32_t gs = gskip[row];
      const int64_t s = rp[row] + gs, e = rp[row + 1];
      AT acc = spmv_part<VT, XT, AT, kWave>(s, e, lane, row, col, val, x);
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
      if (lane == 0) *out.template row<PERM>(row, 1) = static_cast<YT>(gs ? static_cast<AT>(y[row]) + acc : acc);
    }
  }
}

// SpMM, Y = S K S X (S = diag(scale), or K X without scale), k <= 32 columns of
// a row-major block with leading dimension ld.  Blocks of 32 aligned columns take
// the row quads (k_spmm_quad) and, for rows of more than kLongRow entries, a
// block per row (k_spmm_long); fewer columns take k_spmm_rows.

// orders the LDS accesses of one wave (its own slice; no block barrier)
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T>
__device__ __forceinline__ T shfl_any(T v, int src) {
  return __shfl(v, src, kWave);
}

// lane l stages entry j0 + l of [j0, e): its column id q (self when past the
// end) and weight v (0 past the end)
template <typename VT, typename T, bool SCALE>
__device__ __forceinline__ void spmm_stage(int64_t j0, int64_t e, int32_t self, const int32_t* __restrict__ col,
                                           const VT* __restrict__ val, const T* __restrict__ scale, int lane,
                                           int32_t& q, T& v) {
  const int64_t j = j0 + lane;
  q = self;
  v = 0;
  if (j < e) {
    q = col[j];
    v = static_cast<T>(val[j]);
    if constexpr (SCALE) v *= scale[q];
  }
}

// Sum over the m staged entries of v * X[q, columns] with 16-byte X loads, for
// blocks whose rows hold at least 32 values at 16-byte alignment: lane l works
// on the kCpl consecutive columns
// kCpl (l % kLpe) ... of entry slot l / kLpe, so one load instruction serves
// kWave / kLpe entries.  Returns the lane's kCpl partial sums; the slots are
// added by the caller.
template <typename T>
struct Vec16 {
  static constexpr int kCpl = 16 / sizeof(T);   // columns per lane
  static constexpr int kLpe = 32 / kCpl;         // lanes per entry
  static constexpr int kEpi = kWave / kLpe;      // entries per load instruction
  T v[kCpl];
};
constexpr int kUq = 4;

template <typename T>
__device__ __forceinline__ Vec16<T> spmm_consume16(int32_t q, T v, int m, const T* __restrict__ X, int ld,
                                                    int lane) {
  using V = Vec16<T>;
  const int g = lane / V::kLpe, cp = lane % V::kLpe;
  const int nq = (m + V::kEpi - 1) / V::kEpi;
  V acc;
#pragma unroll
  for (int u = 0; u < V::kCpl; ++u) acc.v[u] = 0;
  for (int i0 = 0; i0 < nq; i0 += kUq) {
    int32_t qq[kUq];
    T vv[kUq];
#pragma unroll
    for (int u = 0; u < kUq; ++u) {
      const int src = (V::kEpi * (i0 + u) + g) & (kWave - 1);  // entries past m carry weight 0
      qq[u] = shfl_any(q, src);
      vv[u] = shfl_any(v, src);
      if (i0 + u >= nq) vv[u] = 0;
    }
    V xv[kUq];
#pragma unroll
    for (int u = 0; u < kUq; ++u) __builtin_memcpy(xv[u].v, X + static_cast<int64_t>(qq[u]) * ld + cp * V::kCpl, 16);
#pragma unroll
    for (int u = 0; u < kUq; ++u)
#pragma unroll
      for (int t = 0; t < V::kCpl; ++t) acc.v[t] += vv[u] * xv[u].v[t];
  }
  return acc;
}

// adds the entry slots of spmm_consume16 (lanes l, l + kLpe, ...), fixed order
template <typename T>
__device__ __forceinline__ void slot_sum(Vec16<T>& a) {
#pragma unroll
  for (int off = Vec16<T>::kLpe; off < kWave; off <<= 1)
#pragma unroll
    for (int t = 0; t < Vec16<T>::kCpl; ++t) a.v[t] += __shfl_xor(a.v[t], off, kWave);
}

// Rows of more than kLongRow entries past their group part, a block each: a wave
// stages 64 consecutive entries at a time (lane l entry l, column id and value *
// scale[column], one coalesced access), wave w the chunks w, w + 4, ...; all X
// gathers of a chunk are independent, so kUq of them are in flight per lane.  The
// four partial rows are added in a fixed order, after the group part already in Y.
template <typename VT, typename T, bool SCALE, bool PERM>
__global__ void __launch_bounds__(kThreads) k_spmm_long(int64_t nlong, const int32_t* __restrict__ rows, int k, int ld,
                                                        const int64_t* __restrict__ rp,
                                                        const int32_t* __restrict__ gskip,
                                                        const int32_t* __restrict__ col, const VT* __restrict__ val,
                                                        const T* __restrict__ X, const T* Y,
                                                        RowDest<T> out, const T* __restrict__ scale,
                                                        const double* __restrict__ colscale) {
  using V = Vec16<T>;
  __shared__ T part[kThreads / kWave][32];
  const int lane = lane_id(), w = threadIdx.x / kWave;
  const int64_t li = xcd_remap(blockIdx.x, gridDim.x);
  if (li >= nlong) return;  // uniform over the block
  const int32_t row = rows[li];
  const int32_t gs = gskip[row];
  const int64_t s = rp[row] + gs, e = rp[row + 1];
  V acc;
#pragma unroll
  for (int t = 0; t < V::kCpl; ++t) acc.v[t] = 0;
  for (int64_t j0 = s + static_cast<int64_t>(w) * kWave; j0 < e; j0 += kThreads) {
    int32_t q;
    T v;
    spmm_stage<VT, T, SCALE>(j0, e, row, col, val, scale, lane, q, v);
    const V a = spmm_consume16<T>(q, v, static_cast<int>(min<int64_t>(e - j0, kWave)), X, ld, lane);
#pragma unroll
    for (int t = 0; t < V::kCpl; ++t) acc.v[t] += a.v[t];
  }
  slot_sum<T>(acc);
  if (lane < V::kLpe)
#pragma unroll
    for (int t = 0; t < V::kCpl; ++t) part[w][lane * V::kCpl + t] = acc.v[t];
  __syncthreads();
  const int c = threadIdx.x;
  if (c >= k) return;
  T t = part[0][c];
#pragma unroll
  for (int i = 1; i < kThreads / kWave; ++i) t += part[i][c];
  if (gs) t = Y[static_cast<int64_t>(row) * ld + c] + t;
  if constexpr (SCALE) t *= scale[row];
  if (colscale) t *= colscale[c];
  out.template row<PERM>(row, ld)[c] = t;
}

// CSR part of the product with fewer than 32 columns (any k <= W, any ld).  A row
// is the work of L lanes in slots of W, a lane per column.  The L lanes stage L
// consecutive entries (a lane each: id and weight) in their LDS slice; each slot
// then takes its entries from there and its lanes read their column of the X row,
// so an entry costs one read of its id and value and one of its k columns.  Two
// columns leave too few steps to a chunk for that to pay: there a slot takes four
// consecutive entries itself, as in the one-column product.
// Blocks [0, nb_long) take the listed long rows, a block each; the others rows
// row0 .. n - 1.
// Bound by the gathers of X through the caches.  A wave per row and 32 columns
// whatever k was, as before, took as long for 2 columns as for 31; the whole
// product by columns, before -> now: n = 100,003 (mixture, FP64) 2: 187 -> 65 us, 8: 183 -> 88,
// 16: 184 -> 116, 31: 197 -> 173; n = 1,095,000 (space-time, mixed) 2: 1062 -> 286, 8: 1058 -> 476,
// 16: 1134 -> 728, 31: 1332 -> 1264.  Reading an entry in every lane of its slot
// instead of staging: 8: 107 and 539 us, 16: 153 and 901.
template <int W>
constexpr int row_lanes() { return W <= 8 ? 16 : 2 * W; }  // lanes of a row
constexpr int kRowUq = 4;  // X rows a lane has in flight
// Blocks of a launch at most (whole eighths, see xcd_remap): a grid of 2^32 threads
// or more loses its upper bits without an error.
constexpr int64_t kLaunchBlocks = (int64_t(1) << 32) / kThreads - 8;
template <int W, int L>
constexpr int row_chunk() { return W < kRowUq ? L / W * kRowUq : L; }  // entries the lanes take at a time

template <int W, int L, typename VT, typename T, bool SCALE>
__device__ __forceinline__ T spmm_part(int64_t s, int64_t e, int64_t stride, int32_t self, int32_t* sq, T* sv,
                                       const int32_t* __restrict__ col, const int16_t* __restrict__ off16,
                                       const VT* __restrict__ val, const T* __restrict__ X, int64_t ld,
                                       const T* __restrict__ scale) {
  constexpr int kSlots = L / W, kU = kRowUq;
  const int l = lane_id() % L, slot = l / W;
  T acc = 0;
  if constexpr (W < kU) {
    for (int64_t j1 = s + kU * slot; j1 < e; j1 += stride) {
      // (a load may run up to three entries past the row, into the padding at most)
      int32_t q[kU];
      VT raw[kU];
      if (off16) {
        int16_t o[kU];
        __builtin_memcpy(o, off16 + j1, sizeof(o));
#pragma unroll
        for (int u = 0; u < kU; ++u) q[u] = self + static_cast<int32_t>(o[u]);
      } else {
        __builtin_memcpy(q, col + j1, sizeof(q));
      }
      __builtin_memcpy(raw, val + j1, sizeof(raw));
      T xv[kU], wv[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const bool in = j1 + u < e;
        q[u] = in ? q[u] : self;
        wv[u] = in ? static_cast<T>(raw[u]) : T(0);
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        xv[u] = X[q[u] * ld];
        if constexpr (SCALE) wv[u] *= scale[q[u]];
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) acc += wv[u] * xv[u];
    }
  } else {
    int32_t q = self;
    T v = 0;
    auto load = [&](int64_t j0) {
      const int64_t j = j0 + l;
      q = self;
      v = 0;
      if (j < e) {
        q = off16 ? self + static_cast<int32_t>(off16[j]) : col[j];
        v = static_cast<T>(val[j]);
        if constexpr (SCALE) v *= scale[q];
      }
    };
    load(s);
    for (int64_t j0 = s; j0 < e; j0 += stride) {
      wave_sync_lds();  // the previous entries have been read
      sq[l] = q;
      sv[l] = v;
      wave_sync_lds();
      const int m = static_cast<int>(min<int64_t>(L, e - j0));
      load(j0 + stride);  // in flight while these are consumed
      for (int u0 = 0; u0 * kSlots < m; u0 += kU) {
        T xv[kU], wv[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int i = (u0 + u) * kSlots + slot;  // past m: the row itself, weight 0
          wv[u] = sv[i];
          xv[u] = X[sq[i] * ld];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) acc += wv[u] * xv[u];
      }
    }
  }
#pragma unroll
  for (int off = W; off < L; off <<= 1) acc += __shfl_xor(acc, off, kWave);
  return acc;
}

template <typename VT, typename T, bool SCALE, bool PERM, int W>
__global__ void __launch_bounds__(kThreads) k_spmm_rows(int64_t row0, int64_t n, unsigned nb_long, int64_t nlong,
                                                        const int32_t* __restrict__ rows, int k, int ld,
                                                        const int64_t* __restrict__ rp,
                                                        const int32_t* __restrict__ gskip,
                                                        const int32_t* __restrict__ col,
                                                        const int16_t* __restrict__ off16,
                                                        const VT* __restrict__ val, const T* __restrict__ X,
                                                        const T* Y, RowDest<T> out,
                                                        const T* __restrict__ scale,
                                                        const double* __restrict__ colscale) {
  constexpr int kL = row_lanes<W>();
  __shared__ int32_t sq[kThreads];
  __shared__ T sv[kThreads];
  const int lane = lane_id(), c = lane % W;
  const T* Xc = X + min(c, k - 1);  // lanes past k re-read column k - 1 and store nothing
  auto finish = [&](int64_t row, int32_t gs, T t) {
    if (gs) t = Y[row * ld + c] + t;
    if constexpr (SCALE) t *= scale[row];
    if (colscale) t *= colscale[c];
    out.template row<PERM>(row, ld)[c] = t;
  };
  if (blockIdx.x >= nb_long) {
    const unsigned b = xcd_remap(blockIdx.x - nb_long, gridDim.x - nb_long);
    const int64_t row = row0 + (b * static_cast<int64_t>(kThreads) + threadIdx.x) / kL;
    if (row >= n) return;
    const int32_t gs = gskip[row];
    const int64_t s = rp[row] + gs, e = rp[row + 1];
    if (e - s > kLongRow) return;  // uniform over the row's lanes
    const int base = threadIdx.x / kL * kL;
    const T acc = spmm_part<W, kL, VT, T, SCALE>(s, e, row_chunk<W, kL>(), static_cast<int32_t>(row), sq + base,
                                                 sv + base, col, off16, val, Xc, ld, scale);
    if (lane % kL < k) finish(row, gs, acc);
  } else {
    __shared__ T part[kThreads / kWave][W];
    const int64_t li = xcd_remap(blockIdx.x, nb_long);
    if (li >= nlong) return;  // uniform over the block
    const int32_t row = rows[li];
    const int32_t gs = gskip[row];
    constexpr int kChunk = row_chunk<W, kWave>();
    const int w = threadIdx.x / kWave, base = w * kWave;
    const T acc = spmm_part<W, kWave, VT, T, SCALE>(rp[row] + gs + w * kChunk, rp[row + 1], kThreads / kWave * kChunk,
                                                    row, sq + base, sv + base, col, nullptr, val, Xc, ld, scale);
    if (lane < W) part[w][lane] = acc;
    __syncthreads();
    if (static_cast<int>(threadIdx.x) >= k) return;
    T t = part[0][c];
#pragma unroll
    for (int i = 1; i < kThreads / kWave; ++i) t += part[i][c];
    finish(row, gs, t);
  }
}

// Group-block part of the product: for the rows of one tile (same mask M,
// at most kTileRows rows) y[row] = sum_k val[row, k] x[U_M[k]] over the
// row's leading |U_M| entries.  x[U_M] is staged in LDS one chunk at a time
// and each staged value serves the four rows a wave owns.
constexpr int kGChunk = 1024;

constexpr int kWaves = kThreads / kWave;
constexpr int kWaveRows = kTileRows / kWaves;  // rows of a tile a wave owns: w, w + kWaves, ...

// The sums of the wave's rows of tile t over their leading |U_M| entries, in
// every lane (0 for rows the tile does not have).
template <typename VT, typename XT, typename AT>
__device__ __forceinline__ void tile_gemv(const int4& t, const int32_t* __restrict__ grows,
                                          const int64_t* __restrict__ uoff, const int32_t* __restrict__ ulist,
                                          const int64_t* __restrict__ rp, const VT* __restrict__ val,
                                          const XT* __restrict__ x, AT (&acc)[kWaveRows]) {
  __shared__ AT xs[kGChunk];
  const int32_t* U = ulist + uoff[t.x];
  const int64_t nU = uoff[t.x + 1] - uoff[t.x];
  const int w = threadIdx.x / kWave, lane = lane_id();
  int64_t base[kWaveRows];
  bool has[kWaveRows];
#pragma unroll
  for (int r = 0; r < kWaveRows; ++r) {
    const int i = w + r * kWaves;
    has[r] = i < t.z;
    base[r] = has[r] ? rp[grows[t.y + i]] : 0;
  }
#pragma unroll
  for (int r = 0; r < kWaveRows; ++r) acc[r] = 0;
  constexpr int kPer = kGChunk / kThreads;
  AT xr[kPer];
  auto load = [&](int64_t c0) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int64_t k = c0 + threadIdx.x + i * kThreads;
      xr[i] = k < nU ? static_cast<AT>(x[U[k]]) : AT(0);
    }
  };
  load(0);
  for (int64_t c0 = 0; c0 < nU; c0 += kGChunk) {
    const int clen = static_cast<int>(min<int64_t>(kGChunk, nU - c0));
    __syncthreads();  // the previous chunk has been consumed
#pragma unroll
    for (int i = 0; i < kPer; ++i) xs[threadIdx.x + i * kThreads] = xr[i];
    __syncthreads();
    if (c0 + kGChunk < nU) load(c0 + kGChunk);   // in flight while this chunk is consumed
    // lane takes entries k .. k + 3 (one 16-byte load per row for float32
    // values; a load may run past the row's group entries, into the row's
    // CSR part, the next row or the zeroed padding after the last row, and
    // those entries get weight 0); one such group per row at a time
    // keeps the kernel at 80 registers (6 waves per SIMD), which measured
    // faster than two groups in flight at 4 waves per SIMD
    for (int k = 4 * lane; k < clen; k += 4 * kWave) {
      VT v[kWaveRows][4];
#pragma unroll
      for (int r = 0; r < kWaveRows; ++r) __builtin_memcpy(v[r], val + base[r] + c0 + k, 4 * sizeof(VT));
      AT xk[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) xk[u] = k + u < clen ? xs[min(k + u, kGChunk - 1)] : AT(0);
#pragma unroll
      for (int r = 0; r < kWaveRows; ++r)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[r] += (has[r] ? static_cast<AT>(v[r][u]) : AT(0)) * xk[u];
    }
  }
#pragma unroll
  for (int r = 0; r < kWaveRows; ++r)
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) acc[r] += __shfl_xor(acc[r], off, kWave);
}

template <typename VT, typename XT, typename AT, typename YT>
__global__ void __launch_bounds__(kThreads) k_group_spmv(const int32_t* __restrict__ tiles,
                                                         const int32_t* __restrict__ grows,
                                                         const int64_t* __restrict__ uoff,
                                                         const int32_t* __restrict__ ulist,
                                                         const int64_t* __restrict__ rp, const VT* __restrict__ val,
                                                         const XT* __restrict__ x, YT* __restrict__ y,
                                                         const int* __restrict__ skip) {
  if (skip && *skip) return;  // uniform over the launch
  solve_wave_priority();
  // tiles come largest first; block b runs on XCD b % 8, so every XCD gets an
  // equal share of large and small tiles and the small ones fill the tail
  const int4 t = reinterpret_cast<const int4*>(tiles)[blockIdx.x];
  AT acc[kWaveRows];
  tile_gemv<VT, XT, AT>(t, grows, uoff, ulist, rp, val, x, acc);
  const int w = threadIdx.x / kWave;
#pragma unroll
  for (int r = 0; r < kWaveRows; ++r)
    if (lane_id() == 0 && w + r * kWaves < t.z) y[grows[t.y + w + r * kWaves]] = static_cast<YT>(acc[r]);
}

// Both parts in one launch, for products short enough that the second launch,
// and not the memory, is what they wait for (kOneLaunchEntries).  A tile's
// block adds its rows' CSR parts to their group parts; the long rows without a
// group part take a wave each, the other rows kG lanes.  Every row is summed in
// the order of the two kernels.  Blocks: tiles, then nb_long, then rows.
//
// WAVES: waves per SIMD its registers are held to (one_waves).
template <typename VT, bool PERM, int WAVES>
__global__ void __launch_bounds__(kThreads, WAVES) k_spmv_one(int64_t n, unsigned ntiles, unsigned nb_long, int64_t nlong,
                                                       const int32_t* __restrict__ tiles,
                                                       const int32_t* __restrict__ grows,
                                                       const int64_t* __restrict__ uoff,
                                                       const int32_t* __restrict__ ulist,
                                                       const int32_t* __restrict__ long_rows,
                                                       const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ gskip,
                                                       const int32_t* __restrict__ col, const VT* __restrict__ val,
                                                       const double* __restrict__ x, RowDest<double> out,
                                                       const int16_t* __restrict__ off16,
                                                       const int* __restrict__ skip) {
  if (skip && *skip) return;  // uniform over the launch
  solve_wave_priority();
  const int w = threadIdx.x / kWave, lane = lane_id(), sub = threadIdx.x & (kG - 1);
  auto short_row = [&](int64_t s, int64_t e, int32_t row) {  // by kG lanes
    double acc = off16 ? spmv_part16<VT, double, double, kG>(s, e, sub, row, off16, val, x)
                       : spmv_part<VT, double, double, kG>(s, e, sub, row, col, val, x);
#pragma unroll
    for (int off = kG / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kG);
    return acc;
  };
  auto long_row = [&](int64_t s, int64_t e, int32_t row) {  // by the wave
    double acc = spmv_part<VT, double, double, kWave>(s, e, lane, row, col, val, x);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
    return acc;
  };
  if (blockIdx.x < ntiles) {
    const int4 t = reinterpret_cast<const int4*>(tiles)[blockIdx.x];
    // lanes kG r .. kG r + kG - 1 take the CSR part of the wave's row r
    const int r8 = lane / kG;
    const bool own = r8 < kWaveRows && w + r8 * kWaves < t.z;
    int32_t row = 0;
    int64_t s = 0, e = 0;
    if (own) {
      row = grows[t.y + w + r8 * kWaves];
      s = rp[row] + gskip[row];
      e = rp[row + 1];
    }
    const bool lng = e - s > kLongRow;
    double csr = short_row(s, lng ? s : e, row);
    for (uint64_t todo = __ballot(lng && sub == 0); todo; todo &= todo - 1) {  // uniform
      const int src = __builtin_ctzll(todo);
      const double a = long_row(__shfl(s, src, kWave), __shfl(e, src, kWave), __shfl(row, src, kWave));
      if (lane == src) csr = a;
    }
    double acc[kWaveRows], mine = 0.0;
    tile_gemv<VT, double, double>(t, grows, uoff, ulist, rp, val, x, acc);
#pragma unroll
    for (int r = 0; r < kWaveRows; ++r)
      if (r == r8) mine = acc[r];
    if (own && sub == 0) *out.template row<PERM>(row, 1) = mine + csr;
  } else if (blockIdx.x < ntiles + nb_long) {
    const int64_t i = static_cast<int64_t>(blockIdx.x - ntiles) * kWaves + w;
    if (i < nlong) {
      const int32_t row = long_rows[i];
      if (gskip[row] == 0) {
        const double a = long_row(rp[row], rp[row + 1], row);
        if (lane == 0) *out.template row<PERM>(row, 1) = a;
      }
    }
  } else {
    const unsigned b = xcd_remap(blockIdx.x - ntiles - nb_long, gridDim.x - ntiles - nb_long);
    const int64_t row = (b * static_cast<int64_t>(kThreads) + threadIdx.x) / kG;
    if (row < n) {
      const int64_t s = rp[row], e = rp[row + 1];
      if (gskip[row] == 0 && e - s <= kLongRow) {  // uniform within the group
        const double a = short_row(s, e, static_cast<int32_t>(row));
        if (sub == 0) *out.template row<PERM>(row, 1) = a;
      }
    }
  }
}

// offsets col - row of the CSR part (flag 1 when one does not fit in int16);
// kG lanes per row, four consecutive entries each, as in the product
__global__ void __launch_bounds__(kThreads) k_col16(int64_t n, const int64_t* __restrict__ rp,
                                                    const int32_t* __restrict__ gskip, const int32_t* __restrict__ col,
                                                    int16_t* __restrict__ off, int* __restrict__ err) {
  const unsigned b = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t row = (b * static_cast<int64_t>(kThreads) + threadIdx.x) / kG;
  if (row >= n) return;
  const int32_t self = static_cast<int32_t>(row);
  const int64_t s = rp[row] + gskip[row], e = rp[row + 1];
  bool bad = false;
  auto put = [&](const int32_t* c, int64_t j) {
    int16_t o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t d = c[u] - self;
      if (j + u < e) bad = bad || d < -32768 || d > 32767;
      o[u] = static_cast<int16_t>(d);
    }
    if (j + 4 <= e) {
      __builtin_memcpy(off + j, o, sizeof(o));
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (j + u < e) off[j + u] = o[u];
    }
  };
  constexpr int kB = 2;  // groups of four requested at once (rows of up to 64 entries: all)
  for (int64_t j0 = s + 4 * (threadIdx.x & (kG - 1)); j0 < e; j0 += 4 * kG * kB) {
    int32_t c[kB][4];
#pragma unroll
    for (int h = 0; h < kB; ++h)
      if (j0 + 4 * kG * h < e) __builtin_memcpy(c[h], col + j0 + 4 * kG * h, sizeof(c[h]));
#pragma unroll
    for (int h = 0; h < kB; ++h)
      if (j0 + 4 * kG * h < e) put(c[h], j0 + 4 * kG * h);
  }
  if (bad) atomicOr(err, 1);
}

// Entries up to which the product takes one launch.  Two launches -> one, per
// product: 0.3M entries (FP64) 10.5 -> 8.0 us, 2.0M (mixture n = 30,011, mixed)
// 13.7 -> 9.6, 5.0M 21.4 -> 16.2, 42M 52.5 -> 49.0 and 87.5 -> 79.2 (FP64).  At 87M
// entries the CSR rows want the waves that the tile code's registers cost them:
// FP64 239 -> 243 us (gp_matvec); mixed (6 waves, see one_waves) 183 -> 180, but a
// likelihood with the log det's products beside it 114.6 -> 116.6 ms; one limit holds
// for both.
constexpr int64_t kOneLaunchEntries = int64_t(64) << 20;

// Waves per SIMD the one-launch product is compiled for.  The tile code is at its
// best with the registers it asks for (float32 values 96: 5 waves; FP64 113: 4), the
// CSR rows with more waves, which hide their gathers.  Held to 6 waves (80
// registers, float32), per CG iteration: 0.3M to 3.7M entries 17.66 -> 17.89 and 20.1 ->
// 20.8 us, 5M 26.1 -> 25.2, 14M (eight problems) 36.4 -> 35.4, 42M 55.8 -> 52.1, 46M 59.7 -> 58.9.  To
// 5 waves (96, FP64), by the share of group entries: 0.18 29.3 -> 28.2, 0.35 23.5 -> 22.9,
// 0.84 103.1 -> 100.5, 0.93 89.9 -> 90.3 and 78.6 -> 80.2.  (6 waves spill there.)
template <typename VT>
int one_waves(const gp_matrix* m) {
  if (sizeof(VT) == 4) return m->nnz > (int64_t(4) << 20) ? 6 : 1;
  return 8 * m->nnz_group < 7 * m->nnz ? 5 : 1;
}

template <typename VT, typename XT, typename AT, typename YT, bool PERM>
void spmv_launch_to(gp_ctx* c, const gp_matrix* m, const XT* x, YT* y, const int* skip, RowDest<YT> out) {
  const VT* val = static_cast<const VT*>(m->val);
  // long-row blocks padded to a multiple of the XCD count so that both block
  // ranges start on XCD 0 (see xcd_remap)
  const unsigned nb_short = grid_for(m->n * kG, kThreads);
  if constexpr (std::is_same<XT, double>::value && std::is_same<YT, double>::value) {
    if (m->ntiles > 0 && m->nnz <= kOneLaunchEntries) {
      const unsigned nt = static_cast<unsigned>(m->ntiles);
      const unsigned nl = m->n_long > 0 ? grid_for(m->n_long, kWaves) : 0;
      auto one = [&](auto waves) {
        hipLaunchKernelGGL((k_spmv_one<VT, PERM, decltype(waves)::value>), dim3(nt + nl + nb_short), dim3(kThreads), 0,
                           c->stream, m->n, nt, nl, m->n_long, m->g_tiles, m->g_rows, m->g_uoff, m->g_ulist,
                           m->long_rows, m->row_ptr, m->gskip, m->col, val, x, out, m->col16, skip);
      };
      if (one_waves<VT>(m) > 1)
        one(std::integral_constant<int, sizeof(VT) == 4 ? 6 : 5>{});
      else
        one(std::integral_constant<int, 1>{});
      check_launch("spmv");
      return;
    }
  }
  const unsigned nb_long = m->n_long > 0 ? round_up8(grid_for(m->n_long * kWave, kThreads)) : 0;
  if (m->ntiles > 0)
    hipLaunchKernelGGL((k_group_spmv<VT, XT, AT, YT>), dim3(static_cast<unsigned>(m->ntiles)), dim3(kThreads), 0,
                       c->stream, m->g_tiles, m->g_rows, m->g_uoff, m->g_ulist, m->row_ptr, val, x, y, skip);
  hipLaunchKernelGGL((k_spmv<VT, XT, AT, YT, PERM>), dim3(nb_short + nb_long), dim3(kThreads), 0, c->stream, m->n,
                     nb_long, m->n_long, m->long_rows, m->row_ptr, m->gskip, m->col, val, x, y, out, m->col16, skip);
  check_launch("spmv");
}

template <typename VT, typename XT, typename AT, typename YT>
void spmv_launch(gp_ctx* c, const gp_matrix* m, const XT* x, YT* y, const int* skip, RowDest<YT> out) {
  if (!out.y) out.y = y;
  if (out.perm)
    spmv_launch_to<VT, XT, AT, YT, true>(c, m, x, y, skip, out);
  else
    spmv_launch_to<VT, XT, AT, YT, false>(c, m, x, y, skip, out);
}

template <typename VT, typename XT, typename AT, typename YT>
void spmv_impl(gp_ctx* c, const gp_matrix* m, const XT* x, YT* y, const int* skip, RowDest<YT> out) {
  ProfScope ps(c, sizeof(VT) == 4 ? (sizeof(XT) == 4 ? "spmv_f32" : "spmv_f32val_f64") : "spmv_f64");
  spmv_launch<VT, XT, AT, YT>(c, m, x, y, skip, out);
}

}  // namespace

void free_col16(gp_ctx* c, gp_matrix* m) {
  if (m->col16) dev_free(c, m->col16, sizeof(int16_t) * (m->nnz + kCsrPad));
  m->col16 = nullptr;
}

static void build_col16(gp_ctx* c, gp_matrix* m) {
  if (m->col16_tried) return;
  m->col16_tried = true;
  ProfScope ps(c, "col16_build");
  // the offsets are a cache: without room for them (allocator or context
  // budget) the products keep reading the int32 column ids
  try {
    m->col16 = dev_new<int16_t>(c, m->nnz + kCsrPad);
  } catch (const Error& e) {
    if (e.st != GP_ENOMEM) throw;
    m->col16 = nullptr;
    return;
  }
  GPS_HIP(hipMemsetAsync(c->err_flag, 0, sizeof(int), c->stream));
  hipLaunchKernelGGL(k_col16, dim3(grid_for(m->n * kG, kThreads)), dim3(kThreads), 0, c->stream, m->n, m->row_ptr,
                     m->gskip, m->col, m->col16, c->err_flag);
  check_launch("col16");
  int* h = static_cast<int*>(pinned(c, sizeof(int)));
  GPS_HIP(hipMemcpyAsync(h, c->err_flag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  sync(c);
  if (*h)
    free_col16(c, m);
  else
    m->bytes += sizeof(int16_t) * (m->nnz + kCsrPad);
}

// The same product with whatever caches the matrix already holds: nothing is
// built, allocated, timed or waited for (the int16 offsets are read when an
// earlier product built them; both column forms give bitwise equal sums).
void spmv_f64_enqueue(gp_ctx* c, const gp_matrix* m, const double* x, double* y, RowDest<double> out) {
  if (m->prec == GP_MIXED)
    spmv_launch<float, double, double, double>(c, m, x, y, nullptr, out);
  else
    spmv_launch<double, double, double, double>(c, m, x, y, nullptr, out);
}

void spmv_f64(gp_ctx* c, const gp_matrix* m, const double* x, double* y, const int* skip, RowDest<double> out) {
  build_col16(c, const_cast<gp_matrix*>(m));
  if (m->prec == GP_MIXED)
    spmv_impl<float, double, double, double>(c, m, x, y, skip, out);
  else
    spmv_impl<double, double, double, double>(c, m, x, y, skip, out);
}


namespace {

// Group-block part of the SpMM on the matrix cores.  For the rows of one
// super-tile (same mask M, at most kSuperRows rows) the product is the dense
// contraction Y[rows, 0:32] = V[rows, U_M] (S X)[U_M, 0:32] (the row scaling is
// applied by the CSR part).  One block takes one piece: the super-tile's rows
// times at most kPiece consecutive entries of U_M, so that every block does a
// similar amount of work whatever |U_M| is.  The piece's column ids and
// scales are read into LDS first; then chunks of kMChunk rows of S X are
// staged in LDS (double-buffered) and shared by the eight waves: waves w and
// w + 4 own the 16 rows 16 w ... 16 w + 15 and take the first and second half
// of the k-steps of each chunk on the 16x16x4 MFMA.  Lane (i, kk) = (lane %
// 16, lane / 16) holds A[i][kk] = V[row 16 w + i, 4 s + kk] and B[kk][i] =
// (S X)[U_M[4 s + kk], i] (a second MFMA covers columns 16-31).  The halves
// are added in a fixed order; a super-tile of one piece writes Y, otherwise
// each piece writes its partial block and k_group_reduce adds the pieces in
// order, so the result is deterministic.  Lane l of an MFMA result holds
// four entries v = 0..3 of column l % 16: rows l / 16 + 4 v.
typedef double mfma_d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ mfma_d4 mfma16x16x4(double a, double b, mfma_d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <typename T>
struct MfmaAcc;
template <>
struct MfmaAcc<double> {
  using type = mfma_d4;
  static __device__ __forceinline__ int row(int kk, int v) { return kk + 4 * v; }
};

constexpr int kMThreads = 512;                   // 8 waves: 4 row groups x 2 halves of each chunk
constexpr int kMChunk = 64;                      // U_M entries per staged chunk
constexpr int kMSteps = kMChunk / 4 / 2;         // MFMA k-steps per wave per chunk
static_assert(kSuperRows == 4 * 16, "one row group of 16 per wave pair");
static_assert(kMSteps == 8 && kMChunk == 64, "lane (i, kk) of a wave half takes 8 consecutive entries");
static_assert(kPiece % kMChunk == 0 && kPiece <= kMThreads, "piece = whole chunks, ids loaded in one pass");

template <typename VT, typename T, bool SCALE, int NB>
__global__ void __launch_bounds__(kMThreads) k_group_spmm_mfma(const int32_t* __restrict__ pieces,
                                                               const int32_t* __restrict__ grows,
                                                               const int64_t* __restrict__ uoff,
                                                               const int32_t* __restrict__ ulist, int k, int ld,
                                                               const int64_t* __restrict__ rp,
                                                               const VT* __restrict__ val, const T* __restrict__ X,
                                                               T* __restrict__ Y, const T* __restrict__ scale,
                                                               T* __restrict__ part) {
  using Acc = typename MfmaAcc<T>::type;
  constexpr int kCols = 16 * NB;                      // columns: one or two blocks of 16
  constexpr int kXPer = kMChunk * kCols / kMThreads;  // X values staged per thread
  __shared__ T xs[2][kMChunk][kCols + 1];
  __shared__ int32_t us[kPiece];
  __shared__ T ss[SCALE ? kPiece : 1];
  const unsigned pid = xcd_remap(blockIdx.x, gridDim.x);
  const int4 t = reinterpret_cast<const int4*>(pieces)[pid];
  const int nUall = static_cast<int>(uoff[t.x + 1] - uoff[t.x]);
  const int kstart = t.w;
  const int len = min(kPiece, nUall - kstart);
  const bool whole = kstart == 0 && len == nUall;   // the only piece of its super-tile
  if (threadIdx.x < kPiece) {
    int32_t q = 0;
    if (static_cast<int>(threadIdx.x) < len) q = ulist[uoff[t.x] + kstart + threadIdx.x];
    us[threadIdx.x] = q;
    if constexpr (SCALE) ss[threadIdx.x] = static_cast<int>(threadIdx.x) < len ? scale[q] : T(0);
  }
  const int w = threadIdx.x / kWave, lane = lane_id();
  const int rg = w & 3, half = w >> 2;   // rows 16 rg ... 16 rg + 15; steps of this half of each chunk
  const int i = lane & 15, kk = lane >> 4;
  const bool wave_rows = 16 * rg < t.z;  // uniform over the wave
  // chunk entry of k-step s for this lane (the A and B operands agree on it):
  // lane (i, kk) takes 8 consecutive entries, loaded with one vector load
  auto ent = [&](int s) { return half * (kMChunk / 2) + 8 * kk + s; };
  // A operands, V[row 16 rg + i, kstart + c0 + ent(s)]; rows past the tile read
  // row 0 of the tile and are zeroed.  The loads are clamped into the row's
  // leading U_M entries; a vector load may run up to 7 entries further, which
  // stays inside the value array (its length carries kCsrPad entries of
  // padding).
  const int r = 16 * rg + i;
  const bool rvalid = r < t.z;
  const VT* vrow = val + rp[grows[t.y + (rvalid ? r : 0)]] + kstart;
  VT areg[kMSteps], acur[kMSteps];
  auto load_a = [&](int c0) {
    const int e0 = c0 + ent(0);
    VT v[kMSteps];
    __builtin_memcpy(v, vrow + min(e0, len - 1), sizeof(v));
#pragma unroll
    for (int s = 0; s < kMSteps; ++s) areg[s] = (rvalid && e0 + s < len) ? v[s] : VT(0);
  };
  load_a(0);
  __syncthreads();
  // staging of X: thread -> (chunk row, kXPer consecutive columns); rows of
  // at least kCols values are read with vector loads (columns past k are read
  // but only feed output columns that are never stored)
  constexpr int kSegs = kCols / kXPer;
  const int xr = threadIdx.x / kSegs, xc0 = (threadIdx.x % kSegs) * kXPer;
  const bool xvec = ld >= kCols;
  T xreg[kXPer];
  auto load_x = [&](int c0) {
    const int e = min(c0 + xr, len - 1);
    const T* xp = X + static_cast<int64_t>(us[e]) * ld;
    if (xvec) {
      __builtin_memcpy(xreg, xp + xc0, sizeof(xreg));
    } else {
#pragma unroll
      for (int u = 0; u < kXPer; ++u) xreg[u] = xp[min(xc0 + u, k - 1)];
    }
    T sq = c0 + xr < len ? T(1) : T(0);
    if constexpr (SCALE) sq *= ss[e];
#pragma unroll
    for (int u = 0; u < kXPer; ++u) xreg[u] *= sq;
  };
  auto store_x = [&](int buf) {
#pragma unroll
    for (int u = 0; u < kXPer; ++u) xs[buf][xr][xc0 + u] = xreg[u];
  };
  Acc acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = Acc{0, 0, 0, 0};
  load_x(0);
  store_x(0);
#pragma unroll
  for (int s = 0; s < kMSteps; ++s) acur[s] = areg[s];
  __syncthreads();
  for (int c0 = 0, buf = 0; c0 < len; c0 += kMChunk, buf ^= 1) {
    const bool more = c0 + kMChunk < len;  // uniform over the block
    if (more) {
      load_x(c0 + kMChunk);
      load_a(c0 + kMChunk);
    }
    if (wave_rows) {
      T bx[NB][kMSteps];
#pragma unroll
      for (int s = 0; s < kMSteps; ++s)
#pragma unroll
        for (int b = 0; b < NB; ++b) bx[b][s] = xs[buf][ent(s)][i + 16 * b];
#pragma unroll
      for (int s = 0; s < kMSteps; ++s) {
        const T a = static_cast<T>(acur[s]);
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = mfma16x16x4(a, bx[b][s], acc[b]);
      }
    }
    if (more) {
      store_x(buf ^ 1);
#pragma unroll
      for (int s = 0; s < kMSteps; ++s) acur[s] = areg[s];
    }
    __syncthreads();
  }
  // the second half adds into the first in a fixed order (xs is free now)
  T(*red)[16][kCols + 1] = reinterpret_cast<T(*)[16][kCols + 1]>(&xs[0][0][0]);
  static_assert(sizeof(xs) >= 4 * 16 * (kCols + 1) * sizeof(T), "reduction buffer fits in the staging buffer");
  if (half == 1 && wave_rows) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int rr = MfmaAcc<T>::row(kk, v);
#pragma unroll
      for (int b = 0; b < NB; ++b) red[rg][rr][i + 16 * b] = acc[b][v];
    }
  }
  __syncthreads();
  if (half == 0 && wave_rows) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int rr = MfmaAcc<T>::row(kk, v);
      const int row = 16 * rg + rr;
      if (row >= t.z) continue;
      T* yr = whole ? Y + static_cast<int64_t>(grows[t.y + row]) * ld
                    : part + (static_cast<int64_t>(pid) * kSuperRows + row) * 32;
      const int kc = whole ? k : 32;
#pragma unroll
      for (int b = 0; b < NB; ++b)
        if (i + 16 * b < kc) yr[i + 16 * b] = acc[b][v] + red[rg][rr][i + 16 * b];
    }
  }
}

// Adds the partial blocks of the pieces of each super-tile with more than one
// piece, in piece order, into Y.  Block (super-tile, group of kRedRows rows),
// thread -> (row, column).
constexpr int kRedRows = kThreads / 32;

template <typename T>
__global__ void __launch_bounds__(kThreads) k_group_reduce(const int32_t* __restrict__ stiles,
                                                           const int32_t* __restrict__ grows, int k, int ld,
                                                           const T* __restrict__ part, T* __restrict__ Y) {
  constexpr int kGroups = kSuperRows / kRedRows;
  const int4 t = reinterpret_cast<const int4*>(stiles)[blockIdx.x / kGroups];
  const int row = (blockIdx.x % kGroups) * kRedRows + threadIdx.x / 32, col = threadIdx.x & 31;
  if (t.w <= 1 || row >= t.y || col >= k) return;  // single pieces write Y themselves
  const T* pp = part + (static_cast<int64_t>(t.z) * kSuperRows + row) * 32 + col;
  constexpr int64_t kStride = static_cast<int64_t>(kSuperRows) * 32;
  T acc = pp[0];
  int p = 1;
  for (; p + 4 <= t.w; p += 4) {
    const T a0 = pp[p * kStride], a1 = pp[(p + 1) * kStride], a2 = pp[(p + 2) * kStride], a3 = pp[(p + 3) * kStride];
    acc += a0;
    acc += a1;
    acc += a2;
    acc += a3;
  }
  for (; p < t.w; ++p) acc += pp[p * kStride];
  Y[static_cast<int64_t>(grows[t.x + row]) * ld + col] = acc;
}

}  // namespace

namespace {

// ------------------------------------------------------------ row quads
// The CSR part of the 32-column product reads one 256-byte row of X per
// stored entry.  Rows next to each other along the grid axis with the most
// cells (at the space-time workload: one station on consecutive days) share
// most of their columns, so the rows are listed along that axis (a line: the
// cells with all other cell coordinates fixed, binned order within a cell),
// in segments of kSlabCells cells of a line, and every four consecutive
// listed rows of a segment form a quad that stores the ascending union of its
// rows' columns once, with the four rows' values per entry: one gather of an
// X row serves four rows.  Consecutive quads share many X rows, which then
// come from the caches (k_line_rows gives the order of the segments).
constexpr int kQuad = 4;
constexpr int kLineThreads = 256;
constexpr int kSlabCells = 16;  // cells of a line per listed segment

struct LineGeom {
  int a;            // axis along which a line runs
  int nother;       // number of other axes
  int o[2];         // the other axes, fastest first
  int32_t g[3];     // cells per axis
  int64_t stride[3];
  int64_t nlines;   // lines of the grid
  int64_t lpr;      // lines per region (the lines are cut into kXcds contiguous regions)
  int32_t slab;     // cells of a line per segment
  int32_t nslab;    // segments per line
};

// exclusive prefix sum over the block of v (kLineThreads threads); *total
// receives the block's sum
__device__ __forceinline__ int32_t block_excl_scan(int32_t v, int32_t* total) {
  __shared__ int32_t wsum[kLineThreads / kWave];
  const int lane = lane_id(), w = threadIdx.x / kWave;
  int32_t x = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t y = __shfl_up(x, off, kWave);
    if (lane >= off) x += y;
  }
  __syncthreads();  // wsum of an earlier call has been read
  if (lane == kWave - 1) wsum[w] = x;
  __syncthreads();
  int32_t before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kLineThreads / kWave; ++i) {
    if (i < w) before += wsum[i];
    all += wsum[i];
  }
  *total = all;
  return before + x - v;
}

// The rows are listed segment by segment: a segment is the rows of lg.slab
// consecutive cells of one line (binned order within a cell), padded to a
// multiple of four.  Segments are ordered by region (kXcds contiguous ranges
// of lines), then slab, then line: the 32-column product gives each XCD a
// contiguous range of quads, so an XCD sweeps its region slab by slab and the
// X rows that neighbouring lines share are read while they are in its L2.
// Block per segment.  PASS 0: the segment's row count padded to a multiple of
// four (lpad).  PASS 1: its rows, then the padding (-1).
template <int PASS>
__global__ void __launch_bounds__(kLineThreads) k_line_rows(LineGeom lg, const int32_t* __restrict__ cell_start,
                                                             int32_t* __restrict__ lpad, const int64_t* __restrict__ loff,
                                                             int32_t* __restrict__ trow) {
  const int64_t S = blockIdx.x;
  const int64_t j = S % lg.lpr, rs = S / lg.lpr;
  const int64_t region = rs / lg.nslab;
  const int slab = static_cast<int>(rs % lg.nslab);
  const int64_t L = region * lg.lpr + j;
  int64_t running = 0;
  const int64_t out0 = PASS == 1 ? loff[S] : 0;
  if (L < lg.nlines) {
    int64_t base = 0, r = L;
    for (int k = 0; k < lg.nother; ++k) {
      const int ax = lg.o[k];
      base += (r % lg.g[ax]) * lg.stride[ax];
      r /= lg.g[ax];
    }
    const int64_t sa = lg.stride[lg.a];
    const int c0 = slab * lg.slab, c1 = min(c0 + lg.slab, lg.g[lg.a]);
    for (int i0 = c0; i0 < c1; i0 += kLineThreads) {
      const int i = i0 + static_cast<int>(threadIdx.x);
      int32_t cs = 0, cnt = 0;
      if (i < c1) {
        const int64_t key = base + i * sa;
        cs = cell_start[key];
        cnt = cell_start[key + 1] - cs;
      }
      int32_t total;
      const int32_t ex = block_excl_scan(cnt, &total);
      if constexpr (PASS == 1)
        for (int32_t t = 0; t < cnt; ++t) trow[out0 + running + ex + t] = cs + t;
      running += total;
    }
  }
  const int64_t pad = (running + kQuad - 1) / kQuad * kQuad;
  if constexpr (PASS == 0) {
    if (threadIdx.x == 0) lpad[S] = static_cast<int32_t>(pad);
  } else {
    for (int64_t t = running + threadIdx.x; t < pad; t += kLineThreads) trow[out0 + t] = -1;
  }
}

// The CSR-part column lists of the rows of quad g (listed rows 4g .. 4g+3;
// padding and rows with more than kLongRow entries count as empty): begin and
// end of each.
__device__ __forceinline__ void quad_lists(int64_t g, const int32_t* __restrict__ trow,
                                           const int64_t* __restrict__ rp, const int32_t* __restrict__ gskip,
                                           int64_t (&h)[kQuad], int64_t (&e)[kQuad]) {
#pragma unroll
  for (int i = 0; i < kQuad; ++i) {
    const int32_t r = trow[g * kQuad + i];
    h[i] = e[i] = 0;
    if (r >= 0) {
      const int64_t s = rp[r] + gskip[r], t = rp[r + 1];
      if (t - s <= kLongRow) {
        h[i] = s;
        e[i] = t;
      }
    }
  }
}

// first index of list[0, len) with list[i] >= c (lower) or > c (upper)
template <bool UPPER>
__device__ __forceinline__ int list_bound(const int32_t* lst, int len, int32_t c) {
  int lo = 0, hi = len;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (UPPER ? lst[mid] <= c : lst[mid] < c)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// One wave per quad.  The four rows' CSR-part column lists (ascending, at
// most kLongRow each) are loaded into the wave's LDS slice; every entry (row
// i, position j, column c) finds its place in the merged order by (column,
// row): j plus, in each other row k, the number of columns < c (k > i) or
// <= c (k < i).  Equal columns are then adjacent, at most one per row; the
// first of each run starts a quad entry, numbered by a ballot scan.
// PASS 0 writes the number of entries of each quad, PASS 1 the ascending
// column ids with the four rows' values (0 where a row lacks the column).
constexpr int kQuadMax = kQuad * kLongRow;

template <typename VT, int PASS>
__global__ void __launch_bounds__(kThreads) k_quad_build(int64_t ngroups, const int32_t* __restrict__ trow,
                                                         const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ gskip,
                                                         const int32_t* __restrict__ col, const VT* __restrict__ val,
                                                         int32_t* __restrict__ cnt, const int64_t* __restrict__ qptr,
                                                         int32_t* __restrict__ qcol, VT* __restrict__ qval) {
  __shared__ int32_t lc[kThreads / kWave][kQuad][kLongRow];
  __shared__ int32_t mc[kThreads / kWave][kQuadMax];
  __shared__ int16_t mij[kThreads / kWave][kQuadMax];  // row * kLongRow + position
  const int lane = lane_id(), w = threadIdx.x / kWave;
  const int64_t g = blockIdx.x * static_cast<int64_t>(kThreads / kWave) + w;
  if (g >= ngroups) return;  // uniform over the wave
  int64_t h[kQuad], e[kQuad];
  quad_lists(g, trow, rp, gskip, h, e);
  int len[kQuad], off[kQuad + 1];
  off[0] = 0;
#pragma unroll
  for (int i = 0; i < kQuad; ++i) {
    len[i] = static_cast<int>(e[i] - h[i]);
    off[i + 1] = off[i] + len[i];
  }
  const int T = off[kQuad];
#pragma unroll
  for (int i = 0; i < kQuad; ++i)
    for (int j = lane; j < len[i]; j += kWave) lc[w][i][j] = col[h[i] + j];
  wave_sync_lds();
  for (int t = lane; t < T; t += kWave) {
    int i = 0;
#pragma unroll
    for (int k = 1; k < kQuad; ++k)
      if (t >= off[k]) i = k;
    const int j = t - off[i];
    const int32_t c = lc[w][i][j];
    int pos = j;
#pragma unroll
    for (int k = 0; k < kQuad; ++k) {
      if (k < i) pos += list_bound<true>(lc[w][k], len[k], c);
      if (k > i) pos += list_bound<false>(lc[w][k], len[k], c);
    }
    mc[w][pos] = c;
    mij[w][pos] = static_cast<int16_t>(i * kLongRow + j);
  }
  wave_sync_lds();
  int64_t out0 = PASS == 1 ? qptr[g] : 0;
  int running = 0;
  for (int b = 0; b < T; b += kWave) {
    const int p = b + lane;
    const bool first = p < T && (p == 0 || mc[w][p] != mc[w][p - 1]);
    const uint64_t bal = __ballot(first);
    if constexpr (PASS == 1) {
      if (first) {
        const int64_t out = out0 + running + __popcll(bal & lanes_below());
        const int32_t c = mc[w][p];
        VT v[kQuad];
#pragma unroll
        for (int i = 0; i < kQuad; ++i) v[i] = VT(0);
#pragma unroll
        for (int d = 0; d < kQuad; ++d) {
          if (p + d < T && mc[w][p + d] == c) {
            const int ij = mij[w][p + d];
            const int row = ij / kLongRow, j = ij % kLongRow;
#pragma unroll
            for (int i = 0; i < kQuad; ++i)
              if (row == i) v[i] = val[h[i] + j];
          }
        }
        qcol[out] = c;
#pragma unroll
        for (int i = 0; i < kQuad; ++i) qval[out * kQuad + i] = v[i];
      }
    }
    running += __popcll(bal);
  }
  if constexpr (PASS == 0)
    if (lane == 0) cnt[g] = running;
}

// Row codes of the listed rows for the product: -1 for padding and for rows
// with more than kLongRow entries past their group part, the row for a row
// without a group part, -(row + 2) for a row with one.
__global__ void __launch_bounds__(kThreads) k_quad_codes(int64_t ntrow, const int32_t* __restrict__ trow,
                                                         const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ gskip, int32_t* __restrict__ code) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x;
  if (i >= ntrow) return;
  const int32_t r = trow[i];
  int32_t c = -1;
  if (r >= 0) {
    const int32_t gs = gskip[r];
    if (rp[r + 1] - rp[r] - gs <= kLongRow) c = gs ? -r - 2 : r;
  }
  code[i] = c;
}

// CSR part of Y = S K S X D for the short rows, one quad at a time (four
// consecutive listed rows share most of their local columns): lane l
// stages union entry j0 + l of the group (column id and the four rows'
// weights, times the column's scale) in the wave's LDS slice; then each
// 16-byte load of an X row serves all four rows.  The same column split as
// spmm_consume16 (lane l: kCpl columns of entry slot l / kLpe), slot sums in
// a fixed order, group part added from Y.
constexpr int kQuadsPerWave = 2;
constexpr int kQuadUq = 2;  // X loads in flight per lane (two keep the kernel at 68 registers)
// Beside another stream's kernels the row-quad product takes 15 KB of dynamic
// LDS more per block: with its 9 KB of static LDS, six blocks (six waves per
// SIMD) fit in a CU's 160 KB instead of the seven its registers allow, and the
// other stream's waves find free slots (measured beside the solve: 6.88 ->
// 6.94 likelihood evaluations per second; alone the product is 2% slower).
constexpr unsigned kShareLds = 15 * 1024;

template <typename VT, bool SCALE, bool PERM>
__global__ void __launch_bounds__(kThreads) k_spmm_quad(int64_t ngroups, const int64_t* __restrict__ qptr,
                                                        const int32_t* __restrict__ qcol,
                                                        const VT* __restrict__ qval, const int32_t* __restrict__ code,
                                                        int k, int ld,
                                                        const double* __restrict__ X, double* __restrict__ Y,
                                                        double* __restrict__ dest, const int32_t* __restrict__ perm,
                                                        const double* __restrict__ scale,
                                                        const double* __restrict__ colscale) {
  using V = Vec16<double>;
  __shared__ int32_t sq[kThreads / kWave][kWave];
  __shared__ double sv[kThreads / kWave][kWave][kQuad];
  const int lane = lane_id(), w = threadIdx.x / kWave;
  const int gs_lane = lane / V::kLpe, cp = lane % V::kLpe;
  double csv[V::kCpl];
#pragma unroll
  for (int t = 0; t < V::kCpl; ++t) csv[t] = colscale ? colscale[min(cp * V::kCpl + t, k - 1)] : 1.0;
  const int64_t wave = static_cast<int64_t>(xcd_remap(blockIdx.x, gridDim.x)) * (kThreads / kWave) + w;
  for (int gi = 0; gi < kQuadsPerWave; ++gi) {
    const int64_t g = wave * kQuadsPerWave + gi;
    if (g >= ngroups) return;  // uniform over the wave
    const int64_t s = qptr[g], e = qptr[g + 1];
    V acc[kQuad];
#pragma unroll
    for (int r = 0; r < kQuad; ++r)
#pragma unroll
      for (int t = 0; t < V::kCpl; ++t) acc[r].v[t] = 0;
    for (int64_t j0 = s; j0 < e; j0 += kWave) {
      const int m = static_cast<int>(min<int64_t>(kWave, e - j0));
      wave_sync_lds();  // the previous chunk has been read
      // Column ids are staged first and the first X rows requested while the
      // column scales are still on their way; the weights (value times the
      // column's scale) follow through the second stage.
      int32_t q = 0;
      VT raw[kQuad];
      double sc = 1.0;
#pragma unroll
      for (int r = 0; r < kQuad; ++r) raw[r] = VT(0);
      if (lane < m) {
        q = qcol[j0 + lane];
#pragma unroll
        for (int r = 0; r < kQuad; ++r) raw[r] = qval[(j0 + lane) * kQuad + r];
      }
      sq[w][lane] = q;
      if (SCALE && lane < m) sc = scale[q];
      wave_sync_lds();
      const int nq = (m + V::kEpi - 1) / V::kEpi;
      int32_t qn[kQuadUq];
      V xn[kQuadUq];
#pragma unroll
      for (int u = 0; u < kQuadUq; ++u) {
        qn[u] = sq[w][(V::kEpi * u + gs_lane) & (kWave - 1)];
        __builtin_memcpy(xn[u].v, X + static_cast<int64_t>(qn[u]) * ld + cp * V::kCpl, 16);
      }
#pragma unroll
      for (int r = 0; r < kQuad; ++r) sv[w][lane][r] = static_cast<double>(raw[r]) * sc;
      wave_sync_lds();
      for (int i0 = 0; i0 < nq; i0 += kQuadUq) {
        int32_t qq[kQuadUq];
        double vv[kQuadUq][kQuad];
#pragma unroll
        for (int u = 0; u < kQuadUq; ++u) {
          const int idx = (V::kEpi * (i0 + u) + gs_lane) & (kWave - 1);  // past m: q = 0, weights 0
          qq[u] = sq[w][idx];
#pragma unroll
          for (int r = 0; r < kQuad; ++r) vv[u][r] = (i0 + u < nq) ? sv[w][idx][r] : 0.0;
        }
        V xv[kQuadUq];
        if (i0 == 0) {
#pragma unroll
          for (int u = 0; u < kQuadUq; ++u) xv[u] = xn[u];
        } else {
#pragma unroll
          for (int u = 0; u < kQuadUq; ++u)
            __builtin_memcpy(xv[u].v, X + static_cast<int64_t>(qq[u]) * ld + cp * V::kCpl, 16);
        }
#pragma unroll
        for (int u = 0; u < kQuadUq; ++u)
#pragma unroll
          for (int r = 0; r < kQuad; ++r)
#pragma unroll
            for (int t = 0; t < V::kCpl; ++t) acc[r].v[t] += vv[u][r] * xv[u].v[t];
      }
    }
#pragma unroll
    for (int r = 0; r < kQuad; ++r) {
      slot_sum<double>(acc[r]);
      const int32_t cr = code[g * kQuad + r];
      if (cr == -1) continue;  // padding, or a row written by the long-row blocks
      const bool grow = cr < -1;
      const int64_t row = grow ? -static_cast<int64_t>(cr) - 2 : cr;
      if (lane < V::kLpe) {
        // (Y and not a copy of the pointer where the rows stay: with two the kernel
        // takes 74 registers and loses its seventh wave)
        double* yg = Y + row * ld + lane * V::kCpl;
        double* yr = PERM ? dest + static_cast<int64_t>(perm[row]) * ld + lane * V::kCpl : yg;
#pragma unroll
        for (int t = 0; t < V::kCpl; ++t) {
          if (lane * V::kCpl + t >= k) break;
          double a = acc[r].v[t];
          if (grow) a = yg[t] + a;
          if constexpr (SCALE) a *= scale[row];
          if (colscale) a *= csv[t];
          yr[t] = a;
        }
      }
    }
  }
}

}  // namespace

void free_quads(gp_ctx* c, gp_matrix* m) {
  const size_t vbytes = m->prec == GP_MIXED ? sizeof(float) : sizeof(double);
  const int64_t ng = m->ntrow / kQuad;
  if (m->trow) dev_free(c, m->trow, sizeof(int32_t) * std::max<int64_t>(m->ntrow, 1));
  if (m->qptr) dev_free(c, m->qptr, sizeof(int64_t) * (ng + 1));
  if (m->qcol) dev_free(c, m->qcol, sizeof(int32_t) * std::max<int64_t>(m->nquad, 1));
  if (m->qval) dev_free(c, m->qval, vbytes * kQuad * std::max<int64_t>(m->nquad, 1));
  m->trow = nullptr;
  m->qptr = nullptr;
  m->qcol = nullptr;
  m->qval = nullptr;
  m->ntrow = m->nquad = 0;
}

static void build_quads(gp_ctx* c, gp_matrix* m) {
  if (m->qptr) return;
  ProfScope ps(c, "quad_build");
  const gp_dataset* ds = m->ds;
  try {
    // lines along the axis with the most cells (ties: the lowest axis)
    LineGeom lg{};
    lg.a = 0;
    for (int k = 1; k < ds->d; ++k)
      if (ds->g[k] > ds->g[lg.a]) lg.a = k;
    int64_t st = 1;
    for (int k = 0; k < 3; ++k) {
      lg.g[k] = k < ds->d ? ds->g[k] : 1;
      lg.stride[k] = st;
      st *= lg.g[k];
    }
    lg.nother = 0;
    for (int k = 0; k < ds->d; ++k)
      if (k != lg.a) lg.o[lg.nother++] = k;
    const int64_t nlines = ds->ncells / lg.g[lg.a];
    GPS_REQUIRE(nlines * lg.g[lg.a] == ds->ncells, GP_EDEVICE, "quad build: grid does not match the dataset's cells");
    lg.nlines = nlines;
    lg.lpr = (nlines + kXcds - 1) / kXcds;
    lg.slab = kSlabCells;
    lg.nslab = (lg.g[lg.a] + kSlabCells - 1) / kSlabCells;
    const int64_t nseg = static_cast<int64_t>(kXcds) * lg.nslab * lg.lpr;
    GPS_REQUIRE(nseg < (int64_t(1) << 31), GP_ENOMEM, "quad build: too many segments");
    TmpBuf lpad(c, sizeof(int32_t) * nseg), loff(c, sizeof(int64_t) * (nseg + 1));
    hipLaunchKernelGGL((k_line_rows<0>), dim3(static_cast<unsigned>(nseg)), dim3(kLineThreads), 0, c->stream, lg,
                       ds->cell_start, lpad.as<int32_t>(), nullptr, nullptr);
    check_launch("line rows");
    scan_i32_to_i64(c, lpad.as<int32_t>(), loff.as<int64_t>(), nseg);
    m->ntrow = read_i64(c, loff.as<int64_t>() + nseg);
    GPS_REQUIRE(m->ntrow < (int64_t(1) << 31), GP_ENOMEM, "quad build: too many rows");
    m->trow = dev_new<int32_t>(c, std::max<int64_t>(m->ntrow, 1));
    TmpBuf trow(c, sizeof(int32_t) * std::max<int64_t>(m->ntrow, 1));
    hipLaunchKernelGGL((k_line_rows<1>), dim3(static_cast<unsigned>(nseg)), dim3(kLineThreads), 0, c->stream, lg,
                       ds->cell_start, nullptr, loff.as<int64_t>(), trow.as<int32_t>());
    check_launch("line rows");
    const int64_t ng = m->ntrow / kQuad;
    TmpBuf cnt(c, sizeof(int32_t) * std::max<int64_t>(ng, 1));
    m->qptr = dev_new<int64_t>(c, ng + 1);
    auto go = [&](auto vt) {
      using VT = decltype(vt);
      const VT* val = static_cast<const VT*>(m->val);
      const unsigned nbb = grid_for(ng, kThreads / kWave);
      hipLaunchKernelGGL((k_quad_build<VT, 0>), dim3(nbb), dim3(kThreads), 0, c->stream, ng, trow.as<int32_t>(),
                         m->row_ptr, m->gskip, m->col, val, cnt.as<int32_t>(), nullptr, nullptr, nullptr);
      check_launch("quad count");
      scan_i32_to_i64(c, cnt.as<int32_t>(), m->qptr, ng);
      m->nquad = read_i64(c, m->qptr + ng);
      m->qcol = dev_new<int32_t>(c, std::max<int64_t>(m->nquad, 1));
      m->qval = dev_alloc(c, sizeof(VT) * kQuad * std::max<int64_t>(m->nquad, 1));
      hipLaunchKernelGGL((k_quad_build<VT, 1>), dim3(nbb), dim3(kThreads), 0, c->stream, ng, trow.as<int32_t>(),
                         m->row_ptr, m->gskip, m->col, val, nullptr, m->qptr, m->qcol, static_cast<VT*>(m->qval));
      check_launch("quad fill");
      hipLaunchKernelGGL(k_quad_codes, dim3(grid_for(m->ntrow, kThreads)), dim3(kThreads), 0, c->stream, m->ntrow,
                         trow.as<int32_t>(), m->row_ptr, m->gskip, m->trow);
      check_launch("quad row codes");
      sync(c);  // the temporaries are released when their scopes end
      m->bytes += sizeof(int32_t) * m->ntrow + sizeof(int64_t) * (ng + 1) + (sizeof(int32_t) + sizeof(VT) * kQuad) * m->nquad;
    };
    if (m->prec == GP_MIXED)
      go(float{});
    else
      go(double{});
  } catch (...) {
    free_quads(c, m);
    throw;
  }
}

// the work space of a 32-column product (partial blocks of multi-piece super-tiles)
static size_t spmm_part_bytes(const gp_matrix* m) { return sizeof(double) * kSuperRows * 32 * m->npieces; }

void spmm_reserve(gp_ctx* c, const gp_matrix* m) {
  if (m->npieces > 0) (void)workspace(c, 55, spmm_part_bytes(m));
}

template <typename T>
void spmm(gp_ctx* c, const gp_matrix* m, int k, int ld, const T* X, T* Y, const T* scale, const double* colscale,
          bool share, RowDest<T> out) {
  if (!out.y) out.y = Y;
  static_assert(std::is_same<T, double>::value, "the products take float64 vectors");
  if (k > 32 || ld < k) throw Error{GP_EINVAL, "spmm: at most 32 right-hand sides per call"};
  // 16-byte X loads need rows of at least 32 values at 16-byte alignment
  const bool vec = ld >= 32 && (ld * sizeof(T)) % 16 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
  gp_matrix* mm = const_cast<gp_matrix*>(m);  // the quads are a cache of the matrix
  if (vec) build_quads(c, mm);
  ProfScope ps(c, "spmm");
  // partial blocks of the pieces of multi-piece super-tiles
  T* part = m->npieces > 0 ? static_cast<T*>(workspace(c, 55, spmm_part_bytes(m))) : nullptr;
  auto go = [&](auto vt, auto sc, auto pm) {
    using VT = decltype(vt);
    constexpr bool SC = decltype(sc)::value, PM = decltype(pm)::value;
    if (m->npieces > 0) {
      const int32_t* st = m->g_tiles + 4 * m->ntiles;
      auto group = [&](auto nb) {
        hipLaunchKernelGGL((k_group_spmm_mfma<VT, T, SC, decltype(nb)::value>),
                           dim3(static_cast<unsigned>(m->npieces)), dim3(kMThreads), 0, c->stream,
                           st + 4 * m->nstiles, m->g_rows, m->g_uoff, m->g_ulist, k, ld, m->row_ptr,
                           static_cast<const VT*>(m->val), X, Y, scale, part);
      };
      if (k <= 16)
        group(std::integral_constant<int, 1>{});
      else
        group(std::integral_constant<int, 2>{});
      hipLaunchKernelGGL((k_group_reduce<T>), dim3(static_cast<unsigned>(m->nstiles * (kSuperRows / kRedRows))),
                         dim3(kThreads), 0, c->stream,
                         st, m->g_rows, k, ld, part, Y);
    }
    if (vec) {
      // short rows over the row quads; the long rows by k_spmm_long
      const int64_t ng = mm->ntrow / kQuad;
      if (ng > 0) {
        const unsigned nbq =
            static_cast<unsigned>(round_up8(grid_for((ng + kQuadsPerWave - 1) / kQuadsPerWave, kThreads / kWave)));
        hipLaunchKernelGGL((k_spmm_quad<VT, SC, PM>), dim3(nbq), dim3(kThreads), share ? kShareLds : 0, c->stream, ng,
                           mm->qptr, mm->qcol,
                           static_cast<const VT*>(mm->qval), mm->trow, k, ld, X, Y, out.y, out.perm, scale, colscale);
      }
      if (m->n_long > 0)
        hipLaunchKernelGGL((k_spmm_long<VT, T, SC, PM>), dim3(static_cast<unsigned>(m->n_long)), dim3(kThreads), 0,
                           c->stream, m->n_long, m->long_rows, k, ld, m->row_ptr, m->gskip, m->col,
                           static_cast<const VT*>(m->val), X, Y, out, scale, colscale);
    } else {
      unsigned nb_long = m->n_long > 0 ? round_up8(static_cast<unsigned>(m->n_long)) : 0;
      auto rows = [&](auto w) {
        constexpr int W = decltype(w)::value, kRows = kThreads / row_lanes<W>();  // rows of a block
        for (int64_t row0 = 0, row1; row0 < m->n; row0 = row1, nb_long = 0) {
          row1 = std::min<int64_t>(m->n, row0 + std::max<int64_t>(kLaunchBlocks - nb_long, 1) * kRows);
          hipLaunchKernelGGL((k_spmm_rows<VT, T, SC, PM, W>), dim3(nb_long + grid_for(row1 - row0, kRows)),
                             dim3(kThreads), 0, c->stream, row0, row1, nb_long, m->n_long, m->long_rows, k, ld,
                             m->row_ptr, m->gskip, m->col, m->col16, static_cast<const VT*>(m->val), X, Y, out, scale,
                             colscale);
        }
      };
      if (k <= 2)
        rows(std::integral_constant<int, 2>{});
      else if (k <= 4)
        rows(std::integral_constant<int, 4>{});
      else if (k <= 8)
        rows(std::integral_constant<int, 8>{});
      else if (k <= 16)
        rows(std::integral_constant<int, 16>{});
      else
        rows(std::integral_constant<int, 32>{});
    }
  };
  auto with_dest = [&](auto vt, auto sc) {
    if (out.perm)
      go(vt, sc, std::true_type{});
    else
      go(vt, sc, std::false_type{});
  };
  if (m->prec == GP_MIXED) {
    if (scale)
      with_dest(float{}, std::true_type{});
    else
      with_dest(float{}, std::false_type{});
  } else {
    if (scale)
      with_dest(double{}, std::true_type{});
    else
      with_dest(double{}, std::false_type{});
  }
  check_launch("spmm");
}

template void spmm<double>(gp_ctx*, const gp_matrix*, int, int, const double*, double*, const double*,
                           const double*, bool, RowDest<double>);

void build_product_caches(gp_ctx* c, gp_matrix* m) {
  build_col16(c, m);
  build_quads(c, m);
}

}  // namespace gps
