// Kriging mean at test points (Sec. 3.2): m(x*) = sum_q C_y(x*, x_q) alpha_q.
//
// The cross-covariance is evaluated and applied in one pass (never stored):
//   local part: each test point searches the training cells within R rings of
//     its cell and adds s0 f0(u) alpha_q for every q with u0^2 < 1;
//   bump part: sum_q [M_i(x*) M_i(q)] f_i(x*) f_i(q) alpha_q
//            = sum_{i in M(x*)} f_i(x*) c_i,   c_i = sum_q f_i(x_q) alpha_q,
//     the rank-n1 structure of the bump term (Proposition 1's proof), with
//     c_i computed once per (theta, alpha) when the predictor is created.
// With a core kernel (Eq. sparseCov) both parts are multiplied by
// C_core(x*, x_q) inside the sums.  The bump part then no longer factors
// through c_i: a wave per test point with a group bit sums
//   sum_q C_core(x*, x_q) sum_{i in M(x*) & M(q)} f_i(x*) f_i(x_q) alpha_q
// over the members of its groups (the masked training points' data and the
// groups' member lists are kept when the predictor is created).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>

#include "device.hpp"

struct gp_predictor {
  const gp_dataset* ds = nullptr;
  gps::Bump* bumps = nullptr;
  int nbumps = 0;
  gps::KernelTheta kt{};
  gps::Grid grid{};
  double* alpha_b = nullptr;  // n, binned order
  double* coef = nullptr;     // n1 (at least 1)
  // coordinates and alpha of each training point side by side (binned order,
  // kPackOf(d) doubles a point), or null: read from the data set and alpha_b
  double* pack = nullptr;
  // core kernel: basis of the nonstationary fields, the fields of the training
  // points (binned order), and the masked training points' data
  gps::CoreBasis cb{};
  double* sig = nullptr;      // n (nonstationary core)
  double* Sig = nullptr;      // n
  int64_t nm = 0;
  int32_t* mlist = nullptr;   // nm binned ids of the masked training points
  uint64_t* mmask = nullptr;  // nm group masks
  double* mF = nullptr;       // nm x n1 values f_i
  // members of each group, one list after another (null: every masked point is tested)
  int64_t nlist = 0;
  int32_t* goff = nullptr;    // n1 + 1 offsets
  int32_t* gk = nullptr;      // nlist masked indices (ascending in a group)
  int32_t* gq = nullptr;      // nlist binned ids
  uint64_t* gmask = nullptr;  // nlist group masks
};

namespace gps {
namespace {

constexpr int kThreads = 256;

// c_i = sum over masked points k of F[k, i] * alpha[mlist[k]]; one block per group.
__global__ void __launch_bounds__(kThreads) k_group_coef(int64_t nm, int n1, const double* __restrict__ F,
                                                         const int32_t* __restrict__ mlist,
                                                         const double* __restrict__ alpha, double* __restrict__ coef) {
  const int i = blockIdx.x;
  double s = 0;
  for (int64_t k = threadIdx.x; k < nm; k += kThreads) s += F[k * n1 + i] * alpha[mlist[k]];
  __shared__ double sh[kThreads];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int st = kThreads / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) coef[i] = sh[0];
}

// Doubles per point of the packed training data: (x, alpha) or (x, y, z or 0, alpha).
constexpr int kPackOf(int d) { return d == 1 ? 2 : 4; }

__global__ void __launch_bounds__(kThreads) k_pack(int64_t n, int d, const double* __restrict__ xb,
                                                   const double* __restrict__ alpha, double* __restrict__ pack) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x;
  if (i >= n) return;
  const int w = kPackOf(d);
  for (int k = 0; k + 1 < w; ++k) pack[i * w + k] = k < d ? xb[k * n + i] : 0.0;
  pack[i * w + w - 1] = alpha[i];
}

// Member lists of the bump groups, one block per group i: the masked points
// with bit i, ascending.  FILL = false: their number into off[i + 1];
// FILL = true: the lists, from off[i] on.
constexpr int kListThreads = 1024;

template <bool FILL>
__global__ void __launch_bounds__(kListThreads) k_group_members(int64_t nm, const uint64_t* __restrict__ mmask,
                                                            const int32_t* __restrict__ mlist,
                                                            int32_t* __restrict__ off, int32_t* __restrict__ gk,
                                                            int32_t* __restrict__ gq, uint64_t* __restrict__ gmask) {
  __shared__ int32_t wcount[kListThreads / kWave];
  const int i = blockIdx.x, w = threadIdx.x / kWave;
  int32_t running = FILL ? off[i] : 0;
  for (int64_t b = 0; b < nm; b += kListThreads) {
    const int64_t k = b + threadIdx.x;
    const uint64_t mk = k < nm ? mmask[k] : 0;
    const bool hit = (mk >> i) & 1;
    const uint64_t bal = __ballot(hit);
    if (lane_id() == 0) wcount[w] = __popcll(bal);
    __syncthreads();
    int32_t before = 0, total = 0;
    for (int j = 0; j < kListThreads / kWave; ++j) {
      if (j < w) before += wcount[j];
      total += wcount[j];
    }
    if (FILL && hit) {
      const int32_t o = running + before + __popcll(bal & lanes_below());
      gk[o] = static_cast<int32_t>(k);
      gq[o] = mlist[k];
      gmask[o] = mk;
    }
    running += total;
    __syncthreads();
  }
  if (!FILL && threadIdx.x == 0) off[i + 1] = running;
}

struct PredArgs {
  KernelTheta kt;
  int64_t n;
  const double* xb;
  const int32_t* cell_start;
  double lo[3], cell[3];
  int32_t g[3], R[3];
  const double* alpha;
  const double* pack;
  const double* coef;
  // core kernel: masked training points
  int64_t nm;
  const int32_t* mlist;
  const uint64_t* mmask;
  const double* mF;
  const int32_t* goff;
  const int32_t* gk;
  const int32_t* gq;
  const uint64_t* gmask;
};

// coordinates and alpha of training point q
template <int D>
__device__ __forceinline__ void load_train(const PredArgs& a, int32_t q, double* x, double& alpha) {
  if (a.pack) {  // uniform over the launch
    double v[kPackOf(D)];
    __builtin_memcpy(v, __builtin_assume_aligned(a.pack + static_cast<int64_t>(q) * kPackOf(D), 16), sizeof(v));
#pragma unroll
    for (int k = 0; k < D; ++k) x[k] = v[k];
    alpha = v[kPackOf(D) - 1];
  } else {
    x[0] = a.xb[q];
    if constexpr (D >= 2) x[1] = a.xb[a.n + q];
    if constexpr (D >= 3) x[2] = a.xb[2 * a.n + q];
    alpha = a.alpha[q];
  }
}

// Lanes per test point.  A test point's window holds 100 - 250 candidates in a
// few to a few dozen pencils (cell rows along x).  Walked by one thread they
// are a chain of as many dependent loads, and 1000 points fill four blocks.
// Sixteen lanes share the point: they read the bounds of up to 32 pencils at
// once, lay their candidates out as one list in LDS and take its entries in
// turn, so the loads are independent and no lane idles on a short pencil.
// About a quarter of the candidates lies within the support; their values
// (a square root and a degree-11 polynomial, or a core kernel) would be formed
// with three lanes of four idle, so the hits are gathered first, in place of
// the list, and evaluated by full groups.  What is left is the gather of the
// training points from beyond L2 (random sites), which the packed layout
// halves: one 32-byte read a candidate instead of four 8-byte ones.
// Calls on the n = 1,095,000 space-time set, thread per point -> this: 1009
// points (mixed) 245 -> 28 us, other sites each time (the same again 24, the very
// first call after the data was made about 90); 200,003 points in 12 requests
// (FP64) 1360 -> 300 us (384 us before the hits were gathered and the data packed).
// The split is the same for every m, so a row's value does not depend on the
// request it arrives in.
constexpr int kPl = 16;
constexpr int kPointsPerBlock = kThreads / kPl;
constexpr int kPencils = 2;     // pencils per lane and round
constexpr int kCandList = 256;  // candidates listed at a time
constexpr int kCandUnroll = 4;  // candidates whose loads a lane has in flight
constexpr int kHitUnroll = 2;

// Rows a launch takes: a grid of 2^32 threads or more loses its upper bits without
// an error, and the group kernels take a wave per row (2^31 threads here).
constexpr int64_t kLaunchRows = int64_t(1) << 25;

// orders the LDS accesses of a point's lanes (one wave; no block barrier)
__device__ __forceinline__ void lanes_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The cells lo .. hi of the point's window; false: none
template <int D>
__device__ __forceinline__ bool point_window(const PredArgs& a, const double* xp, int* lo, int* hi) {
  bool some = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    lo[k] = hi[k] = 0;
    if (k < D) {
      const int c = cell_coord(xp[k], a.lo[k], a.cell[k]);
      lo[k] = max(c - a.R[k], 0);
      hi[k] = min(c + a.R[k], a.g[k] - 1);
      some = some && lo[k] <= hi[k];
    }
  }
  return some;
}

// acc += C_core(x*, x_q) s0 f0(u) alpha_q, u2 = u^2 < 1
template <int D, bool MIXED, int CK>
__device__ __forceinline__ void add_hit(const PredArgs& a, const double* xp, double sp, double Sp, int32_t q,
                                        const double* xq, double u2, double al, double& acc) {
  double v = a.kt.s0 * wendland(u2, a.kt.variant);
  if constexpr (CK == 1) v = core_value<D, 1>(a.kt.core, xp, xq, 0.0, 0.0, 0.0, 0.0) * v;
  if constexpr (CK == 2) v = core_value<D, 2>(a.kt.core, xp, xq, sp, Sp, a.kt.core.sig[q], a.kt.core.Sig[q]) * v;
  // the mixed form: the value and alpha rounded to float32, their product in float32
  if constexpr (MIXED)
    acc += static_cast<double>(static_cast<float>(v) * static_cast<float>(al));
  else
    acc += v * al;
}

// acc += f_i(x*) c_i where the point lies in a bump of group i
template <int D>
__device__ __forceinline__ void add_bumps(const PredArgs& a, const double* xp, int i, double& acc) {
  double f = 0.0;
  bool in_group = false;
  for (int j = 0; j < a.kt.n2; ++j) {
    const Bump& bp = a.kt.bumps[i * a.kt.n2 + j];
    const double ub2 = scaled_sq<D>(xp, bp.h, bp.inv);
    if (bp.a > 0.0 && ub2 < 1.0) {
      in_group = true;
      f = f + bp.a * exp(bp.b * (1.0 - 1.0 / (1.0 - ub2)));
    }
  }
  if (in_group) acc += f * a.coef[i];
}

// The mean at one test point xp (local part over the cell window, plus the
// bump groups through c_i when there is no core kernel), by the kPl lanes of a
// point; lane: 0 .. kPl - 1, ids: the point's kCandList words of LDS.  Every lane
// returns the mean.
template <int D, bool MIXED, int CK>
__device__ __forceinline__ double predict_point(const PredArgs& a, const CoreBasis& cb, const double* xp, int lane,
                                                int32_t* ids) {
  double sp = 0.0, Sp = 0.0;
  if constexpr (CK == 2) core_point_fields<D>(cb, xp, &sp, &Sp);
  int lo_[3], hi_[3];
  const bool empty = !point_window<D>(a, xp, lo_, hi_);
  const int shift = lane_id() & ~(kPl - 1);  // the point's first lane of the wave
  const uint32_t below = (1u << lane) - 1;
  double acc = 0.0;
  const int ny = hi_[1] - lo_[1] + 1;
  const int64_t npen = empty ? 0 : static_cast<int64_t>(ny) * (hi_[2] - lo_[2] + 1);
  for (int64_t p0 = 0; p0 < npen; p0 += kPl * kPencils) {  // the same trips for the point's lanes
    // this lane's pencils: candidates s[j] .. s[j] + cnt[j] - 1
    int32_t s[kPencils], cnt[kPencils], own = 0;
#pragma unroll
    for (int j = 0; j < kPencils; ++j) {
      const int64_t pk = p0 + j * kPl + lane;
      s[j] = cnt[j] = 0;
      if (pk < npen) {
        const int y = lo_[1] + static_cast<int>(pk % ny), z = lo_[2] + static_cast<int>(pk / ny);
        const int64_t base = (static_cast<int64_t>(z) * a.g[1] + y) * a.g[0];
        s[j] = a.cell_start[base + lo_[0]];
        cnt[j] = a.cell_start[base + hi_[0] + 1] - s[j];
      }
      own += cnt[j];
    }
    int32_t end = own;  // inclusive scan over the point's lanes
#pragma unroll
    for (int off = 1; off < kPl; off <<= 1) {
      const int32_t v = __shfl_up(end, off, kPl);
      if (lane >= off) end += v;
    }
    const int32_t total = __shfl(end, kPl - 1, kPl);
    for (int32_t c0 = 0; c0 < total; c0 += kCandList) {  // dense cells: the list in parts
      const int32_t len = min(kCandList, total - c0);
      lanes_sync_lds();  // the previous part has been read
      int32_t first = end - own - c0;  // list position of the pencil's first candidate
#pragma unroll
      for (int j = 0; j < kPencils; ++j) {
        const int32_t i1 = min(cnt[j], len - first);
        for (int32_t i = max(0, -first); i < i1; ++i) ids[first + i] = s[j] + i;
        first += cnt[j];
      }
      lanes_sync_lds();
      // candidates within the support, kept in place (never ahead of what has been read)
      int32_t nhit = 0;
      for (int32_t t0 = 0; t0 < len; t0 += kPl * kCandUnroll) {
        int32_t q[kCandUnroll];
        double xq[kCandUnroll][3], al;
#pragma unroll
        for (int u = 0; u < kCandUnroll; ++u) {
          const int32_t t = t0 + u * kPl + lane;
          q[u] = ids[t < len ? t : 0];
        }
#pragma unroll
        for (int u = 0; u < kCandUnroll; ++u) load_train<D>(a, q[u], xq[u], al);
        lanes_sync_lds();
#pragma unroll
        for (int u = 0; u < kCandUnroll; ++u) {
          const bool hit = t0 + u * kPl + lane < len && scaled_sq<D>(xp, xq[u], a.kt.inv0) < 1.0;
          const uint32_t bal = static_cast<uint32_t>(__ballot(hit) >> shift) & ((1u << kPl) - 1);
          if (hit) ids[nhit + __popc(bal & below)] = q[u];
          nhit += __popc(bal);
        }
        lanes_sync_lds();
      }
      for (int32_t t0 = 0; t0 < nhit; t0 += kPl * kHitUnroll) {
        int32_t q[kHitUnroll];
        double xq[kHitUnroll][3], al[kHitUnroll];
#pragma unroll
        for (int u = 0; u < kHitUnroll; ++u) {
          const int32_t t = t0 + u * kPl + lane;
          q[u] = ids[t < nhit ? t : 0];
        }
#pragma unroll
        for (int u = 0; u < kHitUnroll; ++u) load_train<D>(a, q[u], xq[u], al[u]);
#pragma unroll
        for (int u = 0; u < kHitUnroll; ++u)
          if (t0 + u * kPl + lane < nhit)
            add_hit<D, MIXED, CK>(a, xp, sp, Sp, q[u], xq[u], scaled_sq<D>(xp, xq[u], a.kt.inv0), al[u], acc);
      }
    }
  }
  // bump groups of the test point, a group per lane (with a core kernel: k_predict_groups)
  for (int i = lane; CK == 0 && i < a.kt.n1; i += kPl) add_bumps<D>(a, xp, i, acc);
#pragma unroll
  for (int off = kPl / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kPl);
  return acc;
}

// The same mean by one thread: acc, kPl words of LDS kThreads apart, holds the sums
// of the sixteen lanes.  Candidates come in the order of the list (lane by lane its
// pencils of a round), and a round's hits go to the lanes in turn.
template <int D, bool MIXED, int CK>
__device__ __forceinline__ double predict_point_alone(const PredArgs& a, const CoreBasis& cb, const double* xp,
                                                      double* acc) {
  double sp = 0.0, Sp = 0.0;
  if constexpr (CK == 2) core_point_fields<D>(cb, xp, &sp, &Sp);
  int lo_[3], hi_[3];
  const bool some = point_window<D>(a, xp, lo_, hi_);
#pragma unroll
  for (int l = 0; l < kPl; ++l) acc[l * kThreads] = 0.0;
  const int ny = hi_[1] - lo_[1] + 1;
  const int64_t npen = some ? static_cast<int64_t>(ny) * (hi_[2] - lo_[2] + 1) : 0;
  for (int64_t p0 = 0; p0 < npen; p0 += kPl * kPencils) {
    int32_t nhit = 0;
    for (int l = 0; l < kPl && p0 + l < npen; ++l)
      for (int64_t pk = p0 + l; pk < min(npen, p0 + kPl * kPencils); pk += kPl) {
        const int y = lo_[1] + static_cast<int>(pk % ny), z = lo_[2] + static_cast<int>(pk / ny);
        const int64_t base = (static_cast<int64_t>(z) * a.g[1] + y) * a.g[0];
        const int32_t e = a.cell_start[base + hi_[0] + 1];
        for (int32_t q = a.cell_start[base + lo_[0]]; q < e; ++q) {
          double xq[3], al;
          load_train<D>(a, q, xq, al);
          const double u2 = scaled_sq<D>(xp, xq, a.kt.inv0);
          if (u2 < 1.0) add_hit<D, MIXED, CK>(a, xp, sp, Sp, q, xq, u2, al, acc[nhit++ % kPl * kThreads]);
        }
      }
  }
  for (int i = 0; CK == 0 && i < a.kt.n1; ++i) add_bumps<D>(a, xp, i, acc[i % kPl * kThreads]);
  double s[kPl];
#pragma unroll
  for (int l = 0; l < kPl; ++l) s[l] = acc[l * kThreads];
#pragma unroll
  for (int off = kPl / 2; off > 0; off >>= 1)
#pragma unroll
    for (int l = 0; l < off; ++l) s[l] += s[l + off];
  return s[0];
}

// rows t0 .. m - 1
template <int D, bool MIXED, int CK>
__global__ void __launch_bounds__(kThreads) k_predict(PredArgs a, CoreBasis cb, int64_t t0, int64_t m,
                                                      const double* __restrict__ xs, double* __restrict__ out) {
  __shared__ int32_t ids[kPointsPerBlock][kCandList];
  const int g = threadIdx.x / kPl, lane = threadIdx.x % kPl;
  const int64_t t = t0 + blockIdx.x * static_cast<int64_t>(kPointsPerBlock) + g;
  if (t >= m) return;
  double xp[3];
  for (int k = 0; k < D; ++k) xp[k] = xs[t * D + k];
  const double v = predict_point<D, MIXED, CK>(a, cb, xp, lane, ids[g]);
  if (lane == 0) out[t] = v;
}

template <int D, bool MIXED, int CK>
__global__ void __launch_bounds__(kThreads) k_predict_alone(PredArgs a, CoreBasis cb, int64_t t0, int64_t m,
                                                            const double* __restrict__ xs,
                                                            double* __restrict__ out) {
  __shared__ double acc[kPl][kThreads];
  const int64_t t = t0 + blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x;
  if (t >= m) return;
  double xp[3];
  for (int k = 0; k < D; ++k) xp[k] = xs[t * D + k];
  out[t] = predict_point_alone<D, MIXED, CK>(a, cb, xp, &acc[0][threadIdx.x]);
}

// Request of row t of a batch: the last r with roff[r] <= t (empty requests
// share their offset with the next one).
__device__ __forceinline__ int batch_request(const int64_t* __restrict__ roff, int nreq, int64_t t) {
  int lo = 0, hi = nreq - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (roff[mid] <= t)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Batched form: the rows of all requests (t0 .. m - 1 of them), each with the
// arguments of its request's predictor.
template <int D, bool MIXED, int CK>
__global__ void __launch_bounds__(kThreads) k_predict_batch(const PredArgs* __restrict__ args,
                                                            const CoreBasis* __restrict__ cbs,
                                                            const int32_t* __restrict__ req_pred,
                                                            const int64_t* __restrict__ roff, int nreq, int64_t t0,
                                                            int64_t m, const double* __restrict__ xs,
                                                            double* __restrict__ out) {
  __shared__ int32_t ids[kPointsPerBlock][kCandList];
  const int g = threadIdx.x / kPl, lane = threadIdx.x % kPl;
  const int64_t t = t0 + blockIdx.x * static_cast<int64_t>(kPointsPerBlock) + g;
  if (t >= m) return;
  const int pi = req_pred[batch_request(roff, nreq, t)];
  double xp[3];
  for (int k = 0; k < D; ++k) xp[k] = xs[t * D + k];
  const double v = predict_point<D, MIXED, CK>(args[pi], cbs[pi], xp, lane, ids[g]);
  if (lane == 0) out[t] = v;
}

template <int D, bool MIXED, int CK>
__global__ void __launch_bounds__(kThreads) k_predict_batch_alone(const PredArgs* __restrict__ args,
                                                                  const CoreBasis* __restrict__ cbs,
                                                                  const int32_t* __restrict__ req_pred,
                                                                  const int64_t* __restrict__ roff, int nreq,
                                                                  int64_t t0, int64_t m,
                                                                  const double* __restrict__ xs,
                                                                  double* __restrict__ out) {
  __shared__ double acc[kPl][kThreads];
  const int64_t t = t0 + blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x;
  if (t >= m) return;
  const int pi = req_pred[batch_request(roff, nreq, t)];
  double xp[3];
  for (int k = 0; k < D; ++k) xp[k] = xs[t * D + k];
  out[t] = predict_point_alone<D, MIXED, CK>(args[pi], cbs[pi], xp, &acc[0][threadIdx.x]);
}

// Bump part with a core kernel: one wave per test point.  Lane i < n1 forms
// f_i(x*) (bumps of group i in j order) into LDS; the lanes then stride over
// the members of the point's groups and the wave adds its lanes in a fixed
// order.
template <int D, int CK>
__device__ __forceinline__ void predict_groups_point(const PredArgs& a, const CoreBasis& cb, int64_t t,
                                                     const double* __restrict__ xs, double* __restrict__ out,
                                                     double* f) {
  const int lane = lane_id();
  double xp[3];
  for (int k = 0; k < D; ++k) xp[k] = xs[t * D + k];
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
  if (mask == 0) return;  // uniform
  f[lane] = fi;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  double sp = 0.0, Sp = 0.0;
  if constexpr (CK == 2) core_point_fields<D>(cb, xp, &sp, &Sp);
  double acc = 0.0;
  // masked training point k (binned id q) with shared groups sh
  auto add = [&](int64_t k, int32_t q, uint64_t sh) {
    double bsum = 0.0;
    while (sh) {
      const int i = __builtin_ctzll(sh);
      sh &= sh - 1;
      bsum += f[i] * a.mF[k * a.kt.n1 + i];
    }
    double xq[3], al;
    load_train<D>(a, q, xq, al);
    double cv;
    if constexpr (CK == 1)
      cv = core_value<D, 1>(a.kt.core, xp, xq, 0.0, 0.0, 0.0, 0.0);
    else
      cv = core_value<D, 2>(a.kt.core, xp, xq, sp, Sp, a.kt.core.sig[q], a.kt.core.Sig[q]);
    acc += cv * bsum * al;
  };
  if (a.goff) {
    // the members of the point's groups, each taken in the lowest group it
    // shares: a few thousand points instead of all masked ones
    for (uint64_t mm = mask; mm; mm &= mm - 1) {
      const int i = __builtin_ctzll(mm);
      const int32_t e = a.goff[i + 1];
#pragma unroll 2
      for (int32_t j = a.goff[i] + lane; j < e; j += kWave) {
        const uint64_t sh = a.gmask[j] & mask;
        if (__builtin_ctzll(sh) == i) add(a.gk[j], a.gq[j], sh);
      }
    }
  } else {
    for (int64_t j = lane; j < a.nm; j += kWave) {
      const uint64_t sh = a.mmask[j] & mask;
      if (sh) add(j, a.mlist[j], sh);
    }
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
  if (lane == 0) out[t] += acc;
}

template <int D, int CK>
__global__ void __launch_bounds__(kThreads) k_predict_groups(PredArgs a, CoreBasis cb, int64_t t0, int64_t m,
                                                             const double* __restrict__ xs, double* __restrict__ out) {
  __shared__ double fs[kThreads / kWave][kWave];
  const int64_t t = t0 + (blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x) / kWave;
  if (t >= m) return;  // uniform per wave
  predict_groups_point<D, CK>(a, cb, t, xs, out, fs[threadIdx.x / kWave]);
}

template <int D, int CK>
__global__ void __launch_bounds__(kThreads) k_predict_groups_batch(const PredArgs* __restrict__ args,
                                                                   const CoreBasis* __restrict__ cbs,
                                                                   const int32_t* __restrict__ req_pred,
                                                                   const int64_t* __restrict__ roff, int nreq,
                                                                   int64_t t0, int64_t m,
                                                                   const double* __restrict__ xs,
                                                                   double* __restrict__ out) {
  __shared__ double fs[kThreads / kWave][kWave];
  const int64_t t = t0 + (blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x) / kWave;
  if (t >= m) return;  // uniform per wave
  const int pi = req_pred[batch_request(roff, nreq, t)];
  if (args[pi].nm == 0) return;  // no masked training points: no group part (uniform per wave)
  predict_groups_point<D, CK>(args[pi], cbs[pi], t, xs, out, fs[threadIdx.x / kWave]);
}

}  // namespace

void destroy_predictor(gp_ctx* c, gp_predictor* p);

// device memory for a copy the predictor can do without: null when there is no room
template <typename T>
static T* cache_new(gp_ctx* c, int64_t count) {
  try {
    return dev_new<T>(c, static_cast<size_t>(count));
  } catch (const Error& e) {
    if (e.st != GP_ENOMEM) throw;
    return nullptr;
  }
}

// the lists in one allocation: masks, then indices, ids and offsets
static size_t member_words(const gp_predictor* p) {
  return static_cast<size_t>(p->nlist) * 2 + (p->kt.n1 + 2) / 2;
}

static void free_member_lists(gp_ctx* c, gp_predictor* p) {
  if (p->gmask) dev_free(c, p->gmask, sizeof(uint64_t) * member_words(p));
  p->goff = p->gk = p->gq = nullptr;
  p->gmask = nullptr;
}

// Masked points from which on the lists are made: they cost gp_predictor_create 45 - 60 us
// (a read-back, an allocation, two passes), which a few thousand masks tested by a wave
// do not.  Create, 1, 1009 and 100,003 sites without -> with, us (mixture, Matern core):
//   2858 masked 90 -> 137, 22 -> 22, 68 -> 59, 233 -> 195
//   4787        95 -> 139, 40 -> 28, 88 -> 87, 277 -> 249
//   26,644     140 -> 199, 30 -> 29, 259 -> 250, 1666 -> 1268
constexpr int64_t kListMembers = 4096;

// Member lists of the groups from the predictor's masked points (nm > 0).
static void make_member_lists(gp_ctx* c, gp_predictor* p, int n1) {
  int32_t* size = static_cast<int32_t*>(workspace(c, 122, sizeof(int32_t) * (kMaxGroups + 1)));
  hipLaunchKernelGGL((k_group_members<false>), dim3(n1), dim3(kListThreads), 0, c->stream, p->nm, p->mmask, p->mlist,
                     size, nullptr, nullptr, nullptr);
  check_launch("group sizes");
  int32_t* h = static_cast<int32_t*>(pinned_for_write(c, sizeof(int32_t) * (n1 + 1)));
  GPS_HIP(hipMemcpyAsync(h, size, sizeof(int32_t) * (n1 + 1), hipMemcpyDeviceToHost, c->stream));
  sync(c);
  int64_t total = 0;
  for (int i = 0; i <= n1; ++i) {
    if (i > 0) total += h[i];
    h[i] = static_cast<int32_t>(total);
  }
  if (total >= (int64_t(1) << 31)) return;
  p->nlist = total;  // > 0: every masked point is in a group
  p->gmask = cache_new<uint64_t>(c, static_cast<int64_t>(member_words(p)));
  if (!p->gmask) return;
  p->gk = reinterpret_cast<int32_t*>(p->gmask + total);
  p->gq = p->gk + total;
  p->goff = p->gq + total;
  h2d_async(c, p->goff, h, sizeof(int32_t) * (n1 + 1));
  hipLaunchKernelGGL((k_group_members<true>), dim3(n1), dim3(kListThreads), 0, c->stream, p->nm, p->mmask, p->mlist,
                     p->goff, p->gk, p->gq, p->gmask);
  check_launch("group members");
}

gp_predictor* make_predictor(gp_ctx* c, const gp_dataset* ds, const gp_theta* th, const double* alpha) {
  // a failure part-way releases whatever device memory the predictor holds by then
  auto release = [c](gp_predictor* x) { destroy_predictor(c, x); };
  std::unique_ptr<gp_predictor, decltype(release)> p(new gp_predictor(), release);
  p->ds = ds;
  Bump* tmp_bumps = nullptr;
  KernelTheta kt{};
  upload_theta(c, th, &tmp_bumps, &kt);
  const int nb = std::max(th->n1 * th->n2, 1);
  p->nbumps = nb;
  p->bumps = dev_new<Bump>(c, nb);
  GPS_HIP(hipMemcpyAsync(p->bumps, tmp_bumps, sizeof(Bump) * nb, hipMemcpyDeviceToDevice, c->stream));
  kt.bumps = p->bumps;
  p->kt = kt;
  p->grid = make_grid(ds, th);
  const int64_t n = ds->n;
  p->alpha_b = dev_new<double>(c, n);
  p->coef = dev_new<double>(c, std::max(th->n1, 1));
  permute_to_binned<double>(c, ds, 1, alpha, p->alpha_b);
  KernelCore kc;
  core_params(th, &kc, &p->cb);
  if (kc.kind == GP_CORE_PACIOREK) {
    p->sig = dev_new<double>(c, n);
    p->Sig = dev_new<double>(c, n);
    core_fields(c, ds, p->cb, p->sig, p->Sig);
    kc.sig = p->sig;
    kc.Sig = p->Sig;
  }
  p->kt.core = kc;
  if (th->n1 > 0) {
    Features f;
    compute_features(c, ds, kt, &f, 60);
    hipLaunchKernelGGL(k_group_coef, dim3(th->n1), dim3(kThreads), 0, c->stream, f.nm, th->n1, f.F, f.mlist,
                       p->alpha_b, p->coef);
    check_launch("group coefficients");
    if (kc.kind != GP_CORE_NONE && f.nm > 0) {
      // the feature arrays live in workspace slots: keep copies
      p->nm = f.nm;
      p->mlist = dev_new<int32_t>(c, f.nm);
      p->mmask = dev_new<uint64_t>(c, f.nm);
      p->mF = dev_new<double>(c, f.nm * th->n1);
      GPS_HIP(hipMemcpyAsync(p->mlist, f.mlist, sizeof(int32_t) * f.nm, hipMemcpyDeviceToDevice, c->stream));
      GPS_HIP(hipMemcpyAsync(p->mmask, f.mmask, sizeof(uint64_t) * f.nm, hipMemcpyDeviceToDevice, c->stream));
      GPS_HIP(hipMemcpyAsync(p->mF, f.F, sizeof(double) * f.nm * th->n1, hipMemcpyDeviceToDevice, c->stream));
    }
  }
  // Read-only copies of what the predictor holds, made once it is complete.  A
  // context with an HBM budget, whose later calls are to have the room they had,
  // does without them, as one without the room does: 200,003 sites then take 482 us
  // instead of 300, 1009 sites with a Matern core 232 instead of 86.
  if (c->budget == 0) {
    p->pack = cache_new<double>(c, kPackOf(ds->d) * n);
    if (p->pack)
      hipLaunchKernelGGL(k_pack, dim3(grid_for(n, kThreads)), dim3(kThreads), 0, c->stream, n, ds->d, ds->xb,
                         p->alpha_b, p->pack);
    check_launch("pack training data");
    if (p->nm >= kListMembers) make_member_lists(c, p.get(), th->n1);
  }
  sync(c);
  return p.release();
}

void destroy_predictor(gp_ctx* c, gp_predictor* p) {
  if (!p) return;
  const int64_t n = p->ds->n;
  dev_free(c, p->bumps, sizeof(Bump) * p->nbumps);
  dev_free(c, p->alpha_b, sizeof(double) * n);
  dev_free(c, p->pack, sizeof(double) * kPackOf(p->ds->d) * n);
  free_member_lists(c, p);
  dev_free(c, p->coef, sizeof(double) * std::max(p->kt.n1, 1));
  if (p->sig) dev_free(c, p->sig, sizeof(double) * n);
  if (p->Sig) dev_free(c, p->Sig, sizeof(double) * n);
  if (p->mlist) dev_free(c, p->mlist, sizeof(int32_t) * p->nm);
  if (p->mmask) dev_free(c, p->mmask, sizeof(uint64_t) * p->nm);
  if (p->mF) dev_free(c, p->mF, sizeof(double) * p->nm * p->kt.n1);
  delete p;
}

static PredArgs pred_args(const gp_predictor* p) {
  const gp_dataset* ds = p->ds;
  PredArgs a{};
  a.kt = p->kt;
  a.n = ds->n;
  a.xb = ds->xb;
  a.cell_start = ds->cell_start;
  for (int k = 0; k < 3; ++k) {
    a.lo[k] = ds->lo[k];
    a.cell[k] = ds->cell[k];
    a.g[k] = ds->g[k];
    a.R[k] = p->grid.Rt[k];
  }
  a.alpha = p->alpha_b;
  a.pack = p->pack;
  a.coef = p->coef;
  a.nm = p->nm;
  a.mlist = p->mlist;
  a.mmask = p->mmask;
  a.mF = p->mF;
  a.goff = p->goff;
  a.gk = p->gk;
  a.gq = p->gq;
  a.gmask = p->gmask;
  return a;
}

// Whether a request of m rows takes a thread per point.  Where a window holds a dozen
// candidates, sixteen lanes have little to share, and a thread per point
// (predict_point_alone; the same value bitwise, so that the choice is free) is the better
// form once the points fill the chip.  A thread's chain is its pencils' bounds and its
// candidates; where the forms meet (thousands of rows) the rows are 2500 to 4000 times
// that: one dimension 1 / 6 / 24 candidates 12 / 28 / 62, two 20 / 32 / 75, three 60 / 62 /
// 110, two with a core kernel 23 / 50 / 180.  At two million rows, sixteen lanes -> a thread, us:
// 327 -> 57, 344 -> 118, 403 -> 330; 454 -> 101, 458 -> 132, 469 -> 291; 517 -> 225, 560 -> 240, 572
// -> 339; 48 candidates 520 -> 609, 521 -> 517, 604 -> 510 (10^5 training points; 10^6: 822 -> 899).
// Without the packed data the forms meet earlier (three dimensions, 12 candidates: 10^5
// points 623 -> 401, 10^6 0.88x).
constexpr double kAloneCands = 30, kAlonePlain = 16;  // candidates of a mean window, packed and not
constexpr double kAloneDense = 8;                     // times that: of a window of the fullest cells
constexpr double kAloneRows = 2560;
static_assert(kAloneCands * kAloneDense <= kCandList, "the list of such a window has one part");

static bool alone(const gp_predictor* p, int64_t m) {
  const gp_dataset* ds = p->ds;
  double cells = 1.0, pencils = 1.0;  // of a window inside the grid
  for (int k = 0; k < ds->d; ++k) {
    const double w = std::min(2.0 * p->grid.R[k] + 1.0, static_cast<double>(ds->g[k]));
    cells *= w;
    if (k > 0) pencils *= w;
  }
  const double cands = cells * static_cast<double>(ds->n) / static_cast<double>(ds->ncells);
  if (cands > (p->pack ? kAloneCands : kAlonePlain) || cells * ds->max_cell > kAloneCands * kAloneDense) return false;
  const double chain = 2.0 * pencils + (p->kt.core.kind != GP_CORE_NONE ? 2.0 : 1.0) * cands;
  return static_cast<double>(m) >= kAloneRows * chain;
}

void predict(gp_ctx* c, const gp_predictor* p, int64_t m, const double* xs, int prec, double* out) {
  if (m == 0) return;
  const gp_dataset* ds = p->ds;
  const PredArgs a = pred_args(p);
  const dim3 B(kThreads);
  const bool one = alone(p, m);
  ProfScope ps(c, prec == GP_MIXED ? "predict_f32" : "predict_f64");
  auto go = [&](auto DD) {
    constexpr int D = decltype(DD)::value;
    auto with_core = [&](auto CC) {
      constexpr int CK = decltype(CC)::value;
      for (int64_t t0 = 0; t0 < m; t0 += kLaunchRows) {
        const int64_t t1 = std::min(m, t0 + kLaunchRows);
        const dim3 G(grid_for(t1 - t0, one ? kThreads : kPointsPerBlock));
        auto rows = [&](auto kernel) {
          hipLaunchKernelGGL(kernel, G, B, 0, c->stream, a, p->cb, t0, t1, xs, out);
        };
        if (prec == GP_MIXED)
          rows(one ? k_predict_alone<D, true, CK> : k_predict<D, true, CK>);
        else
          rows(one ? k_predict_alone<D, false, CK> : k_predict<D, false, CK>);
        if constexpr (CK != 0) {
          if (p->nm > 0)
            hipLaunchKernelGGL((k_predict_groups<D, CK>), dim3(grid_for((t1 - t0) * kWave, kThreads)), B, 0,
                               c->stream, a, p->cb, t0, t1, xs, out);
        }
      }
    };
    if (p->kt.core.kind == GP_CORE_MATERN)
      with_core(std::integral_constant<int, 1>{});
    else if (p->kt.core.kind == GP_CORE_PACIOREK)
      with_core(std::integral_constant<int, 2>{});
    else
      with_core(std::integral_constant<int, 0>{});
  };
  if (ds->d == 1)
    go(std::integral_constant<int, 1>{});
  else if (ds->d == 2)
    go(std::integral_constant<int, 2>{});
  else
    go(std::integral_constant<int, 3>{});
  check_launch("predict");
}

void predict_batch(gp_ctx* c, int32_t nreq, const gp_predictor* const* preds, const int64_t* roff_host,
                   const double* xs, int prec, double* out) {
  for (int32_t r = 0; r < nreq; ++r) {
    GPS_REQUIRE(preds[r]->ds->d == preds[0]->ds->d, GP_EINVAL,
                "gp_predict_batch: all predictors must have the same dimension");
    GPS_REQUIRE(preds[r]->kt.core.kind == preds[0]->kt.core.kind, GP_EINVAL,
                "gp_predict_batch: all predictors must have the same core kernel kind");
  }
  const int64_t m = roff_host[nreq];
  if (m == 0) return;
  // distinct predictors, in order of first appearance
  std::vector<const gp_predictor*> uniq;
  std::vector<int32_t> req_pred(nreq);
  for (int32_t r = 0; r < nreq; ++r) {
    int32_t k = 0;
    while (k < static_cast<int32_t>(uniq.size()) && uniq[k] != preds[r]) ++k;
    if (k == static_cast<int32_t>(uniq.size())) uniq.push_back(preds[r]);
    req_pred[r] = k;
  }
  const int d = uniq[0]->ds->d;
  const int ck = uniq[0]->kt.core.kind;
  bool any_nm = false, one = true;
  for (const gp_predictor* p : uniq) {
    any_nm = any_nm || p->nm > 0;
    one = one && alone(p, m);
  }
  const size_t np = uniq.size();
  const size_t b_args = sizeof(PredArgs) * np, b_cb = sizeof(CoreBasis) * np;
  const size_t b_req = sizeof(int32_t) * nreq, b_off = sizeof(int64_t) * (nreq + 1);
  auto up = [](size_t b) { return (b + 255) & ~size_t(255); };
  const size_t total = up(b_args) + up(b_cb) + up(b_req) + up(b_off);
  char* dbuf = static_cast<char*>(workspace(c, 123, total));
  char* hbuf = static_cast<char*>(pinned_for_write(c, total));
  PredArgs* ha = reinterpret_cast<PredArgs*>(hbuf);
  CoreBasis* hc = reinterpret_cast<CoreBasis*>(hbuf + up(b_args));
  for (size_t k = 0; k < np; ++k) {
    ha[k] = pred_args(uniq[k]);
    hc[k] = uniq[k]->cb;
  }
  std::memcpy(hbuf + up(b_args) + up(b_cb), req_pred.data(), b_req);
  std::memcpy(hbuf + up(b_args) + up(b_cb) + up(b_req), roff_host, b_off);
  h2d_async(c, dbuf, hbuf, total);
  const PredArgs* da = reinterpret_cast<const PredArgs*>(dbuf);
  const CoreBasis* dc = reinterpret_cast<const CoreBasis*>(dbuf + up(b_args));
  const int32_t* dreq = reinterpret_cast<const int32_t*>(dbuf + up(b_args) + up(b_cb));
  const int64_t* droff = reinterpret_cast<const int64_t*>(dbuf + up(b_args) + up(b_cb) + up(b_req));
  const dim3 B(kThreads);
  ProfScope ps(c, prec == GP_MIXED ? "predict_batch_f32" : "predict_batch_f64");
  auto go = [&](auto DD) {
    constexpr int D = decltype(DD)::value;
    auto with_core = [&](auto CC) {
      constexpr int CK = decltype(CC)::value;
      for (int64_t t0 = 0; t0 < m; t0 += kLaunchRows) {
        const int64_t t1 = std::min(m, t0 + kLaunchRows);
        const dim3 G(grid_for(t1 - t0, one ? kThreads : kPointsPerBlock));
        auto rows = [&](auto kernel) {
          hipLaunchKernelGGL(kernel, G, B, 0, c->stream, da, dc, dreq, droff, nreq, t0, t1, xs, out);
        };
        if (prec == GP_MIXED)
          rows(one ? k_predict_batch_alone<D, true, CK> : k_predict_batch<D, true, CK>);
        else
          rows(one ? k_predict_batch_alone<D, false, CK> : k_predict_batch<D, false, CK>);
        if constexpr (CK != 0) {
          if (any_nm)
            hipLaunchKernelGGL((k_predict_groups_batch<D, CK>), dim3(grid_for((t1 - t0) * kWave, kThreads)), B, 0,
                               c->stream, da, dc, dreq, droff, nreq, t0, t1, xs, out);
        }
      }
    };
    if (ck == GP_CORE_MATERN)
      with_core(std::integral_constant<int, 1>{});
    else if (ck == GP_CORE_PACIOREK)
      with_core(std::integral_constant<int, 2>{});
    else
      with_core(std::integral_constant<int, 0>{});
  };
  if (d == 1)
    go(std::integral_constant<int, 1>{});
  else if (d == 2)
    go(std::integral_constant<int, 2>{});
  else
    go(std::integral_constant<int, 3>{});
  check_launch("predict batch");
}

}  // namespace gps
