// FMM evaluation pass (stage order of Sec. III.A: sort, P2M, M2M, M2L, L2L,
// L2P, P2P), hand-written HIP kernels for gfx950.
//
// Coefficients are kept normalised (tables.h) and scaled per box by its
// radius rho (multipole degree n divided by rho^n, local degree n multiplied
// by rho^{n+1}), box-major: [box][(P+1)^2].  With this scaling every
// translation below multiplies by ratios of lengths that are at most 1
// (child/parent radius, centre offset/parent radius, radius/distance of an
// admissible pair), so single precision cannot overflow.
// All translations are rotation based (Sec. II.D, App. B): for a shift from
// an old centre to a new one with b = old - new = r (sin B cos A,
// sin B sin A, cos B), the coefficients are rotated so that b points along
// +z, shifted with the diagonal z-axis operators of App. B.3 and rotated
// back.  The rotation about y by B is factored as
//   Rz(-pi/2) Ry(-pi/2) Rz(B) Ry(pi/2) Rz(pi/2)
// so each interaction needs four products with the fixed per-degree block
// Y_n (or its transpose) and azimuthal 2x2 rotations (App. B.1) by angles
// built from A and B; the Rz(+-pi/2) next to the z-axis operator cancel
// because that operator commutes with rotations about z.  One thread owns
// one interaction (all of its coefficients sit in registers); the operator
// tables are wave-uniform and are read through the scalar cache.
//
//   M2L item: thread = (target box, up to a dozen of its sources); the
//             items of one target share a block and their sums are added
//             in lane order, so results do not depend on scheduling (the
//             only atomics are adds to lane-private LDS slots).
//   M2M:      thread = child box; the 2^s children of a parent sit in
//             adjacent lanes and are summed with cross-lane shuffles.
//   L2L:      two launches for all levels: the leaves' parents get their M2L
//             sum plus the shifted M2L sums of all their ancestors, one lane
//             per ancestor (local re-centring is exact), summed across
//             lanes; each leaf then adds its parent's shifted local.
//   P2M:      block = leaf, thread = point, LDS reduction over points.
//   L2P:      block = target leaf, thread = target point; writes outputs.
// The near field (P2P) is in near.hip.  This file is compiled once per
// expansion order (FMM_ORDER), so that the orders' kernels build in parallel.
#include <cmath>

#include <type_traits>

#include "internal.h"
#include "ops.h"
#include "tables.h"

namespace fmm {
namespace {

using namespace ops;

// ---------------------------------------------------------------- P2M
// C_leaf = normc * sum_i q_i R-hat((x_i - c) / rho)  (scaled multipole).
// G leaves per wave (LW = 64/G lanes each, lane = point).  The per-lane
// terms go to LDS in chunks of kP2MRows coefficients (row r of lane l at
// r * kRow + l); each chunk is then summed over every leaf's lanes by one
// lane per (leaf, coefficient), in a fixed order (two interleaved partial
// sums).  The kernel also does the
// sort stage: it reads each charge in input order and writes the leaf's
// 32-byte source records that P2P reads.
constexpr int kRow = 65;       // LDS row stride: a lane's rows fall in different banks
constexpr int kP2MRows = 16;   // coefficients per chunk

// Row r of buf holds coefficient rowk[r] (or k0 + r when rowk is NULL) of
// every lane; cs[leaf][coefficient] = the sum over the leaf's LW lanes.
template <int LW, int K, typename T>
__device__ __forceinline__ void leaf_sums(const T* buf, const int* rowk, int nr, int k0,
                                          T (*cs)[K], int G) {
  for (int t = threadIdx.x; t < G * nr; t += 64) {
    const int hh = t / nr, r = t - hh * nr;
    const T* row = buf + r * kRow + hh * LW;
    T s0 = T(0), s1 = T(0);
#pragma unroll
    for (int l = 0; l < LW; l += 2) {
      s0 += row[l];
      s1 += row[l + 1];
    }
    cs[hh][rowk ? rowk[r] : k0 + r] = s0 + s1;
  }
}

template <int P, typename T, int G>
__global__ __launch_bounds__(64) void k_p2m(
    int64_t nleaf, const int32_t* __restrict__ leaf_box,
    const int32_t* __restrict__ leaf_start, const double* __restrict__ xs,
    const double* __restrict__ ys, const double* __restrict__ zs,
    const int32_t* __restrict__ perm, const T* __restrict__ q, Src<T>* __restrict__ src,
    const double* __restrict__ cx, const double* __restrict__ cy,
    const double* __restrict__ cz, const double* __restrict__ scale,
    const T* __restrict__ tab, T* __restrict__ C) {
  constexpr int K = K_<P>::value;
  constexpr int LW = 64 / G;
  __shared__ T cs[G][K];  // finished sums, stored coalesced at the end
  __shared__ T buf[(kP2MRows - 1) * kRow + 64];
  __shared__ int rowk[kP2MRows];  // coefficient held by each row
  const int lane = threadIdx.x;
  const int h = lane / LW, l = lane % LW;
  const int64_t leaf = (int64_t)blockIdx.x * G + h;
  const bool has = leaf < nleaf;
  const int64_t g = has ? leaf_box[leaf] : 0;
  const int st = has ? leaf_start[leaf] : 0, en = has ? leaf_start[leaf + 1] : 0;
  const double ox = cx[g], oy = cy[g], oz = cz[g], ir = 1.0 / scale[g];
  if (G > 1) {
    // at most one point per lane: every term goes to LDS as it is formed
    // (the basis comes order by order, so rows record their coefficient)
    const int j = st + l;
    const bool pt = j < en;
    const int jj = pt ? j : st;
    const T qj = pt ? q[perm[j]] : T(0);
    if (pt) src[j] = Src<T>{xs[j], ys[j], zs[j], qj};
    int e = 0;  // terms emitted so far (the same in every lane)
    regular_basis<P, T>(T((xs[jj] - ox) * ir), T((ys[jj] - oy) * ir), T((zs[jj] - oz) * ir),
                        [&](int k, T v) {
                          const int r = e % kP2MRows;
                          buf[r * kRow + lane] = qj * v;
                          if (lane == 0) rowk[r] = k;
                          ++e;
                          if (r == kP2MRows - 1 || e == K) {
                            __syncthreads();
                            leaf_sums<LW, K, T>(buf, rowk, r + 1, 0, cs, G);
                            __syncthreads();
                          }
                        });
  } else {
    T acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = T(0);
    for (int j = st + l; j < en; j += LW) {
      const T qj = q[perm[j]];
      src[j] = Src<T>{xs[j], ys[j], zs[j], qj};
      regular_basis<P, T>(T((xs[j] - ox) * ir), T((ys[j] - oy) * ir), T((zs[j] - oz) * ir),
                          [&](int k, T v) { acc[k] = fma(qj, v, acc[k]); });
    }
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += kP2MRows) {
#pragma unroll
      for (int r = 0; r < kP2MRows; ++r)
        if (k0 + r < K) buf[r * kRow + lane] = acc[k0 + r];
      __syncthreads();
      leaf_sums<LW, K, T>(buf, nullptr, (K - k0 < kP2MRows ? K - k0 : kP2MRows), k0, cs, 1);
      __syncthreads();
    }
  }
  for (int idx = lane; idx < G * K; idx += 64) {
    const int hh = idx / K, k = idx - hh * K;
    const int64_t lf = (int64_t)blockIdx.x * G + hh;
    if (lf < nleaf) C[(int64_t)leaf_box[lf] * K + k] = cs[hh][k] * tab[tab_normc(P) + k];
  }
}

// ------------------------------------------- translations shared by waves
// One translation (rotate, z-shift, rotate back) split over the NW waves of
// a block, lane l of every wave working on the same translation.  The
// rotations act degree by degree and the z-shift order by order, so wave w
// rotates the degrees of share_mask(P, NW, w, false, kind) and z-shifts the
// orders of share_mask(P, NW, w, true, kind), the coefficients passing
// between the two through a 64-lane LDS tile (three barriers).  Every
// coefficient undergoes the same operations in the same order as in
// rotate_shift, so the results are identical to the one-lane form; each
// wave holds a fraction of the coefficients and runs a fraction of the
// chain of dependent operations, which raises the occupancy where the
// one-lane form runs out of registers and cuts the latency of launches with
// few translations (the level chains).

// Multiply-adds of the two rotation phases on degree n (Y products and
// azimuth steps) and of the z-shift of orders +-am (M2L: full blocks; M2M,
// L2L: triangles).
__host__ __device__ constexpr int rot_cost(int n) { return 4 * (n * n + n + 1) + 16 * n; }
__host__ __device__ constexpr int shift_cost(int P, int am, int kind) {
  const int d = P + 1 - am;
  return (am > 0 ? 2 : 1) * (kind == kM2L ? d * d : d * (d + 1));
}

// Degrees (orders: false/true) of wave w: largest cost first, each onto the
// least loaded wave (the first of equals).
__host__ __device__ constexpr unsigned share_mask(int P, int NW, int w, bool orders, int kind) {
  int load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  unsigned mask[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  unsigned done = 0;
  for (int step = 0; step <= P; ++step) {
    int pick = -1, pc = -1;
    for (int x = 0; x <= P; ++x) {
      if ((done >> x) & 1u) continue;
      const int c = orders ? shift_cost(P, x, kind) : rot_cost(x);
      if (c > pc) {
        pc = c;
        pick = x;
      }
    }
    done |= 1u << pick;
    int best = 0;
    for (int j = 1; j < NW; ++j)
      if (load[j] < load[best]) best = j;
    load[best] += pc;
    mask[best] |= 1u << pick;
  }
  return mask[w];
}

// coefficient loops over (n, m), k = cidx(n, m): the degrees of mask DM,
// the orders of mask OM
#define FMM_DEG_LOOP(DM, stmt)                        \
  _Pragma("unroll") for (int n = 0; n <= P; ++n) {    \
    if (!(((DM) >> n) & 1u)) continue;                \
    _Pragma("unroll") for (int m = -n; m <= n; ++m) { \
      const int k = cidx(n, m);                       \
      stmt;                                           \
    }                                                 \
  }
#define FMM_ORD_LOOP(OM, stmt)                                \
  _Pragma("unroll") for (int n = 0; n <= P; ++n) {            \
    _Pragma("unroll") for (int m = -n; m <= n; ++m) {         \
      if (!(((OM) >> (m < 0 ? -m : m)) & 1u)) continue;       \
      const int k = cidx(n, m);                               \
      stmt;                                                   \
    }                                                         \
  }

// Wave W's part of one translation per lane: v holds the wave's degrees on
// entry and the translated coefficients of those degrees on return.  All
// waves of the block call it together (barriers inside; lanes with act
// false take no part but reach them).  X: LDS tile of (K - 1) kRow + 64
// entries, free again on return.
template <int P, int KIND, typename T, int NW, int W>
__device__ __forceinline__ void turn_shared(T* v, bool act, const Turn<P, KIND, T>& g,
                                            const T* __restrict__ tab, T* X, int lane) {
  constexpr int K = K_<P>::value;
  constexpr unsigned DM = share_mask(P, NW, W, false, KIND);
  constexpr unsigned OM = share_mask(P, NW, W, true, KIND);
  if (act) {
    turn_forward<P, KIND, T, DM>(v, g, tab);
    FMM_DEG_LOOP(DM, X[k * kRow + lane] = v[k])
  }
  __syncthreads();
  if (act) {
    T z[K];
    FMM_ORD_LOOP(OM, z[k] = X[k * kRow + lane])
    zshift<P, KIND, T, OM>(z, g.a, g.b, tab);
    FMM_ORD_LOOP(OM, X[k * kRow + lane] = z[k])
  }
  __syncthreads();
  if (act) FMM_DEG_LOOP(DM, v[k] = X[k * kRow + lane])
  __syncthreads();
  if (act) turn_back<P, KIND, T, DM>(v, g, tab);
}

// ---------------------------------------------------------------- M2M
template <int P, typename T>
__global__ __launch_bounds__(64) void k_m2m(
    int64_t nchild, const int32_t* __restrict__ par, const int32_t* __restrict__ child0,
    int s, const double* __restrict__ cx, const double* __restrict__ cy,
    const double* __restrict__ cz, const double* __restrict__ scale,
    const T* __restrict__ tab, T* C) {
  constexpr int K = K_<P>::value;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = i < nchild;
  const int64_t ii = live ? i : 0;
  const int64_t c = child0[ii >> s] + (ii & ((1 << s) - 1));
  const int64_t pa = par[ii >> s];
  T v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = live ? C[c * K + k] : T(0);
  rotate_shift<P, kM2M, T>(v, cx[c] - cx[pa], cy[c] - cy[pa], cz[c] - cz[pa], scale[c],
                           scale[pa], tab);
  const int nch = 1 << s;
  for (int off = 1; off < nch; off <<= 1) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += __shfl_xor(v[k], off, 64);
  }
  if (live && (i & (nch - 1)) == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) C[pa * K + k] = v[k];
  }
}

// k_m2m with each translation shared by the kShareWaves waves of a block
// (turn_shared); the same results.
template <int P, typename T, int W>
__device__ __forceinline__ void m2m_wave(int lane, int64_t i, bool live, int64_t c, int64_t pa,
                                         int s, const Turn<P, kM2M, T>& g,
                                         const T* __restrict__ tab, T* C, T* X) {
  constexpr int K = K_<P>::value;
  constexpr unsigned DM = share_mask(P, kShareWaves, W, false, kM2M);
  T v[K];
  FMM_DEG_LOOP(DM, v[k] = live ? C[c * K + k] : T(0))
  turn_shared<P, kM2M, T, kShareWaves, W>(v, true, g, tab, X, lane);
  const int nch = 1 << s;
  for (int off = 1; off < nch; off <<= 1) FMM_DEG_LOOP(DM, v[k] += __shfl_xor(v[k], off, 64))
  if (live && (i & (nch - 1)) == 0) FMM_DEG_LOOP(DM, C[pa * K + k] = v[k])
}

template <int P, typename T>
__global__ __launch_bounds__(64 * kShareWaves) void k_m2m_shared(
    int64_t nchild, const int32_t* __restrict__ par, const int32_t* __restrict__ child0,
    int s, const double* __restrict__ cx, const double* __restrict__ cy,
    const double* __restrict__ cz, const double* __restrict__ scale,
    const T* __restrict__ tab, T* C) {
  constexpr int K = K_<P>::value;
  __shared__ T X[(K - 1) * kRow + 64];
  const int lane = threadIdx.x % 64;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const bool live = i < nchild;
  const int64_t ii = live ? i : 0;
  const int64_t c = child0[ii >> s] + (ii & ((1 << s) - 1));
  const int64_t pa = par[ii >> s];
  const Turn<P, kM2M, T> g(cx[c] - cx[pa], cy[c] - cy[pa], cz[c] - cz[pa], scale[c], scale[pa]);
  switch (w) {
    case 0: m2m_wave<P, T, 0>(lane, i, live, c, pa, s, g, tab, C, X); break;
    case 1: m2m_wave<P, T, 1>(lane, i, live, c, pa, s, g, tab, C, X); break;
    case 2: m2m_wave<P, T, 2>(lane, i, live, c, pa, s, g, tab, C, X); break;
    default: m2m_wave<P, T, 3>(lane, i, live, c, pa, s, g, tab, C, X); break;
  }
}

// ---------------------------------------------------------------- M2L
// For every target segment of this block (seg_tgt[g], lanes
// [seg_lanes[g] & 255, seg_lanes[g] >> 8), g in [sb, se)), adds the K rows
// (coefficients; row r of lane l at r * STRIDE + l, an odd stride, so that
// reads of different rows of one lane hit different banks) over the
// segment's lanes in lane order and stores the sums as the target's local.
template <int K, int STRIDE, typename T>
__device__ __forceinline__ void segment_sums(const T* buf, int sb, int se,
                                             const int32_t* __restrict__ seg_tgt,
                                             const int32_t* __restrict__ seg_lanes, T* D) {
  const int n = (se - sb) * K;
  for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
    const int g = sb + idx / K, r = idx % K;
    const int info = seg_lanes[g];
    T acc = T(0);
    for (int l = info & 255; l < (info >> 8); ++l) acc += buf[r * STRIDE + l];
    D[(int64_t)seg_tgt[g] * K + r] = acc;
  }
}

// Waves of a block of the one-lane form: they share the block's accumulators.
constexpr int m2l_block_waves(bool fp64) { return fp64 ? 2 : 4; }
// Waves per SIMD it is held to: the most that the registers of a translation
// (one expansion, the products' partial results, the geometry) allow without
// spilling.
constexpr int m2l_waves_per_simd(int p, bool fp64) {
  return fp64 ? (p <= 5 ? 4 : p == 6 ? 3 : p <= 8 ? 2 : 1)
              : (p <= 5 ? 6 : p == 6 ? 5 : p <= 8 ? 4 : p == 9 ? 3 : 2);
}

// Lane l of the W waves of a block = work item l (a run of at most a dozen
// source boxes of one target); wave w translates the item's pairs w, w + W,
// w + 2 W, ... and adds them to the item's row of accumulators in LDS, the
// waves one after another (barriers), so that an item's pairs are added in
// list order.  The items of one target share the block and their sums are
// added in lane order into the target's local, D_t = sum of its M2L
// translations, written once (no partial rows in memory).
// Bound by the latencies of one wave: the operator tables come through the
// scalar unit about every 16 (FP64) multiply-adds, and a lane's expansion
// fills the registers, so what counts is the number of waves on a SIMD.
// Accumulators shared by W waves and registers held to one expansion (pins
// in the translation steps) give two waves in FP64 at p = 8 (81 x 63
// accumulators of 8 bytes, 40 KB for two waves) and four in FP32, where one
// wave per accumulator set gave one and two.  Measured (uniform cube 2^20,
// 3.4 M pairs, p = 8; one wave per accumulator set before): FP64 0.50 -> 0.40
// ms, FP32 0.29 -> 0.27 ms; 100000 points, FP32, p = 10 (four waves a
// translation) 118 -> 91 us, but 2800 points 63.0 -> 63.5 us and M2M there 17.6
// -> 18.2 us (without the pins in M2M's shares 17.9, the pass no shorter).
template <int P, typename T, int W>
__global__ __launch_bounds__(kM2LBlock* W)
    __attribute__((amdgpu_waves_per_eu(m2l_waves_per_simd(P, sizeof(T) == 8)))) void k_m2l(
        const int32_t* __restrict__ item_tgt, const int32_t* __restrict__ item_begin,
        const int32_t* __restrict__ item_end, const int32_t* __restrict__ seg_ptr,
        const int32_t* __restrict__ seg_tgt, const int32_t* __restrict__ seg_lanes,
        const int32_t* __restrict__ src, const BoxGeo* __restrict__ geo,
        const T* __restrict__ C, const T* __restrict__ tab, T* __restrict__ D) {
  constexpr int K = K_<P>::value;
  constexpr int S = m2l_lanes(P, sizeof(T) == 8) | 1;  // row stride (odd)
  __shared__ T acc[(K - 1) * S + m2l_lanes(P, sizeof(T) == 8)];
  const int64_t b = xcd_block(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x % kM2LBlock;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kM2LBlock);
  for (int e = threadIdx.x; e < (int)(sizeof(acc) / sizeof(T)); e += kM2LBlock * W) acc[e] = T(0);
  const int64_t i = b * kM2LBlock + lane;
  const int tgt = max(item_tgt[i], 0);
  const int jb = item_begin[i], len = item_end[i] - jb;  // len 0 for idle lanes
  // pairs of the longest item of the block (the same in every wave)
  int longest = len;
#pragma unroll
  for (int off = 1; off < kM2LBlock; off <<= 1)
    longest = max(longest, __shfl_xor(longest, off, 64));
  longest = __builtin_amdgcn_readfirstlane(longest);
  for (int j = w; j - w < longest; j += W) {
    // lanes past their item's end translate its last pair (or the list's
    // first) once more and add nothing: no divergence around the translation
    const int sb = src[jb + max(min(j, len - 1), 0)];
    int tb = tgt;
    pin(tb);  // read again every round: no registers for it in between
    const BoxGeo gs = geo[sb], gt = geo[tb];
    T v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = C[(int64_t)sb * K + k];
    rotate_shift<P, kM2L, T>(v, gs.x - gt.x, gs.y - gt.y, gs.z - gt.z, gs.scale, gt.scale, tab);
    // finished here, not moved behind the barriers
#pragma unroll
    for (int k = 0; k < K; ++k) pin(v[k]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < W; ++u) {
      if (w == u && j < len) {
        int at = lane;
        pin(at);  // no addresses held over the translation
#pragma unroll
        for (int k = 0; k < K; ++k) {
          if (sizeof(T) == 8)  // an LDS add needs no register
            __hip_atomic_fetch_add(&acc[k * S + at], v[k], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
          else  // (in FP32 it would be a compare-and-swap loop)
            acc[k * S + at] += v[k];
        }
      }
      if (u + 1 < W) __syncthreads();
    }
  }
  __syncthreads();
  segment_sums<K, S, T>(acc, seg_ptr[b], seg_ptr[b + 1], seg_tgt, seg_lanes, D);
}

template <int P, typename T, int NW, int W>
__device__ __forceinline__ void m2l_share(int lane, int jb, int je, int iters, double tx,
                                          double ty, double tz, double rt,
                                          const int32_t* __restrict__ src,
                                          const double* __restrict__ cx,
                                          const double* __restrict__ cy,
                                          const double* __restrict__ cz,
                                          const double* __restrict__ scale,
                                          const T* __restrict__ C, const T* __restrict__ tab,
                                          T* X) {
  constexpr int K = K_<P>::value;
  constexpr unsigned DM = share_mask(P, NW, W, false, kM2L);
  T acc[K];
  FMM_DEG_LOOP(DM, acc[k] = T(0))
  for (int it = 0; it < iters; ++it) {
    const int j = jb + it;
    const bool act = j < je;
    const int sidx = act ? src[j] : 0;
    const Turn<P, kM2L, T> g(cx[sidx] - tx, cy[sidx] - ty, cz[sidx] - tz, scale[sidx], rt);
    T v[K];
    if (act) FMM_DEG_LOOP(DM, v[k] = C[(int64_t)sidx * K + k])
    turn_shared<P, kM2L, T, NW, W>(v, act, g, tab, X, lane);
    if (act) {
      // a plain add, as in k_m2l
#pragma clang fp contract(off)
      FMM_DEG_LOOP(DM, acc[k] += v[k])
    }
  }
  FMM_DEG_LOOP(DM, X[k * kRow + lane] = acc[k])
}

// The same M2L items with the translation of each item shared by the NW
// waves of a block (turn_shared): lane l of every wave works on item l.
// Gives the same results as k_m2l.  Built where the one-lane form is left
// with two waves per SIMD in FP32 (p = 10: 0.64 against 0.72 ms for 4.2 M
// pairs; at p = 9 it is the slower one, 0.57 against 0.49, as in FP64 at
// p = 6 and 7, 0.43 against 0.29 and 0.68 against 0.45).
template <int P, typename T, int NW>
__global__ __launch_bounds__(kM2LBlock * NW) void k_m2l_shared(
    const int32_t* __restrict__ item_tgt,
    const int32_t* __restrict__ item_begin, const int32_t* __restrict__ item_end,
    const int32_t* __restrict__ seg_ptr, const int32_t* __restrict__ seg_tgt,
    const int32_t* __restrict__ seg_lanes, const int32_t* __restrict__ src,
    const double* __restrict__ cx, const double* __restrict__ cy,
    const double* __restrict__ cz, const double* __restrict__ scale,
    const T* __restrict__ C, const T* __restrict__ tab, T* __restrict__ D) {
  constexpr int K = K_<P>::value;
  __shared__ T X[(K - 1) * kRow + kM2LBlock];
  const int64_t b = xcd_block(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x % kM2LBlock;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kM2LBlock);
  const int64_t i = b * kM2LBlock + lane;
  const int t = item_tgt[i];
  const int jb = item_begin[i], je = item_end[i];  // empty for idle lanes
  const int tt = t < 0 ? 0 : t;
  const double tx = cx[tt], ty = cy[tt], tz = cz[tt], rt = scale[tt];
  // translations of the longest item of the block (the same in every wave)
  int iters = je - jb;
#pragma unroll
  for (int off = 1; off < kM2LBlock; off <<= 1) iters = max(iters, __shfl_xor(iters, off, 64));
  iters = __builtin_amdgcn_readfirstlane(iters);
#define FMM_M2L_WAVE(W)                                                                   \
  case W:                                                                                 \
    if constexpr (W < NW)                                                                 \
      m2l_share<P, T, NW, W>(lane, jb, je, iters, tx, ty, tz, rt, src, cx, cy, cz, scale, \
                             C, tab, X);                                                  \
    break;
  static_assert(NW <= 4, "at most four waves per translation");
  switch (w) {
    FMM_M2L_WAVE(0)
    FMM_M2L_WAVE(1)
    FMM_M2L_WAVE(2)
    FMM_M2L_WAVE(3)
    default: break;
  }
#undef FMM_M2L_WAVE
  __syncthreads();
  segment_sums<K, kRow, T>(X, seg_ptr[b], seg_ptr[b + 1], seg_tgt, seg_lanes, D);
}

// ---------------------------------------------------------------- L2L
// Final locals of one list of boxes (FinList): GS lanes per box, lane j
// translating the expansion anc[j] of src (re-centring a truncated local
// expansion is exact, so these translations add up to the level-by-level
// chain), the lanes' results added by a butterfly in a fixed order; the
// first lane adds the box's own M2L sum (D) and writes the final local to
// out (the multipole array, free once M2L has run).
template <int P, typename T, int GS>
__global__ __launch_bounds__(64) void k_l2l_fin(
    int64_t nfin, const int32_t* __restrict__ fin_box, const int32_t* __restrict__ fin_own,
    const int32_t* __restrict__ fin_anc, const double* __restrict__ cx,
    const double* __restrict__ cy, const double* __restrict__ cz,
    const double* __restrict__ scale, const T* __restrict__ tab, const T* src,
    const T* __restrict__ D, T* out) {
  constexpr int K = K_<P>::value;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t g = i / GS;
  const int j = (int)(i % GS);
  const bool live = g < nfin;
  const int64_t t = live ? fin_box[g] : 0;
  const int a = live ? fin_anc[i] : -1;
  T v[K];
  if (a >= 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = src[(int64_t)a * K + k];
    rotate_shift<P, kL2L, T>(v, cx[a] - cx[t], cy[a] - cy[t], cz[a] - cz[t], scale[a], scale[t],
                             tab);
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = T(0);
  }
#pragma unroll
  for (int off = 1; off < GS; off <<= 1) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += __shfl_xor(v[k], off, 64);
  }
  if (live && j == 0) {
    const bool own = fin_own[g] != 0;
#pragma unroll
    for (int k = 0; k < K; ++k) out[t * K + k] = (own ? D[t * K + k] : T(0)) + v[k];
  }
}

// k_l2l_fin with each translation shared by the kShareWaves waves of a
// block (turn_shared) and the group size gs a launch argument; the same
// results.
template <int P, typename T, int W>
__device__ __forceinline__ void l2l_fin_wave(int lane, bool live, int j, int gs, int64_t t,
                                             int64_t a, bool own, const Turn<P, kL2L, T>& g,
                                             const T* __restrict__ tab, const T* src,
                                             const T* __restrict__ D, T* out, T* X) {
  constexpr int K = K_<P>::value;
  constexpr unsigned DM = share_mask(P, kShareWaves, W, false, kL2L);
  const bool act = a >= 0;
  T v[K];
  FMM_DEG_LOOP(DM, v[k] = act ? src[a * K + k] : T(0))
  turn_shared<P, kL2L, T, kShareWaves, W>(v, act, g, tab, X, lane);
  for (int off = 1; off < gs; off <<= 1) FMM_DEG_LOOP(DM, v[k] += __shfl_xor(v[k], off, 64))
  if (live && j == 0) FMM_DEG_LOOP(DM, out[t * K + k] = (own ? D[t * K + k] : T(0)) + v[k])
}

template <int P, typename T>
__global__ __launch_bounds__(64 * kShareWaves) void k_l2l_fin_shared(
    int64_t nfin, int gs, const int32_t* __restrict__ fin_box,
    const int32_t* __restrict__ fin_own, const int32_t* __restrict__ fin_anc,
    const double* __restrict__ cx, const double* __restrict__ cy,
    const double* __restrict__ cz, const double* __restrict__ scale,
    const T* __restrict__ tab, const T* src, const T* __restrict__ D, T* out) {
  constexpr int K = K_<P>::value;
  __shared__ T X[(K - 1) * kRow + 64];
  const int lane = threadIdx.x % 64;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const int64_t g = i / gs;
  const int j = (int)(i % gs);
  const bool live = g < nfin;
  const int64_t t = live ? fin_box[g] : 0;
  const int64_t a = live ? fin_anc[i] : -1;
  const bool own = live && fin_own[g] != 0;
  const int64_t aa = a >= 0 ? a : t;  // a valid pair for lanes without a source
  const Turn<P, kL2L, T> tr(cx[aa] - cx[t], cy[aa] - cy[t], cz[aa] - cz[t], scale[aa], scale[t]);
  switch (w) {
    case 0: l2l_fin_wave<P, T, 0>(lane, live, j, gs, t, a, own, tr, tab, src, D, out, X); break;
    case 1: l2l_fin_wave<P, T, 1>(lane, live, j, gs, t, a, own, tr, tab, src, D, out, X); break;
    case 2: l2l_fin_wave<P, T, 2>(lane, live, j, gs, t, a, own, tr, tab, src, D, out, X); break;
    default: l2l_fin_wave<P, T, 3>(lane, live, j, gs, t, a, own, tr, tab, src, D, out, X); break;
  }
}

// ---------------------------------------------------------------- L2P
// L2P: u = -1/(4 pi) (1/rho) sum w_m D R-hat(y), y = (x - c)/rho, and
// field = -grad u (an extra 1/rho from the chain rule), at every point of the
// target leaf, added to the near field P2P left in leaf order; writes the
// outputs in input order.  G leaves per wave, LW = 64/G lanes each, lane =
// point.  The gradient is evaluated from the leaf's gradient expansions
// (grad_coeff, formed once per leaf in LDS), so every point needs only the
// basis values.
template <int P, typename T, bool FIELD, int G>
__global__ __launch_bounds__(64) void k_l2p(
    int64_t nleaf, const int32_t* __restrict__ leaf_box,
    const int32_t* __restrict__ leaf_start, const int32_t* __restrict__ perm,
    const double* __restrict__ xs, const double* __restrict__ ys,
    const double* __restrict__ zs, const double* __restrict__ cx,
    const double* __restrict__ cy, const double* __restrict__ cz,
    const double* __restrict__ scale, const T* __restrict__ D, const T* __restrict__ tab,
    int64_t n, const T* __restrict__ near, T* __restrict__ pot, T* __restrict__ field) {
  constexpr int K = K_<P>::value;
  constexpr int K1 = P * P;  // coefficients of the gradient expansions
  constexpr int LW = 64 / G;
  __shared__ T w[G][K];
  __shared__ T gw[G][3][K1];
  const int lane = threadIdx.x;
  const int h = lane / LW, l = lane % LW;
  for (int idx = lane; idx < G * K; idx += 64) {
    const int hh = idx / K, k = idx - hh * K;
    const int64_t lf = (int64_t)blockIdx.x * G + hh;
    if (lf < nleaf) w[hh][k] = D[(int64_t)leaf_box[lf] * K + k] * tab[tab_l2p(P) + k];
  }
  if (FIELD) {
    __syncthreads();
    for (int idx = lane; idx < G * K1; idx += 64) {
      const int hh = idx / K1, k = idx - hh * K1;
      grad_coeff<P, T>(w[hh], k, gw[hh][0][k], gw[hh][1][k], gw[hh][2][k]);
    }
  }
  __syncthreads();
  const int64_t leaf = (int64_t)blockIdx.x * G + h;
  if (leaf >= nleaf) return;
  const int64_t g = leaf_box[leaf];
  const int st = leaf_start[leaf], en = leaf_start[leaf + 1];
  const double ox = cx[g], oy = cy[g], oz = cz[g], ir = 1.0 / scale[g];
  const T fu = T(-kInv4Pi * ir), ff = T(kInv4Pi * ir * ir);
  for (int i = st + l; i < en; i += LW) {
    T fp = T(0), fx = T(0), fy = T(0), fz = T(0);
    local_eval_grad<P, T>(T((xs[i] - ox) * ir), T((ys[i] - oy) * ir), T((zs[i] - oz) * ir),
                          w[h], gw[h][0], gw[h][1], gw[h][2], fp, fx, fy, fz);
    const int o = perm[i];
    pot[o] = near[i] + fu * fp;
    if (FIELD) {
      const T* f = near + n + 3 * (int64_t)i;
      field[3 * (int64_t)o + 0] = f[0] + ff * fx;
      field[3 * (int64_t)o + 1] = f[1] + ff * fy;
      field[3 * (int64_t)o + 2] = f[2] + ff * fz;
    }
  }
}

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

// One evaluation: P2P writes the near field in leaf order, L2P adds the far
// field and writes the outputs.
template <int P, typename T>
void run_pass(fmm_plan* pl, const Workspace& ws, int dir, const T* q, T* pot, T* field,
              hipStream_t st) {
  const int s = pl->s;
  const T* tab = (const T*)pl->tables;
  Src<T>* src = (Src<T>*)ws.src;
  T* C = (T*)ws.C;
  T* D = (T*)ws.D;
  T* near = (T*)ws.near;
  const int64_t n = pl->n;
  const ListSet& Ls = pl->lists[dir];
  const Side& SS = src_side(pl, dir);  // charges: P2M, M2M
  const Side& TS = tgt_side(pl, dir);  // evaluation points: L2L, P2P, L2P
  StageMarks mk(pl, ws.stages);
  // the sort stage (charges into leaf-ordered source records) is folded
  // into P2M; its timing slot stays empty
  mk.begin(kStSort, st);
  mk.end(kStSort, st);
  // far field
  // leaves per wave for P2M and L2P: every lane holds at most one point
  const int GL = leaves_per_wave(pl);
  const int64_t nls = SS.nleaf, nlt = TS.nleaf;
  mk.begin(kStP2M, st);
  auto p2m = [&](auto kern) {
    kern<<<(unsigned)((nls + GL - 1) / GL), 64, 0, st>>>(
        nls, pl->leaf_box + SS.leaf0, pl->leaf_start + SS.leaf0, pl->xs, pl->ys, pl->zs,
        pl->perm, q, src, pl->cx, pl->cy, pl->cz, pl->scale, tab, C);
  };
  if (GL == 1) p2m(k_p2m<P, T, 1>);
  else if (GL == 2) p2m(k_p2m<P, T, 2>);
  else if (GL == 4) p2m(k_p2m<P, T, 4>);
  else p2m(k_p2m<P, T, 8>);
  mk.end(kStP2M, st);
  // The near field needs only the leaf-ordered source records of P2M: it
  // runs on the plan's second stream beside the far-field chain (M2M, M2L,
  // L2L), so each fills the other's idle issue slots; L2P joins the two.
  // Stage profiling keeps the stages one after another on st.
  const bool fork = pl->side_stream != nullptr && !pl->profiling && pl->near_stream != 1;
  const hipStream_t sp = fork ? pl->side_stream : st;
  if (fork) FMM_HIP(hipEventRecord(pl->ev_fork, st));
  auto near_part = [&] {
    if (fork) FMM_HIP(hipStreamWaitEvent(sp, pl->ev_fork, 0));
    near_field(pl, Ls, src, n, near, field != nullptr, sp, mk);
    if (fork) FMM_HIP(hipEventRecord(pl->ev_join, sp));
  };
  // enqueued after the far-field chain when forked, so that the chain's
  // small level launches are not queued behind the near field's blocks
  if (!fork) near_part();
  mk.begin(kStM2M, st);
  const bool chain_shared = P >= kChainShareMinOrder && chain_waves(pl) > 1;
  for (const Step& S : SS.m2m_steps) {
    const int64_t nchild = S.n << s;
    if constexpr (P >= kChainShareMinOrder) {
      if (chain_shared) {
        k_m2m_shared<P, T><<<blocks(nchild, 64), 64 * kShareWaves, 0, st>>>(
            nchild, S.a, S.b, s, pl->cx, pl->cy, pl->cz, pl->scale, tab, C);
        continue;
      }
    }
    k_m2m<P, T><<<blocks(nchild, 64), 64, 0, st>>>(nchild, S.a, S.b, s, pl->cx, pl->cy, pl->cz,
                                                   pl->scale, tab, C);
  }
  mk.end(kStM2M, st);
  mk.begin(kStM2L, st);
  if (Ls.n_blocks > 0) {
    [[maybe_unused]] auto shared_form = [&](auto kern, int nw) {
      kern<<<(unsigned)Ls.n_blocks, kM2LBlock * nw, 0, st>>>(
          Ls.item_tgt, Ls.item_begin, Ls.item_end, Ls.seg_ptr, Ls.seg_tgt, Ls.seg_lanes,
          Ls.m2l_src, pl->cx, pl->cy, pl->cz, pl->scale, C, tab, D);
    };
    auto one_lane = [&] {
      constexpr int W = m2l_block_waves(sizeof(T) == 8);
      k_m2l<P, T, W><<<(unsigned)Ls.n_blocks, kM2LBlock * W, 0, st>>>(
          Ls.item_tgt, Ls.item_begin, Ls.item_end, Ls.seg_ptr, Ls.seg_tgt, Ls.seg_lanes,
          Ls.m2l_src, pl->geo, C, tab, D);
    };
    if constexpr (m2l_shared_built(P, sizeof(T) == 8)) {
      constexpr int NW = m2l_share_waves(P, sizeof(T) == 8);
      if (m2l_waves(pl) > 1)
        shared_form(k_m2l_shared<P, T, NW>, NW);
      else
        one_lane();
    } else {
      one_lane();
    }
  }
  mk.end(kStM2L, st);
  mk.begin(kStL2L, st);
  // final locals, written over the multipoles: the leaves' parents from all
  // their ancestors, then the leaves from their parents
  T* Dfin = C;
  for (int k = 0; k < 2; ++k) {
    const FinList& F = Ls.fin[k];
    if (F.n == 0) continue;
    const T* from = k == 0 ? D : Dfin;
    if constexpr (P >= kChainShareMinOrder) {
      if (chain_shared) {
        k_l2l_fin_shared<P, T><<<blocks(F.n * F.gs, 64), 64 * kShareWaves, 0, st>>>(
            F.n, F.gs, F.box, F.own, F.anc, pl->cx, pl->cy, pl->cz, pl->scale, tab, from, D,
            Dfin);
        continue;
      }
    }
    auto l2l = [&](auto kern) {
      kern<<<blocks(F.n * F.gs, 64), 64, 0, st>>>(F.n, F.box, F.own, F.anc, pl->cx, pl->cy,
                                                 pl->cz, pl->scale, tab, from, D, Dfin);
    };
    switch (F.gs) {
      case 1: l2l(k_l2l_fin<P, T, 1>); break;
      case 2: l2l(k_l2l_fin<P, T, 2>); break;
      case 4: l2l(k_l2l_fin<P, T, 4>); break;
      case 8: l2l(k_l2l_fin<P, T, 8>); break;
      default: l2l(k_l2l_fin<P, T, 16>); break;
    }
  }
  mk.end(kStL2L, st);
  if (fork) {
    near_part();
    FMM_HIP(hipStreamWaitEvent(st, pl->ev_join, 0));
  }
  mk.begin(kStL2P, st);
  auto l2p = [&](auto kern) {
    kern<<<(unsigned)((nlt + GL - 1) / GL), 64, 0, st>>>(
        nlt, pl->leaf_box + TS.leaf0, pl->leaf_start + TS.leaf0, pl->perm, pl->xs, pl->ys,
        pl->zs, pl->cx, pl->cy, pl->cz, pl->scale, Dfin, tab, n, near, pot, field);
  };
  if (field) {
    if (GL == 1) l2p(k_l2p<P, T, true, 1>);
    else if (GL == 2) l2p(k_l2p<P, T, true, 2>);
    else if (GL == 4) l2p(k_l2p<P, T, true, 4>);
    else l2p(k_l2p<P, T, true, 8>);
  } else {
    if (GL == 1) l2p(k_l2p<P, T, false, 1>);
    else if (GL == 2) l2p(k_l2p<P, T, false, 2>);
    else if (GL == 4) l2p(k_l2p<P, T, false, 4>);
    else l2p(k_l2p<P, T, false, 8>);
  }
  mk.end(kStL2P, st);
  FMM_HIP(hipGetLastError());
}

template void run_pass<FMM_ORDER, double>(fmm_plan*, const Workspace&, int, const double*, double*,
                                          double*, hipStream_t);
template void run_pass<FMM_ORDER, float>(fmm_plan*, const Workspace&, int, const float*, float*,
                                         float*, hipStream_t);

}  // namespace fmm
