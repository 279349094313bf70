// Near field (P2P, Sec. III.A "evdir") of the evaluation pass: direct sums
// over the plan's balanced work items, hand-written HIP kernels for gfx950.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "ops.h"

namespace fmm {
namespace {

using namespace ops;

// One source point against the lane's target at (xi, yi, zi): the
// difference is taken in FP64 and rounded to T.  In FP64 the Newton step
// gives 2 / r, one operation less than 1 / r (near_scale takes the powers of
// two out again: 16 instead of 17 operations and the root).  SAFE: pairs at distance 0
// contribute nothing (needed within a leaf, and between leaves when the
// point set has points at a distance that is 0 in T); otherwise the pair is
// known to be apart.
template <typename T, bool FIELD, bool SAFE>
__device__ __forceinline__ void p2p_pair(const Src<T>& s, double xi, double yi, double zi,
                                         T& u, T& gx, T& gy, T& gz) {
  const T dx = T(xi - s.x), dy = T(yi - s.y), dz = T(zi - s.z);
  const T r2 = dx * dx + dy * dy + dz * dz;
  const T inv0 = inv_sqrt2(r2);
  const T inv = SAFE ? (r2 > T(0) ? inv0 : T(0)) : inv0;
  const T qi = s.q * inv;
  u += qi;
  if (FIELD) {
    const T q3 = qi * inv * inv;
    gx = fma(q3, dx, gx);
    gy = fma(q3, dy, gy);
    gz = fma(q3, dz, gz);
  }
}

// Factor of the near field's sums: -1/(4 pi), and 1/2 or 1/8 for the factor
// of inv_sqrt2 in the potential and the field.
template <typename T>
__device__ __forceinline__ constexpr T near_scale(bool field) {
  return sizeof(T) == 4 ? -T(kInv4Pi) : -T(kInv4Pi) * T(field ? 0.125 : 0.5);
}

constexpr int kChunk = 8;

// P2P: writes -1/(4 pi) sum q/r and the matching field over the direct list,
// in leaf order (near[i] and near[n + 3 i + c]); L2P adds the far field and
// writes the outputs in input order.
// Block = one near-field work item (a run of a target leaf's direct list;
// most leaves have one), lane = target point (position from the plan's
// leaf-ordered coordinates; the sources' records are this pass's, written
// by P2M).  A leaf's only item writes its near field; the items of a split
// leaf write partial rows that k_p2p_sum adds in item order.  G source groups: lanes
// [g*64/G, (g+1)*64/G) share targets with the other groups but walk every
// G-th source point starting at point g.  G = 1 keeps all source reads
// wave-uniform (scalar loads).  G = 2, 4 fill the wave when leaves hold at
// most 32 or 16 points; each source leaf is then first copied into LDS with
// one coalesced 16-byte load per lane, and the groups read their records
// from there (a per-lane global read of every record would saturate the
// texture address unit).  Per source leaf the partial sums are added to the
// running sums with Neumaier compensation (FP32 form); group sums are then
// combined with cross-lane shuffles in a fixed order.
template <typename T, bool FIELD, int G>
__global__ __launch_bounds__(64) void k_p2p(
    int64_t n, const int32_t* __restrict__ item_leaf,
    const int32_t* __restrict__ item_kb, const int32_t* __restrict__ item_ke,
    const int64_t* __restrict__ item_out, const int32_t* __restrict__ leaf_start,
    const double* __restrict__ xs, const double* __restrict__ ys, const double* __restrict__ zs,
    const Src<T>* __restrict__ src, const int32_t* __restrict__ p2p_src, int dup,
    T* __restrict__ near, T* __restrict__ part) {
  constexpr int TL = 64 / G;  // targets per pass
  constexpr bool kComp = sizeof(T) == 4;  // FP32: compensated sums
  // G > 1: one source leaf (at most TL points) staged as 16-byte words
  __shared__ __align__(32) double2 stage[G > 1 ? 2 * TL : 1];
  // items in target-leaf order, handed to the XCDs in runs of 64:
  // neighbouring target leaves share most source leaves, so their records
  // stay in one XCD's L2, while leaves of unequal cost (several problems,
  // clustered points) spread over all XCDs
  const int item = (int)xcd_chunked<64>(blockIdx.x, gridDim.x);
  const int leaf = item_leaf[item];
  const int lane = threadIdx.x;
  const int g = G == 1 ? 0 : lane / TL;
  const int st = leaf_start[leaf], en = leaf_start[leaf + 1];
  const int pb = item_kb[item], pe = item_ke[item];
  const int64_t po = item_out[item];
  for (int i0 = st; i0 < en; i0 += TL) {
    const int i = i0 + lane % TL;
    const bool live = i < en;
    const int ia = live ? i : st;
    const Src<T> a{xs[ia], ys[ia], zs[ia], T(0)};
    T u = T(0), gx = T(0), gy = T(0), gz = T(0);
    T cu = T(0), cgx = T(0), cgy = T(0), cgz = T(0);
    for (int k = pb; k < pe; ++k) {
      const int sl = p2p_src[k];
      const int js = leaf_start[sl], cnt = leaf_start[sl + 1] - js;
      T lu = T(0), lx = T(0), ly = T(0), lz = T(0);
      const int full = cnt / G;  // points per group present in every group
      // distance-0 guard only where it can matter: the target leaf itself,
      // or every leaf when some points of the set cannot be told apart
      const bool safe = dup || sl == leaf;
      const Src<T>* rec;
      int stride;
      if (G == 1) {
        rec = src + js;
        stride = 1;
      } else {
        // cnt <= TL: the leaf's records are 2 cnt <= 64 words
        const double2* words = reinterpret_cast<const double2*>(src + js);
        __syncthreads();  // previous leaf's reads are done
        if (lane < 2 * cnt) stage[lane] = words[lane];
        __syncthreads();
        rec = reinterpret_cast<const Src<T>*>(stage) + g;
        stride = G;
      }
      auto sweep = [&](auto safe_tag) {
        constexpr bool S = decltype(safe_tag)::value;
        int c = 0;
        for (; c + kChunk <= full; c += kChunk) {
          Src<T> r[kChunk];
#pragma unroll
          for (int t = 0; t < kChunk; ++t) r[t] = rec[(c + t) * stride];
#pragma unroll
          for (int t = 0; t < kChunk; ++t)
            p2p_pair<T, FIELD, S>(r[t], a.x, a.y, a.z, lu, lx, ly, lz);
        }
        for (; c < full; ++c) p2p_pair<T, FIELD, S>(rec[c * stride], a.x, a.y, a.z, lu, lx, ly, lz);
        if (G > 1 && g < cnt - full * G)
          p2p_pair<T, FIELD, S>(rec[full * G], a.x, a.y, a.z, lu, lx, ly, lz);
      };
      if (safe)
        sweep(std::true_type{});
      else
        sweep(std::false_type{});
      if (kComp) {
        neumaier(u, cu, lu);
        if (FIELD) {
          neumaier(gx, cgx, lx);
          neumaier(gy, cgy, ly);
          neumaier(gz, cgz, lz);
        }
      } else {
        u += lu;
        gx += lx;
        gy += ly;
        gz += lz;
      }
    }
    u += cu;
    gx += cgx;
    gy += cgy;
    gz += cgz;
#pragma unroll
    for (int off = TL; off < 64; off <<= 1) {
      u += __shfl_xor(u, off, 64);
      if (FIELD) {
        gx += __shfl_xor(gx, off, 64);
        gy += __shfl_xor(gy, off, 64);
        gz += __shfl_xor(gz, off, 64);
      }
    }
    if (live && g == 0) {
      // field = -grad u;  grad of the near part is +(1/4pi) sum q d/r^3
      if (po < 0) {  // the leaf's only item: its near field
        near[i] = near_scale<T>(false) * u;
        if (FIELD) {
          T* f = near + n + 3 * (int64_t)i;
          f[0] = near_scale<T>(true) * gx;
          f[1] = near_scale<T>(true) * gy;
          f[2] = near_scale<T>(true) * gz;
        }
      } else {  // one of several items of the leaf: rows of its partial sums
        const int nt = en - st, li = i - st;
        T* r = part + po;
        r[li] = near_scale<T>(false) * u;
        if (FIELD) {
          r[nt + li] = near_scale<T>(true) * gx;
          r[2 * nt + li] = near_scale<T>(true) * gy;
          r[3 * nt + li] = near_scale<T>(true) * gz;
        }
      }
    }
  }
}

// The same items with every lane at work (FP32): a thread holds two targets
// (i and i + h of the leaf's nt, h = nt / 2 rounded up) and the W / h groups
// of h threads each take another source leaf of the item's list.  A group's
// threads sum their leaf's points in order, as k_p2p does; the leaf sums then
// pass through LDS to the thread that keeps the running sum of a (component,
// target) pair, which adds them in list order (Neumaier): the results are
// those of k_p2p with one source group, bit for bit.  Lanes stay idle only
// for the remainders of W / h and of the list over the groups, against 64 -
// nt mod 64 lanes of every wave in k_p2p; a record read from LDS (32 bytes a
// lane, the same for a group) serves two pairs, since one pair per read keeps
// the LDS as busy as the VALU.  Bound by VALU issue.  Measured (near field,
// FP32): 200003 Plummer points, 49 a leaf, 3.42 -> 3.00 ms; 16 problems of 22
// to 109 points a leaf 1.61 -> 1.36 ms; 30011 points on a sphere, 779 items,
// 75 -> 33 us with 256 threads an item.
template <bool FIELD, int W>
__global__ __launch_bounds__(W) __attribute__((amdgpu_waves_per_eu(4))) void k_p2p_wide(
    int64_t n, const int32_t* __restrict__ item_leaf,
    const int32_t* __restrict__ item_kb, const int32_t* __restrict__ item_ke,
    const int64_t* __restrict__ item_out, const int32_t* __restrict__ leaf_start,
    const double* __restrict__ xs, const double* __restrict__ ys, const double* __restrict__ zs,
    const Src<float>* __restrict__ src, const int32_t* __restrict__ p2p_src, int dup,
    float* __restrict__ near, float* __restrict__ part) {
  typedef float T;
  constexpr int NC = FIELD ? 4 : 1;
  constexpr int kWideTargets = W;     // targets at a time (two groups or more)
  constexpr int kWideStage = 2 * W;   // staged source records (all groups)
  constexpr int NQ = NC;              // running sums per thread
  constexpr int U = 4;                // records in registers
  __shared__ __align__(32) double2 stage[2 * kWideStage];
  __shared__ T sums[2 * NC][W];
  __shared__ int ljs[W], lcnt[W];  // source leaves: first point, count
  __shared__ int lmax[W / 64], lself[W / 64];
  const int item = (int)xcd_chunked<64>(blockIdx.x, gridDim.x);
  const int tid = threadIdx.x;
  const int leaf = item_leaf[item];
  const int st = leaf_start[leaf], nt = leaf_start[leaf + 1] - st;
  const int pb = item_kb[item], pe = item_ke[item];
  const int64_t po = item_out[item];
  const double2* words = reinterpret_cast<const double2*>(src);
  for (int t0 = 0; t0 < nt; t0 += kWideTargets) {
    const int ntt = min(kWideTargets, nt - t0);
    const int h = (ntt + 1) / 2, ng = W / h;  // threads per group, groups
    const int CS = kWideStage / ng;               // staged points per group
    const int g = tid / h, i = tid - g * h;
    const int ia = st + t0 + min(i, ntt - 1), ib = st + t0 + min(i + h, ntt - 1);
    const double xa = xs[ia], ya = ys[ia], za = zs[ia];
    const double xb = xs[ib], yb = ys[ib], zb = zs[ib];
    // record that this thread stages (the second one W / CS groups on)
    const int g0 = tid / CS, r0 = tid - g0 * CS;
    const int g1 = (tid + W) / CS, r1 = tid + W - g1 * CS;
    // running sums q = tid + W m of (component q / ntt, target q % ntt)
    T s[NQ], c[NQ];
    int at[NQ];
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      const int q = tid + W * m, comp = q / ntt, t = q - comp * ntt;
      s[m] = c[m] = T(0);
      at[m] = q < NC * ntt ? (t < h ? comp * W + t : (NC + comp) * W + t - h) : -1;
    }
    for (int kb = pb; kb < pe; kb += W) {
      const int nk = min(W, pe - kb);
      __syncthreads();  // the previous leaves' entries and sums are done with
      {
        const int sl = p2p_src[kb + min(tid, nk - 1)];
        const int js = leaf_start[sl], cnt = leaf_start[sl + 1] - js;
        ljs[tid] = js;
        lcnt[tid] = cnt;
        // largest leaf and the target leaf's own place (-1: not here)
        int mx = cnt, self = sl == leaf ? min(tid, nk - 1) : -1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          mx = max(mx, __shfl_xor(mx, off, 64));
          self = max(self, __shfl_xor(self, off, 64));
        }
        lmax[tid / 64] = mx;
        lself[tid / 64] = self;
      }
      __syncthreads();
      int most = lmax[0], self = lself[0];
#pragma unroll
      for (int v = 1; v < W / 64; ++v) {
        most = max(most, lmax[v]);
        self = max(self, lself[v]);
      }
      most = __builtin_amdgcn_readfirstlane(most);
      self = __builtin_amdgcn_readfirstlane(self);
      for (int k0 = 0; k0 < nk; k0 += ng) {
        const int kn = min(ng, nk - k0);
        const bool mine = g < kn;
        T ua = T(0), xa_ = T(0), ya_ = T(0), za_ = T(0), ub = T(0), xb_ = T(0), yb_ = T(0),
          zb_ = T(0);
        const bool safe = dup || (self >= k0 && self < k0 + kn);
        for (int c0 = 0; c0 < most; c0 += CS) {
          __syncthreads();  // the staged records and the leaf sums are done with
          if (g0 < kn && c0 + r0 < lcnt[k0 + g0]) {
            const int64_t j = 2 * ((int64_t)ljs[k0 + g0] + c0 + r0);
            const double2 w0 = words[j], w1 = words[j + 1];
            stage[2 * tid] = w0;
            stage[2 * tid + 1] = w1;
          }
          if (g1 < kn && c0 + r1 < lcnt[k0 + g1]) {
            const int64_t j = 2 * ((int64_t)ljs[k0 + g1] + c0 + r1);
            const double2 w0 = words[j], w1 = words[j + 1];
            stage[2 * (tid + W)] = w0;
            stage[2 * (tid + W) + 1] = w1;
          }
          __syncthreads();
          const int cnt = mine ? min(CS, lcnt[k0 + g] - c0) : 0;
          const Src<T>* rec = reinterpret_cast<const Src<T>*>(stage) + (mine ? g * CS : 0);
          auto sweep = [&](auto safe_tag) {
            constexpr bool S = decltype(safe_tag)::value;
            int e = 0;
            for (; e + U <= cnt; e += U) {
              Src<T> r[U];
#pragma unroll
              for (int t = 0; t < U; ++t) r[t] = rec[e + t];
#pragma unroll
              for (int t = 0; t < U; ++t) {
                p2p_pair<T, FIELD, S>(r[t], xa, ya, za, ua, xa_, ya_, za_);
                p2p_pair<T, FIELD, S>(r[t], xb, yb, zb, ub, xb_, yb_, zb_);
              }
            }
            for (; e < cnt; ++e) {
              const Src<T> r = rec[e];
              p2p_pair<T, FIELD, S>(r, xa, ya, za, ua, xa_, ya_, za_);
              p2p_pair<T, FIELD, S>(r, xb, yb, zb, ub, xb_, yb_, zb_);
            }
          };
          if (safe)
            sweep(std::true_type{});
          else
            sweep(std::false_type{});
        }
        {  // leaf sums (the last round's merge ended before a barrier)
          sums[0][tid] = ua;
          sums[NC][tid] = ub;
          if constexpr (FIELD) {
            sums[1][tid] = xa_;
            sums[2][tid] = ya_;
            sums[3][tid] = za_;
            sums[NC + 1][tid] = xb_;
            sums[NC + 2][tid] = yb_;
            sums[NC + 3][tid] = zb_;
          }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < NQ; ++m) {
          if (at[m] < 0) continue;
          const T* x = &sums[0][0] + at[m];
          for (int gg = 0; gg < kn; ++gg) neumaier(s[m], c[m], x[gg * h]);
        }
      }
    }
    const T su = near_scale<T>(false), sg = near_scale<T>(true);
#pragma unroll
    for (int m = 0; m < NQ; ++m) {
      if (at[m] < 0) continue;
      const int q = tid + W * m, comp = q / ntt, li = t0 + q - comp * ntt;
      const T v = (comp == 0 ? su : sg) * (s[m] + c[m]);
      if (po >= 0)
        part[po + (int64_t)comp * nt + li] = v;
      else if (comp == 0)
        near[st + li] = v;
      else
        near[n + 3 * (int64_t)(st + li) + comp - 1] = v;
    }
  }
}

// FP64, where the order of the sums is free: the same threads and targets,
// but the groups share out the points of the item's source leaves (staged
// one after another, group g takes every ng-th record) and every thread sums
// all its points before the groups' sums are added once, so that neither
// leaves nor lists leave groups idle.  Bound by VALU issue (16 FP64
// operations and the reciprocal square root a pair).  Measured (near field
// against k_p2p with two or four groups): 384 charges and 2048 probes 33 ->
// 13 us, uniform cube 2^20 (32 points a leaf) 0.59 -> 0.58 ms.
template <bool FIELD, int W>
__global__ __launch_bounds__(W) __attribute__((amdgpu_waves_per_eu(4))) void k_p2p_flat(
    int64_t n, const int32_t* __restrict__ item_leaf,
    const int32_t* __restrict__ item_kb, const int32_t* __restrict__ item_ke,
    const int64_t* __restrict__ item_out, const int32_t* __restrict__ leaf_start,
    const double* __restrict__ xs, const double* __restrict__ ys, const double* __restrict__ zs,
    const Src<double>* __restrict__ src, const int32_t* __restrict__ p2p_src, int dup,
    double* __restrict__ near, double* __restrict__ part) {
  constexpr int NC = FIELD ? 4 : 1;
  constexpr int U = 4;              // records in registers
  constexpr int kFlatStage = 2 * W;  // staged source records
  // the staged records, and in the end the threads' sums [2 NC][W]
  __shared__ __align__(32) double2 stage[2 * kFlatStage];
  static_assert(2 * NC * W * sizeof(double) <= sizeof(stage), "sums fit the stage");
  __shared__ int ljs[W], lcnt[W];  // source leaves: first point, count
  __shared__ int lpos[W + 1];          // points of the leaves before
  __shared__ int lmax[2], lself[2];
  const int item = (int)xcd_chunked<64>(blockIdx.x, gridDim.x);
  const int tid = threadIdx.x;
  const int leaf = item_leaf[item];
  const int st = leaf_start[leaf], nt = leaf_start[leaf + 1] - st;
  const int pb = item_kb[item], pe = item_ke[item];
  const int64_t po = item_out[item];
  const double2* words = reinterpret_cast<const double2*>(src);
  for (int t0 = 0; t0 < nt; t0 += 2 * W) {
    const int ntt = min(2 * W, nt - t0);
    const int h = (ntt + 1) / 2, ng = W / h;  // threads per group, groups
    const int g = tid / h, i = tid - g * h;
    const bool mine = g < ng;
    const int ia = st + t0 + min(i, ntt - 1), ib = st + t0 + min(i + h, ntt - 1);
    const double xa = xs[ia], ya = ys[ia], za = zs[ia];
    const double xb = xs[ib], yb = ys[ib], zb = zs[ib];
    double a[4] = {0.0, 0.0, 0.0, 0.0}, b[4] = {0.0, 0.0, 0.0, 0.0};
    for (int kb = pb; kb < pe; kb += W) {
      const int nk = min(W, pe - kb);
      __syncthreads();  // the previous leaves' entries are done with
      {
        const int sl = p2p_src[kb + min(tid, nk - 1)];
        const int js = leaf_start[sl], cnt = tid < nk ? leaf_start[sl + 1] - js : 0;
        ljs[tid] = js;
        lcnt[tid] = cnt;
        // largest leaf, the target leaf's own place (-1: not here), and the
        // points before each leaf
        int mx = cnt, self = tid < nk && sl == leaf ? tid : -1, sum = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          mx = max(mx, __shfl_xor(mx, off, 64));
          self = max(self, __shfl_xor(self, off, 64));
          const int left = __shfl_up(sum, off, 64);
          if (tid % 64 >= off) sum += left;
        }
        lmax[tid / 64] = mx;
        lself[tid / 64] = self;
        if (tid == 63) lpos[64] = sum;
        if (tid < 64) lpos[tid] = sum - cnt;
        if (W > 64) {
          __syncthreads();
          if (tid >= 64) lpos[tid + 1] = lpos[64] + sum;
        }
      }
      __syncthreads();
      const int most = __builtin_amdgcn_readfirstlane(max(lmax[0], lmax[W / 64 - 1]));
      const int self = __builtin_amdgcn_readfirstlane(max(lself[0], lself[W / 64 - 1]));
      const int nl = max(kFlatStage / most, 1);  // leaves staged at a time
      const int inv = (1 << 16) / most + 1;      // e / most = e inv >> 16 for e < kFlatStage
      for (int k0 = 0; k0 < nk; k0 += nl) {
        const int kn = min(nl, nk - k0);
        const bool safe = dup || (self >= k0 && self < k0 + kn);
        // leaves of more than kFlatStage points come in pieces
        for (int c0 = 0; c0 < most; c0 += kFlatStage) {
          const int p0 = lpos[k0];
          const int tot = nl > 1 ? lpos[k0 + kn] - p0 : min(kFlatStage, lcnt[k0] - c0);
          __syncthreads();  // the staged records are done with
#pragma unroll
          for (int u = 0; u < kFlatStage / W; ++u) {
            const int e = tid + u * W;
            const int l = nl > 1 ? e * inv >> 16 : 0, r = nl > 1 ? e - l * most : c0 + e;
            if (l < kn && r < lcnt[k0 + l]) {
              const int64_t j = 2 * ((int64_t)ljs[k0 + l] + r);
              const double2 w0 = words[j], w1 = words[j + 1];
              const int to = nl > 1 ? lpos[k0 + l] - p0 + r : e;
              stage[2 * to] = w0;
              stage[2 * to + 1] = w1;
            }
          }
          __syncthreads();
          const Src<double>* rec = reinterpret_cast<const Src<double>*>(stage) + (mine ? g : 0);
          const int full = tot / ng;  // records of every group
          auto sweep = [&](auto safe_tag) {
            constexpr bool S = decltype(safe_tag)::value;
            auto both = [&](const Src<double>& r) {
              p2p_pair<double, FIELD, S>(r, xa, ya, za, a[0], a[1], a[2], a[3]);
              p2p_pair<double, FIELD, S>(r, xb, yb, zb, b[0], b[1], b[2], b[3]);
            };
            int e = 0;
            for (; e + U <= full; e += U) {
              Src<double> r[U];
#pragma unroll
              for (int t = 0; t < U; ++t) r[t] = rec[(e + t) * ng];
#pragma unroll
              for (int t = 0; t < U; ++t) both(r[t]);
            }
            for (; e < full; ++e) both(rec[e * ng]);
            if (mine && g < tot - full * ng) both(rec[full * ng]);
          };
          if (safe)
            sweep(std::true_type{});
          else
            sweep(std::false_type{});
        }
      }
    }
    // the groups' sums added in group order
    double* sums = reinterpret_cast<double*>(stage);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      sums[c * W + tid] = a[c];
      sums[(NC + c) * W + tid] = b[c];
    }
    __syncthreads();
    for (int q = tid; q < NC * ntt; q += W) {
      const int comp = q / ntt, t = q - comp * ntt;
      const double* x = sums + (t < h ? comp * W + t : (NC + comp) * W + t - h);
      double v = 0.0;
      for (int gg = 0; gg < ng; ++gg) v += x[gg * h];
      v *= near_scale<double>(comp > 0);
      const int li = t0 + t;
      if (po >= 0)
        part[po + (int64_t)comp * nt + li] = v;
      else if (comp == 0)
        near[st + li] = v;
      else
        near[n + 3 * (int64_t)(st + li) + comp - 1] = v;
    }
  }
}

// Near field of the leaves whose direct list was split into several items:
// the items' partial rows added in item order (Neumaier-compensated in
// FP32).  Block = 64 columns (component, target) of one split leaf, one
// thread each, so that every wave reads contiguous runs of the rows, which
// lie one after another; kSumDepth rows are loaded before they are added.
// Bound by the latency of the rows (read once, from L2).  Measured on 500009
// clustered points (FP32, 37 items per leaf on average, hundreds for the
// halo's leaves): near field and sums 6.9 -> 3.7 ms against one wave per leaf
// and a load for every addition (2.9 ms of it).
constexpr int kSumDepth = 16;

template <typename T, bool FIELD>
__global__ __launch_bounds__(64) void k_p2p_sum(
    int64_t n, const int32_t* __restrict__ split_leaf, const int32_t* __restrict__ split_first,
    const int32_t* __restrict__ split_cnt, const int64_t* __restrict__ item_out,
    const int32_t* __restrict__ leaf_start, const T* __restrict__ part, T* __restrict__ near) {
  constexpr bool kComp = sizeof(T) == 4;
  const int leaf = split_leaf[blockIdx.x];
  const int f = split_first[blockIdx.x], c = split_cnt[blockIdx.x];
  const int st = leaf_start[leaf], nt = leaf_start[leaf + 1] - st;
  const int cols = (FIELD ? 4 : 1) * nt;
  const int64_t row = 4 * (int64_t)nt;
  for (int col = blockIdx.y * 64 + threadIdx.x; col < cols; col += gridDim.y * 64) {
    const T* x = part + item_out[f] + col;  // item f + j: x[j * row]
    T acc = T(0), cc = T(0);
    auto add = [&](T v) {
      if (kComp)
        neumaier(acc, cc, v);
      else
        acc += v;
    };
    int j = 0;
    for (; j + kSumDepth <= c; j += kSumDepth) {
      T v[kSumDepth];
#pragma unroll
      for (int u = 0; u < kSumDepth; ++u) v[u] = x[(j + u) * row];
#pragma unroll
      for (int u = 0; u < kSumDepth; ++u) add(v[u]);
    }
    for (; j < c; ++j) add(x[j * row]);
    acc += cc;
    const int comp = col / nt;
    const int64_t i = st + col - comp * nt;
    if (comp == 0)
      near[i] = acc;
    else
      near[n + 3 * i + comp - 1] = acc;
  }
}

// Items [first, first + count) of a pass on one form (near_form).
struct NearRun {
  int form;
  int64_t first, count;
};

// The launches of a pass over Ls, each on the form its items were given
// (at most four, some possibly empty); returns their number.
int near_runs(const fmm_plan* pl, const ListSet& Ls, bool field, NearRun (&run)[4]) {
  const NearItems& N = Ls.near;
  int k = 0;
  int64_t at = 0;
  auto add = [&](int form, int64_t count) {
    run[k++] = NearRun{form, at, count};
    at += count;
  };
  // the wide forms take the leaves they were given unless another number of
  // source groups than the plan's own is asked for
  if (p2p_groups(pl) != default_p2p_groups(pl)) {
    add(kNearWave, N.n);
    return k;
  }
  add(kNearWide256, N.n_wide256);
  add(kNearWide, N.n_wide);
  add(kNearWide64, N.n_wide64);
  add(field ? kNearWave : N.rest_pot, N.n - at);
  return k;
}

template <typename T>
void run_near(fmm_plan* pl, const ListSet& Ls, const Src<T>* src, int64_t n, T* near, bool field,
              hipStream_t sp) {
  const NearItems& N = Ls.near;
  const int G = p2p_groups(pl);
  NearRun run[4];
  const int runs = near_runs(pl, Ls, field, run);
  auto all = [&](const NearRun& r, auto field_tag) {
    constexpr bool F = decltype(field_tag)::value;
    // (the run's items by pointer: with their offset as an argument k_p2p of two
    // source groups took 158.7 instead of 154.3 us on 256 items of 17 points)
    auto launch = [&](auto kern, int threads) {
      kern<<<(unsigned)r.count, threads, 0, sp>>>(
          n, N.leaf + r.first, N.kb + r.first, N.ke + r.first, N.out + r.first, pl->leaf_start,
          pl->xs, pl->ys, pl->zs, src, Ls.p2p_src, pl->has_dup ? 1 : 0, near, (T*)N.part);
    };
    if (r.form == kNearWave) {
      if (G == 1) launch(k_p2p<T, F, 1>, 64);
      else if (G == 2) launch(k_p2p<T, F, 2>, 64);
      else launch(k_p2p<T, F, 4>, 64);
    } else if constexpr (sizeof(T) == 8) {
      if (r.form == kNearWide) launch(k_p2p_flat<F, 128>, 128);
      else launch(k_p2p_flat<F, 64>, 64);
    } else {
      if (r.form == kNearWide256) launch(k_p2p_wide<F, 256>, 256);
      else if (r.form == kNearWide) launch(k_p2p_wide<F, 128>, 128);
      else launch(k_p2p_wide<F, 64>, 64);
    }
  };
  for (int k = 0; k < runs; ++k) {
    if (run[k].count == 0) continue;
    if (field) all(run[k], std::true_type{});
    else all(run[k], std::false_type{});
  }
  if (N.n_split > 0) {
    auto sum = [&](auto kern) {
      // a block per 64 columns of the largest leaf (others loop or idle)
      const int64_t tiles = ((field ? 4 : 1) * (int64_t)pl->max_leaf_count + 63) / 64;
      kern<<<dim3((unsigned)N.n_split, (unsigned)std::min<int64_t>(tiles, 1024)), 64, 0, sp>>>(
          n, N.split_leaf, N.split_first, N.split_cnt, N.out, pl->leaf_start, (const T*)N.part,
          near);
    };
    if (field) sum(k_p2p_sum<T, true>);
    else sum(k_p2p_sum<T, false>);
  }
}

}  // namespace

// The near field (P2P) over the direct lists Ls into near, on stream sp:
// one launch over the work items, then the partial sums of the leaves whose
// list was split.
void near_field(fmm_plan* pl, const ListSet& Ls, const void* src, int64_t n, void* near, bool field,
                hipStream_t sp, const StageMarks& mk) {
  mk.begin(kStP2P, sp);
  if (pl->prm.precision == FMM_FP32)
    run_near<float>(pl, Ls, (const Src<float>*)src, n, (float*)near, field, sp);
  else
    run_near<double>(pl, Ls, (const Src<double>*)src, n, (double*)near, field, sp);
  mk.end(kStP2P, sp);
}

}  // namespace fmm

// For the tests, no part of the ABI: the forms of a pass as threads of an
// item's block (0: one wave, one target a lane) and the items of each, up to
// four; returns their number.
extern "C" int fmm_near_runs(const fmm_plan* pl, int transposed, int field, int* threads,
                             int64_t* items) {
  using namespace fmm;
  NearRun run[4];
  const int k = near_runs(pl, pl->lists[transposed ? 1 : 0], field != 0, run);
  for (int j = 0; j < k; ++j) {
    const int f = run[j].form;
    threads[j] = f == kNearWide256 ? 256 : f == kNearWide ? 128 : f == kNearWide64 ? 64 : 0;
    items[j] = run[j].count;
  }
  return k;
}
