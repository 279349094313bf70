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
// difference is taken in FP64 and rounded to T.  SAFE: pairs at distance 0
// contribute nothing (needed within a leaf, and between leaves when the
// point set has coincident points); otherwise the pair is known to be apart.
template <typename T, bool FIELD, bool SAFE>
__device__ __forceinline__ void p2p_pair(const Src<T>& s, double xi, double yi, double zi,
                                         T& u, T& gx, T& gy, T& gz) {
  const T dx = T(xi - s.x), dy = T(yi - s.y), dz = T(zi - s.z);
  const T r2 = dx * dx + dy * dy + dz * dz;
  const T inv0 = inv_sqrt(r2);
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
    int64_t n, const int32_t* __restrict__ item_leaf, const int32_t* __restrict__ item_kb,
    const int32_t* __restrict__ item_ke, const int64_t* __restrict__ item_out,
    const int32_t* __restrict__ leaf_start, const double* __restrict__ xs,
    const double* __restrict__ ys, const double* __restrict__ zs,
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
      // or every leaf when the point set has coincident points
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
        near[i] = -T(kInv4Pi) * u;
        if (FIELD) {
          T* f = near + n + 3 * (int64_t)i;
          f[0] = -T(kInv4Pi) * gx;
          f[1] = -T(kInv4Pi) * gy;
          f[2] = -T(kInv4Pi) * gz;
        }
      } else {  // one of several items of the leaf: rows of its partial sums
        const int nt = en - st, li = i - st;
        T* r = part + po;
        r[li] = -T(kInv4Pi) * u;
        if (FIELD) {
          r[nt + li] = -T(kInv4Pi) * gx;
          r[2 * nt + li] = -T(kInv4Pi) * gy;
          r[3 * nt + li] = -T(kInv4Pi) * gz;
        }
      }
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

template <typename T>
void run_near(fmm_plan* pl, const ListSet& Ls, const Src<T>* src, int64_t n, T* near, bool field,
              hipStream_t sp) {
  const int G = p2p_groups(pl);
  const NearItems& N = Ls.near;
  auto p2p = [&](auto kern) {
    kern<<<(unsigned)N.n, 64, 0, sp>>>(n, N.leaf, N.kb, N.ke, N.out, pl->leaf_start, pl->xs,
                                       pl->ys, pl->zs, src, Ls.p2p_src, pl->has_dup ? 1 : 0, near,
                                       (T*)N.part);
  };
  if (field) {
    if (G == 1) p2p(k_p2p<T, true, 1>);
    else if (G == 2) p2p(k_p2p<T, true, 2>);
    else p2p(k_p2p<T, true, 4>);
  } else {
    if (G == 1) p2p(k_p2p<T, false, 1>);
    else if (G == 2) p2p(k_p2p<T, false, 2>);
    else p2p(k_p2p<T, false, 4>);
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
