// Evaluation pass for up to kRB = 32 charge vectors at once on one plan
// (the paper's cached hierarchy reused for new charges, Sec. II.E), FP32.
//
// Layout: every per-point and per-box array carries the vectors innermost:
// charges qL[n][kRB] in leaf order, expansions C, D [box][(p+1)^2][kRB],
// outputs potL[n][kRB], fldL[n][3][kRB] in leaf order, scattered to the
// caller's [R][n] / [R][n][3] at the end.  Lane r of a 32-lane half-wave
// owns vector r, so every coefficient access is a contiguous 128-byte
// segment, and everything that depends only on the geometry -- rotation
// angles, scale ratios, the operator tables -- is shared by all vectors.
//
//   P2M:  block = leaf; the basis of 64 points goes to LDS, lane r then
//         forms C[k][r] = sum_i B_k(y_i) q_i[r].
//   M2M, M2L, L2L: the single-vector rotate / z-shift / rotate-back code,
//         one (box or work item, vector) per lane, two boxes or items per
//         wave (one per half-wave); M2M translates the children of a parent
//         in parallel waves and adds them in child order.
//   L2P:  block = leaf; basis and gradient of 32 points in LDS, lane r
//         forms the potential and gradient sums.
// The near field and the moves between the caller's layout and leaf order,
// which do not depend on the order, are in batch_near.hip; this file is
// compiled once per expansion order (FMM_ORDER).
#include <cmath>

#include <type_traits>

#include "internal.h"
#include "ops.h"
#include "tables.h"

namespace fmm {
namespace {

using namespace ops;
constexpr int kRB = kBatchWidth;

typedef float floatx16 __attribute__((ext_vector_type(16)));

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// P2M as a contraction on the matrix cores: C[k][r] = normc_k sum_p
// R_k(y_p) q[p][r] for the 32 vectors r.  The basis values of up to 64
// points are formed in LDS (one lane per point); then v_mfma_f32_32x32x2f32
// takes two points per step: A = basis of 32 coefficients (rows, one tile
// of three) x 2 points, B = charges of the 2 points x 32 vectors.
// Accumulator register v of lane l holds coefficient row
// 8 (v / 4) + 4 (l / 32) + v % 4 of the tile, vector l % 32.  One wave per
// tile of 32 coefficients, the basis and charge tiles shared in LDS.  The
// charges come leaf-ordered from k_bgather.
template <int P>
__global__ __launch_bounds__(64 * ((K_<P>::value + 31) / 32)) void k_bp2m(
    const int32_t* __restrict__ leaf_box, const int32_t* __restrict__ leaf_start,
    const double* __restrict__ xs, const double* __restrict__ ys,
    const double* __restrict__ zs, const float* __restrict__ qL,
    const double* __restrict__ cx, const double* __restrict__ cy,
    const double* __restrict__ cz, const double* __restrict__ scale,
    const float* __restrict__ tab, float* __restrict__ C) {
  constexpr int K = K_<P>::value;
  constexpr int NT = (K + 31) / 32;  // coefficient tiles, one wave each
  __shared__ float B[64][NT * 32 + 1];
  __shared__ float Q[64][kRB];  // charges of the chunk's points
  const int leaf = blockIdx.x;
  const int lane = threadIdx.x % 64;
  const int t = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // this wave's tile
  const int col = lane % 32, kh = lane / 32;
  const int64_t g = leaf_box[leaf];
  const int st = leaf_start[leaf], en = leaf_start[leaf + 1];
  const double ox = cx[g], oy = cy[g], oz = cz[g], ir = 1.0 / scale[g];
  floatx16 acc = {};
  for (int c0 = st; c0 < en; c0 += 64) {
    const int cnt = min(64, en - c0);
    __syncthreads();
    if (t == 0) {
      // the first wave forms the basis (lane = point); padding rows and
      // missing points read as zero
      const int j = c0 + lane;
      const bool pt = j < en;
      const int jj = pt ? j : c0;
#pragma unroll
      for (int k = K; k < NT * 32; ++k) B[lane][k] = 0.f;
      regular_basis<P, float>(float((xs[jj] - ox) * ir), float((ys[jj] - oy) * ir),
                              float((zs[jj] - oz) * ir),
                              [&](int k, float v) { B[lane][k] = pt ? v : 0.f; });
    }
    for (int e = threadIdx.x; e < cnt * kRB; e += blockDim.x)
      Q[e / kRB][e % kRB] = qL[(int64_t)c0 * kRB + e];
    __syncthreads();
    for (int p0 = 0; p0 < cnt; p0 += 2) {
      const int pp = p0 + kh;
      const float b = pp < cnt ? Q[pp][col] : 0.f;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(B[pp < 64 ? pp : 0][t * 32 + col], b, acc, 0, 0,
                                                 0);
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int k = t * 32 + 8 * (v / 4) + 4 * kh + v % 4;
    if (k < K) C[(g * K + k) * kRB + col] = acc[v] * tab[tab_normc(P) + k];
  }
}

// parent = sum over its 2^s children of M2M(child), 32 vectors per parent:
// wave c of a block of 2^s waves translates child c of two parents (one
// per half-wave, lane = vector), and the translated children are added in
// child order through an LDS tile (one barrier per child).
template <int P>
__global__ __launch_bounds__(512) void k_bm2m_par(
    int64_t npar, const int32_t* __restrict__ par, const int32_t* __restrict__ child0, int s,
    const double* __restrict__ cx, const double* __restrict__ cy,
    const double* __restrict__ cz, const double* __restrict__ scale,
    const float* __restrict__ tab, float* C) {
  constexpr int K = K_<P>::value;
  __shared__ float A[2][K][kRB];
  const int c = threadIdx.x / 64;  // child (wave-uniform)
  const int lane = threadIdx.x % 64;
  const int h = lane / kRB, r = lane % kRB;
  const int64_t b = (int64_t)blockIdx.x * 2 + h;
  const bool live = b < npar;
  const int64_t pa = live ? par[b] : 0;
  const int64_t ch = live ? child0[b] + c : 0;
  float v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = live ? C[(ch * K + k) * kRB + r] : 0.f;
  if (live)
    rotate_shift<P, kM2M, float>(v, cx[ch] - cx[pa], cy[ch] - cy[pa], cz[ch] - cz[pa],
                                 scale[ch], scale[pa], tab);
  const int nch = 1 << s;
  for (int step = 0; step < nch; ++step) {
    if (c == step) {
#pragma unroll
      for (int k = 0; k < K; ++k) A[h][k][r] = (step == 0 ? 0.f : A[h][k][r]) + v[k];
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < 2 * K * kRB; e += blockDim.x) {
    const int hh = e / (K * kRB), kr = e % (K * kRB);
    const int64_t bb = (int64_t)blockIdx.x * 2 + hh;
    if (bb < npar) C[(int64_t)par[bb] * K * kRB + kr] = A[hh][kr / kRB][kr % kRB];
  }
}

template <int P>
__global__ __launch_bounds__(64) void k_bm2l(
    int cols, int64_t nitems, const int32_t* __restrict__ item_tgt,
    const int32_t* __restrict__ item_begin, const int32_t* __restrict__ item_end,
    const int32_t* __restrict__ src, const double* __restrict__ cx,
    const double* __restrict__ cy, const double* __restrict__ cz,
    const double* __restrict__ scale, const float* __restrict__ C,
    const float* __restrict__ tab, float* __restrict__ partial) {
  constexpr int K = K_<P>::value;
  const int64_t i = (int64_t)blockIdx.x * (64 / cols) + threadIdx.x / cols;
  const int r = threadIdx.x % cols;
  if (i >= nitems) return;
  const int t = item_tgt[i];
  if (t < 0) return;  // idle lane of the packed item layout
  const int jb = item_begin[i], je = item_end[i];
  const double tx = cx[t], ty = cy[t], tz = cz[t], rt = scale[t];
  float acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = 0.f;
  for (int j = jb; j < je; ++j) {
    const int sidx = src[j];
    float v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = C[((int64_t)sidx * K + k) * kRB + r];
    rotate_shift<P, kM2L, float>(v, cx[sidx] - tx, cy[sidx] - ty, cz[sidx] - tz, scale[sidx],
                                 rt, tab);
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] += v[k];
  }
#pragma unroll
  for (int k = 0; k < K; ++k) partial[(i * K + k) * kRB + r] = acc[k];
}

// D[t][0..W) = sum over the M2L work items of box t (in item order) of
// their partial rows, for every box t in boxes[0..nb): one block per box,
// threads over the row.  The far-field local of every box starts here; the
// level-by-level L2L kernels then add the translated parent local.
template <typename T>
__global__ void k_psum(int64_t nb, const int32_t* __restrict__ boxes,
                       const int32_t* __restrict__ item_first, const int32_t* __restrict__ item_cnt,
                       const T* __restrict__ partial, int W, T* __restrict__ D) {
  const int64_t t = boxes[blockIdx.x];
  const int b = item_first[t], e = b + item_cnt[t];
  for (int k = threadIdx.x; k < W; k += blockDim.x) {
    T acc = T(0);
    int it = b;
    // four rows' loads in flight at a time; the sum keeps item order
    for (; it + 4 <= e; it += 4) {
      const T r0 = partial[(int64_t)it * W + k], r1 = partial[(int64_t)(it + 1) * W + k];
      const T r2 = partial[(int64_t)(it + 2) * W + k], r3 = partial[(int64_t)(it + 3) * W + k];
      acc += r0;
      acc += r1;
      acc += r2;
      acc += r3;
    }
    for (; it < e; ++it) acc += partial[(int64_t)it * W + k];
    D[t * W + k] = acc;
  }
}

template <int P>
__global__ __launch_bounds__(64) void k_bl2l(
    int cols, int64_t nb, const int32_t* __restrict__ boxes, const int32_t* __restrict__ parents,
    const double* __restrict__ cx, const double* __restrict__ cy,
    const double* __restrict__ cz, const double* __restrict__ scale,
    const float* __restrict__ tab, float* D) {
  constexpr int K = K_<P>::value;
  const int64_t i = (int64_t)blockIdx.x * (64 / cols) + threadIdx.x / cols;
  const int r = threadIdx.x % cols;
  if (i >= nb) return;
  const int64_t t = boxes[i];
  const int64_t pa = parents[i];
  float v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = D[(pa * K + k) * kRB + r];
  rotate_shift<P, kL2L, float>(v, cx[pa] - cx[t], cy[pa] - cy[t], cz[pa] - cz[t], scale[pa],
                               scale[t], tab);
#pragma unroll
  for (int k = 0; k < K; ++k) D[(t * K + k) * kRB + r] = D[(t * K + k) * kRB + r] + v[k];
}

// L2P as a contraction on the matrix cores: for 32 points at a time,
// u[p][r] = sum_k R_k(y_p) w_k D[k][r] and likewise the three gradient
// components.  The basis and its gradient are formed in LDS (one lane per
// point, first wave); v_mfma_f32_32x32x2f32 then takes two coefficients per
// step: A = basis values of 32 points (rows) x 2 coefficients, B = weighted
// local coefficients (2 x 32 vectors).  The block's four waves share the
// basis tile, wave c forming component c (potential, then the gradient's
// x, y, z), so that a 43 KiB tile serves four waves.  Accumulator register
// v of lane l holds point row 8 (v / 4) + 4 (l / 32) + v % 4, vector l % 32.
template <int P>
__global__ __launch_bounds__(256) void k_bl2p(
    const int32_t* __restrict__ leaf_box, const int32_t* __restrict__ leaf_start,
    const double* __restrict__ xs, const double* __restrict__ ys,
    const double* __restrict__ zs, const double* __restrict__ cx,
    const double* __restrict__ cy, const double* __restrict__ cz,
    const double* __restrict__ scale, const float* __restrict__ D,
    const float* __restrict__ tab, float* __restrict__ potL, float* __restrict__ fldL) {
  constexpr int K = K_<P>::value;
  constexpr int K2 = (K + 1) / 2 * 2;  // coefficient pairs (one zero row padded)
  constexpr int NP = 32;
  __shared__ float Bv[4][K2][NP + 1];
  const int leaf = blockIdx.x;
  const int lane = threadIdx.x % 64;
  const int comp = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);  // component of this wave
  const int col = lane % 32, kh = lane / 32;
  const int64_t g = leaf_box[leaf];
  const int st = leaf_start[leaf], en = leaf_start[leaf + 1];
  const double ox = cx[g], oy = cy[g], oz = cz[g], ir = 1.0 / scale[g];
  const float fu = float(-kInv4Pi * ir), ff = float(kInv4Pi * ir * ir);
  for (int c0 = st; c0 < en; c0 += NP) {
    const int cnt = min(NP, en - c0);
    __syncthreads();
    if (threadIdx.x < NP) {
      const bool pt = lane < cnt;
      const int j = pt ? c0 + lane : c0;
      const float x = float((xs[j] - ox) * ir), y = float((ys[j] - oy) * ir),
                  z = float((zs[j] - oz) * ir);
      basis_with_gradient<P, float>(x, y, z, [&](int k, float v, float gx, float gy, float gz) {
        Bv[0][k][lane] = pt ? v : 0.f;
        Bv[1][k][lane] = pt ? gx : 0.f;
        Bv[2][k][lane] = pt ? gy : 0.f;
        Bv[3][k][lane] = pt ? gz : 0.f;
      });
      if (K2 > K) {
#pragma unroll
        for (int c = 0; c < 4; ++c) Bv[c][K2 - 1][lane] = 0.f;
      }
    }
    __syncthreads();
    floatx16 acc = {};
    for (int k0 = 0; k0 < K2; k0 += 2) {
      const int k = k0 + kh;
      const float b = k < K ? D[(g * K + k) * kRB + col] * tab[tab_l2p(P) + k] : 0.f;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(Bv[comp][k][col], b, acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int pnt = 8 * (v / 4) + 4 * kh + v % 4;
      if (pnt < cnt) {
        const int64_t o = c0 + pnt;
        if (comp == 0)
          potL[o * kRB + col] = fu * acc[v];
        else
          fldL[(o * 3 + comp - 1) * kRB + col] = ff * acc[v];
      }
    }
  }
}

}  // namespace

template <int P>
void run_batch(fmm_plan* pl, const ListSet& Ls, const float* q, int R, float* pot, float* field,
               hipStream_t st) {
  const int s = pl->s;
  const float* tab = (const float*)pl->tables;
  float* qL = (float*)pl->ws.bq;
  float* C = (float*)pl->ws.bC;
  float* D = (float*)pl->ws.bD;
  float* part = (float*)pl->bpart;
  float* potL = (float*)pl->ws.bpot;
  float* fldL = (float*)pl->ws.bfld;
  const int64_t n = pl->n;
  // vectors a wave of M2L and L2L takes of each box (the rows stay kRB wide,
  // what lies beyond R in them is not read by any other vector).  Measured, 16
  // vectors of 30000 points with 32 and with 16 a wave, p = 8: 1377 and 970 us
  const int cols = R <= kRB / 2 ? kRB / 2 : kRB;
  StageMarks mk(pl);
  // the sort stage is folded into P2M; its timing slot stays empty
  mk.begin(kStSort, st);
  mk.end(kStSort, st);
  mk.begin(kStP2M, st);
  batch_gather(pl, q, R, qL, st);
  k_bp2m<P><<<(unsigned)pl->nleaf, 64 * ((K_<P>::value + 31) / 32), 0, st>>>(
      pl->leaf_box, pl->leaf_start, pl->xs, pl->ys, pl->zs, qL, pl->cx, pl->cy, pl->cz,
      pl->scale, tab, C);
  mk.end(kStP2M, st);
  mk.begin(kStM2M, st);
  for (const Step& S : pl->side[0].m2m_steps)
    k_bm2m_par<P><<<blocks(S.n, 2), 64 << s, 0, st>>>(S.n, S.a, S.b, s, pl->cx, pl->cy, pl->cz,
                                                      pl->scale, tab, C);
  mk.end(kStM2M, st);
  mk.begin(kStM2L, st);
  if (Ls.n_items > 0)
    k_bm2l<P><<<blocks(Ls.n_items, 64 / cols), 64, 0, st>>>(
        cols, Ls.n_items, Ls.item_tgt, Ls.item_begin, Ls.item_end, Ls.m2l_src, pl->cx, pl->cy,
        pl->cz, pl->scale, C, tab, part);
  mk.end(kStM2L, st);
  mk.begin(kStL2L, st);
  const Step& all = pl->side[0].l2l_sum;
  if (all.n > 0)
    k_psum<float><<<(unsigned)all.n, 256, 0, st>>>(all.n, all.a, Ls.item_first, Ls.item_cnt,
                                                   part, K_<P>::value * kRB, D);
  for (const Step& S : pl->side[0].l2l_steps)
    k_bl2l<P><<<blocks(S.n, 64 / cols), 64, 0, st>>>(cols, S.n, S.a, S.b, pl->cx, pl->cy, pl->cz,
                                                     pl->scale, tab, D);
  mk.end(kStL2L, st);
  mk.begin(kStL2P, st);
  k_bl2p<P><<<(unsigned)pl->nleaf, 256, 0, st>>>(pl->leaf_box, pl->leaf_start, pl->xs, pl->ys,
                                                pl->zs, pl->cx, pl->cy, pl->cz, pl->scale, D,
                                                tab, potL, fldL);
  mk.end(kStL2P, st);
  mk.begin(kStP2P, st);
  batch_near(pl, Ls, R, qL, potL, fldL, st);
  batch_scatter(pl, R, potL, fldL, pot, field, st);
  mk.end(kStP2P, st);
  FMM_HIP(hipGetLastError());
}

template void run_batch<FMM_ORDER>(fmm_plan*, const ListSet&, const float*, int, float*, float*,
                                   hipStream_t);

}  // namespace fmm
