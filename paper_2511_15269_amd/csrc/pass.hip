// One evaluation pass of a plan: the launch tiles in effect, the choice of
// the order's kernels (eval.hip) and the adjoint's combine step.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace fmm {

bool valid_p2p_groups(const fmm_plan* pl, int g) {
  return g == 1 || ((g == 2 || g == 4) && pl->max_leaf_count <= 64 / g);
}
bool valid_leaves_per_wave(const fmm_plan* pl, int l) {
  return l == 1 || ((l == 2 || l == 4 || l == 8) && pl->max_leaf_count <= 64 / l);
}
int default_p2p_groups(const fmm_plan* pl) {
  const int m = pl->max_leaf_count;
  return m > 32 ? 1 : (m > 16 ? 2 : 4);
}
int p2p_groups(const fmm_plan* pl) {
  if (pl->p2p_groups && valid_p2p_groups(pl, pl->p2p_groups)) return pl->p2p_groups;
  return default_p2p_groups(pl);
}
int near_form(const fmm_plan* pl, int nt, double list, int64_t items, bool field) {
  const int h = (nt + 1) / 2;
  if (pl->prm.precision == FMM_FP64) {
    int form = kNearWave;
    double best = default_p2p_groups(pl) > 1 ? 0.0 : nt / (64.0 * ((nt + 63) / 64));
    for (int W : {64, 128}) {
      if (nt > 2 * W) continue;  // two targets a thread
      // the groups share out the points; the larger block has to be worth
      // its barriers and its set-up
      const double rate = kFlatRate * nt * (W / h) / (2.0 * W);
      if (rate > (form == kNearWide64 ? kFlatGain * best : best)) {
        best = rate;
        form = W == 128 ? kNearWide : kNearWide64;
      }
    }
    return form;
  }
  if (default_p2p_groups(pl) > 1) return kNearWave;
  const WideRates& R = field ? kWideField : kWidePot;
  const double per_simd = items / 1024.0;
  int form = kNearWave;
  double best = nt / (64.0 * ((nt + 63) / 64)) * per_simd / (per_simd + 1.0);
  for (int W : {64, 128, 256}) {
    // two groups of two targets a thread, or more; 256 threads only for fill
    if (nt > W || (W == 256 && per_simd >= kWideFillWaves)) continue;
    const int ng = W / h;
    const double full = std::floor(list / ng), rem = list - full * ng;
    const double waves = full * std::ceil(ng * h / 64.0) + std::ceil(rem * h / 64.0);
    const double x = per_simd * (W / 64);
    const double rate = W == 64 ? R.w64 : (W == 128 ? R.w128 : R.w256);
    const double r = rate * nt * list / (128.0 * waves) * x / (x + 1.0);
    if (r > best) {
      best = r;
      form = W == 256 ? kNearWide256 : (W == 128 ? kNearWide : kNearWide64);
    }
  }
  return form;
}
// A single-vector pass against the pass of up to 16 vectors, both in us as the
// sum of what they wait for: launches, the level chains, M2L (the length of a
// translation or the pairs' throughput), the near field (the length of a list
// or its throughput) and the work per point.  The two were fitted to 474 plans
// on the cube and the sphere: 60 to 260000 points, p = 2 to 10, leaves of 16 to
// 256 points; each is within 20% of the measured time for nine plans in ten.
// Vectors are taken one by one up to kFewVectors while that is estimated at most
// 5% longer.  Against the better of the two ways as measured this loses less than
// 1% on average for 2 to 5 vectors and 10 to 30% at worst; by count alone (3, or 5
// from 2^14 points) it lost 16 to 39% on average, and small plans up to six times:
// 3 vectors of 300 points, leaves of 32, 141 us one by one and 76 together; 5
// vectors of 20000 points, p = 4, 288 and 226; 5 of 130000, p = 10, 1130 and 2400.
bool vectors_one_by_one(const fmm_plan* pl, int R) {
  constexpr int kFewVectors = 5, kFewVectorsSmall = 3;
  constexpr int64_t kFewVectorsPoints = 1 << 14;
  if (R == 1) return true;
  if (R > (pl->n < kFewVectorsPoints ? kFewVectorsSmall : kFewVectors)) return false;
  const double n = (double)pl->n, p = pl->prm.p, K = (p + 1) * (p + 1);
  const double turn = p * p * std::sqrt(p);  // a translation's growth with p
  const double pairs = (double)pl->lists[0].n_m2l, inter = (double)pl->p2p_inter;
  const double far = pairs > 0 ? 1.0 : 0.0, levels = pl->L, list = inter / n;
  const double leaf = std::ceil(n / (double)pl->nleaf);
  const double tiles = std::ceil(leaf / (16.0 * batch_p2p_waves(pl)));
  const double chain1 = levels * 0.071 * p * p +
                        std::max(far * 0.074 * turn, pairs * 1e-6 * (41 + 0.42 * turn));
  // (leaves of up to 32 points are swept by one wave, staged leaf by leaf)
  const double near1 = std::max(leaf <= 32 ? 0.026 * list : 0.0, inter * 0.44e-6);
  const double one = 58 + std::max(chain1, near1) + 0.5 * std::min(chain1, near1) +
                     n * 2.4e-6 * K;
  const double chain16 = far * levels * (9 + 0.24 * p * p);
  const double m2l16 = std::max(far * (19 + 0.31 * turn) * std::min(1.0, pairs / 2500),
                                pairs * 1e-6 * (240 + 10.5 * turn));
  const double near16 = std::max(0.094 * list * tiles, inter * 1.9e-6);
  const double together = 26 + 0.24 * K + chain16 + m2l16 + near16 + n * 1e-6 * (150 + 20 * K);
  return R * one <= 1.05 * together;
}
int chain_waves(const fmm_plan* pl) {
  return pl->prm.p < kChainShareMinOrder || pl->chain_waves == 1 ? 1 : kShareWaves;
}
int m2l_waves(const fmm_plan* pl) {
  const int shared = m2l_share_waves(pl->prm.p, pl->prm.precision == FMM_FP64);
  return pl->m2l_waves == 1 ? 1 : shared;
}
int leaves_per_wave(const fmm_plan* pl) {
  if (pl->leaves_per_wave && valid_leaves_per_wave(pl, pl->leaves_per_wave))
    return pl->leaves_per_wave;
  const int m = pl->max_leaf_count;
  return m > 32 ? 1 : (m > 16 ? 2 : (m > 8 ? 4 : 8));
}

namespace {

// d/dx_k of sum_i g_i u_i: g_k grad u(x_k) (x_k as a target of the forward
// pass) + q_k grad v(x_k) (x_k as a source, v = transposed pass with charges
// g); fields are -grad.
template <typename T>
__global__ void k_adjoint_combine(int64_t n, const T* __restrict__ q, const T* __restrict__ g,
                                  const T* __restrict__ ff, const T* __restrict__ ft,
                                  T* __restrict__ gx) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 3 * n) return;
  const int64_t i = e / 3;
  gx[e] = -(g[i] * ff[e] + q[i] * ft[e]);
}


inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

template <typename T>
void dispatch(int p, fmm_plan* pl, const Workspace& ws, int dir, const T* q, T* pot,
              T* field, hipStream_t st) {
  switch (p) {
#define FMM_CASE(PP) \
  case PP:           \
    run_pass<PP, T>(pl, ws, dir, q, pot, field, st); \
    break;
    FMM_CASE(1) FMM_CASE(2) FMM_CASE(3) FMM_CASE(4) FMM_CASE(5)
    FMM_CASE(6) FMM_CASE(7) FMM_CASE(8) FMM_CASE(9) FMM_CASE(10)
#undef FMM_CASE
    default:
      throw Error{FMM_ENOTSUP, "expansion order without compiled kernels"};
  }
}

}  // namespace

void evaluate(fmm_plan* pl, const Workspace& ws, int dir, const void* q, int nrhs, void* pot,
              void* field, hipStream_t st) {
  // vector r of q has the source side's points, of pot/field the target side's
  const int64_t nq = src_side(pl, dir).npt, nu = tgt_side(pl, dir).npt;
  for (int r = 0; r < nrhs; ++r) {
    if (pl->prm.precision == FMM_FP32) {
      dispatch<float>(pl->prm.p, pl, ws, dir, (const float*)q + r * nq, (float*)pot + r * nu,
                      field ? (float*)field + 3 * r * nu : nullptr, st);
    } else {
      dispatch<double>(pl->prm.p, pl, ws, dir, (const double*)q + r * nq, (double*)pot + r * nu,
                       field ? (double*)field + 3 * r * nu : nullptr, st);
    }
  }
}

void adjoint_combine(fmm_plan* pl, const void* q, const void* g, const void* field_fwd,
                     const void* field_t, void* grad_x, hipStream_t st) {
  const int64_t n = pl->n;
  if (pl->prm.precision == FMM_FP32)
    k_adjoint_combine<float><<<blocks(3 * n, 256), 256, 0, st>>>(
        n, (const float*)q, (const float*)g, (const float*)field_fwd, (const float*)field_t,
        (float*)grad_x);
  else
    k_adjoint_combine<double><<<blocks(3 * n, 256), 256, 0, st>>>(
        n, (const double*)q, (const double*)g, (const double*)field_fwd,
        (const double*)field_t, (double*)grad_x);
  FMM_HIP(hipGetLastError());
}

}  // namespace fmm
