// Direct O(N * T) evaluation of the potential and field (eqs. 1-3): the
// reference against which the paper measures the FMM error (Sec. III.A).
// Lane = source point, R targets per wave in registers: every source that a
// lane loads (coalesced, no LDS) meets R targets, and each lane's sums over
// its n / 64 sources are added across lanes at the end.  A block has
// kWaves waves; groups of `slices` waves share their R targets and take
// every slices-th run of 64 sources, so that a few targets still fill the
// chip (one lane per target left 224 of the 256 CUs idle for 8192 targets).
// Bound by FP64 VALU issue.  Measured: 8192 targets of 2^20 charges, FP64
// potential and field, 99.3 -> 7.8 ms (9.0 ms with two Newton steps a root and
// every run of 64 sources checked against n).
// Pairs at distance 0 contribute nothing.
#include "internal.h"

namespace fmm {
namespace {

constexpr double kInv4Pi = 0.079577471545947667884441881686257181;
constexpr int kWaves = 16;

// 1 / sqrt(r2): the hardware's estimate y with e = 1 - r2 y^2 (2^-24 or so)
// and the series of (1 - e)^(-1/2) up to e^2; five operations, the remainder
// (5/16) e^3 is far below a rounding.
__device__ __forceinline__ double rsq(double r2) {
  const double y = __builtin_amdgcn_rsq(r2);
  const double e = fma(-(r2 * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ float rsq(float r2) { return __builtin_amdgcn_rsqf(r2); }

template <typename T, bool FIELD, int R>
__global__ __launch_bounds__(64 * kWaves) void k_direct(
    int64_t n, const double* __restrict__ pos, const T* __restrict__ q,
    const int64_t* __restrict__ targets, int64_t nt, int slices, T* __restrict__ pot,
    T* __restrict__ field) {
  constexpr int NC = FIELD ? 4 : 1;
  __shared__ T sum[kWaves][R * NC];
  const int lane = threadIdx.x % 64;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int groups = kWaves / slices;  // groups of waves in the block
  const int grp = w / slices, slice = w - grp * slices;
  const int64_t t0 = ((int64_t)blockIdx.x * groups + grp) * R;  // the wave's first target
  double x[R], y[R], z[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    // past the last target or an index outside [0, n): reads point 0
    const int64_t it = t0 + r;
    int64_t t = it < nt ? (targets ? targets[it] : it) : 0;
    if (t < 0 || t >= n) t = 0;
    x[r] = pos[3 * t];
    y[r] = pos[3 * t + 1];
    z[r] = pos[3 * t + 2];
  }
  T s[R][NC];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < NC; ++c) s[r][c] = T(0);
  if (t0 < nt) {
    const int64_t step = (int64_t)slices * 64;
    auto run = [&](int64_t j, bool live) {
      const double sx = pos[3 * j], sy = pos[3 * j + 1], sz = pos[3 * j + 2];
      // a lane past n reads point 0, whose charge must not count even times 0
      // (it may be infinite)
      const T qj = live ? q[j] : T(0);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const T dx = T(x[r] - sx), dy = T(y[r] - sy), dz = T(z[r] - sz);
        const T r2 = dx * dx + dy * dy + dz * dz;
        const T inv = live && r2 > T(0) ? rsq(r2) : T(0);
        const T qi = qj * inv;
        s[r][0] += qi;
        if (FIELD) {
          const T q3 = qi * inv * inv;
          s[r][1] = fma(q3, dx, s[r][1]);
          s[r][2] = fma(q3, dy, s[r][2]);
          s[r][3] = fma(q3, dz, s[r][3]);
        }
      }
    };
    int64_t j0 = (int64_t)slice * 64;
    for (; j0 + 64 <= n; j0 += step) run(j0 + lane, true);
    if (j0 < n) run(j0 + lane < n ? j0 + lane : 0, j0 + lane < n);
  }
  // sums over the lanes: at each step a lane hands on half of the values that it
  // holds and adds the other half of its partner's, until it holds one (19
  // exchanges for 16 values instead of 96, the same sums; with few sources they
  // are what a wave waits for: 10^5 targets of 64 charges, FP64 potential and
  // field, 117 -> 75 us, 91 with one lane per target)
  constexpr int N = R * NC;
  T* const v = &s[0][0];
  int held = 0;  // the value (target, component) that v[0] ends up as
#pragma unroll
  for (int off = 1, half = N / 2; off < 64; off <<= 1, half /= 2) {
    if (half == 0) {
      v[0] += __shfl_xor(v[0], off, 64);
      continue;
    }
    const bool up = lane & off;
#pragma unroll
    for (int k = 0; k < half; ++k) {
      const T keep = up ? v[k + half] : v[k], hand = up ? v[k] : v[k + half];
      v[k] = keep + __shfl_xor(hand, off, 64);
    }
    if (up) held += half;
  }
  if (lane < N) sum[w][held] = v[0];
  __syncthreads();
  // one thread per (target, component): the slices' sums in order
  for (int e = threadIdx.x; e < groups * R * NC; e += 64 * kWaves) {
    const int g = e / (R * NC), rc = e - g * (R * NC);
    const int64_t it = ((int64_t)blockIdx.x * groups + g) * R + rc / NC;
    if (it >= nt) continue;
    T v = T(0);
    for (int k = 0; k < slices; ++k) v += sum[g * slices + k][rc];
    const int64_t t = targets ? targets[it] : it;
    // field = -grad u = -(1/4pi) sum q (x_i - x_j)/r^3
    v = t >= 0 && t < n ? -T(kInv4Pi) * v : T(__builtin_nan(""));
    if (rc % NC == 0)
      pot[it] = v;
    else
      field[3 * it + rc % NC - 1] = v;
  }
}

// Targets per wave: as few as go into one round of kFill blocks (a block fills
// a CU), 4 at most, since a round of 2 takes 1.3 times and of 4 twice as long
// as a round of 1 (2^20 charges, FP64 potential and field: 64 targets 0.48, 512
// 0.64, 1024 1.00 ms; 300 targets with one a wave, two rounds, 0.97 ms);
// slices: as few waves per group as leave kFill blocks.
constexpr int64_t kFill = 256;

template <typename T, int R>
void launch(int64_t n, const double* pos, const void* q, const int64_t* targets,
            int64_t nt, void* pot, void* field, hipStream_t st) {
  int slices = 1;
  while (slices < kWaves && (nt * slices + R * kWaves - 1) / (R * kWaves) < kFill) slices *= 2;
  const int64_t per = (int64_t)R * (kWaves / slices);
  const unsigned nb = (unsigned)((nt + per - 1) / per);
  if (field)
    k_direct<T, true, R><<<nb, 64 * kWaves, 0, st>>>(n, pos, (const T*)q, targets, nt, slices,
                                                     (T*)pot, (T*)field);
  else
    k_direct<T, false, R><<<nb, 64 * kWaves, 0, st>>>(n, pos, (const T*)q, targets, nt, slices,
                                                      (T*)pot, nullptr);
  FMM_HIP(hipGetLastError());
}

template <typename T>
void choose(int64_t n, const double* pos, const void* q, const int64_t* targets, int64_t nt,
            void* pot, void* field, hipStream_t st) {
  if (nt > 2 * kFill)
    launch<T, 4>(n, pos, q, targets, nt, pot, field, st);
  else if (nt > kFill)
    launch<T, 2>(n, pos, q, targets, nt, pot, field, st);
  else
    launch<T, 1>(n, pos, q, targets, nt, pot, field, st);
}

}  // namespace

void direct_sum(int64_t n, const double* pos, const void* q, int precision,
                const int64_t* targets, int64_t nt, void* pot, void* field,
                hipStream_t st) {
  if (nt == 0) return;
  if (precision == FMM_FP32)
    choose<float>(n, pos, q, targets, nt, pot, field, st);
  else
    choose<double>(n, pos, q, targets, nt, pot, field, st);
}

}  // namespace fmm
