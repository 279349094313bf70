// Near field of the 32-vector pass (batch.hip) on the matrix cores, and the
// moves of charges and outputs between the caller's vector-major layout and
// leaf order with the vectors innermost.
//   P2P:  a dense contraction: for a tile of 16 targets and groups of four
//         source points, the kernel entries 1/r and d/r^3 (computed per lane,
//         one entry each) are the A operand and the source charges of the 32
//         vectors the B operand of v_mfma_f32_16x16x4f32; accumulators hold
//         the potential and the three field components for 16 targets x 32
//         vectors.  Each source leaf is accumulated from zero and added to
//         running sums in FP64.
#include <type_traits>

#include "internal.h"
#include "ops.h"

namespace fmm {
namespace {

using namespace ops;
constexpr int kRB = kBatchWidth;

typedef float floatx4 __attribute__((ext_vector_type(4)));

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// s += x, elementwise, s in FP64
__device__ __forceinline__ void add4(double (&s)[4], floatx4 x) {
#pragma unroll
  for (int v = 0; v < 4; ++v) s[v] += double(x[v]);
}

// The sort stage: the caller's charges (vector-major [R][n], input order)
// to leaf order with the 32 vectors innermost ([n][32], zero beyond R), for
// P2M and P2P.  Block = 64 consecutive input indices: their R rows are read
// as 256-byte runs into an LDS tile, then each point's 32 charges go out as
// one 128-byte row at its leaf position (iperm).
__global__ __launch_bounds__(256) void k_bgather(int64_t n, int R,
                                                 const int32_t* __restrict__ iperm,
                                                 const float* __restrict__ q,
                                                 float* __restrict__ qL) {
  __shared__ float T[kRB][64 + 1];
  const int64_t o0 = (int64_t)blockIdx.x * 64;
  for (int e = threadIdx.x; e < kRB * 64; e += blockDim.x) {
    const int r = e / 64, c = e % 64;
    const int64_t o = o0 + c;
    T[r][c] = (r < R && o < n) ? q[(int64_t)r * n + o] : 0.f;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * kRB; e += blockDim.x) {
    const int c = e / kRB, r = e % kRB;
    const int64_t o = o0 + c;
    if (o < n) qL[(int64_t)iperm[o] * kRB + r] = T[r][c];
  }
}

// P2P on the matrix cores (v_mfma_f32_16x16x4f32).  A tile is 16 targets
// (rows) x 32 vectors (columns, two 16-column halves); every step takes four
// source points: lane l computes the kernel entries of target (l % 16) and
// source (l / 16) -- the A operand -- and supplies the charges of source
// (l / 16) for vectors (l % 16) and 16 + (l % 16) -- the B operands of the
// two halves.  Accumulator register v of lane l holds row 4 (l / 16) + v,
// column l % 16 (+16 in the second half).  Source points (positions and the
// 32 charges) are staged in LDS, up to kStage points at a time, with
// coalesced loads.  A block holds TW waves, one 16-target tile each, that
// share every staged chunk.  H: column halves, 1 for up to 16 vectors.  Small
// tiles keep the accumulators to 32 registers per lane; the kernel is held to
// three waves per SIMD (146 registers, no spills), so that the kernel values of
// one wave's next step are computed while another wave's MFMAs run.  Bound by
// issue: the MFMAs take 56% of the SIMDs' cycles and the vector instructions,
// which do not overlap them, the rest.  So the leaf sums go to FP64 running sums
// (two instructions an element; compensated FP32 sums took eight, 16 of the 39
// vector instructions a step) and distance 0 is looked for only in the target
// leaf itself, or everywhere when some points cannot be told apart.  Measured
// (2^18 points, 64 a leaf, theta = 0.8): 32 vectors 1.29 -> 1.20 ms.
constexpr int kStage = 64;

template <int TW, int H>
__global__ __launch_bounds__(64 * TW) __attribute__((amdgpu_waves_per_eu(3))) void k_bp2p(
    const int32_t* __restrict__ leaf_start, const double* __restrict__ xs,
    const double* __restrict__ ys, const double* __restrict__ zs,
    const float* __restrict__ qL, const int32_t* __restrict__ p2p_ptr,
    const int32_t* __restrict__ p2p_src, int dup, float* __restrict__ potL,
    float* __restrict__ fldL) {
  __shared__ double px[kStage], py[kStage], pz[kStage];
  // charge rows padded to 48 floats: the four source rows a step reads sit
  // 16 banks apart, so a half-wave's 32 lanes hit 32 distinct banks
  constexpr int kQS = kRB + 16;
  __shared__ __align__(16) float qs[kStage][kQS];
  const int leaf = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid % 64, wv = tid / 64;
  const int row = lane % 16, kk = lane / 16;
  const int st = leaf_start[leaf], en = leaf_start[leaf + 1];
  const int pb = p2p_ptr[leaf], pe = p2p_ptr[leaf + 1];
  // every wave runs the same number of tiles (barriers inside)
  const int ntile = (en - st + 16 * TW - 1) / (16 * TW);
  for (int tl = 0; tl < ntile; ++tl) {
    const int i0 = st + 16 * (tl * TW + wv);
    const int i = i0 + row;
    const int ii = i < en ? i : st;  // rows past the leaf's end are not stored
    const double xi = xs[ii], yi = ys[ii], zi = zs[ii];
    // running sums for the two column halves (0, 1); each source leaf is
    // accumulated on the matrix cores from zero and then added
    double su0[4] = {}, sx0[4] = {}, sy0[4] = {}, sz0[4] = {};
    double su1[4] = {}, sx1[4] = {}, sy1[4] = {}, sz1[4] = {};
    for (int k = pb; k < pe; ++k) {
      const int sl = p2p_src[k];
      const int js = leaf_start[sl], je = leaf_start[sl + 1];
      const bool safe = dup || sl == leaf;
      floatx4 au0 = {}, ax0 = {}, ay0 = {}, az0 = {}, au1 = {}, ax1 = {}, ay1 = {}, az1 = {};
      for (int c0 = js; c0 < je; c0 += kStage) {
        const int cnt = min(kStage, je - c0);
        __syncthreads();  // the previous chunk's reads are done
        if (tid < cnt) {
          px[tid] = xs[c0 + tid];
          py[tid] = ys[c0 + tid];
          pz[tid] = zs[c0 + tid];
        }
        {
          const float4* from = reinterpret_cast<const float4*>(qL + (int64_t)c0 * kRB);
          for (int e = tid; e < cnt * (kRB / 4); e += 64 * TW)
            *reinterpret_cast<float4*>(&qs[e / (kRB / 4)][4 * (e % (kRB / 4))]) = from[e];
        }
        __syncthreads();
        // one step: four source points j0 .. j0+3 (lane group kk takes j0+kk)
        // CHECK: some of them may be past the chunk; SAFE: pairs at distance 0
        // contribute nothing (otherwise the pairs are known to be apart)
        auto step = [&](int j0, auto check_tag, auto safe_tag) {
          constexpr bool CHECK = decltype(check_tag)::value;
          constexpr bool SAFE = decltype(safe_tag)::value;
          const int j = j0 + kk;
          const bool live_j = !CHECK || j < cnt;
          const int jj = CHECK ? (live_j ? j : 0) : j;
          const float dx = float(xi - px[jj]), dy = float(yi - py[jj]), dz = float(zi - pz[jj]);
          const float r2 = dx * dx + dy * dy + dz * dz;
          const float inv0 = __builtin_amdgcn_rsqf(r2);
          const float inv = !SAFE || (r2 > 0.f && live_j) ? inv0 : 0.f;
          const float inv3 = inv * inv * inv;
          const float q0 = qs[jj][row], q1 = H == 2 ? qs[jj][16 + row] : 0.f;
          const float b0 = live_j ? q0 : 0.f;
          const float b1 = live_j ? q1 : 0.f;
          const float ex = dx * inv3, ey = dy * inv3, ez = dz * inv3;
          au0 = __builtin_amdgcn_mfma_f32_16x16x4f32(inv, b0, au0, 0, 0, 0);
          if (H == 2) au1 = __builtin_amdgcn_mfma_f32_16x16x4f32(inv, b1, au1, 0, 0, 0);
          ax0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ex, b0, ax0, 0, 0, 0);
          if (H == 2) ax1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ex, b1, ax1, 0, 0, 0);
          ay0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ey, b0, ay0, 0, 0, 0);
          if (H == 2) ay1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ey, b1, ay1, 0, 0, 0);
          az0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ez, b0, az0, 0, 0, 0);
          if (H == 2) az1 = __builtin_amdgcn_mfma_f32_16x16x4f32(ez, b1, az1, 0, 0, 0);
        };
        int j0 = 0;
        auto full = [&](auto safe_tag) {
          for (; j0 + 16 <= cnt; j0 += 16) {
#pragma unroll
            for (int u = 0; u < 4; ++u) step(j0 + 4 * u, std::false_type{}, safe_tag);
          }
        };
        if (safe)
          full(std::true_type{});
        else
          full(std::false_type{});
        for (; j0 < cnt; j0 += 4) step(j0, std::true_type{}, std::true_type{});
      }
      add4(su0, au0);
      add4(sx0, ax0);
      add4(sy0, ay0);
      add4(sz0, az0);
      if (H == 2) add4(su1, au1);
      if (H == 2) add4(sx1, ax1);
      if (H == 2) add4(sy1, ay1);
      if (H == 2) add4(sz1, az1);
    }
    const float c = float(kInv4Pi);
#pragma unroll
    for (int hf = 0; hf < H; ++hf) {
      const int col = 16 * hf + row;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int ti = i0 + 4 * kk + v;
        if (ti < en) {
          const int64_t o = ti;
          potL[o * kRB + col] -= c * float(hf ? su1[v] : su0[v]);
          // field = -grad u; grad of the near part is +(1/4pi) sum q d/r^3
          fldL[(o * 3 + 0) * kRB + col] -= c * float(hf ? sx1[v] : sx0[v]);
          fldL[(o * 3 + 1) * kRB + col] -= c * float(hf ? sy1[v] : sy0[v]);
          fldL[(o * 3 + 2) * kRB + col] -= c * float(hf ? sz1[v] : sz0[v]);
        }
      }
    }
  }
}

// Leaf-ordered [n][32] results to the caller's [R][n] and [R][n][3].
// Block = 64 consecutive output (input-order) indices: each point's
// 32-vector rows are read as 128-byte runs from its leaf position (iperm)
// into LDS tiles, then every vector's outputs for the 64 points go out as
// contiguous runs (256 bytes of potential, 768 bytes of field).
__global__ __launch_bounds__(256) void k_bscatter(int64_t n, int R,
                                                  const int32_t* __restrict__ iperm,
                                                  const float* __restrict__ potL,
                                                  const float* __restrict__ fldL,
                                                  float* __restrict__ pot,
                                                  float* __restrict__ field) {
  __shared__ float U[64][kRB + 1];
  __shared__ float F[3 * 64][kRB + 1];
  const int64_t o0 = (int64_t)blockIdx.x * 64;
  for (int e = threadIdx.x; e < 64 * kRB; e += blockDim.x) {
    const int c = e / kRB, r = e % kRB;
    const int64_t o = o0 + c;
    U[c][r] = o < n ? potL[(int64_t)iperm[o] * kRB + r] : 0.f;
  }
  if (field)
    for (int e = threadIdx.x; e < 3 * 64 * kRB; e += blockDim.x) {
      const int ca = e / kRB, r = e % kRB;
      const int64_t o = o0 + ca / 3;
      F[ca][r] = o < n ? fldL[((int64_t)iperm[o] * 3 + ca % 3) * kRB + r] : 0.f;
    }
  __syncthreads();
  for (int e = threadIdx.x; e < kRB * 64; e += blockDim.x) {
    const int r = e / 64, c = e % 64;
    if (r < R && o0 + c < n) pot[(int64_t)r * n + o0 + c] = U[c][r];
  }
  if (field)
    for (int e = threadIdx.x; e < kRB * 3 * 64; e += blockDim.x) {
      const int r = e / (3 * 64), ca = e % (3 * 64);
      if (r < R && o0 + ca / 3 < n) field[((int64_t)r * n + o0) * 3 + ca] = F[ca][r];
    }
}

// iperm[perm[j]] = j: leaf position of every input index
__global__ void k_invert(int64_t n, const int32_t* __restrict__ perm, int32_t* __restrict__ iperm) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) iperm[perm[j]] = (int32_t)j;
}

}  // namespace

int batch_width() { return kRB; }

int batch_p2p_waves(const fmm_plan* pl) {
  const int w = pl->batch_p2p_waves;
  if (w == 1 || w == 2 || w == 4 || w == 8) return w;
  const int mlc = pl->max_leaf_count;
  return mlc > 64 ? 8 : (mlc > 32 ? 4 : (mlc > 16 ? 2 : 1));
}

void make_iperm(fmm_plan* pl, hipStream_t st) {
  k_invert<<<blocks(pl->n, 256), 256, 0, st>>>(pl->n, pl->perm, pl->iperm);
  FMM_HIP(hipGetLastError());
}

void batch_gather(const fmm_plan* pl, const float* q, int R, float* qL, hipStream_t st) {
  k_bgather<<<blocks(pl->n, 64), 256, 0, st>>>(pl->n, R, pl->iperm, q, qL);
}

void batch_near(const fmm_plan* pl, const ListSet& Ls, int R, const float* qL, float* potL,
                float* fldL, hipStream_t st) {
  const int TW = batch_p2p_waves(pl);
  auto p2p = [&](auto kern, int tw) {
    kern<<<(unsigned)pl->nleaf, 64 * tw, 0, st>>>(pl->leaf_start, pl->xs, pl->ys, pl->zs, qL,
                                                   Ls.p2p_ptr, Ls.p2p_src, pl->has_dup ? 1 : 0,
                                                   potL, fldL);
  };
  auto all = [&](auto halves) {
    constexpr int H = decltype(halves)::value;
    if (TW == 1) p2p(k_bp2p<1, H>, 1);
    else if (TW == 2) p2p(k_bp2p<2, H>, 2);
    else if (TW == 4) p2p(k_bp2p<4, H>, 4);
    else p2p(k_bp2p<8, H>, 8);
  };
  if (R <= kRB / 2) all(std::integral_constant<int, 1>{});
  else all(std::integral_constant<int, 2>{});
}

void batch_scatter(const fmm_plan* pl, int R, const float* potL, const float* fldL, float* pot,
                   float* field, hipStream_t st) {
  k_bscatter<<<blocks(pl->n, 64), 256, 0, st>>>(pl->n, R, pl->iperm, potL, fldL, pot, field);
}

void evaluate_batch(fmm_plan* pl, int dir, const float* q, int R, float* pot, float* field,
                    hipStream_t st) {
  const ListSet& Ls = pl->lists[dir];
  switch (pl->prm.p) {
#define FMM_CASE(PP)                                   \
  case PP:                                             \
    run_batch<PP>(pl, Ls, q, R, pot, field, st); \
    break;
    FMM_CASE(1) FMM_CASE(2) FMM_CASE(3) FMM_CASE(4) FMM_CASE(5)
    FMM_CASE(6) FMM_CASE(7) FMM_CASE(8) FMM_CASE(9) FMM_CASE(10)
#undef FMM_CASE
    default:
      throw Error{FMM_ENOTSUP, "expansion order without compiled kernels"};
  }
}

}  // namespace fmm
