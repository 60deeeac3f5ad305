// Gram-Schmidt of the FGMRES step (Sec. 4.2) in two passes over the basis.
//
// Modified Gram-Schmidt subtracts one projection after the other: h_i = (w, v_i) of the w
// that has lost h_0 v_0 .. h_{i-1} v_{i-1}.  With d_i = (w, v_i) of the undiminished w and
// the Gram entries G_ik = (v_i, v_k) that is h_i = d_i - sum_{k<i} G_ik h_k (the
// inverse-compact-WY form of MGS: Swirydowicz, Langou, Ananthan, Yang, Thomas, "Low
// synchronization Gram-Schmidt and generalized minimal residual algorithms", Numer. Linear
// Algebra Appl. 28, 2021), so every dot product of a step can be formed in one pass:
//
//   k_gs_dots     partial sums of d_i = (w, v_i) and of the new Gram row G_ji = (v_j, v_i)
//   k_gs_update   every block adds the partials up in a fixed order, solves for h by the
//                 forward substitution (one wave, lane i = row i), w -= sum_i h_i v_i in the
//                 order of i, and the partial sums of (w, w)
//
// Both are bound by the bytes of the basis (one multiply-add per 4 to 8 bytes) or, for short
// vectors, by launches.  Step j moves 2 (j + 1) + 3 vectors in two launches where one kernel
// per projection moved 4 (j + 1) in j + 1.  Whole solves, before and after: 70,785 unknowns
// (57 cycles a step) 17.6 -> 15.2 ms, 1.0M unknowns 4.66 -> 4.48 ms, 6.4M unknowns (51 MB a
// vector) 62.7 -> 61.7 ms.
#include "mgq1_device.h"

namespace mgq1 {
namespace {

constexpr int kGsMaxBlocks = 256;          // partial sums per dot product: one block per CU

// Partial sums of the NV dot products (w, v_i) (rows 0 .. NV-1 of the group's output) and
// (v_j, v_i) (rows NV .. 2 NV - 1), v_i = V + i * ldv for the group's NV vectors, row q of
// block blk at out[q * gridDim.x + blk].  OWN: v_j is the group's last vector.
template <int NV, bool OWN>
__global__ __launch_bounds__(kRedThreads) void k_gs_dots(int64_t n, const double* __restrict__ w,
                                                         const double* __restrict__ V, int64_t ldv,
                                                         const double* __restrict__ vj, double* __restrict__ out) {
  constexpr int NQ = 2 * NV, P = pow2_above(NQ);
  __shared__ double lds[kMaxWaves][NQ];
  double acc[P];
#pragma unroll
  for (int q = 0; q < P; ++q) acc[q] = 0.0;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride) {
    const double wv = w[i];
    double v[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = V[int64_t(q) * ldv + i];
    const double u = OWN ? v[NV - 1] : vj[i];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      acc[q] += wv * v[q];
      acc[NV + q] += u * v[q];
    }
  }
  const int lane = int(threadIdx.x) % kWave, wv = int(threadIdx.x) / kWave;
  int which = 0;
  wave_sums_step<P, kWave / 2, 1>(acc, lane, which);
  if (which < NQ) lds[wv][which] = acc[0];   // several lanes may hold the same sum
  __syncthreads();
  if (int(threadIdx.x) < NQ) {
    double t = 0.0;
    for (int k = 0; k < int(blockDim.x) / kWave; ++k) t += lds[k][threadIdx.x];
    out[int64_t(threadIdx.x) * gridDim.x + blockIdx.x] = t;
  }
}

// The coefficients h_0 .. h_j from the partials of k_gs_dots (gd of them per sum): d_i and the
// new Gram row (v_j, v_k) are added up by the block's waves, older Gram entries come from
// gram[k * 64 + i] = (v_i, v_k), i < j.  On return sh[i] = h_i for every thread; block 0
// stores h in hout and the new Gram row.  Sum q of group g (vectors g * group ..) sits at
// row 2 * g * group + q (its d's) and behind them its Gram entries.
__device__ __forceinline__ void gs_solve(int j, int group, const double* __restrict__ partials, int gd,
                                         double* __restrict__ gram, double* __restrict__ hout, bool store,
                                         double* sd, double* sg, double* sh) {
  const int lane = int(threadIdx.x) % kWave, wv = int(threadIdx.x) / kWave, nw = int(blockDim.x) / kWave;
  const int nq = 2 * (j + 1);
  for (int q = wv; q < nq; q += nw) {
    // vector i of the step, d (kind 0) or Gram entry (kind 1)
    const int g0 = (q / (2 * group)) * group, in = q - 2 * g0;
    const int gn = min(group, j + 1 - g0);
    const int kind = in >= gn ? 1 : 0, i = g0 + in - kind * gn;
    constexpr int U = kGsMaxBlocks / kWave;  // gd <= kGsMaxBlocks: every load at once
    double p[U], t = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) p[u] = lane + u * kWave < gd ? partials[int64_t(q) * gd + lane + u * kWave] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) t += p[u];
    t = wave_sum(t);
    if (lane == 0) (kind ? sg : sd)[i] = t;
  }
  __syncthreads();
  if (wv == 0) {
    double x = lane <= j ? sd[lane] : 0.0;
    for (int k = 0; k < j; ++k) {
      // row j's entries are this step's sums; the others were stored by their own steps
      const double gk = lane == j ? sg[k] : (lane > k && lane < j ? gram[k * kWave + lane] : 0.0);
      const double hk = __shfl(x, k, kWave);
      if (lane > k && lane <= j) x -= gk * hk;
    }
    if (lane <= j) {
      sh[lane] = x;
      if (store) {
        hout[lane] = x;
        if (lane < j) gram[lane * kWave + j] = sg[lane];
      }
    }
  }
  __syncthreads();
}

// h alone, for steps whose vectors take more than one group
__global__ __launch_bounds__(kRedThreads) void k_gs_solve(int j, int group, const double* __restrict__ partials, int gd,
                                                          double* __restrict__ gram, double* __restrict__ hout) {
  __shared__ double sd[kWave], sg[kWave], sh[kWave];
  gs_solve(j, group, partials, gd, gram, hout, true, sd, sg, sh);
}

// w -= sum_i h_i v_i over the group's NV vectors in the order of i, and the partial sums of
// (w, w) (used of the last group).  SOLVE: the step's vectors are this one group and h is
// formed here from the partials of k_gs_dots; else it is read from h.
template <int NV, bool SOLVE>
__global__ __launch_bounds__(kRedThreads) void k_gs_update(int64_t n, double* __restrict__ w,
                                                           const double* __restrict__ V, int64_t ldv,
                                                           const double* __restrict__ partials, int gd,
                                                           double* gram, double* h, double* __restrict__ pout) {
  __shared__ double lds[kMaxWaves + 1];
  __shared__ double sd[kWave], sg[kWave], sh[kWave];
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  const int64_t first = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  double wv = 0.0, v[NV];
  auto load = [&](int64_t i) {
    wv = w[i];
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = V[int64_t(q) * ldv + i];
  };
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = 0.0;
  // the first elements do not depend on h: their loads overlap the sums
  if (first < n) load(first);
  double c[NV];
  if constexpr (SOLVE) {
    gs_solve(NV - 1, NV, partials, gd, gram, h, blockIdx.x == 0, sd, sg, sh);
#pragma unroll
    for (int q = 0; q < NV; ++q) c[q] = sh[q];
  } else {
#pragma unroll
    for (int q = 0; q < NV; ++q) c[q] = h[q];
  }
  double t = 0.0;
  for (int64_t i = first; i < n; i += stride) {
    if (i != first) load(i);
    double r = wv;
#pragma unroll
    for (int q = 0; q < NV; ++q) r = r - c[q] * v[q];
    w[i] = r;
    t += r * r;
  }
  const double s = block_allsum(t, lds);
  if (threadIdx.x == 0) pout[blockIdx.x] = s;
}

template <int NV>
hipError_t gs_dots_n(int nv, int64_t n, const double* w, const double* V, const double* vj, double* out, unsigned g,
                     unsigned threads, hipStream_t s) {
  if constexpr (NV >= 1) {
    if (nv != NV) return gs_dots_n<NV - 1>(nv, n, w, V, vj, out, g, threads, s);
    if (vj == V + int64_t(NV - 1) * n)
      hipLaunchKernelGGL((k_gs_dots<NV, true>), g, threads, 0, s, n, w, V, n, vj, out);
    else
      hipLaunchKernelGGL((k_gs_dots<NV, false>), g, threads, 0, s, n, w, V, n, vj, out);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <int NV, bool SOLVE>
hipError_t gs_update_n(int nv, int64_t n, double* w, const double* V, const double* partials, int gd, double* gram,
                       double* h, double* pout, unsigned g, hipStream_t s) {
  if constexpr (NV >= 1) {
    if (nv != NV) return gs_update_n<NV - 1, SOLVE>(nv, n, w, V, partials, gd, gram, h, pout, g, s);
    hipLaunchKernelGGL((k_gs_update<NV, SOLVE>), g, kRedThreads, 0, s, n, w, V, n, partials, gd, gram, h, pout);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

// Threads per block of the dot products: 256 while 256 such blocks take the vector with a
// few elements per thread, so that a short vector spreads over as many CUs as it can; 1024
// above.
unsigned gs_dot_threads(int64_t n) { return n <= int64_t(kGsMaxBlocks) * 1024 ? 256u : unsigned(kRedThreads); }

unsigned gs_dot_blocks(int64_t n) {
  const unsigned g = grid_for(n, int(gs_dot_threads(n)));
  return g > unsigned(kGsMaxBlocks) ? unsigned(kGsMaxBlocks) : (g ? g : 1u);
}

// the update's 16 waves share the sums of its prologue; two blocks per CU
unsigned gs_update_blocks(int64_t n) {
  const unsigned g = grid_for(n, kRedThreads);
  return g > 2u * kGsMaxBlocks ? 2u * kGsMaxBlocks : (g ? g : 1u);
}

}  // namespace

int64_t gs_partials_size(int m) { return int64_t(2) * m * kGsMaxBlocks; }

hipError_t launch_gram_schmidt(int64_t n, int j, double* w, const double* V, double* partials, double* gram,
                               double* h, double* pnorm, int* gnorm, hipStream_t s) {
  const unsigned th = gs_dot_threads(n), gd = gs_dot_blocks(n), gu = gs_update_blocks(n);
  *gnorm = int(gu);
  hipError_t e;
  const int nv = j + 1;
  const double* vj = V + int64_t(j) * n;
  for (int i = 0; i < nv; i += kGsGroup)
    if ((e = gs_dots_n<kGsGroup>(nv - i < kGsGroup ? nv - i : kGsGroup, n, w, V + int64_t(i) * n, vj,
                                 partials + int64_t(2) * i * gd, gd, th, s)) != hipSuccess)
      return e;
  if (nv <= kGsGroup) return gs_update_n<kGsGroup, true>(nv, n, w, V, partials, int(gd), gram, h, pnorm, gu, s);
  hipLaunchKernelGGL(k_gs_solve, 1, kRedThreads, 0, s, j, kGsGroup, partials, int(gd), gram, h);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int i = 0; i < nv; i += kGsGroup)
    if ((e = gs_update_n<kGsGroup, false>(nv - i < kGsGroup ? nv - i : kGsGroup, n, w, V + int64_t(i) * n, partials,
                                          int(gd), gram, h + i, pnorm, gu, s)) != hipSuccess)
      return e;
  return hipSuccess;
}

}  // namespace mgq1
