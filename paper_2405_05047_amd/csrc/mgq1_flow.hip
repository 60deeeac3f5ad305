// Kernels of the flow form: operators of four components whose blocks all have the shape
//
//     [ pp  pu  pv  pw ]
//     [ up  a   0   0  ]        one scalar field coupled to a vector field whose own block is a
//     [ vp  0   a   0  ]        multiple of the identity (the linearised flow step: pressure
//     [ wp  0   0   a  ]        first, then the velocity; constrained rows keep the shape)
//
// Setup checks every block of the level bit by bit; 8 of the 16 values are then stored.  The
// sweeps and products of these levels are bound by the operator's bytes: 66 instead of 130 per
// block in FP64, 34 instead of 66 in FP32.
//
// One wavefront runs a slice of 32 nodes, two lanes per node: lane r (r < 32) has rows 0 and 1
// of node r, lane 32 + r its rows 2 and 3.  Value v of slot k sits at val[(k * 8 + v) * 32 + r], so
// both halves of the wave read the same lines.  With one lane per node a 274,625-node level is
// 4,291 waves for 4,096 places; two per node halve what the last ones leave idle.  The
// products run in slot and column order with the zeros multiplied too, so every result has
// the bits of the sliced-ELL kernels (and their NaNs).
//
// Measured, sliced ELL and flow form: 274,625 nodes FP64 sweep 161 and 113 us, product 156 and
// 105 us (474 MB of values and columns at 4.5 TB/s), FP32 79 and 48, 75 and 42 us; 68,921 nodes
// FP32 20.5 and 13.4 us.  2 to 6 slots per batch in FP64 are within 2% of each other.
#include "mgq1_device.h"

namespace mgq1 {
namespace {

constexpr int kFlowValues = 8;

struct FlowLane {
  int slice, r, h, pos, node;   // h: 0 for rows 0 and 1, 1 for rows 2 and 3
  bool valid;
};

__device__ __forceinline__ FlowLane flow_lane(const FlowDev& A, int slice, int lane) {
  FlowLane s;
  s.slice = __builtin_amdgcn_readfirstlane(slice);
  s.r = lane & (kFlowNodes - 1);
  s.h = lane / kFlowNodes;
  const int pos = s.slice * kFlowNodes + s.r;
  s.valid = pos < A.n;
  s.pos = s.valid ? pos : A.n - 1;
  s.node = A.perm ? A.perm[s.pos] : s.pos;
  return s;
}

// NB slots: every index and value first, then the gathers, then the multiply-adds
template <int NB, class XI, class T, bool C16, bool NT>
__device__ __forceinline__ void flow_batch(const FlowDev& A, int k, const FlowLane& s, const XI* __restrict__ x,
                                           T (&acc)[2]) {
  const T* val = static_cast<const T*>(A.val);
  unsigned j[NB];
  T a[NB][6];
  XI v[NB][4];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int64_t e = int64_t(k + q) * kFlowNodes + s.r;
    if constexpr (C16) j[q] = unsigned(A.base[k + q]) + unsigned(stream_load<NT>(A.col16 + e));
    else j[q] = unsigned(stream_load<NT>(A.col + e));
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const T* p = val + int64_t(k + q) * (kFlowValues * kFlowNodes) + s.r;
    a[q][0] = stream_load<NT>(p + (s.h ? 5 : 0) * kFlowNodes);
    a[q][1] = stream_load<NT>(p + (s.h ? 6 : 4) * kFlowNodes);
    a[q][2] = stream_load<NT>(p + 7 * kFlowNodes);
    a[q][3] = stream_load<NT>(p + 1 * kFlowNodes);
    a[q][4] = stream_load<NT>(p + 2 * kFlowNodes);
    a[q][5] = stream_load<NT>(p + 3 * kFlowNodes);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const XI* xj = x + uint64_t(j[q]) * 4;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[q][c] = xj[c];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const T z = T(0), d = a[q][2];
    acc[0] += a[q][0] * T(v[q][0]);
    acc[0] += (s.h ? z : a[q][3]) * T(v[q][1]);
    acc[0] += (s.h ? d : a[q][4]) * T(v[q][2]);
    acc[0] += (s.h ? z : a[q][5]) * T(v[q][3]);
    acc[1] += a[q][1] * T(v[q][0]);
    acc[1] += (s.h ? z : d) * T(v[q][1]);
    acc[1] += z * T(v[q][2]);
    acc[1] += (s.h ? d : z) * T(v[q][3]);
  }
}

template <int N, class XI, class T, bool C16, bool NT>
__device__ __forceinline__ void flow_rest(int rem, const FlowDev& A, int k, const FlowLane& s,
                                          const XI* __restrict__ x, T (&acc)[2]) {
  if constexpr (N >= 1) {
    if (rem == N) flow_batch<N, XI, T, C16, NT>(A, k, s, x, acc);
    else flow_rest<N - 1, XI, T, C16, NT>(rem, A, k, s, x, acc);
  }
}

template <class T> constexpr int flow_slots() { return sizeof(T) == 8 ? 4 : 6; }

// the sums of the lane's two rows
template <class XI, class T, bool C16>
__device__ __forceinline__ void flow_dot(const FlowDev& A, const FlowLane& s, const XI* __restrict__ x, T (&acc)[2]) {
  constexpr int KB = flow_slots<T>();
  acc[0] = acc[1] = T(0);
  int k = A.sptr[s.slice];
  const int k1 = A.sptr[s.slice + 1];
  if (A.nt) {
    for (; k + KB <= k1; k += KB) flow_batch<KB, XI, T, C16, true>(A, k, s, x, acc);
    flow_rest<KB - 1, XI, T, C16, true>(k1 - k, A, k, s, x, acc);
  } else {
    for (; k + KB <= k1; k += KB) flow_batch<KB, XI, T, C16, false>(A, k, s, x, acc);
    flow_rest<KB - 1, XI, T, C16, false>(k1 - k, A, k, s, x, acc);
  }
}

// y = A x (MODE 0), b - A x (MODE 1), M (b - A x) (MODE 2); NORM: partial sums of squares
template <class XI, class XO, int MODE, bool NORM, bool C16>
__global__ __launch_bounds__(kThreads) void k_flow_spmv(FlowDev A, const XO* __restrict__ b, const XI* __restrict__ x,
                                                        XO* __restrict__ y, const uint8_t* __restrict__ mask,
                                                        double* __restrict__ partials) {
  using T = XO;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int slice = bid * kSliceWaves + int(threadIdx.x) / kWave;
  double sq = 0.0;
  if (slice < A.nslices) {
    const FlowLane s = flow_lane(A, slice, int(threadIdx.x) % kWave);
    const int64_t d0 = int64_t(s.node) * 4 + 2 * s.h;
    XO bv[2] = {XO(0), XO(0)};
    uint8_t mk[2] = {0, 0};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      if (MODE != 0) bv[c] = b[d0 + c];
      if (MODE == 2) mk[c] = mask[d0 + c];
    }
    T acc[2];
    flow_dot<XI, T, C16>(A, s, x, acc);
    if (s.valid) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        T out = MODE == 0 ? acc[c] : T(bv[c]) - acc[c];
        if (MODE == 2 && mk[c]) out = T(0);
        y[d0 + c] = XO(out);
        if (NORM) sq += double(out) * double(out);
      }
    }
  }
  if (NORM) {
    __shared__ double lds[kMaxWaves + 1];
    const double p = block_allsum(sq, lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = p;
  }
}

// the smoother rows of the lane: S[(slice * 8 + 4 a + cc) * 64 + lane], a = 0, 1
template <class X>
__device__ __forceinline__ void flow_smoother(const FlowDev& A, int slice, int lane, X (&sv)[2][4]) {
  const X* S = static_cast<const X*>(A.S);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) sv[a][cc] = S[(int64_t(slice) * 8 + 4 * a + cc) * kWave + lane];
}

// row sums of the smoother over the node's four residuals, two in each half of the wave
template <class X, class T>
__device__ __forceinline__ void flow_apply(const X (&sv)[2][4], const T (&res)[2], int h, T (&upd)[2]) {
  T o[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) o[c] = __shfl_xor(res[c], kFlowNodes, kWave);
  const T r0 = h ? o[0] : res[0], r1 = h ? o[1] : res[1], r2 = h ? res[0] : o[0], r3 = h ? res[1] : o[1];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    upd[a] = T(0);
    upd[a] += T(sv[a][0]) * r0;
    upd[a] += T(sv[a][1]) * r1;
    upd[a] += T(sv[a][2]) * r2;
    upd[a] += T(sv[a][3]) * r3;
  }
}

// x_out = x + omega S (b - A x), and the three-term (Chebyshev) form as in sweep_slice
template <class X, bool C16>
__global__ __launch_bounds__(kThreads) void k_flow_sweep(FlowDev A, const X* __restrict__ b, const X* __restrict__ x,
                                                         X* xo, X omega, X beta, int pmode) {
  using T = X;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int slice = bid * kSliceWaves + int(threadIdx.x) / kWave;
  const int lane = int(threadIdx.x) % kWave;
  if (slice >= A.nslices) return;
  const FlowLane s = flow_lane(A, slice, lane);
  const int64_t d0 = int64_t(s.node) * 4 + 2 * s.h;
  const X* pp = pmode == 1 ? static_cast<const X*>(xo) : x;
  X bv[2], xv[2], pv[2], sv[2][4];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    bv[c] = b[d0 + c];
    xv[c] = x[d0 + c];
    pv[c] = pp[d0 + c];
  }
  flow_smoother<X>(A, s.slice, lane, sv);
  T acc[2], res[2], upd[2];
  flow_dot<X, T, C16>(A, s, x, acc);
#pragma unroll
  for (int c = 0; c < 2; ++c) res[c] = T(bv[c]) - acc[c];
  flow_apply<X, T>(sv, res, s.h, upd);
  if (!s.valid) return;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    T nx = T(xv[c]) + omega * upd[c];
    if (pmode != 0) nx = nx + beta * (T(xv[c]) - (pmode == 1 ? T(pv[c]) : T(0)));
    xo[d0 + c] = X(nx);
  }
}

// x_out = omega S b
template <class X>
__global__ __launch_bounds__(kThreads) void k_flow_sweep0(FlowDev A, const X* __restrict__ b, X* __restrict__ xo,
                                                          X omega) {
  using T = X;
  const int slice = int(blockIdx.x) * kSliceWaves + int(threadIdx.x) / kWave;
  const int lane = int(threadIdx.x) % kWave;
  if (slice >= A.nslices) return;
  const FlowLane s = flow_lane(A, slice, lane);
  const int64_t d0 = int64_t(s.node) * 4 + 2 * s.h;
  X sv[2][4];
  flow_smoother<X>(A, s.slice, lane, sv);
  const T res[2] = {T(b[d0]), T(b[d0 + 1])};
  T upd[2];
  flow_apply<X, T>(sv, res, s.h, upd);
  if (!s.valid) return;
#pragma unroll
  for (int c = 0; c < 2; ++c) xo[d0 + c] = X(omega * upd[c]);
}

// S in the lanes' layout from one 4 x 4 block per row position
template <class X>
__global__ __launch_bounds__(256) void k_flow_smoother(int n, int nslices, const X* __restrict__ blocks,
                                                       X* __restrict__ S) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (t >= int64_t(nslices) * 8 * kWave) return;
  const int lane = int(t % kWave), z = int(t / kWave % 8);
  const int64_t pos = t / (8 * kWave) * kFlowNodes + (lane & (kFlowNodes - 1));
  const int row = 2 * (lane / kFlowNodes) + z / 4;
  S[t] = pos < n ? blocks[pos * 16 + row * 4 + z % 4] : X(0);
}

template <class XI, class XO>
hipError_t flow_spmv_t(const FlowDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int mode,
                       double* partials, hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  const XO* bb = static_cast<const XO*>(b);
  const XI* xx = static_cast<const XI*>(x);
  XO* yy = static_cast<XO*>(y);
#define MGQ1_FS(MODE, NORM)                                                                                              \
  if (A.col16) hipLaunchKernelGGL((k_flow_spmv<XI, XO, MODE, NORM, true>), g, kThreads, 0, s, A, bb, xx, yy, mask, partials); \
  else hipLaunchKernelGGL((k_flow_spmv<XI, XO, MODE, NORM, false>), g, kThreads, 0, s, A, bb, xx, yy, mask, partials);
  if (mode == 0 && !partials) { MGQ1_FS(0, false) }
  else if (mode == 1 && partials) { MGQ1_FS(1, true) }
  else if (mode == 1) { MGQ1_FS(1, false) }
  else if (mode == 2 && !partials) { MGQ1_FS(2, false) }
  else return hipErrorInvalidValue;
#undef MGQ1_FS
  return hipGetLastError();
}

template <class X>
hipError_t flow_sweep_t(const FlowDev& A, const void* b, const void* x, void* xo, double omega, double beta, int pmode,
                        hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  const X *bb = static_cast<const X*>(b), *xx = static_cast<const X*>(x);
  X* oo = static_cast<X*>(xo);
  if (A.col16) hipLaunchKernelGGL((k_flow_sweep<X, true>), g, kThreads, 0, s, A, bb, xx, oo, X(omega), X(beta), pmode);
  else hipLaunchKernelGGL((k_flow_sweep<X, false>), g, kThreads, 0, s, A, bb, xx, oo, X(omega), X(beta), pmode);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_flow_spmv(const FlowDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int xk,
                            int yk, int mode, double* partials, hipStream_t s) {
  if (A.tk != yk) return hipErrorInvalidValue;
  if (xk == X_F64 && yk == X_F64) return flow_spmv_t<double, double>(A, b, x, y, mask, mode, partials, s);
  if (xk == X_F32 && yk == X_F64) return flow_spmv_t<float, double>(A, b, x, y, mask, mode, partials, s);
  if (xk == X_F32 && yk == X_F32) return flow_spmv_t<float, float>(A, b, x, y, mask, mode, partials, s);
  return hipErrorInvalidValue;
}

hipError_t launch_flow_sweep(const FlowDev& A, const void* b, const void* x, void* xo, double omega, int xk,
                             hipStream_t s, double beta, int pmode) {
  if (A.tk != xk) return hipErrorInvalidValue;
  return xk == X_F64 ? flow_sweep_t<double>(A, b, x, xo, omega, beta, pmode, s)
                     : flow_sweep_t<float>(A, b, x, xo, omega, beta, pmode, s);
}

hipError_t launch_flow_sweep0(const FlowDev& A, const void* b, void* xo, double omega, int xk, hipStream_t s) {
  if (A.tk != xk) return hipErrorInvalidValue;
  const unsigned g = slice_grid(A.nslices);
  if (xk == X_F64)
    hipLaunchKernelGGL(k_flow_sweep0<double>, g, kThreads, 0, s, A, static_cast<const double*>(b), static_cast<double*>(xo), omega);
  else
    hipLaunchKernelGGL(k_flow_sweep0<float>, g, kThreads, 0, s, A, static_cast<const float*>(b), static_cast<float*>(xo), float(omega));
  return hipGetLastError();
}

hipError_t launch_flow_smoother(int n, int nslices, const void* blocks, void* S, int sk, hipStream_t s) {
  const unsigned g = grid_for(int64_t(nslices) * 8 * kWave, 256);
  if (sk == X_F64)
    hipLaunchKernelGGL(k_flow_smoother<double>, g, 256, 0, s, n, nslices, static_cast<const double*>(blocks), static_cast<double*>(S));
  else
    hipLaunchKernelGGL(k_flow_smoother<float>, g, 256, 0, s, n, nslices, static_cast<const float*>(blocks), static_cast<float*>(S));
  return hipGetLastError();
}

}  // namespace mgq1
