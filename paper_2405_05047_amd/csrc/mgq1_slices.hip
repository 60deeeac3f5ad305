// The slice kernels of the sliced-ELL operators for one block size (MGQ1_B), compiled as one
// object per size: SpMV / defect, smoothing sweep, first sweep from zero, and for one
// component the fused first two sweeps.
#include "mgq1_device.h"

namespace mgq1 {
namespace {

// ------------------------------------------------------------------ grid kernels
// NORM: per-block partial sums of out * out
template <int B, int K, class XI, class XO, class T, int MODE, bool NORM, int KB, bool C16>
__global__ __launch_bounds__(kThreads) void k_spmv(SellDev A, const XO* __restrict__ b, const XI* __restrict__ x,
                                                   XO* __restrict__ y, const uint8_t* __restrict__ mask,
                                                   double* __restrict__ partials) {
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const SliceLane s = slice_lane<B, 1>(A, bid * kSliceWaves + threadIdx.x / kWave, threadIdx.x % kWave);
  const T out = spmv_slice<B, 1, K, XI, XO, T, MODE, KB, C16>(A, b, x, y, mask, s);
  if (NORM) {
    __shared__ double lds[kMaxWaves + 1];
    const double p = block_allsum(double(out) * double(out), lds);
    if (threadIdx.x == 0) partials[blockIdx.x] = p;
  }
}

template <int B, int K, class X, class T, int KB, bool C16>
__global__ __launch_bounds__(kThreads) void k_sweep(SellDev A, const X* __restrict__ S, const X* __restrict__ b,
                                                    const X* __restrict__ x, X* __restrict__ xo, T omega,
                                                    T beta, int pmode) {
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const SliceLane s = slice_lane<B, 1>(A, bid * kSliceWaves + threadIdx.x / kWave, threadIdx.x % kWave);
  sweep_slice<B, 1, K, X, T, KB, C16>(A, S, b, x, xo, omega, s, beta, pmode);
}

// two smoothing sweeps from x = 0 in one pass, one component per node:
// x1 = omega S b (formed per column on the fly), x2 = x1 + omega S (b - A x1)
template <int K, class X, class T, int KB, bool C16>
__global__ __launch_bounds__(kThreads) void k_sweep2z(SellDev A, const X* __restrict__ S, const X* __restrict__ b,
                                                      X* __restrict__ xo, T omega) {
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int slice = bid * kSliceWaves + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  const int64_t i = int64_t(slice) * kWave + lane;
  if (slice >= A.nslices || i >= A.n) return;
  const X si = S[i], bi = b[i];              // issued with the slice bounds
  const int su = __builtin_amdgcn_readfirstlane(slice);
  int k, k1;
  slot_range(A, su, k, k1);
  T acc = T(0);
  const int node = int(i);
  const bool wide = C16 && is_wide(A, su);
  if (A.nt) {
    if (wide) sell_loop_z<KB, K, X, T, false, true>(k, k1, A, lane, node, S, b, omega, acc);
    else sell_loop_z<KB, K, X, T, C16, true>(k, k1, A, lane, node, S, b, omega, acc);
  } else {
    if (wide) sell_loop_z<KB, K, X, T, false, false>(k, k1, A, lane, node, S, b, omega, acc);
    else sell_loop_z<KB, K, X, T, C16, false>(k, k1, A, lane, node, S, b, omega, acc);
  }
  if (K == VK_F16 || K == VK_BF16) acc *= T(ldexpf(1.0f, A.rexp[int64_t(slice) * kWave + lane]));
  const X x1 = X(omega * (T(0) + T(si) * T(bi)));
  const T res = T(bi) - acc;
  const T upd = T(0) + T(si) * res;
  xo[i] = X(T(x1) + omega * upd);
}

template <int B, class X, class T>
__global__ __launch_bounds__(kThreads) void k_sweep0(SellDev A, const X* __restrict__ S, const X* __restrict__ b,
                                                     X* __restrict__ xo, T omega) {
  const SliceLane s = slice_lane<B, 1>(A, blockIdx.x * kSliceWaves + threadIdx.x / kWave, threadIdx.x % kWave);
  sweep0_slice<B, 1, X, T>(S, b, xo, omega, s);
}


template <int B, int K, class XI, class XO, class T>
hipError_t spmv_t(const SellDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int mode,
                  double* partials, hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  if (g == 0) return hipSuccess;
  const XO* bb = static_cast<const XO*>(b);
  const XI* xx = static_cast<const XI*>(x);
  XO* yy = static_cast<XO*>(y);
  // slot batch and column format are runtime properties of the operator
#define MGQ1_SPMV4(MODE, NORM, KB, C16)                                                                     \
  hipLaunchKernelGGL((k_spmv<B, K, XI, XO, T, MODE, NORM, KB, C16>), g, kThreads, 0, s, A, bb, xx, yy, mask, partials)
#define MGQ1_SPMV(MODE, NORM)                                                             \
  if (A.col16) {                                                                          \
    if (A.kb == kb_alt<B>()) MGQ1_SPMV4(MODE, NORM, kb_alt<B>(), true);                   \
    else MGQ1_SPMV4(MODE, NORM, kb_default<B>(), true);                                   \
  } else {                                                                                \
    if (A.kb == kb_alt<B>()) MGQ1_SPMV4(MODE, NORM, kb_alt<B>(), false);                  \
    else MGQ1_SPMV4(MODE, NORM, kb_default<B>(), false);                                  \
  }
  // the combinations the library uses: y = Ax, b - Ax with or without norm partials,
  // masked defect
  if (mode == 0 && !partials) MGQ1_SPMV(0, false)
  else if (mode == 1 && partials) MGQ1_SPMV(1, true)
  else if (mode == 1) MGQ1_SPMV(1, false)
  else if (mode == 2 && !partials) MGQ1_SPMV(2, false)
  else return hipErrorInvalidValue;
#undef MGQ1_SPMV4
#undef MGQ1_SPMV
  return hipGetLastError();
}

}  // namespace

template <int B>
hipError_t spmv_block(const SellDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int xk, int yk,
                  int mode, double* partials, hipStream_t s) {
  if (A.kind == VK_F64) {
    if (xk == X_F64 && yk == X_F64) return spmv_t<B, VK_F64, double, double, double>(A, b, x, y, mask, mode, partials, s);
    if (xk == X_F32 && yk == X_F64) return spmv_t<B, VK_F64, float, double, double>(A, b, x, y, mask, mode, partials, s);
    return hipErrorInvalidValue;
  }
  if (xk != X_F32 || yk != X_F32) return hipErrorInvalidValue;
  switch (A.kind) {
    case VK_F32: return spmv_t<B, VK_F32, float, float, float>(A, b, x, y, mask, mode, partials, s);
    case VK_F16: return spmv_t<B, VK_F16, float, float, float>(A, b, x, y, mask, mode, partials, s);
    case VK_BF16: return spmv_t<B, VK_BF16, float, float, float>(A, b, x, y, mask, mode, partials, s);
    default: return hipErrorInvalidValue;
  }
}

namespace {

template <int B, class X, class T>
hipError_t sweep_t(const SellDev& A, const void* S, const void* b, const void* x, void* xo, double omega,
                   double beta, int pmode, hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  if (g == 0) return hipSuccess;
  const X* SS = static_cast<const X*>(S);
  const X* bb = static_cast<const X*>(b);
  const X* xx = static_cast<const X*>(x);
  X* oo = static_cast<X*>(xo);
#define MGQ1_SWEEP4(KIND, KB, C16) \
  hipLaunchKernelGGL((k_sweep<B, KIND, X, T, KB, C16>), g, kThreads, 0, s, A, SS, bb, xx, oo, T(omega), T(beta), pmode)
#define MGQ1_SWEEP(KIND)                                                   \
  if (A.col16) {                                                           \
    if (A.kb == kb_alt<B>()) MGQ1_SWEEP4(KIND, kb_alt<B>(), true);         \
    else MGQ1_SWEEP4(KIND, kb_default<B>(), true);                         \
  } else {                                                                 \
    if (A.kb == kb_alt<B>()) MGQ1_SWEEP4(KIND, kb_alt<B>(), false);        \
    else MGQ1_SWEEP4(KIND, kb_default<B>(), false);                        \
  }
  // FP64 vectors go with FP64 values only; FP32 vectors with the reduced formats
  if constexpr (sizeof(X) == 8) {
    if (A.kind != VK_F64) return hipErrorInvalidValue;
    MGQ1_SWEEP(VK_F64);
  } else {
    switch (A.kind) {
      case VK_F32: MGQ1_SWEEP(VK_F32); break;
      case VK_F16: MGQ1_SWEEP(VK_F16); break;
      case VK_BF16: MGQ1_SWEEP(VK_BF16); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef MGQ1_SWEEP
#undef MGQ1_SWEEP4
  return hipGetLastError();
}

}  // namespace

template <int B>
hipError_t sweep_block(const SellDev& A, const void* S, const void* b, const void* x, void* xo, double omega,
                       double beta, int pmode, int xk, hipStream_t s) {
  return xk == X_F64 ? sweep_t<B, double, double>(A, S, b, x, xo, omega, beta, pmode, s)
                     : sweep_t<B, float, float>(A, S, b, x, xo, omega, beta, pmode, s);
}

template <int B>
hipError_t sweep0_block(const SellDev& A, const void* S, const void* b, void* xo, double omega, int xk,
                           hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  if (g == 0) return hipSuccess;
  if (xk == X_F64)
    hipLaunchKernelGGL((k_sweep0<B, double, double>), g, kThreads, 0, s, A, static_cast<const double*>(S),
                       static_cast<const double*>(b), static_cast<double*>(xo), omega);
  else
    hipLaunchKernelGGL((k_sweep0<B, float, float>), g, kThreads, 0, s, A, static_cast<const float*>(S),
                       static_cast<const float*>(b), static_cast<float*>(xo), float(omega));
  return hipGetLastError();
}


#if MGQ1_B == 1
hipError_t sweep2z_block(const SellDev& A, const void* S, const void* b, void* xo, double omega, int xk,
                         hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  if (g == 0) return hipSuccess;
#define MGQ1_S2Z4(KIND, X, T, KB, C16)                                                              \
  hipLaunchKernelGGL((k_sweep2z<KIND, X, T, KB, C16>), g, kThreads, 0, s, A, static_cast<const X*>(S), \
                     static_cast<const X*>(b), static_cast<X*>(xo), T(omega))
#define MGQ1_S2Z(KIND, X, T)                                                     \
  if (A.col16) {                                                                 \
    if (A.kb == kb_alt<1>()) MGQ1_S2Z4(KIND, X, T, kb_alt<1>(), true);           \
    else MGQ1_S2Z4(KIND, X, T, kb_default<1>(), true);                           \
  } else {                                                                       \
    if (A.kb == kb_alt<1>()) MGQ1_S2Z4(KIND, X, T, kb_alt<1>(), false);          \
    else MGQ1_S2Z4(KIND, X, T, kb_default<1>(), false);                          \
  }
  if (xk == X_F64) {
    if (A.kind != VK_F64) return hipErrorInvalidValue;
    MGQ1_S2Z(VK_F64, double, double);
  } else {
    switch (A.kind) {
      case VK_F32: MGQ1_S2Z(VK_F32, float, float); break;
      case VK_F16: MGQ1_S2Z(VK_F16, float, float); break;
      case VK_BF16: MGQ1_S2Z(VK_BF16, float, float); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef MGQ1_S2Z
#undef MGQ1_S2Z4
  return hipGetLastError();
}
#endif

template hipError_t spmv_block<MGQ1_B>(const SellDev&, const void*, const void*, void*, const uint8_t*, int, int, int,
                                       double*, hipStream_t);
template hipError_t sweep_block<MGQ1_B>(const SellDev&, const void*, const void*, const void*, void*, double, double,
                                        int, int, hipStream_t);
template hipError_t sweep0_block<MGQ1_B>(const SellDev&, const void*, const void*, void*, double, int, hipStream_t);

}  // namespace mgq1
