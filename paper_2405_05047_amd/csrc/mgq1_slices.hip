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
  dict_stage<K>(A);
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const SliceLane s = slice_lane<B>(A, bid * kSliceWaves + threadIdx.x / kWave, threadIdx.x % kWave);
  const T out = spmv_slice<B, K, XI, XO, T, MODE, KB, C16>(A, b, x, y, mask, s);
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
  dict_stage<K>(A);
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const SliceLane s = slice_lane<B>(A, bid * kSliceWaves + threadIdx.x / kWave, threadIdx.x % kWave);
  sweep_slice<B, K, X, T, KB, C16>(A, S, b, x, xo, omega, s, beta, pmode);
}

// ------------------------------------------------------------------ relay form
// One slice per workgroup: its four waves take a quarter of the slots each, read them all at once
// (one chain of dependent reads instead of one per batch of slots), and pass the row sums on
// in slot order through LDS, so the multiply-adds run in the order of the other kernels and
// give the same bits.  For levels whose slices do not fill the chip and whose rows are long:
// a 27-block row is 4 to 7 batches of two dependent reads each in one wave, and the kernel
// lasts as long as that chain.
constexpr int kRelayBatch = 8;        // slots per wave and round: 32 slots a round

// this wave's slots k .. k + cnt - 1 (cnt <= kRelayBatch, wave-uniform)
template <int B, int K, class XI, bool C16>
__device__ __forceinline__ void relay_load(const SellDev& A, int k, int cnt, int r, int rl, const XI* __restrict__ x,
                                           typename Val<K>::raw (&av)[kRelayBatch][B], XI (&xv)[kRelayBatch][B]) {
  constexpr int R = kWave / B;
  unsigned js[kRelayBatch];
#pragma unroll
  for (int q = 0; q < kRelayBatch; ++q) {
    const int kk = k + (q < cnt ? q : cnt - 1);
    js[q] = slot_col<C16, false>(A, kk, int64_t(kk) * R + r);
#pragma unroll
    for (int cc = 0; cc < B; ++cc) av[q][cc] = Val<K>::template load<false>(A.val, (int64_t(kk) * B + cc) * kWave + rl);
  }
  __builtin_amdgcn_sched_barrier(0);
  // every lane reads all B components of its neighbours (a level this small has read slots to
  // spare; exchanging them between the node's lanes would add a trip through LDS)
#pragma unroll
  for (int q = 0; q < kRelayBatch; ++q)
#pragma unroll
    for (int cc = 0; cc < B; ++cc) xv[q][cc] = x[uint64_t(js[q]) * B + cc];
  __builtin_amdgcn_sched_barrier(0);
}

// the row sums of slice s, valid in the last wave
template <int B, int K, class XI, class T, bool C16>
__device__ __forceinline__ T relay_dot(const SellDev& A, const SliceLane& s, const XI* __restrict__ x) {
  __shared__ T sums[kWave];
  constexpr int R = kWave / B;
  const int lane = s.lane, w = int(threadIdx.x) / kWave;
  // lanes past the last row of the slice read a row that exists
  const int r = lane / B < R ? lane / B : R - 1;
  const int rl = lane < R * B ? lane : R * B - 1;
  const int su = __builtin_amdgcn_readfirstlane(s.slice);
  int k0, k1;
  slot_range(A, su, k0, k1);
  const bool wide = C16 && is_wide(A, su);
  T acc = T(0);
  for (int k = k0; k < k1; k += kSliceWaves * kRelayBatch) {
    const int left = k1 - k < kSliceWaves * kRelayBatch ? k1 - k : kSliceWaves * kRelayBatch;
    const int per = (left + kSliceWaves - 1) / kSliceWaves;
    const int first = w * per < left ? w * per : left;
    const int cnt = left - first < per ? left - first : per;
    typename Val<K>::raw av[kRelayBatch][B];
    XI xv[kRelayBatch][B];
    if (cnt > 0) {
      if (wide) relay_load<B, K, XI, false>(A, k + first, cnt, r, rl, x, av, xv);
      else relay_load<B, K, XI, C16>(A, k + first, cnt, r, rl, x, av, xv);
    }
    for (int turn = 0; turn < kSliceWaves; ++turn) {
      if (turn == w) {
        if (k > k0 || w > 0) acc = sums[lane];
#pragma unroll
        for (int q = 0; q < kRelayBatch; ++q)
          if (q < cnt) {
#pragma unroll
            for (int cc = 0; cc < B; ++cc) acc += T(Val<K>::dec(av[q][cc])) * T(xv[q][cc]);
          }
        sums[lane] = acc;
      }
      __syncthreads();
    }
  }
  if (K == VK_F16 || K == VK_BF16) acc *= T(ldexpf(1.0f, A.rexp[int64_t(su) * kWave + rl]));
  return acc;
}

// y = A x (MODE 0), b - A x (MODE 1), M (b - A x) (MODE 2)
template <int B, int K, class XI, class XO, class T, int MODE, bool C16>
__global__ __launch_bounds__(kThreads) void k_spmv_relay(SellDev A, const XO* __restrict__ b, const XI* __restrict__ x,
                                                         XO* __restrict__ y, const uint8_t* __restrict__ mask) {
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const SliceLane s = slice_lane<B>(A, bid, int(threadIdx.x) % kWave);
  const bool last = int(threadIdx.x) / kWave == kSliceWaves - 1 && s.valid;
  XO bv = XO(0);
  uint8_t mk = 0;
  if (MODE != 0 && last) {
    bv = b[s.dof];
    if (MODE == 2) mk = mask[s.dof];
  }
  const T acc = relay_dot<B, K, XI, T, C16>(A, s, x);
  if (!last) return;
  T out = MODE == 0 ? acc : T(bv) - acc;
  if (MODE == 2 && mk) out = T(0);
  y[s.dof] = XO(out);
}

// x_out = x + omega S (b - A x) and its three-term form, as sweep_slice
template <int B, int K, class X, class T, bool C16>
__global__ __launch_bounds__(kThreads) void k_sweep_relay(SellDev A, const X* __restrict__ S, const X* __restrict__ b,
                                                          const X* __restrict__ x, X* __restrict__ xo, T omega,
                                                          T beta, int pmode) {
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const SliceLane s = slice_lane<B>(A, bid, int(threadIdx.x) % kWave);
  const bool mine = int(threadIdx.x) / kWave == kSliceWaves - 1;
  const bool last = mine && s.valid;
  X bv = X(0), xv = X(0), pv = X(0), sv[B];
#pragma unroll
  for (int cc = 0; cc < B; ++cc) sv[cc] = X(0);
  if (last) {
    bv = b[s.dof];
    xv = x[s.dof];
    pv = (pmode == 1 ? static_cast<const X*>(xo) : x)[s.dof];
#pragma unroll
    for (int cc = 0; cc < B; ++cc) sv[cc] = S[(int64_t(s.slice) * B + cc) * kWave + s.lane];
  }
  const T acc = relay_dot<B, K, X, T, C16>(A, s, x);
  if (!mine) return;                       // the whole wave stays together for the exchange
  const T res = last ? T(bv) - acc : T(0);
  const int base = (s.lane / B) * B;
  T upd = T(0);
#pragma unroll
  for (int cc = 0; cc < B; ++cc) {
    const T rc = __shfl(res, (base + cc) & (kWave - 1), kWave);
    if (last) upd += T(sv[cc]) * rc;
  }
  if (last) {
    T nx = T(xv) + omega * upd;
    if (pmode != 0) nx = nx + beta * (T(xv) - (pmode == 1 ? T(pv) : T(0)));
    xo[s.dof] = X(nx);
  }
}

// two smoothing sweeps from x = 0 in one pass, one component per node:
// x1 = omega S b (formed per column on the fly), x2 = x1 + omega S (b - A x1)
template <int K, class X, class T, int KB, bool C16>
__global__ __launch_bounds__(kThreads) void k_sweep2z(SellDev A, const X* __restrict__ S, const X* __restrict__ b,
                                                      X* __restrict__ xo, T omega) {
  dict_stage<K>(A);                          // before a wave past the last slice leaves
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
  const SliceLane s = slice_lane<B>(A, blockIdx.x * kSliceWaves + threadIdx.x / kWave, threadIdx.x % kWave);
  sweep0_slice<B, X, T>(S, b, xo, omega, s);
}


// The relay form where a level's slices (4 waves each then) do not fill the chip and its rows
// take more than one batch.  Sweep, one wave per slice and relay (4,913 nodes is 234 to 308
// slices): 3 components 729 nodes 6.0 and 3.9 us, 4,913 nodes 6.2 and 4.1 us, 14,620 nodes with
// FP16 values (697 slices) 6.4 and 5.5 us; 4 components 4,913 nodes 6.6 and 5.7 us; one component
// with 27-point rows 9,537 nodes 3.8 and 3.0 us, 70,785 nodes (1,107 slices) 5.7 and 5.7 us.  At
// 1,712 slices (35,937 nodes, 3 components) it loses: 13.2 and 15.4 us; the limit is kRelaySlices.
template <int B>
inline bool relay_level(const SellDev& A) {
  return !A.nt && A.nslices <= kRelaySlices && A.slots >= int64_t(B == 1 ? 12 : 5) * A.nslices;
}

template <int B, int K, class XI, class XO, class T>
hipError_t spmv_t(const SellDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int mode,
                  double* partials, hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  if (g == 0) return hipSuccess;
  const XO* bb = static_cast<const XO*>(b);
  const XI* xx = static_cast<const XI*>(x);
  XO* yy = static_cast<XO*>(y);
  if constexpr (K != VK_DICT) {
    if (!partials && relay_level<B>(A)) {
#define MGQ1_RELAY4(MODE, C16) \
    hipLaunchKernelGGL((k_spmv_relay<B, K, XI, XO, T, MODE, C16>), unsigned(A.nslices), kThreads, 0, s, A, bb, xx, yy, mask)
#define MGQ1_RELAY(MODE)                  \
    if (A.col16) MGQ1_RELAY4(MODE, true);   \
    else MGQ1_RELAY4(MODE, false)
      if (mode == 0) { MGQ1_RELAY(0); }
      else if (mode == 1) { MGQ1_RELAY(1); }
      else if (mode == 2) { MGQ1_RELAY(2); }
      else return hipErrorInvalidValue;
      return hipGetLastError();
#undef MGQ1_RELAY
#undef MGQ1_RELAY4
    }
  }
  // slot batch and column format are runtime properties of the operator
#define MGQ1_SPMV4(MODE, NORM, KB, C16)                                                                               \
  hipLaunchKernelGGL((k_spmv<B, K, XI, XO, T, MODE, NORM, KB, C16>), g, kThreads, dict_lds_bytes<K>(A), s, A, bb, xx, yy, mask, \
                     partials)
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
  if (A.kind == VK_DICT) {
    if (xk == X_F64 && yk == X_F64) return spmv_t<B, VK_DICT, double, double, double>(A, b, x, y, mask, mode, partials, s);
    return hipErrorInvalidValue;
  }
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
  const bool relay = relay_level<B>(A);
#define MGQ1_SWEEPR(KIND, C16) \
  hipLaunchKernelGGL((k_sweep_relay<B, KIND, X, T, C16>), unsigned(A.nslices), kThreads, 0, s, A, SS, bb, xx, oo, T(omega), T(beta), pmode)
#define MGQ1_SWEEP4(KIND, KB, C16) \
  hipLaunchKernelGGL((k_sweep<B, KIND, X, T, KB, C16>), g, kThreads, dict_lds_bytes<KIND>(A), s, A, SS, bb, xx, oo, T(omega), T(beta), pmode)
#define MGQ1_SWEEP1(KIND)                                                  \
  if (A.col16) {                                                           \
    if (A.kb == kb_alt<B>()) MGQ1_SWEEP4(KIND, kb_alt<B>(), true);         \
    else MGQ1_SWEEP4(KIND, kb_default<B>(), true);                         \
  } else {                                                                 \
    if (A.kb == kb_alt<B>()) MGQ1_SWEEP4(KIND, kb_alt<B>(), false);        \
    else MGQ1_SWEEP4(KIND, kb_default<B>(), false);                        \
  }
#define MGQ1_SWEEP(KIND)                                                   \
  if (relay) {                                                             \
    if (A.col16) MGQ1_SWEEPR(KIND, true);                                  \
    else MGQ1_SWEEPR(KIND, false);                                         \
  } else {                                                                 \
    MGQ1_SWEEP1(KIND)                                                      \
  }
  // FP64 vectors go with FP64 values only; FP32 vectors with the reduced formats
  if constexpr (sizeof(X) == 8) {
    if (A.kind == VK_DICT) {
      MGQ1_SWEEP1(VK_DICT)
    } else if (A.kind == VK_F64) {
      MGQ1_SWEEP(VK_F64)
    } else {
      return hipErrorInvalidValue;
    }
  } else {
    switch (A.kind) {
      case VK_F32: MGQ1_SWEEP(VK_F32); break;
      case VK_F16: MGQ1_SWEEP(VK_F16); break;
      case VK_BF16: MGQ1_SWEEP(VK_BF16); break;
      default: return hipErrorInvalidValue;
    }
  }
#undef MGQ1_SWEEP
#undef MGQ1_SWEEP1
#undef MGQ1_SWEEP4
#undef MGQ1_SWEEPR
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
  hipLaunchKernelGGL((k_sweep2z<KIND, X, T, KB, C16>), g, kThreads, dict_lds_bytes<KIND>(A), s, A, static_cast<const X*>(S), \
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
    if (A.kind == VK_DICT) {
      MGQ1_S2Z(VK_DICT, double, double);
    } else if (A.kind == VK_F64) {
      MGQ1_S2Z(VK_F64, double, double);
    } else {
      return hipErrorInvalidValue;
    }
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
