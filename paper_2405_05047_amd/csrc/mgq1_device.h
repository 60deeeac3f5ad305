// Device-side building blocks shared by the HIP translation units of the multigrid
// library (internal linkage: each unit keeps its own copies): value decoding, the slot
// batches of the sliced-ELL operators, the per-slice row bodies, the sliced transfers,
// deterministic block reductions and launch-size helpers.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "mgq1_internal.h"


namespace mgq1 {
namespace {


constexpr int kThreads = kWave * kSliceWaves;   // 256
constexpr int kTailThreads = 1024;
constexpr int kMaxWaves = 16;

__device__ __forceinline__ int xcd_remap(int bid, int nb) {
  // hardware dispatch sends workgroup w to XCD w % 8; give XCD x a contiguous range
  const int q = nb >> 3, r = nb & 7;
  const int x = bid & 7, k = bid >> 3;
  return x * q + (x < r ? x : r) + k;
}

// Loads of the operator streams (values, column indices, transfer weights): non-temporal
// (NT) on levels too large to stay in the memory-side cache between kernels, where they
// would only evict the gathered vectors; ordinary loads on the smaller levels, whose
// operators the next kernels read again from that cache.
template <bool NT, class P>
__device__ __forceinline__ P stream_load(const P* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

// stored matrix values: load() fetches the raw stored word, dec() widens it to FP32/FP64.  FP16/BF16 values are a_ij / s_i with the
// power-of-two row scale s_i applied once to the finished row sum (exact: scaling by 2^e
// commutes with rounding away from overflow and underflow).
template <int K> struct Val;
template <> struct Val<VK_F64> {
  using raw = double;
  template <bool NT>
  __device__ __forceinline__ static raw load(const void* p, int64_t i) {
    return stream_load<NT>(static_cast<const double*>(p) + i);
  }
  __device__ __forceinline__ static double dec(raw u) { return u; }
};
template <> struct Val<VK_F32> {
  using raw = float;
  template <bool NT>
  __device__ __forceinline__ static raw load(const void* p, int64_t i) {
    return stream_load<NT>(static_cast<const float*>(p) + i);
  }
  __device__ __forceinline__ static float dec(raw u) { return u; }
};
template <> struct Val<VK_F16> {
  using raw = unsigned short;
  template <bool NT>
  __device__ __forceinline__ static raw load(const void* p, int64_t i) {
    return stream_load<NT>(static_cast<const unsigned short*>(p) + i);
  }
  __device__ __forceinline__ static float dec(raw u) { return __half2float(__ushort_as_half(u)); }
};
// FP64 blocks from the level's dictionary (loaded in sell_batch, not through load())
template <> struct Val<VK_DICT> {
  using raw = double;
  __device__ __forceinline__ static double dec(raw u) { return u; }
};
template <> struct Val<VK_BF16> {
  using raw = unsigned short;
  template <bool NT>
  __device__ __forceinline__ static raw load(const void* p, int64_t i) {
    return stream_load<NT>(static_cast<const unsigned short*>(p) + i);
  }
  __device__ __forceinline__ static float dec(raw u) { return __uint_as_float(static_cast<uint32_t>(u) << 16); }
};

// NB block slots k .. k+NB-1 of a slice: the column indices first, then every value and
// x load of the batch, then the FMAs, so the batch costs two memory round trips.  NB is a
// compile-time constant, so no load sits in a conditional block (a conditional load whose
// result is widened inside the block would force a wait per slot).
// C16: column indices are stored as 16-bit offsets from a per-slot base (the smallest
// column of that slot in the slice, wave-uniform, so a scalar load).
template <bool C16, bool NT>
__device__ __forceinline__ unsigned slot_col(const SellDev& A, int k, int64_t idx) {
  if constexpr (C16) return unsigned(A.colbase[k]) + unsigned(stream_load<NT>(A.col16 + idx));
  else return unsigned(stream_load<NT>(A.col + idx));
}

// slot range [k, k1) of slice su (wave-uniform): computed for uniform-width slices, else
// read from the slice pointers (one dependent round trip before the first slot load)
template <class M>
__device__ __forceinline__ void slot_range(const M& A, int su, int& k, int& k1) {
  if (A.ell > 0) {
    k = su * A.ell;
    k1 = k + A.ell;
  } else {
    k = A.sptr[su];
    k1 = A.sptr[su + 1];
  }
}

// slice su (wave-uniform) of a 16-bit-column operator reads the 32-bit columns instead
__device__ __forceinline__ bool is_wide(const SellDev& A, int su) {
  return A.wide != nullptr && ((A.wide[su >> 5] >> (su & 31)) & 1u);
}

// bytes of LDS that hold a VK_DICT operator's blocks (0: they are read through the caches)
__host__ __device__ __forceinline__ int dict_lds_size(const SellDev& A) {
  const int64_t bytes = int64_t(A.ndict) * A.B * A.B * int64_t(sizeof(double));
  return bytes <= kDictLdsBytes ? int(bytes) : 0;
}

template <int NB, int B, int K, class XI, class T, bool C16, bool NT>
__device__ __forceinline__ void sell_batch(const SellDev& A, int k, int r, int node, int rl,
                                           const XI* __restrict__ x, T& acc) {
  constexpr int R = kWave / B;
  using VR = typename Val<K>::raw;
  // phase 1: column indices and values (independent of each other); phase 2: the x
  // gathers; phase 3: the FMAs.  Scheduling barriers keep the phases apart, otherwise the
  // scheduler interleaves the FMA chain with the loads and adds round trips.
  unsigned js[NB];                         // unsigned: widening needs no sign extension
  VR av[NB][B];
  XI xv[NB][B];
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) js[qq] = slot_col<C16, NT>(A, k + qq, int64_t(k + qq) * R + r);
  if constexpr (K == VK_DICT) {
    // column and block numbers first, then the block's row from the (cached) dictionary together
    // with the x gathers
    unsigned short di[NB];
#pragma unroll
    for (int qq = 0; qq < NB; ++qq) di[qq] = stream_load<NT>(A.didx + int64_t(k + qq) * R + r);
    __builtin_amdgcn_sched_barrier(0);
    const int c = rl % B;
    if (dict_lds_size(A) > 0) {
      extern __shared__ double dict_lds[];
#pragma unroll
      for (int qq = 0; qq < NB; ++qq)
#pragma unroll
        for (int cc = 0; cc < B; ++cc) av[qq][cc] = dict_lds[(int(di[qq]) * B + c) * B + cc];
    } else {
#pragma unroll
      for (int qq = 0; qq < NB; ++qq)
#pragma unroll
        for (int cc = 0; cc < B; ++cc)
          av[qq][cc] = static_cast<const double*>(A.val)[(int64_t(di[qq]) * B + c) * B + cc];
    }
  } else {
#pragma unroll
    for (int qq = 0; qq < NB; ++qq) {
      const int64_t vb = int64_t(k + qq) * B * kWave + rl;
#pragma unroll
      for (int cc = 0; cc < B; ++cc) av[qq][cc] = Val<K>::template load<NT>(A.val, vb + cc * kWave);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (B > 1) {
    // each lane gathers only its own component of the neighbour node (the B lanes of a
    // node read one contiguous B-vector together) and takes the others from its node's
    // lanes by wave shuffles
    const int c = rl % B, base = rl - c;
    XI xo[NB];
#pragma unroll
    for (int qq = 0; qq < NB; ++qq) xo[qq] = x[uint64_t(js[qq]) * B + c];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int qq = 0; qq < NB; ++qq)
#pragma unroll
      for (int cc = 0; cc < B; ++cc) xv[qq][cc] = __shfl(xo[qq], base + cc, kWave);
  } else {
#pragma unroll
    for (int qq = 0; qq < NB; ++qq) xv[qq][0] = x[js[qq]];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int qq = 0; qq < NB; ++qq)
#pragma unroll
    for (int cc = 0; cc < B; ++cc) acc += T(Val<K>::dec(av[qq][cc])) * T(xv[qq][cc]);
}

// small dictionaries: the workgroup copies them into LDS before any slice work (all threads
// reach the barrier); launched with dict_lds_bytes of dynamic shared memory
template <int K>
__device__ __forceinline__ void dict_stage(const SellDev& A) {
  if constexpr (K == VK_DICT) {
    const int n = dict_lds_size(A) / int(sizeof(double));
    if (n > 0) {
      extern __shared__ double dict_lds[];
      for (int i = int(threadIdx.x); i < n; i += int(blockDim.x)) dict_lds[i] = static_cast<const double*>(A.val)[i];
      __syncthreads();
    }
  }
}

template <int K>
inline size_t dict_lds_bytes(const SellDev& A) {
  return K == VK_DICT ? size_t(dict_lds_size(A)) : 0;
}

// The same batch for the second of two sweeps from x = 0 with b = 1: the iterate after the
// first sweep, x1_j = omega * (S_j * b_j), is formed on the fly from S and b instead of being
// read (S of node j sits at S[j] for one component and one right-hand side), with the
// rounding of the stored value, so the result is bitwise that of the two separate sweeps.
template <int NB, int K, class X, class T, bool C16, bool NT>
__device__ __forceinline__ void sell_batch_z(const SellDev& A, int k, int rl, int node, const X* __restrict__ S,
                                             const X* __restrict__ b, T omega, T& acc) {
  using VR = typename Val<K>::raw;
  unsigned js[NB];
  VR av[NB];
  X sv[NB], bv[NB];
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) js[qq] = slot_col<C16, NT>(A, k + qq, int64_t(k + qq) * kWave + rl);
  if constexpr (K == VK_DICT) {
    unsigned short di[NB];
#pragma unroll
    for (int qq = 0; qq < NB; ++qq) di[qq] = stream_load<NT>(A.didx + int64_t(k + qq) * kWave + rl);
    __builtin_amdgcn_sched_barrier(0);
    if (dict_lds_size(A) > 0) {
      extern __shared__ double dict_lds[];
#pragma unroll
      for (int qq = 0; qq < NB; ++qq) av[qq] = dict_lds[di[qq]];
    } else {
#pragma unroll
      for (int qq = 0; qq < NB; ++qq) av[qq] = static_cast<const double*>(A.val)[di[qq]];
    }
  } else {
#pragma unroll
    for (int qq = 0; qq < NB; ++qq) av[qq] = Val<K>::template load<NT>(A.val, int64_t(k + qq) * kWave + rl);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) {
    sv[qq] = S[js[qq]];
    bv[qq] = b[js[qq]];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) {
    const X x1 = X(omega * (T(0) + T(sv[qq]) * T(bv[qq])));
    acc += T(Val<K>::dec(av[qq])) * T(x1);
  }
}

template <int N, int K, class X, class T, bool C16, bool NT>
__device__ __forceinline__ void sell_rest_z(int rem, const SellDev& A, int k, int rl, int node,
                                            const X* __restrict__ S, const X* __restrict__ b, T omega, T& acc) {
  if constexpr (N >= 1) {
    if (rem == N) sell_batch_z<N, K, X, T, C16, NT>(A, k, rl, node, S, b, omega, acc);
    else sell_rest_z<N - 1, K, X, T, C16, NT>(rem, A, k, rl, node, S, b, omega, acc);
  }
}

// the slots [k, k1) of one slice for the second of two sweeps from 0
template <int KB, int K, class X, class T, bool C16, bool NT>
__device__ __forceinline__ void sell_loop_z(int k, int k1, const SellDev& A, int rl, int node,
                                            const X* __restrict__ S, const X* __restrict__ b, T omega, T& acc) {
  for (; k + KB <= k1; k += KB) sell_batch_z<KB, K, X, T, C16, NT>(A, k, rl, node, S, b, omega, acc);
  sell_rest_z<KB - 1, K, X, T, C16, NT>(k1 - k, A, k, rl, node, S, b, omega, acc);
}

// the remaining rem < KB slots of a slice as one batch of exactly rem slots
template <int N, int B, int K, class XI, class T, bool C16, bool NT>
__device__ __forceinline__ void sell_rest(int rem, const SellDev& A, int k, int r, int node, int rl,
                                          const XI* __restrict__ x, T& acc) {
  if constexpr (N >= 1) {
    if (rem == N) sell_batch<N, B, K, XI, T, C16, NT>(A, k, r, node, rl, x, acc);
    else sell_rest<N - 1, B, K, XI, T, C16, NT>(rem, A, k, r, node, rl, x, acc);
  }
}

// the slots [k, k1) of one slice: batches of KB, then the remainder as one batch
template <int KB, int B, int K, class XI, class T, bool C16, bool NT>
__device__ __forceinline__ void sell_loop(int k, int k1, const SellDev& A, int r, int node, int rl,
                                          const XI* __restrict__ x, T& acc) {
  for (; k + KB <= k1; k += KB) sell_batch<KB, B, K, XI, T, C16, NT>(A, k, r, node, rl, x, acc);
  sell_rest<KB - 1, B, K, XI, T, C16, NT>(k1 - k, A, k, r, node, rl, x, acc);
}

template <int B> constexpr int kb_default() { return B <= 2 ? 8 : 4; }
template <int B> constexpr int kb_alt() { return B <= 2 ? 16 : 8; }

// per-lane row dot product of a slice: sum_k sum_cc a(k, cc) x[col_k * B + cc], lane = r * B + c,
// values at val[(k * B + cc) * 64 + lane].  Slots are consumed in batches of KB, the remainder in
// one shorter batch (slice-uniform branch); the FMAs run in slot order whatever KB is, so
// every KB gives the same bits.
// LK: load kind of the operator stream — 0 as the operator says (A.nt), 1 always
// non-temporal (batched form), 2 always ordinary (single-workgroup tail)
template <int B, int K, class XI, class T, int KB = kb_default<B>(), bool C16 = false, int LK = 0>
__device__ __forceinline__ T sell_dot(const SellDev& A, int slice, int lane, bool valid,
                                      const XI* __restrict__ x) {
  constexpr int R = kWave / B;
  T acc = T(0);
  if (!valid) return acc;
  const int rl = lane, r = lane / B;
  // the slice is the same for the whole wave: keep it (and the slot range, the load bases)
  // in scalar registers
  slice = __builtin_amdgcn_readfirstlane(slice);
  const int node = slice * R + r;
  int k, k1;
  slot_range(A, slice, k, k1);
  const bool wide = C16 && is_wide(A, slice);
  if (LK == 1 || (LK == 0 && A.nt)) {
    if constexpr (LK != 2) {
      if (wide) sell_loop<KB, B, K, XI, T, false, true>(k, k1, A, r, node, rl, x, acc);
      else sell_loop<KB, B, K, XI, T, C16, true>(k, k1, A, r, node, rl, x, acc);
    }
  } else {
    if constexpr (LK != 1) {
      if (wide) sell_loop<KB, B, K, XI, T, false, false>(k, k1, A, r, node, rl, x, acc);
      else sell_loop<KB, B, K, XI, T, C16, false>(k, k1, A, r, node, rl, x, acc);
    }
  }
  if (K == VK_F16 || K == VK_BF16) acc *= T(ldexpf(1.0f, A.rexp[int64_t(slice) * kWave + rl]));
  return acc;
}

template <class T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, kWave);
  return v;
}

// The sums over the lanes of equal lane % OMIN of P values per lane (P a power of two up to
// 32): at every step each half of the lanes keeps one half of the values and hands over the
// other (P - 1 shuffles and then one per remaining step, instead of one per value and
// step).  On return v[0], v[1] .. are the sums of the values number `which`, `which` + 1 ..
// (P * OMIN / 64 of them, at least one); the order of the additions is fixed.
template <int P, int O, int OMIN, int NT>
__device__ __forceinline__ void wave_sums_step(double (&v)[NT], int lane, int& which) {
  if constexpr (O >= OMIN) {
    if constexpr (P > 1) {
      constexpr int H = P / 2;
      const bool up = (lane & O) != 0;
#pragma unroll
      for (int i = 0; i < H; ++i) {
        const double send = up ? v[i] : v[i + H];
        v[i] = (up ? v[i + H] : v[i]) + __shfl_xor(send, O, kWave);
      }
      which += up ? H : 0;
      wave_sums_step<H, O / 2, OMIN, NT>(v, lane, which);
    } else {
      v[0] = v[0] + __shfl_xor(v[0], O, kWave);
      wave_sums_step<1, O / 2, OMIN, NT>(v, lane, which);
    }
  }
}

constexpr int pow2_above(int n) { int p = 1; while (p < n) p *= 2; return p; }

// sum over the block in a fixed order, returned to every thread
__device__ __forceinline__ double block_allsum(double v, double* lds) {
  v = wave_sum(v);
  const int w = threadIdx.x / kWave, ln = threadIdx.x % kWave;
  const int nw = blockDim.x / kWave;
  if (ln == 0) lds[w] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < nw; ++q) t += lds[q];
    lds[kMaxWaves] = t;
  }
  __syncthreads();
  const double r = lds[kMaxWaves];
  __syncthreads();
  return r;
}

// sum of partials[0..g) in a fixed order (every block computes the same value)
__device__ __forceinline__ double sum_partials(const double* __restrict__ p, int g, double* lds) {
  constexpr int U = 8;                     // loads issued together, summed in index order
  double t = 0.0;
  for (int q0 = threadIdx.x; q0 < g; q0 += blockDim.x * U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u * int(blockDim.x);
      v[u] = q < g ? p[q] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) t += v[u];
  }
  return block_allsum(t, lds);
}

// ------------------------------------------------------------------ per-slice bodies
// geometry of one wave-slice
struct SliceLane {
  int slice, lane, node;
  int64_t dof;            // node * B + c
  bool valid;
};

template <int B>
__device__ __forceinline__ SliceLane slice_lane(const SellDev& A, int slice, int lane) {
  constexpr int R = kWave / B;
  SliceLane s;
  s.slice = slice;
  s.lane = lane;
  const int pos = slice * R + lane / B;   // row position of the lane's node
  s.valid = slice < A.nslices && lane < R * B && pos < A.n;
  s.node = (A.perm != nullptr && s.valid) ? A.perm[pos] : pos;
  s.dof = int64_t(s.node) * B + lane % B;
  return s;
}

// y = A x (MODE 0), b - A x (MODE 1), M (b - A x) (MODE 2); returns the written value
template <int B, int K, class XI, class XO, class T, int MODE, int KB = kb_default<B>(), bool C16 = false,
          int LK = 0>
__device__ __forceinline__ T spmv_slice(const SellDev& A, const XO* __restrict__ b, const XI* __restrict__ x,
                                        XO* __restrict__ y, const uint8_t* __restrict__ mask, const SliceLane& s) {
  XO bv = XO(0);
  uint8_t mk = 0;
  if (MODE != 0 && s.valid) {              // loaded before the row sum (latency overlap)
    bv = b[s.dof];
    if (MODE == 2) mk = mask[s.dof];
  }
  const T acc = sell_dot<B, K, XI, T, KB, C16, LK>(A, s.slice, s.lane, s.valid, x);
  T out = T(0);
  if (s.valid) {
    if (MODE == 0) {
      out = acc;
    } else {
      out = T(bv) - acc;
      if (MODE == 2 && mk) out = T(0);
    }
    y[s.dof] = XO(out);
  }
  return out;
}

// x_out = x + omega S (b - A x), and with pmode != 0 the three-term (Chebyshev) form
// x_out = x + omega S (b - A x) + beta (x - x_prev): pmode 1 reads x_prev from x_out
// itself (each lane reads its own entry before it overwrites it), pmode 2 takes x_prev = 0
template <int B, int K, class X, class T, int KB = kb_default<B>(), bool C16 = false, int LK = 0>
__device__ __forceinline__ void sweep_slice(const SellDev& A, const X* __restrict__ S, const X* __restrict__ b,
                                            const X* __restrict__ x, X* __restrict__ xo, T omega,
                                            const SliceLane& s, T beta = T(0), int pmode = 0) {
  // the lane's own b, x and smoother row are loaded before the row sum, so their latency
  // overlaps the slot batches
  X bv = X(0), xv = X(0), pv = X(0), sv[B];
#pragma unroll
  for (int cc = 0; cc < B; ++cc) sv[cc] = X(0);
  if (s.valid) {
    bv = b[s.dof];
    xv = x[s.dof];
    // unconditional load (a load inside a branch would make the slot loop wait for it);
    // with pmode != 1 it rereads x and the value is not used
    pv = (pmode == 1 ? static_cast<const X*>(xo) : x)[s.dof];
#pragma unroll
    for (int cc = 0; cc < B; ++cc) sv[cc] = S[(int64_t(s.slice) * B + cc) * kWave + s.lane];
  }
  const T acc = sell_dot<B, K, X, T, KB, C16, LK>(A, s.slice, s.lane, s.valid, x);
  const T res = s.valid ? T(bv) - acc : T(0);
  const int base = (s.lane / B) * B;
  T upd = T(0);
#pragma unroll
  for (int cc = 0; cc < B; ++cc) {
    const T rc = __shfl(res, (base + cc) & (kWave - 1), kWave);
    if (s.valid) upd += T(sv[cc]) * rc;
  }
  if (s.valid) {
    T nx = T(xv) + omega * upd;
    if (pmode != 0) nx = nx + beta * (T(xv) - (pmode == 1 ? T(pv) : T(0)));
    xo[s.dof] = X(nx);
  }
}

template <int B, class X, class T>
__device__ __forceinline__ void sweep0_slice(const X* __restrict__ S, const X* __restrict__ b, X* __restrict__ xo,
                                             T omega, const SliceLane& s) {
  if (!s.valid) return;
  T upd = T(0);
#pragma unroll
  for (int cc = 0; cc < B; ++cc)
    upd += T(S[(int64_t(s.slice) * B + cc) * kWave + s.lane]) * T(b[int64_t(s.node) * B + cc]);
  xo[s.dof] = X(omega * upd);
}

__device__ __forceinline__ double weight(const CsrDev& M, int k) {
  return M.f32 ? double(static_cast<const float*>(M.val)[k]) : static_cast<const double*>(M.val)[k];
}

// d[dof] = M_c sum_k R_jk (M_f r)[k], dof = j * B + c
template <int B, class X, class T>
__device__ __forceinline__ void restrict_dof(const CsrDev& R, const X* __restrict__ r, X* __restrict__ d,
                                             const uint8_t* __restrict__ mask_c, const uint8_t* __restrict__ mask_f,
                                             int64_t dof) {
  const int j = int(dof / B), c = int(dof % B);
  T acc = T(0);
  if (!mask_c[dof]) {
    for (int k = R.rowptr[j]; k < R.rowptr[j + 1]; ++k) {
      const int64_t fd = int64_t(R.col[k]) * B + c;
      if (mask_f == nullptr || !mask_f[fd]) acc += T(weight(R, k)) * T(r[fd]);
    }
  }
  d[dof] = X(acc);
}

// x[dof] += M_f sum_k P_ik (M_c y)[k]
template <int B, class X, class T>
__device__ __forceinline__ void prolong_dof(const CsrDev& P, const X* __restrict__ y, X* __restrict__ x,
                                            const uint8_t* __restrict__ mask_f, const uint8_t* __restrict__ mask_c,
                                            int64_t dof) {
  if (mask_f[dof]) return;
  const int i = int(dof / B), c = int(dof % B);
  T acc = T(0);
  for (int k = P.rowptr[i]; k < P.rowptr[i + 1]; ++k) {
    const int64_t cd = int64_t(P.col[k]) * B + c;
    if (!mask_c[cd]) acc += T(weight(P, k)) * T(y[cd]);
  }
  x[dof] = X(T(x[dof]) + acc);
}

// ---- sliced transfers: NB slots of one node row, loads first (straight-line), then the
// weighted sum in slot order.  MC: apply the column mask (entries whose column DoF is
// masked contribute 0).
template <int NB, int B, class X, class T, class WT, bool MC, bool NT>
__device__ __forceinline__ void tsell_batch(const TSellDev& M, int k, int r, int c,
                                            const X* __restrict__ in, const uint8_t* __restrict__ mcol,
                                            T& acc) {
  const int R = M.R;
  unsigned js[NB];
  WT ws[NB];
  X vs[NB];
  uint8_t ms[NB];
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) {
    js[qq] = unsigned(stream_load<NT>(M.col + int64_t(k + qq) * R + r));
    ws[qq] = stream_load<NT>(static_cast<const WT*>(M.w) + int64_t(k + qq) * R + r);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) {
    const uint64_t d = uint64_t(js[qq]) * B + c;
    vs[qq] = in[d];
    ms[qq] = MC ? mcol[d] : uint8_t(0);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) acc += T(ws[qq]) * (ms[qq] ? T(0) : T(vs[qq]));
}

template <int N, int B, class X, class T, class WT, bool MC, bool NT>
__device__ __forceinline__ void tsell_rest(int rem, const TSellDev& M, int k, int r, int c,
                                           const X* __restrict__ in, const uint8_t* __restrict__ mcol, T& acc) {
  if constexpr (N >= 1) {
    if (rem == N) tsell_batch<N, B, X, T, WT, MC, NT>(M, k, r, c, in, mcol, acc);
    else tsell_rest<N - 1, B, X, T, WT, MC, NT>(rem, M, k, r, c, in, mcol, acc);
  }
}

// one lane of a sliced transfer.  MODE 0: out = restriction sum (zero on masked rows);
// MODE 1: out += prolongation sum (rows whose DoF is masked are left unchanged)
template <int B, class X, class T, class WT, bool MC, int MODE>
__device__ __forceinline__ void tsell_lane(const TSellDev& M, int slice, int lane, const X* __restrict__ in,
                                           X* __restrict__ out, const uint8_t* __restrict__ mrow,
                                           const uint8_t* __restrict__ mcol) {
  constexpr int KB = 8;
  const int R = M.R;
  const int r = lane / B, c = lane % B;
  const int node = slice * R + r;
  if (slice >= M.nslices || lane >= R * B || node >= M.nrows) return;
  const int64_t dof = int64_t(node) * B + c;
  // the row mask and (prolongation) the old value are loaded with the first slots; masked
  // rows run the sum too (their columns are valid indices) and drop it at the end, so no
  // branch waits for the mask before the slot loads are issued
  const uint8_t masked = mrow[dof];
  X old = X(0);
  if (MODE == 1) old = out[dof];
  const int su = __builtin_amdgcn_readfirstlane(slice);
  int k, k1;
  slot_range(M, su, k, k1);
  T acc = T(0);
  if (M.nt) {
    for (; k + KB <= k1; k += KB) tsell_batch<KB, B, X, T, WT, MC, true>(M, k, r, c, in, mcol, acc);
    tsell_rest<KB - 1, B, X, T, WT, MC, true>(k1 - k, M, k, r, c, in, mcol, acc);
  } else {
    for (; k + KB <= k1; k += KB) tsell_batch<KB, B, X, T, WT, MC, false>(M, k, r, c, in, mcol, acc);
    tsell_rest<KB - 1, B, X, T, WT, MC, false>(k1 - k, M, k, r, c, in, mcol, acc);
  }
  if (MODE == 0) out[dof] = masked ? X(0) : X(acc);
  else if (!masked) out[dof] = X(T(old) + acc);
}

template <int B, class X, class T, class WT, bool MC, int MODE>
__global__ __launch_bounds__(kThreads) void k_tsell(TSellDev M, const X* __restrict__ in, X* __restrict__ out,
                                                    const uint8_t* __restrict__ mrow,
                                                    const uint8_t* __restrict__ mcol) {
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  tsell_lane<B, X, T, WT, MC, MODE>(M, bid * kSliceWaves + threadIdx.x / kWave, threadIdx.x % kWave, in, out,
                                        mrow, mcol);
}

// ---- node form of the sliced transfers: one lane per node computes its B components.  Per
// slot one packed 32-bit entry (16-bit column offset, 8-bit weight code w * 128, the column
// DoFs' mask bits) and B gathers of the column node's vector; the FMAs run in slot order
// with the same operands as the per-DoF form, so the sums are the same bit for bit.  A
// wave issues one entry load per slot for 64 nodes where the per-DoF form issues an index,
// a weight and a mask load per slot for 64 / B nodes.
//
// WIDE: levels with a slot whose columns span 2^16 and more (adaptive 3D meshes) keep the
// column in 32 bits and weight code and mask bits in another 16: 6 bytes per entry.
template <int NB, int B, class X, bool WIDE>
__device__ __forceinline__ void tnode_load(const TSellDev& M, int k, int last, int lane, const X* __restrict__ in,
                                           uint32_t (&e)[NB], X (&v)[NB][B]) {
  uint32_t j[NB];
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) {
    const int kk = k + qq < last ? k + qq : last;          // past the end: the last slot again, not used
    if constexpr (WIDE) {
      j[qq] = uint32_t(M.col[int64_t(kk) * kWave + lane]);
      e[qq] = uint32_t(M.cw[int64_t(kk) * kWave + lane]) << 16;
    } else {
      e[qq] = M.ent[int64_t(kk) * kWave + lane];
      j[qq] = uint32_t(M.colbase[kk]);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) {
    const uint64_t c0 = uint64_t(WIDE ? j[qq] : j[qq] + (e[qq] & 0xffffu)) * B;
#pragma unroll
    for (int c = 0; c < B; ++c) v[qq][c] = in[c0 + c];
  }
  __builtin_amdgcn_sched_barrier(0);
}

// the weighted sum of slot entry e in slot order
template <int B, class X, class T, bool MC>
__device__ __forceinline__ void tnode_add(uint32_t e, const X (&v)[B], T (&acc)[B]) {
  const T w = T(float((e >> 16) & 0xffu) * 0.0078125f);
#pragma unroll
  for (int c = 0; c < B; ++c) {
    const bool ms = MC && ((e >> (24 + c)) & 1u);
    acc[c] += w * (ms ? T(0) : T(v[c]));
  }
}

template <int NB, int B, class X, class T, bool MC, bool WIDE>
__device__ __forceinline__ void tnode_batch(const TSellDev& M, int k, int lane, const X* __restrict__ in,
                                            T (&acc)[B]) {
  uint32_t e[NB];
  X v[NB][B];
  tnode_load<NB, B, X, WIDE>(M, k, k + NB - 1, lane, in, e, v);
#pragma unroll
  for (int qq = 0; qq < NB; ++qq) tnode_add<B, X, T, MC>(e[qq], v[qq], acc);
}

template <int N, int B, class X, class T, bool MC, bool WIDE>
__device__ __forceinline__ void tnode_rest(int rem, const TSellDev& M, int k, int lane, const X* __restrict__ in,
                                           T (&acc)[B]) {
  if constexpr (N >= 1) {
    if (rem == N) tnode_batch<N, B, X, T, MC, WIDE>(M, k, lane, in, acc);
    else tnode_rest<N - 1, B, X, T, MC, WIDE>(rem, M, k, lane, in, acc);
  }
}

// MODE 0: out = restriction sum (zero on masked row DoFs); MODE 1: out += prolongation sum
// (masked row DoFs left unchanged)
template <int B, class X, class T, bool MC, int MODE, bool WIDE>
__device__ __forceinline__ void tnode_lane(const TSellDev& M, int slice, int lane, const X* __restrict__ in,
                                           X* __restrict__ out) {
  // slot batch: restriction rows hold up to 3^d entries (27 on 3D box meshes), prolongation
  // rows at most 2^d; a batch is one dependent round trip (entries, then gathers)
  constexpr int KB = MODE == 0 ? 8 : 4;
  const int node = slice * kWave + lane;
  if (slice >= M.nslices || node >= M.nrows) return;
  const int64_t d0 = int64_t(node) * B;
  const uint8_t rm = M.rmask[node];
  X old[B];
  if (MODE == 1) {
#pragma unroll
    for (int c = 0; c < B; ++c) old[c] = out[d0 + c];
  }
  const int su = __builtin_amdgcn_readfirstlane(slice);
  int k, k1;
  slot_range(M, su, k, k1);
  T acc[B];
#pragma unroll
  for (int c = 0; c < B; ++c) acc[c] = T(0);
  for (; k + KB <= k1; k += KB) tnode_batch<KB, B, X, T, MC, WIDE>(M, k, lane, in, acc);
  tnode_rest<KB - 1, B, X, T, MC, WIDE>(k1 - k, M, k, lane, in, acc);
#pragma unroll
  for (int c = 0; c < B; ++c) {
    const bool masked = (rm >> c) & 1u;
    if (MODE == 0) out[d0 + c] = masked ? X(0) : X(acc[c]);
    else if (!masked) out[d0 + c] = X(T(old[c]) + acc[c]);
  }
}

// Restriction of a level with few slices: one slice per workgroup, a quarter of the slots per
// wave, the sums passed on in slot order (the relay of the slice kernels).
template <int B, class X, class T, bool MC, bool WIDE>
__global__ __launch_bounds__(kThreads) void k_tnode_relay(TSellDev M, const X* __restrict__ in, X* __restrict__ out) {
  constexpr int NB = 8;
  __shared__ T sums[B][kWave];
  const int slice = xcd_remap(blockIdx.x, gridDim.x);
  const int lane = int(threadIdx.x) % kWave, w = int(threadIdx.x) / kWave;
  const int node = slice * kWave + lane;
  uint8_t rm = 0;
  if (w == kSliceWaves - 1 && node < M.nrows) rm = M.rmask[node];
  const int su = __builtin_amdgcn_readfirstlane(slice);
  int k0, k1;
  slot_range(M, su, k0, k1);
  T acc[B];
#pragma unroll
  for (int c = 0; c < B; ++c) acc[c] = T(0);
  for (int k = k0; k < k1; k += kSliceWaves * NB) {
    const int left = k1 - k < kSliceWaves * NB ? k1 - k : kSliceWaves * NB;
    const int per = (left + kSliceWaves - 1) / kSliceWaves;
    const int first = w * per < left ? w * per : left;
    const int cnt = left - first < per ? left - first : per;
    uint32_t e[NB];
    X v[NB][B];
    if (cnt > 0) tnode_load<NB, B, X, WIDE>(M, k + first, k + first + cnt - 1, lane, in, e, v);
    for (int turn = 0; turn < kSliceWaves; ++turn) {
      if (turn == w) {
        if (k > k0 || w > 0) {
#pragma unroll
          for (int c = 0; c < B; ++c) acc[c] = sums[c][lane];
        }
#pragma unroll
        for (int qq = 0; qq < NB; ++qq)
          if (qq < cnt) tnode_add<B, X, T, MC>(e[qq], v[qq], acc);
#pragma unroll
        for (int c = 0; c < B; ++c) sums[c][lane] = acc[c];
      }
      __syncthreads();
    }
  }
  if (w != kSliceWaves - 1 || node >= M.nrows) return;
#pragma unroll
  for (int c = 0; c < B; ++c) out[int64_t(node) * B + c] = ((rm >> c) & 1u) ? X(0) : X(acc[c]);
}

template <int B, class X, class T, bool MC, int MODE, bool WIDE>
__global__ __launch_bounds__(kThreads) void k_tnode(TSellDev M, const X* __restrict__ in, X* __restrict__ out) {
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  tnode_lane<B, X, T, MC, MODE, WIDE>(M, bid * kSliceWaves + threadIdx.x / kWave, threadIdx.x % kWave, in, out);
}

// Gauss-Jordan with row pivoting on [M | I]; the right half becomes the inverse.  false: singular
template <int B>
__device__ __forceinline__ bool invert_augmented(double (&m)[B][2 * B]) {
  for (int k = 0; k < B; ++k) {
    int p = k;
    for (int i = k + 1; i < B; ++i)
      if (fabs(m[i][k]) > fabs(m[p][k])) p = i;
    if (m[p][k] == 0.0) return false;
    if (p != k)
      for (int c = 0; c < 2 * B; ++c) { const double t = m[k][c]; m[k][c] = m[p][c]; m[p][c] = t; }
    const double inv = 1.0 / m[k][k];
    for (int c = 0; c < 2 * B; ++c) m[k][c] *= inv;
    for (int i = 0; i < B; ++i) {
      if (i == k) continue;
      const double f = m[i][k];
      for (int c = 0; c < 2 * B; ++c) m[i][c] -= f * m[k][c];
    }
  }
  return true;
}

inline unsigned grid_for(int64_t n, int threads) { return unsigned((n + threads - 1) / threads); }
inline unsigned slice_grid(int nslices) { return unsigned((nslices + kSliceWaves - 1) / kSliceWaves); }

}  // namespace
}  // namespace mgq1
