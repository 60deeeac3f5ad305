// HIP kernels of the batched form: every V-cycle step and Krylov vector operation of many
// independent problems (1 or 8 right-hand sides each) in one launch.  With one right-hand side
// the per-slice bodies are those of the single-problem kernels; a wave finds its problem
// entry with one compare of 64 entries, and segmented reductions keep one partial per
// block and right-hand side, re-summed in a fixed order by the consumer kernel.
#include "mgq1_device.h"

#include <algorithm>
#include <climits>

namespace mgq1 {

// ======================================================================== batched form
namespace {

// the entry of block blk: the largest e with E[e].first <= blk (entries are sorted by
// first and E[0].first = 0).  Called by the whole first wave: each lane tests one entry, so
// 64 entries cost one round trip instead of a chain of dependent loads.
__device__ __forceinline__ int find_entry_wave(const BEntry* __restrict__ E, int n, int blk) {
  const int lane = threadIdx.x % kWave;
  int cnt = 0;
  for (int e0 = 0; e0 < n; e0 += kWave) {
    const int e = e0 + lane;
    const bool le = e < n && E[e].first <= blk;
    cnt += __popcll(__ballot(le));
    if (cnt < e0 + kWave) break;           // this chunk holds the first entry past blk
  }
  return cnt - 1;
}

__device__ __forceinline__ void block_entry(const BEntry* __restrict__ E, int n, int& se) {
  if (threadIdx.x < kWave) {
    const int e = find_entry_wave(E, n, blockIdx.x);
    if (threadIdx.x == 0) se = e;
  }
  __syncthreads();
}

// ---- work of a launch: blocks of kSliceWaves slices, those of inactive problems left out.
// A launch of more than kBatchGrid blocks (and up to 64 entries, one per lane) starts
// kBatchGrid workgroups that share the active problems' blocks, each XCD a contiguous range,
// so that the gathered neighbours of a slice come from its own L2 and problems that have
// converged cost nothing.  Smaller launches start one workgroup per block.
struct BatchWork {
  int start, total;                        // first block of the lane's entry; blocks of all entries
  bool strided;
};

__device__ __forceinline__ BatchWork batch_work(const BEntry* __restrict__ E, int ne, int nb,
                                                const int* __restrict__ active) {
  BatchWork w;
  w.strided = int(gridDim.x) < nb;
  w.start = INT_MAX;
  w.total = nb;
  if (!w.strided) return w;
  const int lane = int(threadIdx.x) % kWave;
  int n = 0;
  bool off = false;
  if (lane < ne) {
    w.start = E[lane].first;
    n = (lane + 1 < ne ? E[lane + 1].first : nb) - w.start;
    off = active && !active[E[lane].prob];
  }
  if (__ballot(off) == 0) return w;
  int sum = off ? 0 : n;                   // inclusive prefix sums over the entries
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int v = __shfl_up(sum, o, kWave);
    if (lane >= o) sum += v;
  }
  w.total = __shfl(sum, kWave - 1, kWave);
  if (lane < ne) w.start = sum - (off ? 0 : n);
  return w;
}

// entry and block of work item v: the last entry that starts at or before v (an inactive one
// starts where the next one does)
__device__ __forceinline__ int work_entry(const BatchWork& w, int v, int* blk) {
  const int e = __popcll(__ballot(w.start <= v)) - 1;
  *blk = v - __shfl(w.start, e, kWave);
  return __builtin_amdgcn_readfirstlane(e);
}

// f(entry, block of the entry) for this workgroup's share
template <class F>
__device__ __forceinline__ void for_batch(const BEntry* __restrict__ E, int ne, int nb,
                                          const int* __restrict__ active, F f) {
  const BatchWork w = batch_work(E, ne, nb, active);
  for (int v = int(blockIdx.x); v < w.total; v += int(gridDim.x)) {
    int e, blk;
    if (w.strided) {
      e = work_entry(w, xcd_remap(v, w.total), &blk);
    } else {
      e = __builtin_amdgcn_readfirstlane(find_entry_wave(E, ne, v));
      if (active && !active[E[e].prob]) return;
      blk = v - E[e].first;
    }
    f(E[e], __builtin_amdgcn_readfirstlane(blk));
  }
}

// ---- eight right-hand sides of one component: kRowLanes lanes per row, each with kRowRhs of the
// row's values, which lie together in memory.  With one lane per value every wave load of
// operator values brought 64 bytes for 64 lanes, and the vector memory pipe bound the sweep.
//
// Measured on 16 problems, 1.96M nodes together, 8 right-hand sides, FP64 (560 MB that a sweep
// moves): sweep 265 us with one lane per value and workgroups over all XCDs in turn, 169 us with 4
// lanes per row and the work shared as above; product 207 and 139, prolongation 110 and 68; with
// one of the problems left 28 and 14.8 us.  Whole solve 62.0 ms; 49.0 with 4 lanes per row, 45.6 with
// 2, 51.7 with 1.  Grids of 2,048 and 8,192 workgroups are within 0.5% of 4,096.
constexpr int kRowRhs = 8 / kRowLanes;
constexpr int kRows = kWave / kRowLanes;

template <class X>
struct RowVec {
  X v[kRowRhs];
};
template <class X>
__device__ __forceinline__ RowVec<X> row_load(const X* p) {      // 8-byte alignment is enough
  RowVec<X> r;
  __builtin_memcpy(&r, p, sizeof(r));
  return r;
}
template <class X>
__device__ __forceinline__ void row_store(X* p, const RowVec<X>& r) {
  __builtin_memcpy(p, &r, sizeof(r));
}

struct RowLane {
  int slice, r, node;
  int64_t at;                              // the lane's first value in a vector
  int q;                                   // its first right-hand side
  bool valid;
};
__device__ __forceinline__ RowLane row_lane(int n, int nslices, const int32_t* perm, int slice, int lane) {
  RowLane s;
  s.slice = __builtin_amdgcn_readfirstlane(slice);
  s.r = lane / kRowLanes;
  s.q = lane % kRowLanes * kRowRhs;
  const int pos = s.slice * kRows + s.r;
  s.valid = s.slice < nslices && pos < n;
  s.node = s.valid ? (perm ? perm[pos] : pos) : 0;
  s.at = int64_t(s.node) * 8 + s.q;
  return s;
}

// NB slots as in sell_batch: indices and values, then the gathers, then the multiply-adds
template <int NB, int K, class XI, class T, bool C16>
__device__ __forceinline__ void rows_batch(const SellDev& A, int k, const RowLane& s, const XI* __restrict__ x,
                                           T (&acc)[kRowRhs]) {
  unsigned js[NB];
  typename Val<K>::raw av[NB];
  RowVec<XI> xv[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int64_t e = int64_t(k + u) * kRows + s.r;
    js[u] = slot_col<C16, true>(A, k + u, e);
    av[u] = Val<K>::template load<true>(A.val, e);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < NB; ++u) xv[u] = row_load(x + uint64_t(js[u]) * 8 + s.q);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int i = 0; i < kRowRhs; ++i) acc[i] += T(Val<K>::dec(av[u])) * T(xv[u].v[i]);
}
template <int N, int K, class XI, class T, bool C16>
__device__ __forceinline__ void rows_rest(int rem, const SellDev& A, int k, const RowLane& s,
                                          const XI* __restrict__ x, T (&acc)[kRowRhs]) {
  if constexpr (N >= 1) {
    if (rem == N) rows_batch<N, K, XI, T, C16>(A, k, s, x, acc);
    else rows_rest<N - 1, K, XI, T, C16>(rem, A, k, s, x, acc);
  }
}
template <int K, class XI, class T, int KB, bool C16>
__device__ __forceinline__ void rows_loop(const SellDev& A, const RowLane& s, const XI* __restrict__ x,
                                          T (&acc)[kRowRhs]) {
  // The lane holds kRowRhs values per slot.  The default slot batch takes half the slots at a
  // time, for occupancy on large levels; the other one all 16, a 9-point row in one dependent
  // read, for small levels (16,641 nodes and two of 1,000, 16-bit values: sweep 5.4 and 4.4 us,
  // solve 3.86 and 3.64 ms); the setup times both.
  constexpr int NB = KB == kb_alt<1>() ? KB : KB / 2;
  int k, k1;
  slot_range(A, s.slice, k, k1);
  for (; k + NB <= k1; k += NB) rows_batch<NB, K, XI, T, C16>(A, k, s, x, acc);
  rows_rest<NB - 1, K, XI, T, C16>(k1 - k, A, k, s, x, acc);
}
template <int K, class XI, class T, int KB, bool C16>
__device__ __forceinline__ void rows_dot(const SellDev& A, const RowLane& s, const XI* __restrict__ x,
                                         T (&acc)[kRowRhs]) {
#pragma unroll
  for (int i = 0; i < kRowRhs; ++i) acc[i] = T(0);
  if (!s.valid) return;
  if (C16 && is_wide(A, s.slice)) rows_loop<K, XI, T, KB, false>(A, s, x, acc);
  else rows_loop<K, XI, T, KB, C16>(A, s, x, acc);
  if (K == VK_F16 || K == VK_BF16) {
    const T f = T(ldexpf(1.0f, A.rexp[int64_t(s.slice) * kRows + s.r]));
#pragma unroll
    for (int i = 0; i < kRowRhs; ++i) acc[i] *= f;
  }
}

// spmv_slice of one component for the lane's right-hand sides
template <int K, class XI, class XO, class T, int MODE, int KB, bool C16>
__device__ __forceinline__ RowVec<XO> rows_spmv(const SellDev& A, const XO* __restrict__ b, const XI* __restrict__ x,
                                          XO* __restrict__ y, const uint8_t* __restrict__ mask, int slice) {
  const RowLane s = row_lane(A.n, A.nslices, A.perm, slice, int(threadIdx.x) % kWave);
  RowVec<XO> bv = {};
  uint8_t mk = 0;
  if (MODE != 0 && s.valid) {
    bv = row_load(b + s.at);
    if (MODE == 2) mk = mask[s.node];
  }
  T acc[kRowRhs];
  rows_dot<K, XI, T, KB, C16>(A, s, x, acc);
  RowVec<XO> o;
#pragma unroll
  for (int i = 0; i < kRowRhs; ++i) {
    T out = T(0);
    if (s.valid) out = MODE == 0 ? acc[i] : T(bv.v[i]) - acc[i];
    if (MODE == 2 && mk) out = T(0);
    o.v[i] = XO(out);
  }
  if (s.valid) row_store(y + s.at, o);
  return o;
}

template <int K, class X, class T, int KB, bool C16>
__device__ __forceinline__ void rows_sweep(const SellDev& A, const X* __restrict__ S, const X* __restrict__ b,
                                           const X* __restrict__ x, X* __restrict__ xo, T omega, int slice) {
  const RowLane s = row_lane(A.n, A.nslices, A.perm, slice, int(threadIdx.x) % kWave);
  RowVec<X> bv = {}, xv = {};
  X sv = X(0);
  if (s.valid) {
    bv = row_load(b + s.at);
    xv = row_load(x + s.at);
    sv = S[int64_t(s.slice) * kRows + s.r];
  }
  T acc[kRowRhs];
  rows_dot<K, X, T, KB, C16>(A, s, x, acc);
  RowVec<X> o;
#pragma unroll
  for (int i = 0; i < kRowRhs; ++i) {
    T upd = T(0);
    upd += T(sv) * (T(bv.v[i]) - acc[i]);
    o.v[i] = X(T(xv.v[i]) + omega * upd);
  }
  if (s.valid) row_store(xo + s.at, o);
}

template <class X, class T>
__device__ __forceinline__ void rows_sweep0(const SellDev& A, const X* __restrict__ S, const X* __restrict__ b,
                                            X* __restrict__ xo, T omega, int slice) {
  const RowLane s = row_lane(A.n, A.nslices, A.perm, slice, int(threadIdx.x) % kWave);
  if (!s.valid) return;
  const RowVec<X> bv = row_load(b + s.at);
  const X sv = S[int64_t(s.slice) * kRows + s.r];
  RowVec<X> o;
#pragma unroll
  for (int i = 0; i < kRowRhs; ++i) {
    T upd = T(0);
    upd += T(sv) * T(bv.v[i]);
    o.v[i] = X(omega * upd);
  }
  row_store(xo + s.at, o);
}

// transfers, as tsell_lane
template <int NB, class X, class T, class WT, bool MC, bool NT>
__device__ __forceinline__ void trows_batch(const TSellDev& M, int k, const RowLane& s, const X* __restrict__ in,
                                            const uint8_t* __restrict__ mcol, T (&acc)[kRowRhs]) {
  unsigned js[NB];
  WT ws[NB];
  RowVec<X> vs[NB];
  uint8_t ms[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int64_t e = int64_t(k + u) * kRows + s.r;
    js[u] = unsigned(stream_load<NT>(M.col + e));
    ws[u] = stream_load<NT>(static_cast<const WT*>(M.w) + e);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    vs[u] = row_load(in + uint64_t(js[u]) * 8 + s.q);
    ms[u] = MC ? mcol[js[u]] : uint8_t(0);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int i = 0; i < kRowRhs; ++i) acc[i] += T(ws[u]) * (ms[u] ? T(0) : T(vs[u].v[i]));
}
template <int N, class X, class T, class WT, bool MC, bool NT>
__device__ __forceinline__ void trows_rest(int rem, const TSellDev& M, int k, const RowLane& s,
                                           const X* __restrict__ in, const uint8_t* __restrict__ mcol,
                                           T (&acc)[kRowRhs]) {
  if constexpr (N >= 1) {
    if (rem == N) trows_batch<N, X, T, WT, MC, NT>(M, k, s, in, mcol, acc);
    else trows_rest<N - 1, X, T, WT, MC, NT>(rem, M, k, s, in, mcol, acc);
  }
}
template <class X, class T, class WT, bool MC, bool NT>
__device__ __forceinline__ void trows_loop(const TSellDev& M, const RowLane& s, const X* __restrict__ in,
                                           const uint8_t* __restrict__ mcol, T (&acc)[kRowRhs]) {
  constexpr int KB = 4;
  int k, k1;
  slot_range(M, s.slice, k, k1);
  for (; k + KB <= k1; k += KB) trows_batch<KB, X, T, WT, MC, NT>(M, k, s, in, mcol, acc);
  trows_rest<KB - 1, X, T, WT, MC, NT>(k1 - k, M, k, s, in, mcol, acc);
}
template <class X, class T, class WT, bool MC, int MODE>
__device__ __forceinline__ void trows(const TSellDev& M, int slice, const X* __restrict__ in, X* __restrict__ out,
                                      const uint8_t* __restrict__ mrow, const uint8_t* __restrict__ mcol) {
  const RowLane s = row_lane(M.nrows, M.nslices, nullptr, slice, int(threadIdx.x) % kWave);
  if (!s.valid) return;
  const uint8_t masked = mrow[s.node];
  RowVec<X> old = {};
  if (MODE == 1) old = row_load(out + s.at);
  T acc[kRowRhs];
#pragma unroll
  for (int i = 0; i < kRowRhs; ++i) acc[i] = T(0);
  if (M.nt) trows_loop<X, T, WT, MC, true>(M, s, in, mcol, acc);
  else trows_loop<X, T, WT, MC, false>(M, s, in, mcol, acc);
  RowVec<X> o;
#pragma unroll
  for (int i = 0; i < kRowRhs; ++i) o.v[i] = MODE == 0 ? (masked ? X(0) : X(acc[i])) : X(T(old.v[i]) + acc[i]);
  if (MODE == 0 || !masked) row_store(out + s.at, o);
}

// V-cycle steps on slices (sweep0, sweep, masked defect) for every problem of the batch
template <int B, int NR, int K, class X, class T, int KIND, int KB, bool C16>
__global__ __launch_bounds__(kThreads) void k_bsell(const BEntry* __restrict__ E, int ne, int nb, T omega,
                                                    const int* __restrict__ active) {
  for_batch(E, ne, nb, active, [&](const BEntry& e, int blk) {
    const int slice = blk * kSliceWaves + int(threadIdx.x) / kWave;
    const X *S = static_cast<const X*>(e.S), *in0 = static_cast<const X*>(e.in0), *in1 = static_cast<const X*>(e.in1);
    X* out = static_cast<X*>(e.out);
    if constexpr (NR == 8) {
      if (KIND == BK_SWEEP0) rows_sweep0<X, T>(e.A, S, in0, out, omega, slice);
      else if (KIND == BK_SWEEP) rows_sweep<K, X, T, KB, C16>(e.A, S, in0, in1, out, omega, slice);
      else rows_spmv<K, X, X, T, 2, KB, C16>(e.A, in0, in1, out, e.mask, slice);
    } else {
      const SliceLane s = slice_lane<B>(e.A, slice, threadIdx.x % kWave);
      if (KIND == BK_SWEEP0) sweep0_slice<B, X, T>(S, in0, out, omega, s);
      else if (KIND == BK_SWEEP) sweep_slice<B, K, X, T, KB, C16, 1>(e.A, S, in0, in1, out, omega, s);
      else spmv_slice<B, K, X, X, T, 2, KB, C16, 1>(e.A, in0, in1, out, e.mask, s);
    }
  });
}

// fixed-order sum over the block of values that belong to rhs q = tid % NR; thread q of
// the result gets the sum for q
__device__ __forceinline__ double block_sum_rhs(double v, int NR, double* lds) {
  // inside each wave a fixed shuffle tree combines the lanes of equal lane % NR, then
  // thread q adds the per-wave results in wave order
  for (int o = kWave / 2; o >= NR; o >>= 1) v += __shfl_down(v, o, kWave);
  const int wv = threadIdx.x / kWave, ln = threadIdx.x % kWave;
  if (ln < NR) lds[wv * NR + ln] = v;
  __syncthreads();
  double t = 0.0;
  if (int(threadIdx.x) < NR)
    for (int k = 0; k < int(blockDim.x) / kWave; ++k) t += lds[k * NR + threadIdx.x];
  __syncthreads();
  return t;
}

// outer-loop products with the FP64 operator: w = A z (KIND SPMV64) or r = b - A x with
// partial sums of squares per (block, rhs) (KIND DEFECT64)
template <int B, int NR, class XI, int KIND, int KB, bool C16>
__global__ __launch_bounds__(kThreads) void k_bsell64(const BEntry* __restrict__ E, int ne, int nb,
                                                      const int* __restrict__ active, double* __restrict__ partials) {
  __shared__ double lds[kThreads];
  constexpr int MODE = KIND == BK_SPMV64 ? 0 : 1;
  for_batch(E, ne, nb, active, [&](const BEntry& e, int blk) {
    const int slice = blk * kSliceWaves + int(threadIdx.x) / kWave;
    const double* b = static_cast<const double*>(e.in0);
    const XI* x = static_cast<const XI*>(e.in1);
    double* y = static_cast<double*>(e.out);
    if constexpr (NR == 8) {
      const RowVec<double> out = rows_spmv<VK_F64, XI, double, double, MODE, KB, C16>(e.A, b, x, y, nullptr, slice);
      if (KIND == BK_DEFECT64) {
        // wave sums of equal right-hand sides, then the waves in order
        const int wv = int(threadIdx.x) / kWave, ln = int(threadIdx.x) % kWave;
#pragma unroll
        for (int i = 0; i < kRowRhs; ++i) {
          double v = out.v[i] * out.v[i];
          for (int o = kWave / 2; o >= kRowLanes; o >>= 1) v += __shfl_down(v, o, kWave);
          if (ln < kRowLanes) lds[wv * 8 + ln * kRowRhs + i] = v;
        }
        __syncthreads();
        if (threadIdx.x < 8) {
          double t = 0.0;
          for (int w = 0; w < kSliceWaves; ++w) t += lds[w * 8 + threadIdx.x];
          partials[int64_t(e.first + blk) * 8 + threadIdx.x] = t;
        }
        __syncthreads();
      }
    } else {
      const SliceLane s = slice_lane<B>(e.A, slice, threadIdx.x % kWave);
      const double out = spmv_slice<B, VK_F64, XI, double, double, MODE, KB, C16, 1>(e.A, b, x, y, nullptr, s);
      if (KIND == BK_DEFECT64) {
        const double t = block_sum_rhs(out * out, NR, lds);
        if (threadIdx.x < NR) partials[int64_t(e.first + blk) * NR + threadIdx.x] = t;
      }
    }
  });
}

template <int B, int NR, class X, class T, int KIND>
__global__ __launch_bounds__(kThreads) void k_belem(const BEntry* __restrict__ E, int ne,
                                                    const int* __restrict__ active) {
  __shared__ int se;
  block_entry(E, ne, se);
  const BEntry& e = E[se];
  if (active && !active[e.prob]) return;
  const int64_t t = int64_t(blockIdx.x - e.first) * kThreads + threadIdx.x;
  if (t < int64_t(e.A.n) * B * NR) static_cast<X*>(e.out)[t] = X(0);   // BK_FILL0
}

// restriction (rows = coarse nodes, row mask M_c) and prolongation + correction (rows =
// fine nodes, row mask M_f, column mask M_c) of every problem with the sliced transfers
template <int B, int NR, class X, class T, int KIND>
__global__ __launch_bounds__(kThreads) void k_btsell(const BEntry* __restrict__ E, int ne, int nb,
                                                     const int* __restrict__ active) {
  for_batch(E, ne, nb, active, [&](const BEntry& e, int blk) {
    const int slice = blk * kSliceWaves + int(threadIdx.x) / kWave;
    const int lane = int(threadIdx.x) % kWave;
    const X* in = static_cast<const X*>(e.in0);
    X* out = static_cast<X*>(e.out);
    if constexpr (NR == 8) {
      if (KIND == BK_RESTRICT) {
        if (e.Ts.f32) trows<X, T, float, false, 0>(e.Ts, slice, in, out, e.mask_c, nullptr);
        else trows<X, T, double, false, 0>(e.Ts, slice, in, out, e.mask_c, nullptr);
      } else {
        if (e.Ts.f32) trows<X, T, float, true, 1>(e.Ts, slice, in, out, e.mask, e.mask_c);
        else trows<X, T, double, true, 1>(e.Ts, slice, in, out, e.mask, e.mask_c);
      }
    } else if (KIND == BK_RESTRICT) {
      if (e.Ts.f32) tsell_lane<B, X, T, float, false, 0>(e.Ts, slice, lane, in, out, e.mask_c, nullptr);
      else tsell_lane<B, X, T, double, false, 0>(e.Ts, slice, lane, in, out, e.mask_c, nullptr);
    } else {
      if (e.Ts.f32) tsell_lane<B, X, T, float, true, 1>(e.Ts, slice, lane, in, out, e.mask, e.mask_c);
      else tsell_lane<B, X, T, double, true, 1>(e.Ts, slice, lane, in, out, e.mask, e.mask_c);
    }
  });
}

// coarse solve x = Ainv b for NR right-hand sides, one wavefront per row
template <int NR, class X>
__global__ __launch_bounds__(kThreads) void k_bcoarse(const BEntry* __restrict__ E, int ne,
                                                      const int* __restrict__ active) {
  __shared__ int se;
  block_entry(E, ne, se);
  const BEntry& e = E[se];
  if (active && !active[e.prob]) return;
  const int i = (blockIdx.x - e.first) * kSliceWaves + threadIdx.x / kWave;
  if (i >= e.n0) return;
  const int lane = threadIdx.x % kWave, q = lane % NR;
  const X* b = static_cast<const X*>(e.in0);
  constexpr int U = 8;
  double acc = 0.0;
  const double* row = e.Ainv + int64_t(i) * e.n0;
  for (int k0 = lane / NR; k0 < e.n0; k0 += (kWave / NR) * U) {
    double av[U];
    X bv[U];                                 // widened when used (no wait per element)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u * (kWave / NR);
      av[u] = k < e.n0 ? row[k] : 0.0;
      bv[u] = k < e.n0 ? b[int64_t(k) * NR + q] : X(0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc += av[u] * double(bv[u]);
  }
#pragma unroll
  for (int o = kWave / 2; o >= NR; o >>= 1) acc += __shfl_down(acc, o, kWave);
  if (lane < NR) static_cast<X*>(e.out)[int64_t(i) * NR + lane] = X(acc);
}

// The same product for the matrices of whole small levels (FP64): a workgroup has
// kDenseBlockRows rows, its lanes (waves side by side) the columns, so that a matrix row is read
// in full lines, the right-hand sides once for four rows, and 512 columns are one round of loads.
constexpr int kDenseBlockRows = 4;

template <int NR>
__global__ __launch_bounds__(kThreads) void k_bdense(const BEntry* __restrict__ E, int ne, int nb,
                                                     const int* __restrict__ active) {
  constexpr int P = kDenseBlockRows * NR, U = 2;
  __shared__ double lds[kSliceWaves][P];
  for_batch(E, ne, nb, active, [&](const BEntry& e, int blk) {
    const int n = e.n0, lane = int(threadIdx.x) % kWave, wave = int(threadIdx.x) / kWave;
    const int i0 = blk * kDenseBlockRows;
    const double* b = static_cast<const double*>(e.in0);
    const double* row[kDenseBlockRows];
#pragma unroll
    for (int r = 0; r < kDenseBlockRows; ++r) row[r] = e.Ainv + int64_t(min(i0 + r, n - 1)) * n;
    double acc[P];
#pragma unroll
    for (int q = 0; q < P; ++q) acc[q] = 0.0;
    for (int k0 = int(threadIdx.x); k0 < n; k0 += U * kThreads) {
      double a[U][kDenseBlockRows], bv[U][NR];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(k0 + u * kThreads, n - 1);
        const bool ok = k0 + u * kThreads < n;
#pragma unroll
        for (int r = 0; r < kDenseBlockRows; ++r) a[u][r] = ok ? row[r][k] : 0.0;
#pragma unroll
        for (int q = 0; q < NR; ++q) bv[u][q] = ok ? b[int64_t(k) * NR + q] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int r = 0; r < kDenseBlockRows; ++r)
#pragma unroll
          for (int q = 0; q < NR; ++q) acc[r * NR + q] += a[u][r] * bv[u][q];
    }
    int which = 0;
    wave_sums_step<P, kWave / 2, 1>(acc, lane, which);
    if (lane % (kWave / P) == 0) lds[wave][which] = acc[0];
    __syncthreads();
    if (int(threadIdx.x) < P && i0 + int(threadIdx.x) / NR < n) {
      double t = 0.0;
      for (int w = 0; w < kSliceWaves; ++w) t += lds[w][threadIdx.x];
      static_cast<double*>(e.out)[int64_t(i0) * NR + threadIdx.x] = t;
    }
    __syncthreads();
  });
}

// ---- segmented vector kernels: block -> problem segment, thread keeps rhs q = tid % NR
struct SegPos {
  int p, lb, nb, first;
  int64_t off, len;
  bool on;                                 // the problem takes part in this launch
};

__device__ __forceinline__ SegPos seg_pos(const BSegs& g) {
  SegPos s;
  s.p = g.blk_prob[blockIdx.x];
  s.first = g.vfirst[s.p];
  s.lb = blockIdx.x - s.first;
  s.nb = g.vcount[s.p];
  s.off = g.off[s.p];
  s.len = g.len[s.p];
  s.on = !g.on || g.on[s.p];
  return s;
}

// every block of problem p computes the per-rhs sums of the problem's partials
__device__ __forceinline__ void seg_sums(const double* __restrict__ pin, const SegPos& sp, int NR, double* lds,
                                         double* out) {
  constexpr int U = 8;                     // partial loads issued together
  double t = 0.0;
  const int q = threadIdx.x % NR;
  const int step = int(blockDim.x) / NR;
  const int first = sp.first, nb = sp.nb;
  for (int b0 = threadIdx.x / NR; b0 < nb; b0 += step * U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int b = b0 + u * step;
      v[u] = b < nb ? pin[int64_t(first + b) * NR + q] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) t += v[u];
  }
  const double r = block_sum_rhs(t, NR, lds);
  if (int(threadIdx.x) < NR) out[threadIdx.x] = r;
  __syncthreads();
}

__global__ __launch_bounds__(kThreads) void k_bdot(BSegs g, const double* __restrict__ a,
                                                   const double* __restrict__ b, double* __restrict__ out) {
  __shared__ double lds[kThreads];
  const SegPos sp = seg_pos(g);
  if (!sp.on) return;                      // uniform over the block
  constexpr int U = 4;
  double t = 0.0;
  const int64_t stride = int64_t(sp.nb) * blockDim.x;
  for (int64_t i0 = int64_t(sp.lb) * blockDim.x + threadIdx.x; i0 < sp.len; i0 += stride * U) {
    double av[U], bv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      av[u] = i < sp.len ? a[sp.off + i] : 0.0;
      bv[u] = (b && i < sp.len) ? b[sp.off + i] : av[u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) t += av[u] * bv[u];
  }
  const double r = block_sum_rhs(t, g.NR, lds);
  if (int(threadIdx.x) < g.NR) out[int64_t(blockIdx.x) * g.NR + threadIdx.x] = r;
}

// Gram-Schmidt in two passes over the basis, as for the single problem (mgq1_gs.hip):
//
//   k_bgs_dots     per block and right-hand side the partial sums of (w, v_i) and (v_j, v_i)
//   k_bgs_solve    adds them up per instance, h by the forward substitution
//   k_bgs_update   w -= sum_i h_i v_i in the order of i, partial sums of (w, w)
//
// Step j moves 2 (j + 1) + 4 vectors in 3 launches where a kernel per projection moved
// 4 (j + 1) + 2 in j + 2.  16 problems with 8 right-hand sides (126 MB a vector, 56 steps of a
// solve): 45.7 -> 42.1 ms.
template <int NV>
constexpr int bgs_unroll() { return NV <= 2 ? 4 : NV <= 5 ? 2 : 1; }

// sum q of block blk and right-hand side r at out[(q * NR + r) * blocks + blk]; q < NV: (w, v_q),
// else (v_j, v_{q - NV})
template <int NV, int NR>
__global__ __launch_bounds__(kThreads) void k_bgs_dots(BSegs g, const double* __restrict__ w,
                                                       const double* __restrict__ V, int64_t ldv,
                                                       const double* __restrict__ vj, double* __restrict__ out) {
  constexpr int NQ = 2 * NV, P = pow2_above(NQ), U = bgs_unroll<NV>();
  __shared__ double lds[kSliceWaves][NQ * NR];
  const SegPos sp = seg_pos(g);
  if (!sp.on) return;                      // uniform over the block
  double acc[P];
#pragma unroll
  for (int q = 0; q < P; ++q) acc[q] = 0.0;
  const int64_t stride = int64_t(sp.nb) * blockDim.x;
  for (int64_t i0 = int64_t(sp.lb) * blockDim.x + threadIdx.x; i0 < sp.len; i0 += stride * U) {
    double wv[U], uv[U], v[U][NV];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      const bool ok = i < sp.len;
      const int64_t e = sp.off + i;
      wv[u] = ok ? w[e] : 0.0;
      uv[u] = ok ? vj[e] : 0.0;
#pragma unroll
      for (int q = 0; q < NV; ++q) v[u][q] = ok ? V[int64_t(q) * ldv + e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        acc[q] += wv[u] * v[u][q];
        acc[NV + q] += uv[u] * v[u][q];
      }
  }
  const int lane = int(threadIdx.x) % kWave, wave = int(threadIdx.x) / kWave;
  int which = 0;
  wave_sums_step<P, kWave / 2, NR>(acc, lane, which);
  constexpr int left = P * NR / kWave > 1 ? P * NR / kWave : 1;
#pragma unroll
  for (int i = 0; i < left; ++i)           // several lanes may hold the same sum
    if (which + i < NQ) lds[wave][(which + i) * NR + lane % NR] = acc[i];
  __syncthreads();
  if (int(threadIdx.x) < NQ * NR) {
    double t = 0.0;
    for (int k = 0; k < kSliceWaves; ++k) t += lds[k][threadIdx.x];
    out[int64_t(threadIdx.x) * gridDim.x + blockIdx.x] = t;
  }
}

// h_0 .. h_j of every instance of the active problems, one block each; gram[k * m + i] of an
// instance is (v_i, v_k).  The sums of the vectors g0 .. of a group start at row 2 * g0.
__global__ __launch_bounds__(512) void k_bgs_solve(BSegs g, int j, int m, int group, const double* __restrict__ partials,
                                                   double* __restrict__ gram, double* __restrict__ H, int64_t hstride) {
  __shared__ double sd[kWave], sg[kWave];
  const int NR = g.NR, p = int(blockIdx.x) / NR, r = int(blockIdx.x) % NR;
  if (g.on && !g.on[p]) return;
  const int lane = int(threadIdx.x) % kWave, wv = int(threadIdx.x) / kWave, nw = int(blockDim.x) / kWave;
  const int first = g.vfirst[p], nb = g.vcount[p];
  for (int q = wv; q < 2 * (j + 1); q += nw) {
    const int g0 = (q / (2 * group)) * group, in = q - 2 * g0;
    const int gn = min(group, j + 1 - g0);
    const int kind = in >= gn ? 1 : 0, i = g0 + in - kind * gn;
    const double* row = partials + (int64_t(q) * NR + r) * g.n_blocks + first;
    constexpr int U = kSegBlocksMax / kWave;
    double v[U], t = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = lane + u * kWave < nb ? row[lane + u * kWave] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) t += v[u];
    t = wave_sum(t);
    if (lane == 0) (kind ? sg : sd)[i] = t;
  }
  __syncthreads();
  if (wv != 0) return;
  double* G = gram + int64_t(blockIdx.x) * m * m;
  double x = lane <= j ? sd[lane] : 0.0;
  for (int k = 0; k < j; ++k) {
    // row j's entries are this step's sums; the others were stored by their own steps
    const double gk = lane == j ? sg[k] : (lane > k && lane < j ? G[k * m + lane] : 0.0);
    const double hk = __shfl(x, k, kWave);
    if (lane > k && lane <= j) x -= gk * hk;
  }
  if (lane <= j) H[int64_t(blockIdx.x) * hstride + lane] = x;
  if (lane < j) G[lane * m + j] = sg[lane];
}

template <int NV>
__global__ __launch_bounds__(kThreads) void k_bgs_update(BSegs g, double* __restrict__ w, const double* __restrict__ V,
                                                         int64_t ldv, const double* __restrict__ H, int64_t hstride,
                                                         double* __restrict__ pout) {
  __shared__ double lds[kThreads];
  const SegPos sp = seg_pos(g);
  if (!sp.on) return;                      // uniform over the block
  constexpr int U = bgs_unroll<NV>();
  const double* h = H + int64_t(sp.p * g.NR + int(threadIdx.x) % g.NR) * hstride;
  double c[NV], t = 0.0;
#pragma unroll
  for (int q = 0; q < NV; ++q) c[q] = h[q];
  const int64_t stride = int64_t(sp.nb) * blockDim.x;
  for (int64_t i0 = int64_t(sp.lb) * blockDim.x + threadIdx.x; i0 < sp.len; i0 += stride * U) {
    double wv[U], v[U][NV];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      const bool ok = i < sp.len;
      const int64_t e = sp.off + i;
      wv[u] = ok ? w[e] : 0.0;
#pragma unroll
      for (int q = 0; q < NV; ++q) v[u][q] = ok ? V[int64_t(q) * ldv + e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      double x = wv[u];
#pragma unroll
      for (int q = 0; q < NV; ++q) x = x - c[q] * v[u][q];
      if (i < sp.len) {
        w[sp.off + i] = x;
        t += x * x;
      }
    }
  }
  const double s = block_sum_rhs(t, g.NR, lds);
  if (int(threadIdx.x) < g.NR) pout[int64_t(blockIdx.x) * g.NR + threadIdx.x] = s;
}

__global__ __launch_bounds__(kThreads) void k_bmgs_normalize(BSegs g, double* __restrict__ w,
                                                             const double* __restrict__ pin, double* __restrict__ H,
                                                             int64_t hstride, float* __restrict__ wc) {
  __shared__ double lds[kThreads];
  __shared__ double hq[64];
  const SegPos sp = seg_pos(g);
  if (!sp.on) return;                      // uniform over the block
  constexpr int U = 4;
  const int64_t stride = int64_t(sp.nb) * blockDim.x;
  double wv[U];
  auto load = [&](int64_t i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      wv[u] = i < sp.len ? w[sp.off + i] : 0.0;
    }
  };
  const int64_t first = int64_t(sp.lb) * blockDim.x + threadIdx.x;
  load(first);                             // independent of the norm (latency overlap)
  seg_sums(pin, sp, g.NR, lds, hq);
  if (int(threadIdx.x) < g.NR) hq[threadIdx.x] = sqrt(hq[threadIdx.x]);
  __syncthreads();
  if (sp.lb == 0 && int(threadIdx.x) < g.NR) H[int64_t(sp.p * g.NR + threadIdx.x) * hstride] = hq[threadIdx.x];
  const double nrm = hq[threadIdx.x % g.NR];
  if (nrm == 0.0) {
    if (wc)
      for (int64_t i = first; i < sp.len; i += stride) wc[sp.off + i] = float(w[sp.off + i]);
    return;
  }
  for (int64_t i0 = first; i0 < sp.len; i0 += stride * U) {
    if (i0 != first) load(i0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      if (i < sp.len) {
        const double v = wv[u] / nrm;
        w[sp.off + i] = v;
        if (wc) wc[sp.off + i] = float(v);
      }
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_bscale(BSegs g, double* __restrict__ y, const double* __restrict__ x,
                                                     const double* __restrict__ beta, const int* __restrict__ iact,
                                                     float* __restrict__ yc) {
  const SegPos sp = seg_pos(g);
  if (!sp.on) return;                      // uniform over the block
  const int inst = sp.p * g.NR + threadIdx.x % g.NR;
  const double bt = beta[inst];
  const bool on = iact[inst] && bt != 0.0;
  const int64_t stride = int64_t(sp.nb) * blockDim.x;
  for (int64_t i = int64_t(sp.lb) * blockDim.x + threadIdx.x; i < sp.len; i += stride) {
    const double v = on ? x[sp.off + i] / bt : 0.0;
    y[sp.off + i] = v;
    if (yc) yc[sp.off + i] = float(v);
  }
}

template <class Z>
__global__ __launch_bounds__(kThreads) void k_bupdate(BSegs g, double* __restrict__ x, const Z* __restrict__ Zm,
                                                      int64_t ldz, const double* __restrict__ yv, int m,
                                                      const int* __restrict__ kk) {
  const SegPos sp = seg_pos(g);
  if (!sp.on) return;                      // uniform over the block
  const int inst = sp.p * g.NR + threadIdx.x % g.NR;
  const int k = kk[inst];
  if (k == 0) return;
  const double* y = yv + int64_t(inst) * m;
  const int64_t stride = int64_t(sp.nb) * blockDim.x;
  for (int64_t i = int64_t(sp.lb) * blockDim.x + threadIdx.x; i < sp.len; i += stride) {
    const int64_t e = sp.off + i;
    double acc = x[e];
    for (int c = 0; c < k; ++c) acc += y[c] * double(Zm[int64_t(c) * ldz + e]);
    x[e] = acc;
  }
}

__global__ __launch_bounds__(kThreads) void k_bfinish(const double* __restrict__ p, const int* __restrict__ pfirst,
                                                      const int* __restrict__ pcount, int NR, double* out, int sq) {
  __shared__ double lds[kMaxWaves + 1];
  const int inst = blockIdx.x, pr = inst / NR, q = inst % NR;
  double t = 0.0;
  for (int b = threadIdx.x; b < pcount[pr]; b += blockDim.x) t += p[int64_t(pfirst[pr] + b) * NR + q];
  const double s = block_allsum(t, lds);
  if (threadIdx.x == 0) out[inst] = sq ? sqrt(s) : s;
}

__global__ void k_bgivens(int j, int m, int n_inst, double* H, double* cs, double* sn, double* g, double* st,
                          const double* __restrict__ tol, int* kk, const int* __restrict__ iact) {
  const int inst = blockIdx.x * blockDim.x + threadIdx.x;
  // rotations after the instance's cycle has closed are never used
  if (inst >= n_inst || !iact[inst] || kk[inst] != 0) return;
  const int ld = m + 1;
  double* h = H + int64_t(inst) * ld * m + int64_t(j) * ld;
  double* c = cs + int64_t(inst) * m;
  double* s = sn + int64_t(inst) * m;
  double* gg = g + int64_t(inst) * ld;
  const bool breakdown = h[j + 1] == 0.0;
  for (int i = 0; i < j; ++i) {
    const double t = c[i] * h[i] + s[i] * h[i + 1];
    h[i + 1] = -s[i] * h[i] + c[i] * h[i + 1];
    h[i] = t;
  }
  const double den = hypot(h[j], h[j + 1]);
  c[j] = h[j] / den;
  s[j] = h[j + 1] / den;
  h[j] = den;
  h[j + 1] = 0.0;
  gg[j + 1] = -s[j] * gg[j];
  gg[j] = c[j] * gg[j];
  st[2 * inst] = fabs(gg[j + 1]);
  st[2 * inst + 1] = breakdown ? 1.0 : 0.0;
  // closes on breakdown, on the tolerance, or on a non-finite estimate (!(x > tol))
  if (kk[inst] == 0 && (breakdown || !(fabs(gg[j + 1]) > tol[inst]))) kk[inst] = j + 1;
}

__global__ void k_bbacksolve(int m, int n_inst, const double* H, const double* g, double* yv, const int* kk) {
  const int inst = blockIdx.x * blockDim.x + threadIdx.x;
  if (inst >= n_inst) return;
  const int k = kk[inst];
  const int ld = m + 1;
  const double* Hh = H + int64_t(inst) * ld * m;
  const double* gg = g + int64_t(inst) * ld;
  double* y = yv + int64_t(inst) * m;
  for (int i = k - 1; i >= 0; --i) {
    double t = gg[i];
    for (int c = i + 1; c < k; ++c) t -= Hh[int64_t(c) * ld + i] * y[c];
    y[i] = t / Hh[int64_t(i) * ld + i];
  }
}

__global__ void k_binit(int m, int n_inst, double* g, const double* beta, int* kk) {
  const int inst = blockIdx.x * blockDim.x + threadIdx.x;
  if (inst >= n_inst) return;
  double* gg = g + int64_t(inst) * (m + 1);
  gg[0] = beta[inst];
  for (int i = 1; i <= m; ++i) gg[i] = 0.0;
  kk[inst] = 0;
}

__global__ void k_bclose(int j, int n_inst, int* kk, const int* iact) {
  const int inst = blockIdx.x * blockDim.x + threadIdx.x;
  if (inst < n_inst && iact[inst] && kk[inst] == 0) kk[inst] = j + 1;
}

template <int B, int NR, int K, class X, class T, int KB, bool C16>
hipError_t batched_sell(int kind, const BEntry* E, int ne, int nb, int g, double omega, const int* active,
                        double* partials, hipStream_t s) {
  switch (kind) {
    case BK_SWEEP: hipLaunchKernelGGL((k_bsell<B, NR, K, X, T, BK_SWEEP, KB, C16>), g, kThreads, 0, s, E, ne, nb, T(omega), active); break;
    case BK_DEFECT: hipLaunchKernelGGL((k_bsell<B, NR, K, X, T, BK_DEFECT, KB, C16>), g, kThreads, 0, s, E, ne, nb, T(omega), active); break;
    case BK_SPMV64: hipLaunchKernelGGL((k_bsell64<B, NR, X, BK_SPMV64, KB, C16>), g, kThreads, 0, s, E, ne, nb, active, partials); break;
    case BK_DEFECT64: hipLaunchKernelGGL((k_bsell64<B, NR, double, BK_DEFECT64, KB, C16>), g, kThreads, 0, s, E, ne, nb, active, partials); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int B, int NR, int K, class X, class T>
hipError_t batched_t(int kind, const BEntry* E, int ne, int nb, int g, double omega, const int* active, double* partials,
                     int kb, hipStream_t s) {
  switch (kind) {
    case BK_SWEEP: case BK_DEFECT: case BK_SPMV64: case BK_DEFECT64:
      // kb < 0 selects the 16-bit column format (every entry of the launch has it)
      if (kb < 0) {
        if (-kb == kb_alt<B>()) return batched_sell<B, NR, K, X, T, kb_alt<B>(), true>(kind, E, ne, nb, g, omega, active, partials, s);
        return batched_sell<B, NR, K, X, T, kb_default<B>(), true>(kind, E, ne, nb, g, omega, active, partials, s);
      }
      if (kb == kb_alt<B>()) return batched_sell<B, NR, K, X, T, kb_alt<B>(), false>(kind, E, ne, nb, g, omega, active, partials, s);
      return batched_sell<B, NR, K, X, T, kb_default<B>(), false>(kind, E, ne, nb, g, omega, active, partials, s);
    case BK_SWEEP0: hipLaunchKernelGGL((k_bsell<B, NR, K, X, T, BK_SWEEP0, kb_default<B>(), false>), g, kThreads, 0, s, E, ne, nb, T(omega), active); break;
    case BK_RESTRICT: hipLaunchKernelGGL((k_btsell<B, NR, X, T, BK_RESTRICT>), g, kThreads, 0, s, E, ne, nb, active); break;
    case BK_PROLONG: hipLaunchKernelGGL((k_btsell<B, NR, X, T, BK_PROLONG>), g, kThreads, 0, s, E, ne, nb, active); break;
    case BK_FILL0: hipLaunchKernelGGL((k_belem<B, NR, X, T, BK_FILL0>), nb, kThreads, 0, s, E, ne, active); break;
    case BK_COARSE: hipLaunchKernelGGL((k_bcoarse<NR, X>), nb, kThreads, 0, s, E, ne, active); break;
    case BK_DENSE:
      if constexpr (sizeof(X) != 8) return hipErrorInvalidValue;
      else hipLaunchKernelGGL(k_bdense<NR>, g, kThreads, 0, s, E, ne, nb, active);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int B, int NR>
hipError_t batched_bn(int kind, const BEntry* E, int ne, int nb, int g, int vkind, int xk, double omega, const int* active,
                      double* partials, int kb, hipStream_t s) {
  if (xk == X_F64) {
    if (vkind != VK_F64) return hipErrorInvalidValue;
    return batched_t<B, NR, VK_F64, double, double>(kind, E, ne, nb, g, omega, active, partials, kb, s);
  }
  switch (vkind) {
    case VK_F32: return batched_t<B, NR, VK_F32, float, float>(kind, E, ne, nb, g, omega, active, partials, kb, s);
    case VK_F16: return batched_t<B, NR, VK_F16, float, float>(kind, E, ne, nb, g, omega, active, partials, kb, s);
    case VK_BF16: return batched_t<B, NR, VK_BF16, float, float>(kind, E, ne, nb, g, omega, active, partials, kb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int batched_blocks(int kind, const SellDev& A, const TSellDev& Ts, int n0, int NR) {
  switch (kind) {
    case BK_SWEEP0: case BK_SWEEP: case BK_DEFECT: case BK_SPMV64: case BK_DEFECT64:
      return int(slice_grid(A.nslices));
    case BK_RESTRICT: case BK_PROLONG:
      return int(slice_grid(Ts.nslices));
    case BK_FILL0:
      return int(grid_for(int64_t(A.n) * A.B * NR, kThreads));
    case BK_COARSE:
      return int(grid_for(n0, kSliceWaves));
    case BK_DENSE:
      return int(grid_for(n0, kDenseBlockRows));
    default:
      return 0;
  }
}

hipError_t launch_batched(int kind, const BEntry* E, int ne, int nb, int B, int NR, int vkind, int xk, double omega,
                          const int* active, double* partials, int kb, int grid, hipStream_t s) {
  if (nb == 0 || ne == 0) return hipSuccess;
  const int g = ne <= kWave && nb > grid ? grid : nb;
  if (NR == 1) {
    switch (B) {
      case 1: return batched_bn<1, 1>(kind, E, ne, nb, g, vkind, xk, omega, active, partials, kb, s);
      case 3: return batched_bn<3, 1>(kind, E, ne, nb, g, vkind, xk, omega, active, partials, kb, s);
      case 4: return batched_bn<4, 1>(kind, E, ne, nb, g, vkind, xk, omega, active, partials, kb, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (NR == 8) {
    switch (B) {
      case 1: return batched_bn<1, 8>(kind, E, ne, nb, g, vkind, xk, omega, active, partials, kb, s);
      default: return hipErrorInvalidValue;
    }
  }
  return hipErrorInvalidValue;
}

hipError_t launch_bdot(const BSegs& g, const double* a, const double* b, double* partials, hipStream_t s) {
  hipLaunchKernelGGL(k_bdot, g.n_blocks, kThreads, 0, s, g, a, b, partials);
  return hipGetLastError();
}

hipError_t launch_bfinish(const double* partials, const int* pfirst, const int* pcount, int n_inst, int NR,
                          double* out, int sqrt_out, hipStream_t s) {
  hipLaunchKernelGGL(k_bfinish, n_inst, kThreads, 0, s, partials, pfirst, pcount, NR, out, sqrt_out);
  return hipGetLastError();
}

namespace {
template <int NV>
hipError_t bgs_dots_n(int nv, const BSegs& g, const double* w, const double* V, int64_t ldv, const double* vj, double* out,
                      hipStream_t s) {
  if constexpr (NV >= 1) {
    if (nv != NV) return bgs_dots_n<NV - 1>(nv, g, w, V, ldv, vj, out, s);
    if (g.NR == 8) hipLaunchKernelGGL((k_bgs_dots<NV, 8>), g.n_blocks, kThreads, 0, s, g, w, V, ldv, vj, out);
    else hipLaunchKernelGGL((k_bgs_dots<NV, 1>), g.n_blocks, kThreads, 0, s, g, w, V, ldv, vj, out);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <int NV>
hipError_t bgs_update_n(int nv, const BSegs& g, double* w, const double* V, int64_t ldv, const double* H, int64_t hstride,
                        double* pout, hipStream_t s) {
  if constexpr (NV >= 1) {
    if (nv != NV) return bgs_update_n<NV - 1>(nv, g, w, V, ldv, H, hstride, pout, s);
    hipLaunchKernelGGL(k_bgs_update<NV>, g.n_blocks, kThreads, 0, s, g, w, V, ldv, H, hstride, pout);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_bgram_schmidt(const BSegs& g, int n_inst, int j, int m, int64_t ldv, double* w, const double* V,
                                double* partials, double* gram, double* H, int64_t hstride, double* pnorm,
                                hipStream_t s) {
  if ((g.NR != 1 && g.NR != 8) || j >= kWave) return hipErrorInvalidValue;
  const int nv = j + 1;
  const double* vj = V + int64_t(j) * ldv;
  hipError_t e;
  for (int i = 0; i < nv; i += kGsGroup)
    if ((e = bgs_dots_n<kGsGroup>(std::min(nv - i, kGsGroup), g, w, V + int64_t(i) * ldv, ldv, vj,
                                  partials + int64_t(2) * i * g.NR * g.n_blocks, s)) != hipSuccess)
      return e;
  hipLaunchKernelGGL(k_bgs_solve, n_inst, 512, 0, s, g, j, m, kGsGroup, partials, gram, H, hstride);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int i = 0; i < nv; i += kGsGroup)
    if ((e = bgs_update_n<kGsGroup>(std::min(nv - i, kGsGroup), g, w, V + int64_t(i) * ldv, ldv, H + i, hstride, pnorm,
                                    s)) != hipSuccess)
      return e;
  return hipSuccess;
}

hipError_t launch_bmgs_normalize(const BSegs& g, double* w, const double* pin, double* H, int64_t hstride,
                                 hipStream_t s, float* wc) {
  hipLaunchKernelGGL(k_bmgs_normalize, g.n_blocks, kThreads, 0, s, g, w, pin, H, hstride, wc);
  return hipGetLastError();
}

hipError_t launch_bscale(const BSegs& g, double* y, const double* x, const double* beta, const int* iact,
                         hipStream_t s, float* yc) {
  hipLaunchKernelGGL(k_bscale, g.n_blocks, kThreads, 0, s, g, y, x, beta, iact, yc);
  return hipGetLastError();
}

hipError_t launch_bupdate(const BSegs& g, double* x, const void* Z, int zk, int64_t ldz, const double* yv, int m,
                          const int* kk, hipStream_t s) {
  if (zk == X_F64)
    hipLaunchKernelGGL(k_bupdate<double>, g.n_blocks, kThreads, 0, s, g, x, static_cast<const double*>(Z), ldz, yv, m, kk);
  else
    hipLaunchKernelGGL(k_bupdate<float>, g.n_blocks, kThreads, 0, s, g, x, static_cast<const float*>(Z), ldz, yv, m, kk);
  return hipGetLastError();
}

hipError_t launch_bgivens(int j, int m, int n_inst, double* H, double* cs, double* sn, double* g, double* st,
                          const double* tol, int* kk, const int* iact, hipStream_t s) {
  hipLaunchKernelGGL(k_bgivens, grid_for(n_inst, 64), 64, 0, s, j, m, n_inst, H, cs, sn, g, st, tol, kk, iact);
  return hipGetLastError();
}

hipError_t launch_bbacksolve(int m, int n_inst, const double* H, const double* g, double* yv, const int* kk,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_bbacksolve, grid_for(n_inst, 64), 64, 0, s, m, n_inst, H, g, yv, kk);
  return hipGetLastError();
}

hipError_t launch_binit(int m, int n_inst, double* g, const double* beta, int* kk, hipStream_t s) {
  hipLaunchKernelGGL(k_binit, grid_for(n_inst, 64), 64, 0, s, m, n_inst, g, beta, kk);
  return hipGetLastError();
}

hipError_t launch_bclose(int j, int n_inst, int* kk, const int* iact, hipStream_t s) {
  hipLaunchKernelGGL(k_bclose, grid_for(n_inst, 64), 64, 0, s, j, n_inst, kk, iact);
  return hipGetLastError();
}

}  // namespace mgq1
