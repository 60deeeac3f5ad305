// Kernels of the node form: operators whose rows repeat (constant coefficients on box cells).
//
// Setup stores each distinct B x B block of such a level once, finds the distinct rows
// (sequences of blocks) and groups 64 node rows of equal content into slices; one wavefront
// runs one slice, one lane one node with its B components.  A slice is of one of these
// kinds, named in its descriptor:
//
//   values   uniform   all its rows have the same blocks: they are read once per wave through
//                      the scalar cache (8 B^2 bytes per slot instead of 64 * 8 B^2) and
//                      enter the multiply-adds as scalar operands
//            general   a 16-bit block number per row and slot, the block read per lane
//   columns  uniform   all rows have the same column offsets: nothing is stored per row, the
//                      64 lanes read the neighbours' vector as one run.  With several
//                      components the runs are staged in LDS: the lanes' B values lie B apart, so
//                      reading them component by component and slot by slot touches every cache
//                      line several times, and the 3 slots of a mesh line read almost the same run
//            16-bit    offsets from the slot's smallest column (32-bit where they do not fit)
//
// The sliced-ELL form of the same operator streams 8 B^2 + 2 bytes per block; here a block
// costs 0 to 4 bytes, and what is left to move is the vectors.  Why one lane per node: the
// scalar operands then serve 64 nodes instead of 64 / B, a lane holds the B residuals that
// the smoother combines, and a neighbour's B components are one contiguous read.  The
// slots run in the row's order and the B products of a block in component order with the
// sliced-ELL kernels' expressions, so every result has the same bits.
//
// Measured, finest-level FP64 sweep, sliced ELL and node form: 129^3 elasticity (staged runs)
// 838 and 66 us, face-refined elasticity (43% of the slices with 16-bit columns) 243 and 51 us
// (FP16 values 96 and 32 us), 1.0M-node 2D annulus mesh 18.7 and 12.8 us, uniform 1025^2 mesh
// 18.8 and 11.3 us.  The 129^3 sweep moves 170 MB of vectors (31 us at the copy rate); the rest
// is the chain of a wave's dependent reads (descriptor, positions, runs, three phases).
#include "mgq1_device.h"

namespace mgq1 {
namespace {

// pointers to data that no kernel of the library writes while one reads it: uniform loads
// through them go through the scalar cache
template <class T> using ConstPtr = const T __attribute__((address_space(4)))*;
template <class T>
__device__ __forceinline__ ConstPtr<T> as_const(const void* p) {
  return (ConstPtr<T>)(reinterpret_cast<unsigned long long>(p));
}

// Slots whose vector loads are issued together.  Deep batches: a 9-point row in one, a 27-point
// row in three.  Shallow ones leave registers for 6 instead of 4 waves per SIMD in the FP64
// kernels of 2 and 3 components: better where most slices read staged runs from LDS
// (129^3 elasticity sweep 66 us, deep 78 us), worse where they gather from memory (face-refined
// elasticity 62 and 51 us); chosen per level by its slices (NodeDev::shallow).
template <bool DEEP> constexpr int node_batch_size() { return DEEP ? 9 : 3; }
template <bool DEEP> constexpr int node_min_waves() { return DEEP ? 1 : 6; }
constexpr int kRunBatch = 3;          // slots read from LDS together
// slots whose uniform blocks are read together: about 56 scalar registers of them
template <int B, class T> constexpr int scalar_group() {
  constexpr int g = 56 / (B * B * int(sizeof(T)) / 4);
  return g < 1 ? 1 : g > 9 ? 9 : g;
}

struct NodeLane {
  int slice, pos, node;     // pos: row position (last row repeated past the end)
  bool valid;
  int width, flags, iv, ic; // the slice's descriptor
};

__device__ __forceinline__ NodeLane node_lane(const NodeDev& A, int slice, int lane) {
  NodeLane s;
  s.slice = __builtin_amdgcn_readfirstlane(slice);
  const int pos = s.slice * kWave + lane;
  s.valid = pos < A.n;
  s.pos = s.valid ? pos : A.n - 1;
  s.node = A.perm ? A.perm[s.pos] : s.pos;
  const ConstPtr<int> d = as_const<int>(A.desc) + int64_t(s.slice) * 4;
  s.width = d[0];
  s.flags = d[1];
  s.iv = d[2];
  s.ic = d[3];
  return s;
}

// what a neighbour contributes: its vector entries, or (Z) those of the first sweep from
// zero x1_j = omega S_j b_j, formed on the fly for one component.  o: the neighbour's byte
// offset in the vector (below 2^32, checked at setup)
template <int B, class X>
struct GatherX {
  const X* x;
  using raw = X;
  static constexpr unsigned kStride = B * sizeof(X);
  __device__ __forceinline__ void load(unsigned o, X (&v)[B]) const {
    const X* p = reinterpret_cast<const X*>(reinterpret_cast<const char*>(x) + o);
#pragma unroll
    for (int c = 0; c < B; ++c) v[c] = p[c];
  }
  template <class T>
  __device__ __forceinline__ T get(const X (&v)[B], int c) const { return T(v[c]); }
};
template <class X, class T>
struct GatherZ {
  const X *S, *b;
  T omega;
  using raw = X;
  static constexpr unsigned kStride = sizeof(X);
  __device__ __forceinline__ void load(unsigned o, X (&v)[2]) const {
    v[0] = *reinterpret_cast<const X*>(reinterpret_cast<const char*>(S) + o);
    v[1] = *reinterpret_cast<const X*>(reinterpret_cast<const char*>(b) + o);
  }
  template <class TT>
  __device__ __forceinline__ TT get(const X (&v)[2], int) const {
    return TT(X(omega * (T(0) + T(v[0]) * T(v[1]))));
  }
};

// NB slots of a slice.  VU: uniform values; CK: 0 uniform columns, 1 16-bit, 2 32-bit.  First
// every index, then every gather of the batch, then the multiply-adds in slot order.
template <int NB, int B, class T, class G, int NR, bool VU, int CK>
__device__ __forceinline__ void node_batch(const NodeDev& A, const NodeLane& s, int lane, int k, const G& gx,
                                           T (&acc)[B]) {
  using X = typename G::raw;
  X v[NB][NR];
  unsigned id[NB];
  if constexpr (CK == 0) {
    const ConstPtr<int> off = as_const<int>(A.opat) + s.ic + k;
#pragma unroll
    for (int q = 0; q < NB; ++q) gx.load(unsigned(s.node) * G::kStride + unsigned(off[q]) * G::kStride, v[q]);
  } else if constexpr (CK == 1) {
    unsigned j[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) j[q] = A.col16[(int64_t(s.ic) + k + q) * kWave + lane];
    if constexpr (!VU) {
#pragma unroll
      for (int q = 0; q < NB; ++q) id[q] = A.didx[(int64_t(s.iv) + k + q) * kWave + lane];
    }
    const ConstPtr<int> base = as_const<int>(A.base) + s.ic + k;
#pragma unroll
    for (int q = 0; q < NB; ++q) gx.load(unsigned(base[q]) * G::kStride + j[q] * G::kStride, v[q]);
  } else {
    unsigned j[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) j[q] = unsigned(A.col32[(int64_t(s.ic) + k + q) * kWave + lane]);
    if constexpr (!VU) {
#pragma unroll
      for (int q = 0; q < NB; ++q) id[q] = A.didx[(int64_t(s.iv) + k + q) * kWave + lane];
    }
#pragma unroll
    for (int q = 0; q < NB; ++q) gx.load(j[q] * G::kStride, v[q]);
  }
  if constexpr (VU) {
    const ConstPtr<T> a = as_const<T>(A.vtab) + (int64_t(s.iv) + k) * (B * B);
    constexpr int G0 = scalar_group<B, T>();
#pragma unroll
    for (int q0 = 0; q0 < NB; q0 += G0) {
      __builtin_amdgcn_sched_barrier(0);   // or every block's load moves up and the registers run out
#pragma unroll
      for (int q = q0; q < (q0 + G0 < NB ? q0 + G0 : NB); ++q)
#pragma unroll
        for (int c = 0; c < B; ++c)
#pragma unroll
          for (int cc = 0; cc < B; ++cc) acc[c] += a[q * B * B + c * B + cc] * gx.template get<T>(v[q], cc);
    }
  } else {
    const T* tab = static_cast<const T*>(A.dtab);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const T* a = tab + uint64_t(id[q]) * (B * B);
#pragma unroll
      for (int c = 0; c < B; ++c)
#pragma unroll
        for (int cc = 0; cc < B; ++cc) acc[c] += a[c * B + cc] * gx.template get<T>(v[q], cc);
    }
  }
}

template <int N, int B, class T, class G, int NR, bool VU, int CK>
__device__ __forceinline__ void node_rest(int rem, const NodeDev& A, const NodeLane& s, int lane, int k, const G& gx,
                                          T (&acc)[B]) {
  if constexpr (N >= 1) {
    if (rem == N) node_batch<N, B, T, G, NR, VU, CK>(A, s, lane, k, gx, acc);
    else node_rest<N - 1, B, T, G, NR, VU, CK>(rem, A, s, lane, k, gx, acc);
  }
}

template <int B, class T, class G, int NR, bool VU, int CK, bool DEEP>
__device__ __forceinline__ void node_loop(const NodeDev& A, const NodeLane& s, int lane, const G& gx, T (&acc)[B]) {
  constexpr int KB = node_batch_size<DEEP>();
  int k = 0;
  for (; k + KB <= s.width; k += KB) node_batch<KB, B, T, G, NR, VU, CK>(A, s, lane, k, gx, acc);
  node_rest<KB - 1, B, T, G, NR, VU, CK>(s.width - k, A, s, lane, k, gx, acc);
}

// One slice whose offsets form runs: per phase up to three runs of consecutive columns are read
// with full cache lines, put into the wave's LDS area, and the phase's slots read from there
// (lane stride B elements: no bank conflicts for B = 3).  The next phase's reads are in flight
// during a phase's products.
template <class X, int B> constexpr int stage_elems() { return kPhaseRuns * kRunStride * B; }

template <int NB, int B, class T, class X>
__device__ __forceinline__ void run_batch(const NodeDev& A, const NodeLane& s, int k, ConstPtr<int> place,
                                          const X* stage, int rel, T (&acc)[B]) {
  X v[NB][B];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int c = 0; c < B; ++c) v[q][c] = stage[place[k + q] * B + rel + c];
  const ConstPtr<T> a = as_const<T>(A.vtab) + (int64_t(s.iv) + k) * (B * B);
  constexpr int G0 = scalar_group<B, T>();
#pragma unroll
  for (int q0 = 0; q0 < NB; q0 += G0) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = q0; q < (q0 + G0 < NB ? q0 + G0 : NB); ++q)
#pragma unroll
      for (int c = 0; c < B; ++c)
#pragma unroll
        for (int cc = 0; cc < B; ++cc) acc[c] += a[q * B * B + c * B + cc] * T(v[q][cc]);
  }
}

template <int N, int B, class T, class X>
__device__ __forceinline__ void run_rest(int rem, const NodeDev& A, const NodeLane& s, int k, ConstPtr<int> place,
                                         const X* stage, int rel, T (&acc)[B]) {
  if constexpr (N >= 1) {
    if (rem == N) run_batch<N, B, T, X>(A, s, k, place, stage, rel, acc);
    else run_rest<N - 1, B, T, X>(rem, A, s, k, place, stage, rel, acc);
  }
}

template <int B, class T, class X>
__device__ __forceinline__ void node_runs(const NodeDev& A, const NodeLane& s, int lane, const X* __restrict__ x,
                                          X* stage, T (&acc)[B]) {
  constexpr int NLD = (kRunStride * B + kWave - 1) / kWave;
  constexpr int KB = kRunBatch;
  const ConstPtr<int> rec = as_const<int>(A.rpat) + s.ic;
  const int nph = rec[0];
  const ConstPtr<int> place = rec + 1 + nph * kPhaseInts;
  const int node0 = __builtin_amdgcn_readlane(s.node, 0);
  const int span = __builtin_amdgcn_readlane(s.node, kWave - 1) - node0 + 1;
  const int rel = (s.node - node0) * B;
  X v[kPhaseRuns][NLD];
  auto load = [&](int p) {
    const ConstPtr<int> ph = rec + 1 + p * kPhaseInts;
#pragma unroll
    for (int q = 0; q < kPhaseRuns; ++q) {
      // columns node0 + start .. node0 + start + span + width - 2: the first is a column of
      // the first row, the last one of the last row, so all are in range
      const int w = ph[2 + 2 * q], cnt = w > 0 ? (span + w - 1) * B : 0;
      const X* src = x + int64_t(node0 + ph[1 + 2 * q]) * B;
#pragma unroll
      for (int u = 0; u < NLD; ++u) {
        const int e = lane + u * kWave;
        if (e < cnt) v[q][u] = src[e];
      }
    }
  };
  load(0);
  int k = 0;
  for (int p = 0; p < nph; ++p) {
    const ConstPtr<int> ph = rec + 1 + p * kPhaseInts;
#pragma unroll
    for (int q = 0; q < kPhaseRuns; ++q) {
      const int w = ph[2 + 2 * q], cnt = w > 0 ? (span + w - 1) * B : 0;
#pragma unroll
      for (int u = 0; u < NLD; ++u) {
        const int e = lane + u * kWave;
        if (e < cnt) stage[q * kRunStride * B + e] = v[q][u];
      }
    }
    // the wave's LDS accesses execute in order; the fences keep the compiler's order too
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (p + 1 < nph) load(p + 1);
    const int k1 = ph[0];
    for (; k + KB <= k1; k += KB) run_batch<KB, B, T, X>(A, s, k, place, stage, rel, acc);
    run_rest<KB - 1, B, T, X>(k1 - k, A, s, k, place, stage, rel, acc);
    k = k1;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// this wave's staging area (none for one component)
template <class X, int B>
__device__ __forceinline__ X* wave_stage() {
  if constexpr (B == 1) {
    return nullptr;
  } else {
    __shared__ X area[kSliceWaves][stage_elems<X, B>()];
    return area[int(threadIdx.x) / kWave];
  }
}

// the B row sums of the lane's node; T is also the type of the block tables
template <int B, class T, class G, int NR, bool DEEP>
__device__ __forceinline__ void node_dot(const NodeDev& A, const NodeLane& s, int lane, const G& gx,
                                         typename G::raw* stage, T (&acc)[B]) {
#pragma unroll
  for (int c = 0; c < B; ++c) acc[c] = T(0);
  if (s.flags & kNodeValUniform) {
    if (B >= 2 && (s.flags & kNodeRuns)) {
      if constexpr (B >= 2) node_runs<B, T, typename G::raw>(A, s, lane, gx.x, stage, acc);
    } else if (s.flags & kNodeColUniform) node_loop<B, T, G, NR, true, 0, DEEP>(A, s, lane, gx, acc);
    else if (s.flags & kNodeCol32) node_loop<B, T, G, NR, true, 2, DEEP>(A, s, lane, gx, acc);
    else node_loop<B, T, G, NR, true, 1, DEEP>(A, s, lane, gx, acc);
  } else {
    if (s.flags & kNodeCol32) node_loop<B, T, G, NR, false, 2, DEEP>(A, s, lane, gx, acc);
    else node_loop<B, T, G, NR, false, 1, DEEP>(A, s, lane, gx, acc);
  }
  if (A.rexp) {
#pragma unroll
    for (int c = 0; c < B; ++c) acc[c] *= T(ldexpf(1.0f, A.rexp[int64_t(s.pos) * B + c]));
  }
}

// row c of the lane's smoother block
template <int B, class X>
__device__ __forceinline__ void node_smoother(const NodeDev& A, const NodeLane& s, X (&sv)[B][B]) {
  if (A.sidx == nullptr) {
    const X* S = static_cast<const X*>(A.sfull) + int64_t(s.node) * (B * B);
#pragma unroll
    for (int c = 0; c < B; ++c)
#pragma unroll
      for (int cc = 0; cc < B; ++cc) sv[c][cc] = S[c * B + cc];
  } else if (s.flags & kNodeValUniform) {
    // rows of equal values also have the same smoother block
    const ConstPtr<X> S = as_const<X>(A.stab) + int64_t(__builtin_amdgcn_readfirstlane(int(A.sidx[s.pos]))) * (B * B);
#pragma unroll
    for (int c = 0; c < B; ++c)
#pragma unroll
      for (int cc = 0; cc < B; ++cc) sv[c][cc] = S[c * B + cc];
  } else {
    const X* S = static_cast<const X*>(A.stab) + int64_t(A.sidx[s.pos]) * (B * B);
#pragma unroll
    for (int c = 0; c < B; ++c)
#pragma unroll
      for (int cc = 0; cc < B; ++cc) sv[c][cc] = S[c * B + cc];
  }
}

// y = A x (MODE 0), b - A x (MODE 1), M (b - A x) (MODE 2); NORM: partial sums of squares
template <int B, class XI, class XO, int MODE, bool NORM, bool DEEP>
__global__ __launch_bounds__(kThreads, node_min_waves<DEEP>()) void k_node_spmv(
    NodeDev A, const XO* __restrict__ b, const XI* __restrict__ x, XO* __restrict__ y,
    const uint8_t* __restrict__ mask, double* __restrict__ partials) {
  using T = XO;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int lane = int(threadIdx.x) % kWave;
  const int slice = bid * kSliceWaves + int(threadIdx.x) / kWave;
  double sq = 0.0;
  if (slice < A.nslices) {
    const NodeLane s = node_lane(A, slice, lane);
    const int64_t d0 = int64_t(s.node) * B;
    XO bv[B];
    uint8_t mk[B];
#pragma unroll
    for (int c = 0; c < B; ++c) {
      bv[c] = MODE != 0 ? b[d0 + c] : XO(0);
      mk[c] = MODE == 2 ? mask[d0 + c] : uint8_t(0);
    }
    T acc[B];
    const GatherX<B, XI> gx{x};
    node_dot<B, T, GatherX<B, XI>, B, DEEP>(A, s, lane, gx, wave_stage<XI, B>(), acc);
    if (s.valid) {
#pragma unroll
      for (int c = 0; c < B; ++c) {
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

// x_out = x + omega S (b - A x), and the three-term (Chebyshev) form as in sweep_slice
template <int B, class X, bool DEEP>
__global__ __launch_bounds__(kThreads, node_min_waves<DEEP>()) void k_node_sweep(
    NodeDev A, const X* __restrict__ b, const X* __restrict__ x, X* xo, X omega, X beta, int pmode) {
  using T = X;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int lane = int(threadIdx.x) % kWave;
  const int slice = bid * kSliceWaves + int(threadIdx.x) / kWave;
  if (slice >= A.nslices) return;
  const NodeLane s = node_lane(A, slice, lane);
  const int64_t d0 = int64_t(s.node) * B;
  X bv[B], xv[B], pv[B], sv[B][B];
  const X* pp = pmode == 1 ? static_cast<const X*>(xo) : x;
#pragma unroll
  for (int c = 0; c < B; ++c) {
    bv[c] = b[d0 + c];
    xv[c] = x[d0 + c];
    pv[c] = pp[d0 + c];
  }
  T acc[B];
  const GatherX<B, X> gx{x};
  node_dot<B, T, GatherX<B, X>, B, DEEP>(A, s, lane, gx, wave_stage<X, B>(), acc);
  node_smoother<B, X>(A, s, sv);
  T res[B];
#pragma unroll
  for (int c = 0; c < B; ++c) res[c] = T(bv[c]) - acc[c];
  if (!s.valid) return;
#pragma unroll
  for (int c = 0; c < B; ++c) {
    T upd = T(0);
#pragma unroll
    for (int cc = 0; cc < B; ++cc) upd += T(sv[c][cc]) * res[cc];
    T nx = T(xv[c]) + omega * upd;
    if (pmode != 0) nx = nx + beta * (T(xv[c]) - (pmode == 1 ? T(pv[c]) : T(0)));
    xo[d0 + c] = X(nx);
  }
}

// x_out = omega S b
template <int B, class X>
__global__ __launch_bounds__(kThreads) void k_node_sweep0(NodeDev A, const X* __restrict__ b, X* __restrict__ xo,
                                                          X omega) {
  using T = X;
  const int slice = int(blockIdx.x) * kSliceWaves + int(threadIdx.x) / kWave;
  if (slice >= A.nslices) return;
  const NodeLane s = node_lane(A, slice, int(threadIdx.x) % kWave);
  const int64_t d0 = int64_t(s.node) * B;
  X bv[B], sv[B][B];
#pragma unroll
  for (int c = 0; c < B; ++c) bv[c] = b[d0 + c];
  node_smoother<B, X>(A, s, sv);
  if (!s.valid) return;
#pragma unroll
  for (int c = 0; c < B; ++c) {
    T upd = T(0);
#pragma unroll
    for (int cc = 0; cc < B; ++cc) upd += T(sv[c][cc]) * T(bv[cc]);
    xo[d0 + c] = X(omega * upd);
  }
}

// two sweeps from x = 0 in one pass, one component per node (as k_sweep2z)
template <class X>
__global__ __launch_bounds__(kThreads) void k_node_sweep2z(NodeDev A, const X* __restrict__ b, X* __restrict__ xo,
                                                           X omega) {
  using T = X;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int lane = int(threadIdx.x) % kWave;
  const int slice = bid * kSliceWaves + int(threadIdx.x) / kWave;
  if (slice >= A.nslices) return;
  const NodeLane s = node_lane(A, slice, lane);
  const X* S = static_cast<const X*>(A.sfull);
  const X si = S[s.node], bi = b[s.node];
  T acc[1];
  const GatherZ<X, T> gz{S, b, omega};
  node_dot<1, T, GatherZ<X, T>, 2, true>(A, s, lane, gz, nullptr, acc);
  if (!s.valid) return;
  const X x1 = X(omega * (T(0) + T(si) * T(bi)));
  const T res = T(bi) - acc[0];
  const T upd = T(0) + T(si) * res;
  xo[s.node] = X(T(x1) + omega * upd);
}

// ---- setup
// inverses of nb FP64 blocks (Gauss-Jordan with row pivoting, as k_block_invert)
template <int B, class ST>
__global__ __launch_bounds__(256) void k_invert_blocks(int nb, const double* __restrict__ blocks, ST* __restrict__ out,
                                                       int* flag) {
  const int i = int(blockIdx.x) * 256 + int(threadIdx.x);
  if (i >= nb) return;
  double m[B][2 * B];
  for (int c = 0; c < B; ++c)
    for (int cc = 0; cc < B; ++cc) {
      m[c][cc] = blocks[(int64_t(i) * B + c) * B + cc];
      m[c][B + cc] = c == cc ? 1.0 : 0.0;
    }
  if (!invert_augmented<B>(m)) { *flag = 1; return; }
  for (int c = 0; c < B; ++c)
    for (int cc = 0; cc < B; ++cc) out[(int64_t(i) * B + c) * B + cc] = ST(m[c][B + cc]);
}

// the smoother block of every node from the table: S[node] = stab[sidx[pos]], node = perm[pos]
template <class X>
__global__ __launch_bounds__(256) void k_expand_smoother(int n, int bb, const int32_t* __restrict__ perm,
                                                         const uint16_t* __restrict__ sidx,
                                                         const X* __restrict__ stab, X* __restrict__ S) {
  const int pos = int(blockIdx.x) * 256 + int(threadIdx.x);
  if (pos >= n) return;
  const int64_t node = perm ? perm[pos] : pos;
  for (int z = 0; z < bb; ++z) S[node * bb + z] = stab[int64_t(sidx[pos]) * bb + z];
}

// the kernels with a choice of batch: FP64 sums of 2 and 3 components (4 exceed the registers of
// 6 waves either way)
template <int B, class T> constexpr bool has_shallow() { return (B == 2 || B == 3) && sizeof(T) == 8; }

template <int B, class XI, class XO, bool DEEP>
hipError_t node_spmv_d(const NodeDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int mode,
                       double* partials, hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  const XO* bb = static_cast<const XO*>(b);
  const XI* xx = static_cast<const XI*>(x);
  XO* yy = static_cast<XO*>(y);
#define MGQ1_NS(MODE, NORM) \
  hipLaunchKernelGGL((k_node_spmv<B, XI, XO, MODE, NORM, DEEP>), g, kThreads, 0, s, A, bb, xx, yy, mask, partials)
  if (mode == 0 && !partials) MGQ1_NS(0, false);
  else if (mode == 1 && partials) MGQ1_NS(1, true);
  else if (mode == 1) MGQ1_NS(1, false);
  else if (mode == 2 && !partials) MGQ1_NS(2, false);
  else return hipErrorInvalidValue;
#undef MGQ1_NS
  return hipGetLastError();
}

template <int B, class XI, class XO>
hipError_t node_spmv_t(const NodeDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int mode,
                       double* partials, hipStream_t s) {
  if constexpr (has_shallow<B, XO>())
    if (A.shallow) return node_spmv_d<B, XI, XO, false>(A, b, x, y, mask, mode, partials, s);
  return node_spmv_d<B, XI, XO, true>(A, b, x, y, mask, mode, partials, s);
}

template <int B>
hipError_t node_spmv_b(const NodeDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int xk, int yk,
                       int mode, double* partials, hipStream_t s) {
  if (A.tk != yk) return hipErrorInvalidValue;
  if (xk == X_F64 && yk == X_F64) return node_spmv_t<B, double, double>(A, b, x, y, mask, mode, partials, s);
  if (xk == X_F32 && yk == X_F64) return node_spmv_t<B, float, double>(A, b, x, y, mask, mode, partials, s);
  if (xk == X_F32 && yk == X_F32) return node_spmv_t<B, float, float>(A, b, x, y, mask, mode, partials, s);
  return hipErrorInvalidValue;
}

template <int B, class X>
hipError_t node_sweep_t(const NodeDev& A, const void* b, const void* x, void* xo, double omega, double beta, int pmode,
                        hipStream_t s) {
  const unsigned g = slice_grid(A.nslices);
  const X *bb = static_cast<const X*>(b), *xx = static_cast<const X*>(x);
  X* oo = static_cast<X*>(xo);
  if constexpr (has_shallow<B, X>()) {
    if (A.shallow) {
      hipLaunchKernelGGL((k_node_sweep<B, X, false>), g, kThreads, 0, s, A, bb, xx, oo, X(omega), X(beta), pmode);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_node_sweep<B, X, true>), g, kThreads, 0, s, A, bb, xx, oo, X(omega), X(beta), pmode);
  return hipGetLastError();
}

template <int B, class X>
hipError_t node_sweep0_t(const NodeDev& A, const void* b, void* xo, double omega, hipStream_t s) {
  hipLaunchKernelGGL((k_node_sweep0<B, X>), slice_grid(A.nslices), kThreads, 0, s, A, static_cast<const X*>(b),
                     static_cast<X*>(xo), X(omega));
  return hipGetLastError();
}

}  // namespace

hipError_t launch_node_spmv(const NodeDev& A, const void* b, const void* x, void* y, const uint8_t* mask, int xk,
                            int yk, int mode, double* partials, hipStream_t s) {
  switch (A.B) {
    case 1: return node_spmv_b<1>(A, b, x, y, mask, xk, yk, mode, partials, s);
    case 2: return node_spmv_b<2>(A, b, x, y, mask, xk, yk, mode, partials, s);
    case 3: return node_spmv_b<3>(A, b, x, y, mask, xk, yk, mode, partials, s);
    case 4: return node_spmv_b<4>(A, b, x, y, mask, xk, yk, mode, partials, s);
    default: return hipErrorInvalidValue;
  }
}

#define MGQ1_NODE_B(F, ...)                                                                  \
  switch (A.B) {                                                                             \
    case 1: return xk == X_F64 ? F<1, double>(__VA_ARGS__) : F<1, float>(__VA_ARGS__);       \
    case 2: return xk == X_F64 ? F<2, double>(__VA_ARGS__) : F<2, float>(__VA_ARGS__);       \
    case 3: return xk == X_F64 ? F<3, double>(__VA_ARGS__) : F<3, float>(__VA_ARGS__);       \
    case 4: return xk == X_F64 ? F<4, double>(__VA_ARGS__) : F<4, float>(__VA_ARGS__);       \
    default: return hipErrorInvalidValue;                                                    \
  }

hipError_t launch_node_sweep(const NodeDev& A, const void* b, const void* x, void* xo, double omega, int xk,
                             hipStream_t s, double beta, int pmode) {
  if (A.tk != xk) return hipErrorInvalidValue;
  MGQ1_NODE_B(node_sweep_t, A, b, x, xo, omega, beta, pmode, s)
}

hipError_t launch_node_sweep0(const NodeDev& A, const void* b, void* xo, double omega, int xk, hipStream_t s) {
  if (A.tk != xk) return hipErrorInvalidValue;
  MGQ1_NODE_B(node_sweep0_t, A, b, xo, omega, s)
}
#undef MGQ1_NODE_B

hipError_t launch_node_sweep2z(const NodeDev& A, const void* b, void* xo, double omega, int xk, hipStream_t s) {
  if (A.B != 1 || A.tk != xk || A.sfull == nullptr) return hipErrorInvalidValue;
  const unsigned g = slice_grid(A.nslices);
  if (xk == X_F64)
    hipLaunchKernelGGL(k_node_sweep2z<double>, g, kThreads, 0, s, A, static_cast<const double*>(b),
                       static_cast<double*>(xo), omega);
  else
    hipLaunchKernelGGL(k_node_sweep2z<float>, g, kThreads, 0, s, A, static_cast<const float*>(b),
                       static_cast<float*>(xo), float(omega));
  return hipGetLastError();
}

hipError_t launch_invert_blocks(int nb, int B, const double* blocks, void* out, int sk, int* flag, hipStream_t s) {
  if (nb == 0) return hipSuccess;
  const unsigned g = grid_for(nb, 256);
#define MGQ1_IB(BB)                                                                                                  \
  case BB:                                                                                                           \
    if (sk == X_F64) hipLaunchKernelGGL((k_invert_blocks<BB, double>), g, 256, 0, s, nb, blocks, static_cast<double*>(out), flag); \
    else hipLaunchKernelGGL((k_invert_blocks<BB, float>), g, 256, 0, s, nb, blocks, static_cast<float*>(out), flag); \
    break;
  switch (B) {
    MGQ1_IB(1)
    MGQ1_IB(2)
    MGQ1_IB(3)
    MGQ1_IB(4)
    default: return hipErrorInvalidValue;
  }
#undef MGQ1_IB
  return hipGetLastError();
}

hipError_t launch_expand_smoother(int n, int B, const int32_t* perm, const uint16_t* sidx, const void* stab, void* S,
                                  int sk, hipStream_t s) {
  const unsigned g = grid_for(n, 256);
  if (sk == X_F64)
    hipLaunchKernelGGL(k_expand_smoother<double>, g, 256, 0, s, n, B * B, perm, sidx, static_cast<const double*>(stab), static_cast<double*>(S));
  else
    hipLaunchKernelGGL(k_expand_smoother<float>, g, 256, 0, s, n, B * B, perm, sidx, static_cast<const float*>(stab), static_cast<float*>(S));
  return hipGetLastError();
}

}  // namespace mgq1
