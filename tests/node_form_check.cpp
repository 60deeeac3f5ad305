// Host walk over the node form's arrays, as the kernels index them: builds the form of a block
// CSR operator with mgq1_nodebuild.h and computes y = A x slice by slice, slot by slot, with
// every index checked against its array.  Returns 1 (built), 0 (refused) or a negative code
// for an index out of range; stats = {slices, slots, slots in general slices, slices of
// uniform values, slices of uniform columns, slices of 32-bit columns, distinct blocks,
// regrouped}.
#include <cmath>
#include <new>

#include "../paper_2405_05047_amd/csrc/mgq1_nodebuild.h"

extern "C" int node_form_check(int32_t n, int32_t B, const int32_t* rowptr, const int32_t* col, const double* val,
                               const int8_t* row_exp, int32_t must, const double* x, double* y, int64_t* stats) {
  using namespace mgq1;
  NodeHost H;
  const bool ok = build_node(n, B, rowptr, col, val, row_exp, must != 0,
                             [](int64_t m, int64_t, auto&& f) { f(int64_t(0), m); }, H);
  if (!ok) return 0;
  const int BB = B * B;
  std::vector<char> seen(size_t(n), 0);
  int64_t vu = 0, cu = 0, c32 = 0;
  if (int64_t(H.desc.size()) != int64_t(H.nslices) * 4) return -1;
  for (int64_t s = 0; s < H.nslices; ++s) {
    const int32_t w = H.desc[size_t(s) * 4], fl = H.desc[size_t(s) * 4 + 1], iv = H.desc[size_t(s) * 4 + 2],
                  ic = H.desc[size_t(s) * 4 + 3];
    vu += (fl & kNodeValUniform) != 0;
    cu += (fl & kNodeColUniform) != 0;
    c32 += (fl & kNodeCol32) != 0;
    if ((fl & kNodeColUniform) && !(fl & kNodeValUniform)) return -2;
    const int first_s = H.sidx[size_t(s) * kWave];
    for (int lane = 0; lane < kWave; ++lane) {
      const int64_t pos = std::min<int64_t>(s * kWave + lane, n - 1);
      const int32_t node = H.perm.empty() ? int32_t(pos) : H.perm[size_t(pos)];
      if (node < 0 || node >= n) return -3;
      if (H.sidx[size_t(pos)] >= H.sblock.size()) return -4;
      if ((fl & kNodeValUniform) && H.sidx[size_t(pos)] != first_s) return -5;
      double acc[4] = {0.0, 0.0, 0.0, 0.0};
      for (int32_t k = 0; k < w; ++k) {
        int64_t j;
        if (fl & kNodeColUniform) {
          if (size_t(ic + k) >= H.opat.size()) return -6;
          j = int64_t(node) + H.opat[size_t(ic + k)];
        } else if (fl & kNodeCol32) {
          if ((size_t(ic) + k) * kWave + lane >= H.col32.size()) return -7;
          j = H.col32[(size_t(ic) + k) * kWave + lane];
        } else {
          if ((size_t(ic) + k) * kWave + lane >= H.col16.size() || size_t(ic + k) >= H.base.size()) return -8;
          j = int64_t(H.base[size_t(ic + k)]) + H.col16[(size_t(ic) + k) * kWave + lane];
        }
        if (j < 0 || j >= n) return -9;
        int64_t e;
        if (fl & kNodeValUniform) {
          if (size_t(iv + k) >= H.vlist.size()) return -10;
          e = H.vlist[size_t(iv + k)];
        } else {
          if ((size_t(iv) + k) * kWave + lane >= H.didx.size()) return -11;
          e = H.didx[(size_t(iv) + k) * kWave + lane];
        }
        if (e < 0 || e >= H.nblocks()) return -12;
        for (int c = 0; c < B; ++c)
          for (int cc = 0; cc < B; ++cc)
            acc[c] = std::fma(H.dict[size_t(e) * BB + c * B + cc], x[j * B + cc], acc[c]);
      }
      if (s * kWave + lane >= n) continue;
      if (seen[size_t(node)]++) return -13;
      for (int c = 0; c < B; ++c) y[int64_t(node) * B + c] = acc[c];
      // the smoother table's entry comes from this row's diagonal block
      for (int32_t k = rowptr[node]; k < rowptr[node + 1]; ++k)
        if (col[k] == node && std::memcmp(&H.dict[size_t(H.sblock[H.sidx[size_t(pos)]]) * BB], val + int64_t(k) * BB,
                                          size_t(BB) * 8) != 0)
          return -15;
    }
  }
  for (char v : seen)
    if (!v) return -14;
  const int64_t st[8] = {H.nslices, H.slots, H.general, vu, cu, c32, H.nblocks(), H.perm.empty() ? 0 : 1};
  for (int q = 0; q < 8; ++q) stats[q] = st[q];
  return 1;
}
