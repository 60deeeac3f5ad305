// Host walk over the node form's arrays, as the kernels index them: builds the form of a block
// CSR operator with mgq1_nodebuild.h and computes y = A x slice by slice, slot by slot, with
// every index checked against its array.  Returns 1 (built), 0 (refused) or a negative code
// for an index out of range; stats = {slices, slots, slots in general slices, slices of
// uniform values, slices of uniform columns, slices of 32-bit columns, distinct blocks,
// regrouped, slices of staged runs}.
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
  int64_t vu = 0, cu = 0, c32 = 0, runs = 0;
  if (int64_t(H.desc.size()) != int64_t(H.nslices) * 4) return -1;
  for (int64_t s = 0; s < H.nslices; ++s) {
    const int32_t w = H.desc[size_t(s) * 4], fl = H.desc[size_t(s) * 4 + 1], iv = H.desc[size_t(s) * 4 + 2],
                  ic = H.desc[size_t(s) * 4 + 3];
    runs += (fl & kNodeRuns) != 0;
    // the staging area of a run slice as the wave fills it, phase by phase: the column that each
    // place holds, and how many slots a phase ends at
    std::vector<std::vector<int64_t>> staged;
    std::vector<int32_t> phase_end;
    const int64_t lastpos = std::min<int64_t>(s * kWave + kWave, n) - 1;
    if (fl & kNodeRuns) {
      const int32_t node0 = H.node_at(s * kWave), span = H.node_at(lastpos) - node0 + 1;
      if (B < 2 || !(fl & kNodeColUniform) || span < 1 || span > kRunSpan || size_t(ic) >= H.rpat.size()) return -16;
      const int32_t nph = H.rpat[size_t(ic)];
      if (size_t(ic) + 1 + size_t(nph) * kPhaseInts + w > H.rpat.size()) return -17;
      for (int32_t p = 0; p < nph; ++p) {
        const int32_t* ph = &H.rpat[size_t(ic) + 1 + size_t(p) * kPhaseInts];
        phase_end.push_back(ph[0]);
        staged.emplace_back(size_t(kPhaseRuns) * kRunStride, -1);
        for (int q = 0; q < kPhaseRuns; ++q) {
          const int32_t wd = ph[2 + 2 * q];
          if (wd < 0 || wd > kRunWidth) return -18;
          for (int32_t e = 0; wd > 0 && e < span + wd - 1; ++e) {
            const int64_t j = int64_t(node0) + ph[1 + 2 * q] + e;
            if (j < 0 || j >= n) return -19;
            staged.back()[size_t(q) * kRunStride + e] = j;
          }
        }
      }
      if (phase_end.empty() || phase_end.back() != w) return -20;
    }
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
        if (fl & kNodeRuns) {
          size_t p = 0;
          while (p < phase_end.size() && k >= phase_end[p]) ++p;
          const int32_t nph = H.rpat[size_t(ic)];
          const int64_t at = int64_t(H.rpat[size_t(ic) + 1 + size_t(nph) * kPhaseInts + k]) + node - H.node_at(s * kWave);
          if (p == phase_end.size() || at < 0 || at >= int64_t(staged[p].size())) return -21;
          j = staged[p][size_t(at)];
        } else if (fl & kNodeColUniform) {
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
  const int64_t st[9] = {H.nslices, H.slots, H.general, vu, cu, c32, H.nblocks(), H.perm.empty() ? 0 : 1, runs};
  for (int q = 0; q < 9; ++q) stats[q] = st[q];
  return 1;
}
