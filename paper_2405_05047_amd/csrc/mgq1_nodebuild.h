// Host side of the node form (NodeDev): the distinct blocks of an operator, its distinct
// rows, their grouping into slices of 64 nodes, and the arrays that the kernels read.
// Host code only; parallel loops run on parallel_for of the runtime and write disjoint
// outputs, and every choice follows row order, so the result does not depend on the
// number of threads.
#pragma once

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <unordered_map>
#include <utility>
#include <vector>

#include "mgq1_internal.h"

namespace mgq1 {

struct NodeHost {
  int32_t n = 0, B = 1, nslices = 0;
  std::vector<int32_t> perm;            // node at each row position (empty: itself)
  std::vector<int32_t> desc;            // 4 per slice
  std::vector<double> dict;             // distinct blocks (number 0: the zero block)
  std::vector<int8_t> dexp;             // their rows' exponents (with_exp), B per block
  std::vector<int32_t> vlist;           // block numbers of the uniform rows, row after row
  std::vector<int32_t> opat, rpat;
  std::vector<uint16_t> didx, col16, sidx;
  std::vector<int32_t> base, col32;
  std::vector<int32_t> sblock;          // block number behind each smoother table entry
  int64_t slots = 0, general = 0;       // slot rows of 64, and those of slices with general values

  // frees what only the device reads once it is there; the rest maps stored values back
  void drop_uploaded() {
    for (auto* v : {&opat, &rpat, &base, &col32, &sblock}) std::vector<int32_t>().swap(*v);
    for (auto* v : {&col16, &sidx}) std::vector<uint16_t>().swap(*v);
    std::vector<int8_t>().swap(dexp);
  }
  int32_t nblocks() const { return int32_t(dict.size()) / (B * B); }
  int32_t node_at(int64_t pos) const { return perm.empty() ? int32_t(pos) : perm[size_t(pos)]; }
  // number of the block in slot k of slice s, lane r
  int32_t block_at(int64_t s, int32_t k, int32_t r) const {
    const int32_t* d = &desc[size_t(s) * 4];
    return (d[1] & kNodeValUniform) ? vlist[size_t(d[2]) + k] : didx[(size_t(d[2]) + k) * kWave + r];
  }
};

namespace nodebuild {

inline uint64_t mix(uint64_t x) {
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebull;
  return x ^ (x >> 31);
}

// open-addressing set of the distinct keys of `words` 64-bit words each
struct BlockSet {
  int words;
  std::vector<uint64_t> keys;           // words per entry, in order of first appearance
  std::vector<int32_t> slot;            // entry + 1, 0 = free
  uint64_t mask = 0;
  explicit BlockSet(int w) : words(w), slot(1024, 0), mask(1023) {}
  int32_t size() const { return int32_t(keys.size() / size_t(words)); }
  uint64_t hash(const uint64_t* k) const {
    uint64_t h = 0x9e3779b97f4a7c15ull;
    for (int i = 0; i < words; ++i) h = (h ^ k[i]) * 0xff51afd7ed558ccdull + (h >> 29);
    return mix(h);
  }
  int32_t find_or_add(const uint64_t* k) {
    uint64_t p = hash(k) & mask;
    while (slot[p]) {
      const int32_t e = slot[p] - 1;
      if (std::memcmp(&keys[size_t(e) * words], k, size_t(words) * 8) == 0) return e;
      p = (p + 1) & mask;
    }
    const int32_t e = size();
    keys.insert(keys.end(), k, k + words);
    slot[p] = e + 1;
    if (uint64_t(e) * 2 >= mask) grow();
    return e;
  }
  void grow() {
    mask = mask * 2 + 1;
    slot.assign(size_t(mask) + 1, 0);
    for (int32_t e = 0; e < size(); ++e) {
      uint64_t p = hash(&keys[size_t(e) * words]) & mask;
      while (slot[p]) p = (p + 1) & mask;
      slot[p] = e + 1;
    }
  }
};

constexpr int32_t kMaxBlocks = 65535;

// chunks of a loop whose chunks each keep a set of their own: a small level is not worth the
// threads
inline int64_t set_chunks(int64_t items, int64_t least) {
  return std::min<int64_t>(64, std::max<int64_t>(1, items / least));
}

struct Always {
  bool operator()(const NodeHost&) const { return true; }
};

}  // namespace nodebuild

// Builds the node form of a block CSR operator (n rows, B x B blocks, rows' exponents in
// row_exp when given: blocks are then distinct with their rows' exponents).  false: more
// than 65,535 distinct blocks, vectors of 4 GiB and more, or (must == false) more than a
// quarter of the slots in slices of general values, where the sliced-ELL form moves fewer
// instructions per block, or pays(H) false of the descriptors and counts.  Throws
// std::bad_alloc.
template <class ParallelFor, class Pays = nodebuild::Always>
bool build_node(int32_t n, int B, const int32_t* rowptr, const int32_t* col, const double* val,
                const int8_t* row_exp, bool must, ParallelFor&& parallel_for, NodeHost& H, Pays pays = Pays()) {
  using namespace nodebuild;
  const int BB = B * B;
  if (B > 4 || n < 1 || int64_t(n) * B * 8 >= (int64_t(1) << 32)) return false;
  const int words = BB + (row_exp ? 1 : 0);
  H.n = n;
  H.B = B;
  H.nslices = int32_t((int64_t(n) + kWave - 1) / kWave);
  const int64_t nnz = rowptr[n];
  std::vector<uint16_t> id(size_t(nnz), 0);
  // ---- distinct blocks: per chunk of rows, then merged in chunk order
  const int64_t nchunk = set_chunks(n, 256), per = (int64_t(n) + nchunk - 1) / nchunk;
  std::vector<BlockSet> sets(static_cast<size_t>(nchunk), BlockSet(words));
  std::vector<int> bad(size_t(nchunk), 0);
  auto key_of = [&](int64_t i, int64_t k, uint64_t* key) {
    std::memcpy(key, val + k * BB, size_t(BB) * 8);
    if (row_exp) {
      uint64_t e = 0;
      std::memcpy(&e, row_exp + i * B, size_t(B));
      key[BB] = e;
    }
  };
  parallel_for(nchunk, 1, [&](int64_t c0, int64_t c1) {
    for (int64_t c = c0; c < c1; ++c) {
      try {
        BlockSet& S = sets[size_t(c)];
        uint64_t key[17];
        for (int z = 0; z < words; ++z) key[z] = 0;
        S.find_or_add(key);
        for (int64_t i = c * per; i < std::min<int64_t>(n, (c + 1) * per); ++i) {
          // a row is mostly like the one before it: compare with that row's block first
          const bool prev = i > c * per && (!row_exp || std::memcmp(row_exp + i * B, row_exp + (i - 1) * B, size_t(B)) == 0);
          const int64_t p0 = prev ? rowptr[i - 1] : 0, plen = prev ? rowptr[i] - p0 : 0;
          for (int64_t k = rowptr[i]; k < rowptr[i + 1]; ++k) {
            const int64_t q = k - rowptr[i];
            if (q < plen && std::memcmp(val + k * BB, val + (p0 + q) * BB, size_t(BB) * 8) == 0) {
              id[size_t(k)] = id[size_t(p0 + q)];
              continue;
            }
            key_of(i, k, key);
            const int32_t e = S.find_or_add(key);
            if (e >= kMaxBlocks) { bad[size_t(c)] = 1; break; }
            id[size_t(k)] = uint16_t(e);
          }
          if (bad[size_t(c)]) break;
        }
      } catch (...) {
        bad[size_t(c)] = 2;
      }
    }
  });
  for (int b : bad)
    if (b == 2) throw std::bad_alloc();
  for (int b : bad)
    if (b) return false;
  BlockSet all(words);
  std::vector<std::vector<uint16_t>> remap(static_cast<size_t>(nchunk));
  for (int64_t c = 0; c < nchunk; ++c) {
    const BlockSet& S = sets[size_t(c)];
    remap[size_t(c)].resize(size_t(S.size()));
    for (int32_t e = 0; e < S.size(); ++e) {
      const int32_t g = all.find_or_add(&S.keys[size_t(e) * words]);
      if (g >= kMaxBlocks) return false;
      remap[size_t(c)][size_t(e)] = uint16_t(g);
    }
  }
  const int32_t nblk = all.size();
  H.dict.resize(size_t(nblk) * BB);
  if (row_exp) H.dexp.assign(size_t(nblk) * B, 0);
  for (int32_t e = 0; e < nblk; ++e) {
    std::memcpy(&H.dict[size_t(e) * BB], &all.keys[size_t(e) * words], size_t(BB) * 8);
    if (row_exp) std::memcpy(&H.dexp[size_t(e) * B], &all.keys[size_t(e) * words + BB], size_t(B));
  }
  // ---- distinct rows by their blocks (with the diagonal's place, which names the smoother
  // block) and by their column offsets: hashes first, then every row against the first row of
  // its hash, so that equal numbers mean equal rows
  std::vector<uint64_t> hv(static_cast<size_t>(n)), ho(static_cast<size_t>(n));
  std::vector<uint16_t> diag(size_t(n), 0);
  parallel_for(nchunk, 1, [&](int64_t c0, int64_t c1) {
    for (int64_t c = c0; c < c1; ++c)
      for (int64_t i = c * per; i < std::min<int64_t>(n, (c + 1) * per); ++i) {
        uint64_t a = uint64_t(rowptr[i + 1] - rowptr[i]), o = a;
        for (int64_t k = rowptr[i]; k < rowptr[i + 1]; ++k) {
          const uint16_t g = remap[size_t(c)][id[size_t(k)]];
          id[size_t(k)] = g;
          if (col[k] == i) diag[size_t(i)] = g;
          a = mix(a * 0x9e3779b97f4a7c15ull + g);
          o = mix(o * 0x9e3779b97f4a7c15ull + uint64_t(int64_t(col[k]) - i));
        }
        hv[size_t(i)] = mix(a * 0x9e3779b97f4a7c15ull + diag[size_t(i)]);
        ho[size_t(i)] = o;
      }
  });
  auto same_values = [&](int64_t i, int64_t j) {
    const int64_t len = rowptr[i + 1] - rowptr[i];
    return len == rowptr[j + 1] - rowptr[j] && diag[size_t(i)] == diag[size_t(j)] &&
           std::memcmp(&id[size_t(rowptr[i])], &id[size_t(rowptr[j])], size_t(len) * 2) == 0;
  };
  auto same_offsets = [&](int64_t i, int64_t j) {
    const int64_t len = rowptr[i + 1] - rowptr[i], d = j - i;
    if (len != rowptr[j + 1] - rowptr[j]) return false;
    for (int64_t k = 0; k < len; ++k)
      if (int64_t(col[rowptr[i] + k]) + d != col[rowptr[j] + k]) return false;
    return true;
  };
  // numbers of the distinct hashes in row order; a row that differs from the first of its hash
  // gets the number -1 (never grouped)
  auto number = [&](const std::vector<uint64_t>& h, auto&& same, std::vector<int32_t>& num, std::vector<int32_t>& rep) {
    std::unordered_map<uint64_t, int32_t> m;
    num.resize(size_t(n));
    uint64_t lasth = 0;
    int32_t last = -1;
    for (int32_t i = 0; i < n; ++i) {
      if (last < 0 || h[size_t(i)] != lasth) {
        const auto it = m.emplace(h[size_t(i)], int32_t(rep.size()));
        if (it.second) rep.push_back(i);
        last = it.first->second;
        lasth = h[size_t(i)];
      }
      num[size_t(i)] = last;
    }
    parallel_for(n, 1 << 14, [&](int64_t a, int64_t b) {
      for (int64_t i = a; i < b; ++i)
        if (!same(i, int64_t(rep[size_t(num[size_t(i)])]))) num[size_t(i)] = -1;
    });
  };
  std::vector<int32_t> vn, on, vrep, orep;
  number(hv, same_values, vn, vrep);
  number(ho, same_offsets, on, orep);
  hv.clear();
  hv.shrink_to_fit();
  ho.clear();
  ho.shrink_to_fit();
  auto len_of = [&](int32_t i) { return rowptr[i + 1] - rowptr[i]; };
  // bytes that the slices of 64 rows order[0 .. n) read per slot row of 64 lanes, times their
  // widths (general values also cost a scattered block read per lane)
  auto cost_of = [&](const std::vector<int32_t>& order) {
    std::vector<int64_t> part(size_t(nchunk), 0);
    const int64_t sper = (H.nslices + nchunk - 1) / nchunk;
    parallel_for(nchunk, 1, [&](int64_t c0, int64_t c1) {
      for (int64_t c = c0; c < c1; ++c)
        for (int64_t s = c * sper; s < std::min<int64_t>(H.nslices, (c + 1) * sper); ++s) {
          const int32_t* node = &order[size_t(s) * kWave];
          const int cnt = int(std::min<int64_t>(kWave, n - s * kWave));
          int32_t w = 0;
          bool vu = vn[size_t(node[0])] >= 0, ou = on[size_t(node[0])] >= 0;
          for (int r = 0; r < cnt; ++r) {
            w = std::max(w, len_of(node[r]));
            vu = vu && vn[size_t(node[r])] == vn[size_t(node[0])];
            ou = ou && on[size_t(node[r])] == on[size_t(node[0])];
          }
          part[size_t(c)] += int64_t(w) * (vu ? (ou ? 8 : 128 + 8) : 256 + 64 * 8 * BB);
        }
    });
    int64_t t = 0;
    for (int64_t v : part) t += v;
    return t;
  };
  // ---- grouping: the rows of equal values and offsets in whole slices of 64, node order inside a
  // group; then the rest of each kind of values in whole slices; what is left by length.  The
  // whole slices follow each other in the order of their first row, so that neighbours in the
  // mesh stay near each other in the launch.  Over the whole level: what is left is then less
  // than a slice per kind of row.  (Inside windows of 4,096 rows 5% of the slots of the 65^3
  // elasticity level were in general slices, whose scattered block reads took a third of the
  // sweep: 23.6 us against 15.9 us with windows of 32,768.)
  std::vector<int32_t> order(static_cast<size_t>(n));
  for (int32_t i = 0; i < n; ++i) order[size_t(i)] = i;
  const int64_t cost0 = cost_of(order);
  {
    std::vector<int32_t> grouped, left, rows(order);
    grouped.reserve(size_t(n));
    for (int pass = 0; pass < 2; ++pass) {
      // group number of every row: values and offsets, then values
      std::unordered_map<uint64_t, int32_t> m;
      std::vector<int32_t> count, gid(rows.size());
      uint64_t lastk = 0;
      int32_t last = -1;
      for (size_t q = 0; q < rows.size(); ++q) {
        const int32_t i = rows[q], v = vn[size_t(i)], o = on[size_t(i)];
        if (v < 0 || (pass == 0 && o < 0)) {
          gid[q] = -1;
          continue;
        }
        const uint64_t k = uint64_t(uint32_t(v)) << 32 | (pass == 0 ? uint32_t(o) : 0u);
        if (last < 0 || k != lastk) {
          const auto it = m.emplace(k, int32_t(count.size()));
          if (it.second) count.push_back(0);
          last = it.first->second;
          lastk = k;
        }
        gid[q] = last;
        ++count[size_t(last)];
      }
      std::vector<int64_t> at(count.size());
      std::vector<int32_t> room(count.size());
      int64_t fill = int64_t(grouped.size());
      for (size_t g = 0; g < count.size(); ++g) {
        at[g] = fill;
        room[g] = count[g] / kWave * kWave;
        fill += room[g];
      }
      grouped.resize(size_t(fill));
      left.clear();
      for (size_t q = 0; q < rows.size(); ++q) {
        const int32_t g = gid[q];
        if (g >= 0 && room[size_t(g)] > 0) {
          grouped[size_t(at[size_t(g)]++)] = rows[q];
          --room[size_t(g)];
        } else {
          left.push_back(rows[q]);
        }
      }
      rows.swap(left);
    }
    const int64_t ns = int64_t(grouped.size()) / kWave;
    std::vector<std::pair<int32_t, int32_t>> first(static_cast<size_t>(ns));
    for (int64_t z = 0; z < ns; ++z) first[size_t(z)] = {grouped[size_t(z) * kWave], int32_t(z)};
    std::sort(first.begin(), first.end());
    for (int64_t z = 0; z < ns; ++z)
      std::memcpy(&order[size_t(z) * kWave], &grouped[size_t(first[size_t(z)].second) * kWave], kWave * sizeof(int32_t));
    std::stable_sort(rows.begin(), rows.end(), [&](int32_t i, int32_t j) { return len_of(i) > len_of(j); });
    std::copy(rows.begin(), rows.end(), order.begin() + ns * kWave);
  }
  // regroup when that saves 3% of what the kernels read (the vectors: about 24 B bytes per
  // row; the position list costs 4)
  const int64_t vec = int64_t(n) * 24 * B;
  if ((cost_of(order) + 4 * int64_t(n) + vec) * 100 <= (cost0 + vec) * 97) H.perm = std::move(order);
  order.clear();
  order.shrink_to_fit();
  // ---- descriptors
  H.desc.assign(size_t(H.nslices) * 4, 0);
  parallel_for(H.nslices, 256, [&](int64_t s0, int64_t s1) {
    for (int64_t s = s0; s < s1; ++s) {
      const int cnt = int(std::min<int64_t>(kWave, n - s * kWave));
      const int32_t i0 = H.node_at(s * kWave);
      int32_t w = 0;
      bool vu = vn[size_t(i0)] >= 0, ou = on[size_t(i0)] >= 0;
      for (int r = 0; r < cnt; ++r) {
        const int32_t i = H.node_at(s * kWave + r);
        w = std::max(w, len_of(i));
        vu = vu && vn[size_t(i)] == vn[size_t(i0)];
        ou = ou && on[size_t(i)] == on[size_t(i0)];
      }
      int32_t flags = (vu ? kNodeValUniform : 0) | (vu && ou ? kNodeColUniform : 0);
      if (!(flags & kNodeColUniform)) {
        for (int32_t k = 0; k < w && !(flags & kNodeCol32); ++k) {
          int32_t lo = INT32_MAX, hi = INT32_MIN;
          for (int r = 0; r < cnt; ++r) {
            const int32_t i = H.node_at(s * kWave + r);
            const int32_t j = k < len_of(i) ? col[rowptr[i] + k] : i;
            lo = std::min(lo, j);
            hi = std::max(hi, j);
          }
          if (int64_t(hi) - lo > 65535) flags |= kNodeCol32;
        }
      }
      H.desc[size_t(s) * 4] = w;
      H.desc[size_t(s) * 4 + 1] = flags;
    }
  });
  // the run record of a row's offsets (see NodeDev), appended to rpat; -1: it has none
  auto run_record = [&](int32_t i) -> int32_t {
    const int32_t len = len_of(i);
    const int32_t* cl = col + rowptr[i];
    std::vector<int32_t> start, end, run(static_cast<size_t>(len));   // runs, first and last slot + 1
    for (int32_t k = 0; k < len; ++k) {
      if (start.empty() || cl[k] - cl[start.back()] >= kRunWidth) {
        start.push_back(k);
        end.push_back(k);
      }
      end.back() = k + 1;
      run[size_t(k)] = int32_t(start.size()) - 1;
    }
    const int32_t nrun = int32_t(start.size()), nph = (nrun + kPhaseRuns - 1) / kPhaseRuns;
    // a run is worth staging when its columns are read more than once
    if (nrun * 2 > len) return -1;
    const int32_t at = int32_t(H.rpat.size());
    H.rpat.push_back(nph);
    for (int32_t p = 0; p < nph; ++p) {
      const int32_t last = std::min(nrun, (p + 1) * kPhaseRuns) - 1;
      H.rpat.push_back(end[size_t(last)]);
      for (int32_t q = 0; q < kPhaseRuns; ++q) {
        const int32_t r = p * kPhaseRuns + q;
        H.rpat.push_back(r < nrun ? cl[start[size_t(r)]] - i : 0);
        H.rpat.push_back(r < nrun ? cl[end[size_t(r)] - 1] - cl[start[size_t(r)]] + 1 : 0);
      }
      H.rpat.push_back(0);
    }
    for (int32_t k = 0; k < len; ++k) {
      const int32_t r = run[size_t(k)];
      H.rpat.push_back((r % kPhaseRuns) * kRunStride + cl[k] - cl[start[size_t(r)]]);
    }
    return at;
  };
  // places in the arrays (sequential), the lists of the uniform rows
  std::vector<int32_t> vstart(vrep.size(), -1), ostart(orep.size(), -1), rstart(orep.size(), -2);
  int64_t nd = 0, n16 = 0, n32 = 0;
  for (int64_t s = 0; s < H.nslices; ++s) {
    int32_t* d = &H.desc[size_t(s) * 4];
    const int32_t i0 = H.node_at(s * kWave), w = d[0];
    H.slots += w;
    if (d[1] & kNodeValUniform) {
      int32_t& v = vstart[size_t(vn[size_t(i0)])];
      if (v < 0) {
        v = int32_t(H.vlist.size());
        for (int64_t k = rowptr[i0]; k < rowptr[i0 + 1]; ++k) H.vlist.push_back(id[size_t(k)]);
      }
      d[2] = v;
    } else {
      d[2] = int32_t(nd);
      nd += w;
      H.general += w;
    }
    if (d[1] & kNodeColUniform) {
      int32_t& o = ostart[size_t(on[size_t(i0)])];
      if (o < 0) {
        o = int32_t(H.opat.size());
        for (int64_t k = rowptr[i0]; k < rowptr[i0 + 1]; ++k) H.opat.push_back(col[k] - i0);
      }
      d[3] = o;
      const int32_t il = H.node_at(std::min<int64_t>(s * kWave + kWave, n) - 1);
      if (B >= 2 && il - i0 < kRunSpan) {
        int32_t& r = rstart[size_t(on[size_t(i0)])];
        if (r == -2) r = run_record(i0);
        if (r >= 0) {
          d[1] |= kNodeRuns;
          d[3] = r;
        }
      }
    } else if (d[1] & kNodeCol32) {
      d[3] = int32_t(n32);
      n32 += w;
    } else {
      d[3] = int32_t(n16);
      n16 += w;
    }
  }
  if (!must && (H.general * 4 > H.slots || !pays(H))) return false;
  H.didx.assign(size_t(nd) * kWave, 0);
  H.col16.assign(size_t(n16) * kWave, 0);
  H.base.assign(size_t(n16), 0);
  H.col32.assign(size_t(n32) * kWave, 0);
  parallel_for(H.nslices, 256, [&](int64_t s0, int64_t s1) {
    for (int64_t s = s0; s < s1; ++s) {
      const int32_t* d = &H.desc[size_t(s) * 4];
      const int cnt = int(std::min<int64_t>(kWave, n - s * kWave));
      for (int32_t k = 0; k < d[0]; ++k) {
        int32_t j[kWave], lo = INT32_MAX;
        for (int r = 0; r < kWave; ++r) {
          const int32_t i = H.node_at(s * kWave + std::min(r, cnt - 1));
          const bool in = k < len_of(i);
          j[r] = in ? col[rowptr[i] + k] : i;
          lo = std::min(lo, j[r]);
          if (!(d[1] & kNodeValUniform))
            H.didx[(size_t(d[2]) + k) * kWave + r] = in ? id[size_t(rowptr[i] + k)] : uint16_t(0);
        }
        if (d[1] & kNodeColUniform) continue;
        const size_t at = size_t(d[3]) + k;
        if (d[1] & kNodeCol32) {
          for (int r = 0; r < kWave; ++r) H.col32[at * kWave + r] = j[r];
        } else {
          H.base[at] = lo;
          for (int r = 0; r < kWave; ++r) H.col16[at * kWave + r] = uint16_t(j[r] - lo);
        }
      }
    }
  });
  // ---- smoother blocks: one per distinct diagonal block
  std::vector<int32_t> smap(size_t(nblk), -1);
  H.sidx.resize(size_t(n));
  for (int64_t pos = 0; pos < n; ++pos) {
    const uint16_t g = diag[size_t(H.node_at(pos))];
    if (smap[g] < 0) {
      smap[g] = int32_t(H.sblock.size());
      H.sblock.push_back(g);
    }
    H.sidx[size_t(pos)] = uint16_t(smap[g]);
  }
  return true;
}

}  // namespace mgq1
