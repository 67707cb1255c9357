// Host-side loading of a sparse polynomial system (see packer.hpp).
//
// Input form: sparse distributed form, only nonzero monomials (Problem
// Statement, Sec. 1); each monomial a coefficient and (variable, exponent)
// pairs with positive exponents (Sec. 2.1, eq. (1)).
#include "packer.hpp"

#include <algorithm>
#include <cstring>
#include <numeric>
#include <vector>

namespace pe {

int lanes_for(int k, int seg) {
  int need = (k + seg - 1) / seg;
  int s = 1;
  while (s < need) s <<= 1;
  return s;
}

// log2 of a monomial's lanes in the value layout: the fewest that leave at most 12
// factors per lane (a lane's factors are one chain of products, the lanes'
// are joined by log2 s more)
static int val_lg_lanes(int k) {
  int lg = 0;
  while (lg < 6 && (k + (1 << lg) - 1) >> lg > 12) ++lg;
  return lg;
}

int validate(const SysInput& in, std::string& msg) {
  // level codes: 1, 2, 4 complex; 8 | 1, 8 | 2, 8 | 4 real (layout.hpp)
  if ((in.level & ~kRealLevel) != 1 && (in.level & ~kRealLevel) != 2 && (in.level & ~kRealLevel) != 4) {
    msg = "level must be 1, 2 or 4, optionally with the real flag 8";
    return kEinval;
  }
  if (in.n_vars < 1) {
    msg = "n_vars must be at least 1";
    return kEinval;
  }
  if (in.n_vars > kMaxVars) {
    msg = "n_vars above 65535 is not supported";
    return kEunsupported;
  }
  if (in.n_polys < 0) {
    msg = "n_polys must be nonnegative";
    return kEinval;
  }
  if (!in.poly_ptr) {
    msg = "poly_ptr is NULL";
    return kEinval;
  }
  if (in.poly_ptr[0] != 0) {
    msg = "poly_ptr[0] must be 0";
    return kEinval;
  }
  for (int p = 0; p < in.n_polys; ++p)
    if (in.poly_ptr[p + 1] < in.poly_ptr[p]) {
      msg = "poly_ptr is not nondecreasing at polynomial " + std::to_string(p);
      return kEinval;
    }
  const int64_t M = in.poly_ptr[in.n_polys];
  if (M > 0 && (!in.mon_ptr || !in.coef)) {
    msg = "mon_ptr or coef is NULL";
    return kEinval;
  }
  if (M > (int64_t(1) << 31)) {
    msg = "more than 2^31 monomials is not supported";
    return kEunsupported;
  }
  if (M > 0 && in.mon_ptr[0] != 0) {
    msg = "mon_ptr[0] must be 0";
    return kEinval;
  }
  for (int64_t t = 0; t < M; ++t)
    if (in.mon_ptr[t + 1] < in.mon_ptr[t]) {
      msg = "mon_ptr is not nondecreasing at monomial " + std::to_string(t);
      return kEinval;
    }
  const int64_t nnz = M > 0 ? in.mon_ptr[M] : 0;
  if (nnz > 0 && (!in.var_idx || !in.exps)) {
    msg = "var_idx or exps is NULL";
    return kEinval;
  }
  if (nnz > (int64_t(1) << 32)) {
    msg = "more than 2^32 occurrences is not supported";
    return kEunsupported;
  }
  std::vector<int32_t> seen(in.n_vars, -1);
  for (int64_t t = 0; t < M; ++t) {
    const int64_t a = in.mon_ptr[t], b = in.mon_ptr[t + 1];
    if (b - a > kMaxMonomialVars) {
      msg = "monomial " + std::to_string(t) + " has more than 1024 variables";
      return kEunsupported;
    }
    for (int64_t o = a; o < b; ++o) {
      const int32_t v = in.var_idx[o], d = in.exps[o];
      if (v < 0 || v >= in.n_vars) {
        msg = "variable index out of range in monomial " + std::to_string(t);
        return kEinval;
      }
      if (d < 1 || d > 65535) {
        msg = "exponent outside 1..65535 in monomial " + std::to_string(t);
        return kEinval;
      }
      if (seen[v] == int32_t(t & 0x7fffffff)) {
        msg = "duplicate variable in monomial " + std::to_string(t);
        return kEinval;
      }
      seen[v] = int32_t(t & 0x7fffffff);
    }
  }
  return kOk;
}

namespace {

struct Occ {
  int var, exp;
  int64_t orig;  // index of the occurrence in the input
};

}  // namespace

int pack_system(const SysInput& in, const PackParams& pp, Packed& out, std::string& msg) {
  int st = validate(in, msg);
  if (st != kOk) return st;
  const int L = in.level & ~kRealLevel, n = in.n_vars, N = in.n_polys;
  const int ncomp = (in.level & kRealLevel) ? 1 : 2;  // real or complex
  const int W = ncomp * L;                             // doubles per number
  const int64_t M = in.poly_ptr[N];
  const int64_t nnz = M > 0 ? in.mon_ptr[M] : 0;
  const int T = pp.threads, seg = pp.seg;
  if (T < 64 || T > 1024 || (T & 63) || seg < 1 || seg > kMaxSeg) {
    msg = "invalid launch shape";
    return kEinval;
  }

  out = Packed();
  out.level = L;
  out.code = in.level;
  out.n = n;
  out.N = N;
  out.M = M;
  out.nnz = nnz;
  out.params = pp;

  // largest exponent and monomial size, mean size
  int emax = 1, kmax = 0;
  for (int64_t o = 0; o < nnz; ++o) emax = std::max(emax, int(in.exps[o]));
  for (int64_t t = 0; t < M; ++t) kmax = std::max<int>(kmax, int(in.mon_ptr[t + 1] - in.mon_ptr[t]));
  out.emax = emax;
  out.kmax = kmax;
  if (lanes_for(std::max(kmax, 1), seg) > kMaxWave) {
    msg = "monomial too large for the segment length";
    return kEunsupported;
  }
  const int max_slots = pp.max_slots;
  if (max_slots < kMaxMonomialVars + 1 || max_slots > 65535) {
    msg = "slot budget must be in 1025..65535";
    return kEinval;
  }

  out.mcoef.resize(size_t(M) * W);
  out.mmeta.resize(size_t(M));
  out.mon_orig.resize(size_t(M));
  out.chunk_ptr.assign(size_t(N) + 1, 0);
  out.poly_cost.assign(size_t(N), 0);

  std::vector<int64_t> order;
  std::vector<Occ> chunk_occ;
  std::vector<int> counts, next_slot;

  int64_t packed_t = 0;
  for (int p = 0; p < N; ++p) {
    const int64_t t0 = in.poly_ptr[p], t1 = in.poly_ptr[p + 1];
    order.resize(size_t(t1 - t0));
    std::iota(order.begin(), order.end(), t0);
    // larger monomials first so that chunks are homogeneous in k
    std::stable_sort(order.begin(), order.end(), [&](int64_t a, int64_t b) {
      return (in.mon_ptr[a + 1] - in.mon_ptr[a]) > (in.mon_ptr[b + 1] - in.mon_ptr[b]);
    });
    out.chunk_ptr[p] = uint32_t(out.chunks.size());
    size_t i = 0;
    while (i < order.size()) {
      const int kfirst = int(in.mon_ptr[order[i] + 1] - in.mon_ptr[order[i]]);
      const int s = lanes_for(std::max(kfirst, 1), seg);
      const int cap = T / s;
      // one slot per partial derivative; slot index `slots` (one past the
      // last) is the chunk's dummy slot, so at most max_slots - 1 are used
      int count = 0, slots = 0;
      size_t j = i;
      while (j < order.size() && count < cap) {
        const int k = int(in.mon_ptr[order[j] + 1] - in.mon_ptr[order[j]]);
        if (slots + k + 1 > max_slots) break;
        slots += k;
        ++count;
        ++j;
      }
      // build the chunk from order[i..j)
      ChunkDesc cd{};
      cd.poly = uint32_t(p);
      cd.count = uint16_t(count);
      cd.s = uint8_t(s);
      cd.width = uint16_t(count * s);
      cd.mon_base = uint32_t(packed_t);
      cd.nslots = uint16_t(slots);
      const int segc = kfirst > 0 ? (kfirst + s - 1) / s : 1;
      cd.seg = uint8_t(segc);
      out.max_seg_used = std::max(out.max_seg_used, segc);
      out.max_slots_used = std::max(out.max_slots_used, slots + 1);
      cd.occ_base = uint32_t(out.occ.size());
      if (out.occ.size() + size_t(segc) * cd.width > (size_t(1) << 32)) {
        msg = "packed occurrence array too large";
        return kEunsupported;
      }
      cd.colptr_base = uint32_t(out.colptr.size());

      // slots by column, then monomial, then position: a counting sort over
      // the columns that keeps the order of the monomials
      chunk_occ.clear();
      counts.assign(size_t(n) + 1, 0);
      for (int g = 0; g < count; ++g) {
        const int64_t t = order[i + g];
        const int64_t a = in.mon_ptr[t], b = in.mon_ptr[t + 1];
        const size_t first = chunk_occ.size();
        bool sorted = true;
        for (int64_t o = a; o < b; ++o) {
          sorted = sorted && (o == a || in.var_idx[o - 1] < in.var_idx[o]);
          chunk_occ.push_back({in.var_idx[o], in.exps[o], o});
          counts[size_t(in.var_idx[o]) + 1]++;
        }
        if (!sorted)
          std::sort(chunk_occ.begin() + int64_t(first), chunk_occ.end(),
                    [](const Occ& x, const Occ& y) { return x.var < y.var; });
      }
      for (int c = 0; c < n; ++c) counts[size_t(c) + 1] += counts[size_t(c)];
      next_slot.assign(counts.begin(), counts.end());
      for (int c = 0; c <= n; ++c) out.colptr.push_back(uint16_t(counts[size_t(c)]));

      // occurrence records, lane-major; positions past a lane's segment hold
      // the neutral record (variable n, whose value is 1, exponent 1, the
      // dummy slot)
      const size_t rec0 = out.occ.size();
      const OccRec pad{uint16_t(n), 1, uint16_t(slots), 0};
      out.occ.resize(rec0 + size_t(segc) * cd.width, pad);
      out.occ_orig.resize(rec0 + size_t(segc) * cd.width, kNoOcc);
      int64_t cost = 0;
      size_t at = 0;
      for (int g = 0; g < count; ++g) {
        const int64_t t = order[i + g];
        const int k = int(in.mon_ptr[t + 1] - in.mon_ptr[t]);
        const Occ* occ_sorted = chunk_occ.data() + at;
        at += size_t(k);
        // lane q of the group takes occurrences q, q + s, q + 2s, ... (in
        // variable order): a wavefront's gathers and slot stores at one step
        // then touch neighbouring variables when a monomial's variables are
        // runs of consecutive indices, instead of addresses a segment apart
        for (int r = 0; r < k; ++r) {
          const Occ& oc = occ_sorted[r];
          const size_t pos = rec0 + size_t(r / s) * cd.width + size_t(g * s + r % s);
          OccRec& rec = out.occ[pos];
          rec.var = uint16_t(oc.var);
          rec.exp = uint16_t(oc.exp);
          rec.slot = uint16_t(next_slot[size_t(oc.var)]++);
          out.occ_orig[pos] = uint32_t(oc.orig);
        }
        // packed monomial: coefficient and metadata
        for (int c = 0; c < ncomp; ++c)
          for (int l = 0; l < L; ++l)
            out.mcoef[size_t(packed_t + g) * W + size_t(c) * L + l] = in.coef[(size_t(c) * L + l) * size_t(M) + size_t(t)];
        out.mmeta[size_t(packed_t + g)] = mon_meta(uint32_t(k));
        out.mon_orig[size_t(packed_t + g)] = uint32_t(t);
        cost += k;
      }
      out.poly_cost[p] += int64_t(segc) * s * count + cost;
      out.chunks.push_back(cd);
      packed_t += count;
      i = j;
    }
  }
  out.chunk_ptr[N] = uint32_t(out.chunks.size());
  out.rowdesc.assign(size_t(N) * kRowDesc, ChunkDesc{});
  for (int p = 0; p < N; ++p)
    for (uint32_t j = 0; j < uint32_t(kRowDesc) && out.chunk_ptr[p] + j < out.chunk_ptr[p + 1]; ++j)
      out.rowdesc[size_t(p) * kRowDesc + j] = out.chunks[out.chunk_ptr[p] + j];
  return kOk;
}

// Lanes join by a shuffle and an addition, as long as about four entries of a
// lane's own sum: a column is split while its halves keep 8 entries and the
// row's columns take at most eight wavefronts.
int val_lg_lanes_per_column(int n, int64_t len) {
  int lg = 0;
  while (lg < 3 && (int64_t(n) << (lg + 1)) <= 512 && len >> (lg + 1) >= 8) ++lg;
  return lg;
}

// A slice is as long as its longest column, 64 lanes wide: a variable that
// occurs in every monomial of a row of many columns would pad the row to 64 / Q
// times its entries, in memory and as a chain of that many additions in one
// wavefront.  More than kValPadding entries per occurrence are refused (1 MB is
// allowed in any case); sorted columns of similar length take 1.1 to 1.5.
static constexpr int64_t kValPadding = 4;

bool pack_values(const SysInput& in, int block_mons, PackedValues& out) {
  const int n = in.n_vars, N = in.n_polys;
  if (n > 32768 || block_mons < 1 || block_mons > 65534) return false;
  out = PackedValues();
  int64_t longest = 0;
  for (int p = 0; p < N; ++p)
    longest = std::max<int64_t>(longest, in.mon_ptr[in.poly_ptr[p + 1]] - in.mon_ptr[in.poly_ptr[p]]);
  out.lgQ = val_lg_lanes_per_column(n, longest / std::max(n, 1));
  const int Q = 1 << out.lgQ;
  const int per = 64 / Q;  // columns of a slice
  const int slices = out.slices = (n + per - 1) / per;
  out.row_block.assign(size_t(N) + 1, 0);
  out.perm.assign(size_t(N) * slices * per, uint16_t(n));
  const int64_t nnz = in.poly_ptr[N] > 0 ? in.mon_ptr[in.poly_ptr[N]] : 0;
  out.rec.reserve(size_t(nnz) + size_t(nnz) / 8);
  out.ell.reserve(size_t(nnz) + size_t(nnz) / 4);
  std::vector<int64_t> order;
  std::vector<int> total, cnt, fill, bucket, place;
  const uint32_t neutral = uint32_t(n), cols = uint32_t(n) + 1;
  uint32_t packed = 0;
  for (int p = 0; p < N; ++p) {
    const int64_t t0 = in.poly_ptr[p], t1 = in.poly_ptr[p + 1];
    const int64_t M = t1 - t0;
    order.resize(size_t(M));
    std::iota(order.begin(), order.end(), t0);
    bool even = true;
    for (int64_t t = t0 + 1; t < t1 && even; ++t)
      even = in.mon_ptr[t + 1] - in.mon_ptr[t] <= in.mon_ptr[t] - in.mon_ptr[t - 1];
    if (!even)
      std::stable_sort(order.begin(), order.end(), [&](int64_t a, int64_t b) {
        return (in.mon_ptr[a + 1] - in.mon_ptr[a]) > (in.mon_ptr[b + 1] - in.mon_ptr[b]);
      });
    // columns in decreasing number of occurrences in the row (counting sort)
    total.assign(size_t(n), 0);
    for (int64_t t = t0; t < t1; ++t)
      for (int64_t o = in.mon_ptr[t]; o < in.mon_ptr[t + 1]; ++o) total[size_t(in.var_idx[o])]++;
    int most = 0;
    for (int c = 0; c < n; ++c) most = std::max(most, total[size_t(c)]);
    bucket.assign(size_t(most) + 2, 0);
    for (int c = 0; c < n; ++c) bucket[size_t(most - total[size_t(c)]) + 1]++;
    for (int b = 0; b <= most; ++b) bucket[size_t(b) + 1] += bucket[size_t(b)];
    uint16_t* perm = out.perm.data() + size_t(p) * slices * per;
    place.resize(size_t(n));
    for (int c = 0; c < n; ++c) {
      const int at = bucket[size_t(most - total[size_t(c)])]++;
      perm[at] = uint16_t(c);
      place[size_t(c)] = at;
    }
    out.row_block[size_t(p)] = uint32_t(out.block.size());
    int64_t done = 0;
    do {
      const int64_t nm = std::min<int64_t>(block_mons, M - done);
      ValBlock blk{};
      blk.unit0 = uint32_t(out.unit.size());
      blk.mon0 = packed;
      blk.nmon = uint32_t(nm);
      // units
      int64_t j = 0;
      while (j < nm) {
        const int64_t tf = order[size_t(done + j)];
        const int kf = int(in.mon_ptr[tf + 1] - in.mon_ptr[tf]);
        const int lgs = val_lg_lanes(kf), s = 1 << lgs;
        ValUnit u{};
        if (out.rec.size() > 0xffffffffu - 64u * 16u) return false;
        u.base = uint32_t(out.rec.size());
        u.mon = uint16_t(j);
        u.lgs = uint8_t(lgs);
        u.seg = uint32_t(std::max(1, (kf + s - 1) / s));
        int count = 0;
        while (j + count < nm && count < 64 / s) {
          const int64_t t = order[size_t(done + j + count)];
          if (val_lg_lanes(int(in.mon_ptr[t + 1] - in.mon_ptr[t])) != lgs) break;
          ++count;
        }
        u.count = uint8_t(count);
        out.rec.resize(out.rec.size() + 64 * size_t(u.seg), neutral);
        for (int g = 0; g < count; ++g) {
          const int64_t t = order[size_t(done + j + g)];
          const int64_t a = in.mon_ptr[t], b = in.mon_ptr[t + 1];
          uint32_t* r = out.rec.data() + u.base + size_t(g) * s;
          for (int64_t o = a; o < b; ++o) {
            const int i = int(o - a);
            r[64 * (i / s) + i % s] = uint32_t(in.var_idx[o]) + uint32_t(in.exps[o] - 1) * cols;
          }
        }
        out.unit.push_back(u);
        j += count;
      }
      blk.unit1 = uint32_t(out.unit.size());
      // column lists
      const std::vector<int>* c_of = &total;
      if (M > block_mons) {
        cnt.assign(size_t(n), 0);
        for (int64_t g = 0; g < nm; ++g) {
          const int64_t t = order[size_t(done + g)];
          for (int64_t o = in.mon_ptr[t]; o < in.mon_ptr[t + 1]; ++o) cnt[size_t(in.var_idx[o])]++;
        }
        c_of = &cnt;
        out.multi = true;
      }
      blk.slice0 = uint32_t(out.slice.size());
      uint32_t rows = uint32_t(out.ell.size() / 64);
      for (int c = 0; c < slices; ++c) {
        out.slice.push_back(rows);
        int len = 0;
        for (int x = 0; x < per && c * per + x < n; ++x)
          len = std::max(len, ((*c_of)[perm[c * per + x]] + Q - 1) / Q);
        rows += uint32_t(len);
      }
      out.slice.push_back(rows);
      if (rows > 0xffffffffu / 64 || int64_t(rows) * 64 > kValPadding * nnz + (1 << 18)) return false;
      out.ell.resize(size_t(rows) * 64, uint32_t(nm));
      fill.assign(size_t(n), 0);
      const uint32_t* sl = out.slice.data() + blk.slice0;
      for (int64_t g = 0; g < nm; ++g) {
        const int64_t t = order[size_t(done + g)];
        for (int64_t o = in.mon_ptr[t]; o < in.mon_ptr[t + 1]; ++o) {
          const int col = in.var_idx[o], at = place[size_t(col)], e = fill[size_t(col)]++;
          out.ell[(size_t(sl[at / per]) + size_t(e / Q)) * 64 + size_t((at % per) * Q + e % Q)] =
              uint32_t(g) | (uint32_t(in.exps[o]) << 16);
        }
      }
      out.max_mon = std::max(out.max_mon, int(nm));
      out.max_units = std::max(out.max_units, int(blk.unit1 - blk.unit0));
      out.block.push_back(blk);
      packed += uint32_t(nm);
      done += nm;
    } while (done < M);
  }
  out.row_block[size_t(N)] = uint32_t(out.block.size());
  // uniform rows
  if (N > 0 && !out.multi && out.block[0].nmon > 0) {
    const ValUnit& f = out.unit[0];
    const uint32_t nm = out.block[0].nmon, per = 64u >> f.lgs, units = (nm + per - 1) / per;
    bool uni = true;
    for (const ValBlock& b : out.block) uni = uni && b.nmon == nm && b.unit1 - b.unit0 == units;
    for (size_t u = 0; u < out.unit.size() && uni; ++u)
      uni = out.unit[u].lgs == f.lgs && out.unit[u].seg == f.seg && out.unit[u].base == uint32_t(u) * 64 * f.seg;
    if (uni) {
      out.uni_mons = int(nm);
      out.uni_lgs = f.lgs;
      out.uni_units = int(units);
      out.uni_seg = int(f.seg);
    }
  }
  return true;
}

}  // namespace pe
