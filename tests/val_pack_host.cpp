// Host build of the value layout's packer for invariant checks from the test
// suite.
#include <cstdint>
#include <cstring>

#include "../paper_1402_2626_amd/csrc/packer.hpp"

using namespace pe;

static PackedValues g_pv;

extern "C" int pe_test_val_pack(int n, int N, const int64_t* poly_ptr, const int64_t* mon_ptr, const int32_t* var_idx,
                                const int32_t* exps, int block_mons, int64_t* sizes /* [13] */) {
  SysInput in;
  in.level = 1;
  in.n_vars = n;
  in.n_polys = N;
  in.poly_ptr = poly_ptr;
  in.mon_ptr = mon_ptr;
  in.var_idx = var_idx;
  in.exps = exps;
  if (!pack_values(in, block_mons, g_pv)) return 0;
  const int64_t s[10] = {1 << g_pv.lgQ, g_pv.slices, g_pv.max_mon, g_pv.max_units, g_pv.multi ? 1 : 0, int64_t(g_pv.rec.size()),
                         int64_t(g_pv.ell.size()), int64_t(g_pv.slice.size()), int64_t(g_pv.unit.size()),
                         int64_t(g_pv.block.size())};
  std::memcpy(sizes, s, sizeof s);
  const int64_t uni[3] = {g_pv.uni_mons, g_pv.uni_mons ? 1 << g_pv.uni_lgs : 0, g_pv.uni_seg};
  std::memcpy(sizes + 10, uni, sizeof uni);
  return 1;
}

// units as 5 int64 (base, mon, count, s, seg), blocks as 6 (unit0, unit1,
// mon0, nmon, slice0, pad)
extern "C" void pe_test_val_get(uint32_t* rec, uint32_t* ell, uint32_t* slice, int64_t* unit, int64_t* block,
                                uint32_t* row_block, uint16_t* perm) {
  std::memcpy(rec, g_pv.rec.data(), g_pv.rec.size() * 4);
  std::memcpy(ell, g_pv.ell.data(), g_pv.ell.size() * 4);
  std::memcpy(slice, g_pv.slice.data(), g_pv.slice.size() * 4);
  std::memcpy(row_block, g_pv.row_block.data(), g_pv.row_block.size() * 4);
  std::memcpy(perm, g_pv.perm.data(), g_pv.perm.size() * 2);
  for (size_t i = 0; i < g_pv.unit.size(); ++i) {
    const ValUnit& u = g_pv.unit[i];
    const int64_t v[5] = {u.base, u.mon, u.count, 1 << u.lgs, u.seg};
    std::memcpy(unit + 5 * i, v, sizeof v);
  }
  for (size_t i = 0; i < g_pv.block.size(); ++i) {
    const ValBlock& b = g_pv.block[i];
    const int64_t v[6] = {b.unit0, b.unit1, b.mon0, b.nmon, b.slice0, b.pad};
    std::memcpy(block + 6 * i, v, sizeof v);
  }
}
