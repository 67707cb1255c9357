// Host build of the finer quad-double products for accuracy checks from the
// test suite.
#include "../paper_1402_2626_amd/csrc/mdarith.hpp"

using namespace pe;

static R<4> at(const double* p) { return R<4>{{p[0], p[1], p[2], p[3]}}; }

// per case: four operands of four limbs in, fine and plain product of the first
// two, fine and plain sum of two products out
extern "C" void pe_test_qd_fine(int count, const double* in, double* out) {
  for (int i = 0; i < count; ++i) {
    const double* p = in + 16 * i;
    const R<4> r[4] = {r_mul_fine(at(p), at(p + 4)), r_mul(at(p), at(p + 4)),
                       qd_dot2_fine(at(p), at(p + 4), at(p + 8), at(p + 12)),
                       qd_dot2(at(p), at(p + 4), at(p + 8), at(p + 12))};
    for (int k = 0; k < 4; ++k)
      for (int l = 0; l < 4; ++l) out[16 * i + 4 * k + l] = r[k].x[l];
  }
}
