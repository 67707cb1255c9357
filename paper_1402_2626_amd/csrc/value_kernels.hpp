// Evaluation and differentiation through monomial values (gfx950).
//
// For a variable x_v that is not zero, every monomial t that contains it
// with exponent d has d V_t / x_v as its partial derivative, V_t the
// monomial's value.  A column of a row of J is therefore
//     J_pv = (1 / x_v) sum over t of d_tv V_t,
// one product per occurrence for the values and one scaled addition per
// occurrence for the column, where the reverse sweep of Sec. 2.2 takes about
// four products: in double double 63 FP64 instructions against 175, in quad
// double 580 against 2000.  The terms of the sum are x_v times the terms of
// J_pv, so the error against the sum of their absolute values is that of the
// monomial values and of one more product.
//
// Zero variables need no division: a monomial's value is formed without its
// zero factors, and their count decides (no zero: as above; one zero variable
// of exponent 1: the value is the partial derivative with respect to that
// variable; otherwise the monomial contributes nothing).  Points with values
// outside 2^-300 .. 2^300 (for large exponents 2^(-750 / emax) .. 2^(900 / emax)),
// infinities or NaN, and rows in which a product of variables or a value (with
// its coefficient and weight) leaves 2^-750 .. 2^900 (below, a quad double's
// last limbs would underflow), form every partial derivative and every term of
// F as its own product instead (val_direct), in the same kernel.  The products
// on the way to a value are tested where the sizes of the variables allow them
// to leave the range (val_ranges).
//
// A COPY of VW threads (a multiple of 64) evaluates rows at one point:
//   1. powers x_v^1 .. x_v^emax of every variable into LDS (and 1 / x_v, by
//      the wavefronts that step 2 leaves idle);
//   2. its wavefronts take the row's units (layout.hpp): products of table
//      entries per lane, joined across a monomial's lanes by a butterfly, the
//      value (times the coefficient, for the adjoint also conj(v_p)) into LDS;
//   3. after a barrier they take the row's column slices: Q lanes add a
//      column's entries, read in coalesced order, and one of them multiplies
//      by 1 / x_v and writes J.  F is the sum of the values by one wavefront.
// Both phases read the occurrence lists from memory and gather from LDS; no
// partial derivatives are stored in between, so that the LDS of a row is the
// table and its values and several workgroups share a CU.  The order of every
// sum depends on the packing only, so a row has the same bits in every
// launch.
//
// A launch that fills the chip is bound by FP64 and address issue (LDS active
// a third of the time), one row per CU by the chain launch, loads, table,
// products, sums.  Reverse sweep -> this: DD n = 256, 256 x 16: 14.9 -> 14.0 us
// at one point, 343 -> 178 us at 64 points of 128 x 16; QD n = 512, 256 x 32:
// 546 -> 146 us; cyclic 192-roots in DD, whose longest rows are 192 monomials
// of 191 variables: 130 -> 45 us; a batch of 24 DD systems: 818 -> 375 us.
#pragma once
#include <hip/hip_runtime.h>

#include "blockls_kernels.hpp"
#include "eval_kernels.hpp"
#include "layout.hpp"
#include "mdarith.hpp"
#include "newton_kernels.hpp"

namespace pe {

struct ValView {
  int n, N, emax;
  int tab;  // powers in the table: emax, or 1 (higher ones formed per factor)
  int inv;  // reciprocals behind them, or formed per column
  int safe;  // monomials of variables within 2^-safe .. 2^safe stay within 2^-350 .. 2^350, whatever the order of the factors
  int lgQ, slices, max_mon;
  int max_units;
  int lgvw;   // log2 of the threads of a copy
  int uni_mons, uni_lgs, uni_seg, uni_units;  // uniform rows (layout.hpp, PackedValues), or 0
  int multi;  // some row has several blocks
  const ValBlock* block;
  const uint32_t* row_block;
  const ValUnit* unit;
  const uint32_t* rec;
  const uint32_t* ell;
  const uint32_t* slice;
  const uint16_t* perm;
  const double* mcoef;
  const uint32_t* row_order;
};

// Element i of an array in global memory.  A batch reads its views, and with
// them these pointers, from memory, and the compiler would use flat accesses.
template <typename T>
__device__ __forceinline__ T val_ld(const T* p, size_t i) {
  typedef uint32_t v4u __attribute__((ext_vector_type(4)));
  typedef uint32_t v2u __attribute__((ext_vector_type(2)));
  T r;
  if constexpr (sizeof(T) == 16) {
    const v4u w = *(const __attribute__((address_space(1))) v4u*)(p + i);
    __builtin_memcpy(&r, &w, 16);
  } else if constexpr (sizeof(T) == 24) {
    const __attribute__((address_space(1))) v2u* q = (const __attribute__((address_space(1))) v2u*)(p + i);
    const v2u w[3] = {q[0], q[1], q[2]};
    __builtin_memcpy(&r, w, 24);
  } else {
    r = *(const __attribute__((address_space(1))) T*)(p + i);
  }
  return r;
}

template <int L>
__device__ __forceinline__ C<L> val_ld_coef(const double* p) {
  C<L> r;
#pragma unroll
  for (int l = 0; l < limbs_of(L); ++l) {
    r.re.x[l] = val_ld(p, l);
    if constexpr (!is_real(L)) r.im.x[l] = val_ld(p, limbs_of(L) + l);
  }
  return r;
}

// doubles of a copy's LDS: [`blocks` (powers, reciprocals) of n + 1 numbers][max_mon + 1
// values][n column sums when rows have several blocks or the sums run over
// rows][zero counts, bytes][4 flags]
template <int L>
__host__ __device__ inline size_t val_copy_doubles(int n, int blocks, int max_mon, bool sums) {
  const size_t d =
      size_t(width_of(L)) * (size_t(blocks) * (n + 1) + max_mon + 1 + (sums ? n : 0)) + size_t(max_mon + 8) / 8 + 2;
  return (d + 1) & ~size_t(1);  // 16-byte words
}

// Numbers in LDS are records of consecutive limbs, read in 16-byte words: one
// address per gather, where planes of 8-byte words need one each (the product
// and column phases are bound by VALU issue, the LDS is active a third of the
// time).  The address space is spelled out: a batch's layout comes from
// memory, and the compiler would fall back to flat accesses.
typedef double val_v2d __attribute__((ext_vector_type(2)));

template <int L>
__device__ __forceinline__ C<L> val_get(const double* base, int i) {
  constexpr int W = width_of(L);
  double w[W];
  if constexpr (W == 1) {
    w[0] = ((const __attribute__((address_space(3))) double*)base)[i];
  } else {
    const __attribute__((address_space(3))) val_v2d* p =
        (const __attribute__((address_space(3))) val_v2d*)base + i * (W / 2);
#pragma unroll
    for (int k = 0; k < W / 2; ++k) {
      const val_v2d t = p[k];
      w[2 * k] = t.x;
      w[2 * k + 1] = t.y;
    }
  }
  return load_aos<L>(w);
}

template <int L>
__device__ __forceinline__ void val_put(double* base, int i, const C<L>& v) {
  constexpr int W = width_of(L);
  double w[W];
  store_aos(w, v);
  if constexpr (W == 1) {
    ((__attribute__((address_space(3))) double*)base)[i] = w[0];
  } else {
    __attribute__((address_space(3))) val_v2d* p = (__attribute__((address_space(3))) val_v2d*)base + i * (W / 2);
#pragma unroll
    for (int k = 0; k < W / 2; ++k) p[k] = val_v2d{w[2 * k], w[2 * k + 1]};
  }
}

template <int L>
struct ValLds {
  double* tab;    // x^e at (e - 1) cols + v, e <= S.tab; 1 / x (1 for x = 0) at S.tab cols + v
  double* val;    // [max_mon + 1]
  double* sum;    // [n]
  uint8_t* zeros;  // [max_mon]
  int* flag;      // [0], of the point: 1 a zero variable, 2 direct products; [1], of the row: direct products; [2], of the point: val_far
  int cols;
};

template <int L>
__device__ __forceinline__ ValLds<L> val_lds(const ValView& S, double* base, bool sums) {
  ValLds<L> M;
  M.cols = S.n + 1;
  M.tab = base;
  M.val = M.tab + size_t(width_of(L)) * (S.tab + S.inv) * M.cols;
  M.sum = M.val + size_t(width_of(L)) * (S.max_mon + 1);
  double* z = M.sum + (sums ? size_t(width_of(L)) * S.n : 0);
  M.zeros = reinterpret_cast<uint8_t*>(z);
  M.flag = reinterpret_cast<int*>(z + (S.max_mon + 8) / 8);
  return M;
}

template <int L>
__device__ __forceinline__ double val_mag(const C<L>& a) {
  return fmax(fabs(a.re.x[0]), fabs(im_lead(a)));
}

template <int L>
__device__ __forceinline__ bool val_nan(const C<L>& a) {
  const double s = a.re.x[0] + im_lead(a);
  return !(s == s);
}

// The product.  A derivative through values takes about three roundings more
// than in the reverse sweep (x_v itself, its reciprocal, the last product).  In
// quad double, where that showed (mean error of J 1.0 to 1.9 times the
// sweep's), the products that join pairs of factors and all later ones are the
// finer ones, and the sums carry a fifth part: 0.6 to 1.2 times, 0.72 on the
// whole (complex), 0.85 (real), for a tenth of the time.
template <int L>
__device__ __forceinline__ C<L> val_mul(const C<L>& a, const C<L>& b) {
  if constexpr (L == 4)
    return C<4>{qd_dot2_fine(a.re, b.re, r_neg(a.im), b.im), qd_dot2_fine(a.re, b.im, a.im, b.re)};
  else if constexpr (limbs_of(L) == 4)
    return C<L>{r_mul_fine(a.re, b.re)};
  else
    return c_mul(a, b);
}

template <int L>
__device__ C<L> val_pow(const C<L>& x, int e) {
  C<L> r = x, b = x;
  e -= 1;
  while (e > 0) {
    if (e & 1) r = val_mul(r, b);
    e >>= 1;
    if (e) b = val_mul(b, b);
  }
  return r;
}

// 1 / a to the last place; quad double by the series z (1 + t + t^2), t = 1 -
// a z, from a double-double z with relative error below 2^-100
template <int NL>
__device__ __forceinline__ R<NL> val_recip(const R<NL>& a) {
  if constexpr (NL == 2) {
    return bl_recip<2>(a);
  } else {
    const R<2> z2 = bl_recip<2>(R<2>{{a.x[0], a.x[1]}});
    const R<4> z{{z2.x[0], z2.x[1], 0.0, 0.0}};
    R<4> t = r_sub(r_from_double<4>(1.0), r_mul_fine(a, z));
    const double lead = t.x[0] + (t.x[1] + t.x[2]);  // the leading limbs may have cancelled
    t = r_add(t, r_from_double<4>(lead * lead));
    return r_add(z, r_mul(z, t));
  }
}

// 1 / x = conj(x) / |x|^2; double forms |x|^2 and its reciprocal with a
// correction term and rounds once.  Complex quad double takes that of two limbs,
// z, and its residual t = 1 - x z: z (1 + t + t^2), whose error is that of t
// alone.
template <int L>
__device__ __forceinline__ C<L> val_inverse(const C<L>& x) {
  C<L> r;
  if constexpr (limbs_of(L) == 1) {
    double h = x.re.x[0] * x.re.x[0], e = PE_FMA(x.re.x[0], x.re.x[0], -h);
    if constexpr (is_real(L)) {
      h = x.re.x[0];
      e = 0.0;
    } else {
      double g, f, s, t;
      two_prod(x.im.x[0], x.im.x[0], g, f);
      two_sum(h, g, s, t);
      h = s;
      e += f + t;
    }
    double y = __builtin_amdgcn_rcp(h);
    y = PE_FMA(y, PE_FMA(-h, y, 1.0), y);
    y = PE_FMA(y, PE_FMA(-h, y, 1.0), y);
    const double c = y * PE_FMA(-e, y, PE_FMA(-h, y, 1.0));
    if constexpr (is_real(L)) {
      r.re.x[0] = y + c;
    } else {
      r.re.x[0] = PE_FMA(x.re.x[0], y, x.re.x[0] * c);
      r.im.x[0] = -PE_FMA(x.im.x[0], y, x.im.x[0] * c);
    }
  } else if constexpr (is_real(L)) {
    r.re = val_recip<limbs_of(L)>(x.re);
  } else if constexpr (L == 2) {
    r = c_mul_r(c_conj(x), val_recip<2>(c_norm2(x)));
  } else {
    const C<2> z2 = val_inverse<2>(C<2>{{{x.re.x[0], x.re.x[1]}}, {{x.im.x[0], x.im.x[1]}}});
    const C<4> z{{{z2.re.x[0], z2.re.x[1], 0.0, 0.0}}, {{z2.im.x[0], z2.im.x[1], 0.0, 0.0}}};
    C<4> t = c_sub(c_one<4>(), val_mul(x, z));
    const double tr = t.re.x[0] + (t.re.x[1] + t.re.x[2]), ti = t.im.x[0] + (t.im.x[1] + t.im.x[2]);
    t.re = r_add(t.re, r_from_double<4>(PE_FMA(tr, tr, -ti * ti)));
    t.im = r_add(t.im, r_from_double<4>(2.0 * tr * ti));
    r = c_add(z, c_mul(z, t));
  }
  return r;
}

// 64 log2 |x| of an x that is not zero, away from zero (by up to 1; 0 within
// 1e-4 of |x| = 1)
template <int L>
__device__ __forceinline__ int val_log(const C<L>& x) {
  const double mag = val_mag(x);
  if (!(mag <= 0x1.fffffffffffffp1023)) return 64 * 1024;
  const int k = __builtin_amdgcn_frexp_exp(mag);
  const double a = __builtin_ldexp(x.re.x[0], -k), b = __builtin_ldexp(im_lead(x), -k);
  const float l = 64.0f * float(k) + 32.0f * __builtin_amdgcn_logf(float(a * a + b * b));
  const int up = int(ceilf(fabsf(l) - 0.01f));
  return l < 0.0f ? -up : up;
}

// The copy's table for the point xpt (x0 = val_first_x, loaded ahead); lv of
// VW threads, flag clear
template <int L>
__device__ __forceinline__ C<L> val_first_x(const ValView& S, const double* __restrict__ xpt, int lv) {
  return lv < S.n ? load_planar<L>(xpt, S.n, lv) : c_one<L>();
}

template <int L>
__device__ __forceinline__ void val_table(const ValView& S, const ValLds<L>& M, const double* __restrict__ xpt, int lv,
                                          int VW, const C<L>& x0) {
  const double big = __builtin_ldexp(1.0, min(300, 900 / S.emax)), small = __builtin_ldexp(1.0, -min(300, 750 / S.emax));
  const double lo = __builtin_ldexp(1.0, -S.safe), hi = __builtin_ldexp(0.5, S.safe);
  int f = 0;
  for (int v = lv; v <= S.n; v += VW) {
    const C<L> x = v == lv ? x0 : (v < S.n ? load_planar<L>(xpt, S.n, v) : c_one<L>());
    C<L> p = x;
    for (int e = 1; e <= S.tab; ++e) {
      if (e > 1) p = val_mul(p, x);
      val_put(M.tab, (e - 1) * M.cols + v, p);
    }
    const double mag = val_mag(x);
    if (mag == 0.0)
      f |= 1;
    else if (__builtin_expect(!(mag >= lo && mag <= hi), 0))
      f |= mag >= small && mag <= big ? 4 : 2;
    if (val_nan(x)) f |= 2;
  }
  if (f) atomicOr(M.flag, f);
  if (__builtin_expect((f & 4) != 0, 0)) {
    // apart from the loop above, whose registers it would take
    int far = 0;
    for (int v = lv; v < S.n; v += VW) {
      const C<L> x = val_get<L>(M.tab, v);
      if (val_mag(x) != 0.0) far += max(abs(val_log(x)) - 64 * S.safe, 0);
    }
    atomicAdd(M.flag + 2, far);
  }
}

// The table's reciprocals, behind its powers.  The column phase is the first
// to read them, so they are formed in the product phase, from the copy's last
// thread down: the wavefronts without a unit take them (in double double a
// reciprocal is a chain of some 60 dependent operations).
template <int L>
__device__ __forceinline__ void val_inverses(const ValView& S, const ValLds<L>& M, int lv, int VW) {
  for (int v = VW - 1 - lv; v < S.n; v += VW) {
    const C<L> x = val_get<L>(M.tab, v);
    val_put(M.tab, S.tab * M.cols + v, val_mag(x) == 0.0 ? c_one<L>() : val_inverse(x));
  }
}

// Block b and unit u of block blk: computed where the rows are uniform, so
// that the records' loads wait for no other load
__device__ __forceinline__ ValBlock val_block(const ValView& S, uint32_t b) {
  if (S.uni_mons == 0) return val_ld(S.block, b);
  ValBlock k;
  k.unit0 = b * uint32_t(S.uni_units);
  k.unit1 = k.unit0 + uint32_t(S.uni_units);
  k.mon0 = b * uint32_t(S.uni_mons);
  k.nmon = uint32_t(S.uni_mons);
  k.slice0 = b * uint32_t(S.slices + 1);
  k.pad = 0;
  return k;
}

__device__ __forceinline__ ValUnit val_unit_of(const ValView& S, const ValBlock& blk, uint32_t u) {
  if (S.uni_mons == 0) return val_ld(S.unit, u);
  const uint32_t per = 64u >> S.uni_lgs, mon = (u - blk.unit0) * per;
  ValUnit k;
  k.base = u * 64u * uint32_t(S.uni_seg);
  k.mon = uint16_t(mon);
  k.count = uint8_t(min(per, blk.nmon - mon));
  k.lgs = uint8_t(S.uni_lgs);
  k.seg = uint32_t(S.uni_seg);
  k.pad = 0;
  return k;
}

__device__ __forceinline__ int val_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// What a wavefront's first steps of a row read from memory, loaded before the
// table is built: the block, the first unit with its first records and
// coefficient, the first slice with its first entries
template <int L>
struct ValPre {
  ValBlock blk;
  ValUnit u;
  uint32_t r[4];
  C<L> cf;
  uint32_t e0, e1;
  int col;
  uint32_t el[4];
};

template <int L>
__device__ __forceinline__ void val_records(const ValView& S, const ValBlock& blk, const ValUnit& u, int lane,
                                            uint32_t (&r)[4], C<L>& cf) {
  const uint32_t* rec = S.rec + u.base + lane;
  const int last = int(u.seg) - 1;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = val_ld(rec, 64 * min(i, last));
  const int g = lane >> u.lgs;
  cf = c_one<L>();
  if ((lane & ((1 << u.lgs) - 1)) == 0 && g < int(u.count))
    cf = val_ld_coef<L>(S.mcoef + size_t(blk.mon0 + u.mon + g) * width_of(L));
}

template <int L>
__device__ __forceinline__ void val_entries(const ValView& S, const ValBlock& blk, uint32_t e0, uint32_t e1, int lane,
                                            uint32_t (&el)[4]) {
  const uint32_t* ell = S.ell + lane;
#pragma unroll
  for (int i = 0; i < 4; ++i) el[i] = e0 + i < e1 ? val_ld(ell, 64 * size_t(e0 + i)) : blk.nmon;
}

// w: the copy's wavefront, of nw
template <int L, int MODE>
__device__ __forceinline__ void val_prefetch(const ValView& S, int p, int w, int lane, ValPre<L>& pre) {
  // one block per row: its index is the row's
  pre.blk = val_block(S, S.multi ? val_ld(S.row_block, p) : uint32_t(p));
  if (pre.blk.unit0 + w < pre.blk.unit1) {
    pre.u = val_unit_of(S, pre.blk, pre.blk.unit0 + w);
    val_records<L>(S, pre.blk, pre.u, lane, pre.r, pre.cf);
  }
  if (MODE != MODE_FONLY && w < S.slices) {
    const int per = 64 >> S.lgQ;
    const uint32_t* sl = S.slice + (S.multi ? size_t(pre.blk.slice0) : size_t(p) * (S.slices + 1)) + w;
    pre.e0 = val_ld(sl, 0);
    pre.e1 = val_ld(sl, 1);
    pre.col = val_ld(S.perm, size_t(p) * S.slices * per + w * per + (lane >> S.lgQ));
    val_entries<L>(S, pre.blk, pre.e0, pre.e1, lane, pre.el);
  }
}

// SMALL (FULL false here): the kernels that also take systems whose table
// holds x alone (apart, since the code costs the others 3 to 9 %)
//
// one factor, x^d of a record; with ZERO a zero variable counts into z and is
// taken as 1
template <int L, bool ZERO, bool FULL>
__device__ __forceinline__ C<L> val_factor(const ValLds<L>& M, uint32_t r, int& z) {
  C<L> f;
  if constexpr (FULL) {
    f = val_get<L>(M.tab, int(r));
  } else {
    const uint32_t e = r / uint32_t(M.cols);
    f = val_get<L>(M.tab, int(r - e * uint32_t(M.cols)));
    if (e > 0) f = val_pow(f, int(e) + 1);
  }
  if constexpr (ZERO) {
    if (val_mag(val_get<L>(M.tab, int(r % uint32_t(M.cols)))) == 0.0) {
      z += r < uint32_t(M.cols) ? 1 : 2;
      f = c_one<L>();
    }
  }
  return f;
}

// Product phase of one unit by one wavefront (its first records and
// coefficient in r, cf): values into LDS.  Four factors at a time, joined as
// (f0 f1)(f2 f3), so that only one product in four is in the lane's chain.
template <int L, bool ZERO, bool FULL>
__device__ __forceinline__ void val_unit(const ValView& S, const ValLds<L>& M, const ValUnit& u, int lane,
                                         uint32_t (&r)[4], const C<L>& cf, bool direct, bool weighted,
                                         const C<L>& weight) {
  const int s = 1 << u.lgs, g = lane >> u.lgs;
  const uint32_t* rec = S.rec + u.base + lane;
  const int seg = int(u.seg);
  int z = 0;
  C<L> A = c_one<L>();
  int i0 = 0;
  for (; i0 + 4 <= seg; i0 += 4) {
    uint32_t nx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) nx[i] = val_ld(rec, 64 * min(i0 + 4 + i, seg - 1));
    const C<L> f0 = val_factor<L, ZERO, FULL>(M, r[0], z), f1 = val_factor<L, ZERO, FULL>(M, r[1], z);
    const C<L> f2 = val_factor<L, ZERO, FULL>(M, r[2], z), f3 = val_factor<L, ZERO, FULL>(M, r[3], z);
    const C<L> B = val_mul(c_mul(f0, f1), c_mul(f2, f3));
    A = i0 == 0 ? B : val_mul(A, B);
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = nx[i];
  }
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (i0 + i < seg) {
      const C<L> f = val_factor<L, ZERO, FULL>(M, r[i], z);
      A = i0 + i == 0 ? f : val_mul(A, f);
    }
  for (int m = 1; m < s; m <<= 1) {
    A = val_mul(A, shfl_xor_c(A, m));
    if constexpr (ZERO) z += __shfl_xor(z, m);
  }
  C<L> V = val_mul(A, cf);
  if (weighted) V = val_mul(V, weight);
  if ((lane & (s - 1)) == 0 && g < int(u.count)) {
    const int t = u.mon + g;
    val_put(M.val, t, V);
    if constexpr (ZERO) M.zeros[t] = uint8_t(min(z, 2));
    // the value is divided by x_v, so it needs its last limbs as the product
    // does, unless it is zero by its coefficient or weight
    const double mag = val_mag(A), vm = val_mag(V);
    const bool none = val_mag(cf) == 0.0 || (weighted && val_mag(weight) == 0.0);
    const bool fine = mag >= 0x1p-750 && mag <= 0x1p900 && (vm >= 0x1p-750 || none) && vm <= 0x1p1000 && !val_nan(V);
    if (!fine && !direct) M.flag[1] = 1;
  }
}

// Whether the variables' sizes let a product of some factors of a monomial leave
// the range: flag[2] is by how many binary orders (times 64) they are beyond
// 2^-safe .. 2^safe in all, a factor takes that up to emax times, and 400 orders
// are left.  In fractions of an order, so that monomials of many hundred
// variables of modulus near 1 stay clear of it (cyclic 512-roots: 0.42 ms in DD
// against 0.68 with val_ranges).
__device__ __forceinline__ bool val_far(const ValView& S, int far) { return far > 64 * 400 / S.emax; }

// Whether some product of factors of a unit's monomials, in whatever order,
// can leave 2^-750 .. 2^900: one that leaves it and comes back has lost its last
// limbs.  By the sums of the factors' negative and positive exponents, apart
// from the products so that those keep their registers (tested product by
// product, a launch of one row per CU took 14.3 us in place of 14.15); only for
// points whose variables are far from 1 (val_far).
template <int L, bool FULL>
__device__ __forceinline__ void val_ranges(const ValView& S, const ValLds<L>& M, const ValUnit& u, int lane) {
  int lo = 0, hi = 0;
#pragma unroll 1
  for (int i = 0; i < int(u.seg); ++i) {
    const uint32_t r = val_ld(S.rec + u.base + lane, 64 * i);
    const uint32_t e = FULL ? 0 : r / uint32_t(M.cols);
    const C<L> x = val_get<L>(M.tab, int(r - e * uint32_t(M.cols)));
    if (val_mag(x) == 0.0) continue;
    const int k = val_log(x);
    lo += min(k, 0) * int(e + 1);
    hi += max(k, 0) * int(e + 1);
  }
  for (int m = 1; m < 1 << u.lgs; m <<= 1) {
    lo += __shfl_xor(lo, m);
    hi += __shfl_xor(hi, m);
  }
  if (lo < -750 * 64 || hi > 900 * 64) M.flag[1] = 1;
}

// ------------------------------------------------------------------ column sums

// running sum of d V: the terms go into error-free cascades (double: one
// compensated sum), the terms dropped are of order u^limbs times the sum of
// absolute values
template <int NL>
struct ValSum {
  double a[NL == 1 ? 2 : (NL == 4 ? 5 : NL)];
};

template <int NL>
__device__ __forceinline__ void val_add(ValSum<NL>& s, const R<NL>& v, double d) {
  if constexpr (NL == 1) {
    double t, e;
    two_sum(s.a[0], v.x[0] * d, t, e);
    s.a[0] = t;
    s.a[1] += e;
  } else if constexpr (NL == 2) {
    const double h = v.x[0] * d;
    const double l = PE_FMA(v.x[1], d, PE_FMA(v.x[0], d, -h));
    double t, e;
    two_sum(s.a[0], h, t, e);
    s.a[0] = t;
    s.a[1] += e + l;
  } else {
    double p[4], q[3], t, e1, e2, f1, f2, f3;
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = v.x[i] * d;
#pragma unroll
    for (int i = 0; i < 3; ++i) q[i] = PE_FMA(v.x[i], d, -p[i]);
    two_sum(s.a[0], p[0], t, e1);
    s.a[0] = t;
    // order 1: p1, q0, e1
    two_sum(p[1], q[0], p[1], f1);
    two_sum(p[1], e1, p[1], f2);
    two_sum(s.a[1], p[1], t, e2);
    s.a[1] = t;
    // order 2: p2, q1, f1, f2, e2
    two_sum(p[2], q[1], p[2], f3);
    double g1, g2, g3, g4;
    two_sum(f1, f2, f1, g1);
    two_sum(p[2], f1, p[2], g2);
    two_sum(p[2], e2, p[2], g3);
    two_sum(s.a[2], p[2], t, g4);
    s.a[2] = t;
    two_sum(s.a[3], (p[3] + q[2]) + ((f3 + g1) + (g2 + g3)) + g4, t, f1);
    s.a[3] = t;
    s.a[4] += f1;
  }
}

// carries the parts' overlap up, so that the error of later additions stays
// that of the level; after every fourth term
template <int NL>
__device__ __forceinline__ void val_carry(ValSum<NL>& s) {
  if constexpr (NL == 2) {
    two_sum(s.a[0], s.a[1], s.a[0], s.a[1]);
  } else if constexpr (NL == 4) {
    const R<4> r = renorm5(s.a[0], s.a[1], s.a[2], s.a[3], s.a[4]);
#pragma unroll
    for (int l = 0; l < 4; ++l) s.a[l] = r.x[l];
    s.a[4] = 0.0;
  }
}

template <int NL>
__device__ __forceinline__ R<NL> val_total(const ValSum<NL>& s) {
  R<NL> r;
  if constexpr (NL == 1)
    r.x[0] = s.a[0] + s.a[1];
  else if constexpr (NL == 2)
    two_sum(s.a[0], s.a[1], r.x[0], r.x[1]);
  else
    r = renorm5(s.a[0], s.a[1], s.a[2], s.a[3], s.a[4]);
  return r;
}

// r 2^e with the leading limb of r's larger part in 2^-128 .. 2^128; zeros and
// what is not finite stay as they are
template <int L>
__device__ __forceinline__ void val_norm(C<L>& r, int& e) {
  const double mag = val_mag(r);
  if (mag >= 0x1p-128 && mag <= 0x1p128) return;
  if (!(mag > 0.0 && mag <= 0x1.fffffffffffffp1023)) return;
  const int k = __builtin_amdgcn_frexp_exp(mag);
  r = bl_ldexp(r, -k);
  e += k;
}

// partial derivative of monomial t with respect to column v (exponent d), or
// for v < 0 its value (d = 1), every factor in turn: the definition, for points
// the division does not suit.  The product is kept as r 2^e, so that no order
// of the factors leaves the range on the way to a result within it.  Powers come
// from the table where they are in range there (a NaN among 512 polynomials of
// 256 monomials of 32 variables up to the third power, quad double: 3.2 ms; each
// formed here: 10.0; among 256 x 256 x 16 up to the fourth, double double: 0.15
// and 0.24).  wt: the row's weight v_p (planes N apart), whose conjugate
// multiplies the product, or null; read here, so that the common path need not
// keep it.
template <int L>
__device__ C<L> val_direct(const ValView& S, const ValLds<L>& M, const ValBlock& blk, uint32_t t, int v, int d,
                           const double* wt) {
  uint32_t u = blk.unit0;
  while (u + 1 < blk.unit1 && val_ld(S.unit, u + 1).mon <= t) ++u;
  const ValUnit U = val_ld(S.unit, u);
  const int g = int(t) - int(U.mon);
  int e = 0;
  C<L> r = val_ld_coef<L>(S.mcoef + size_t(blk.mon0 + t) * width_of(L));
  val_norm(r, e);
  if (wt) {
    C<L> weight;
#pragma unroll
    for (int l = 0; l < limbs_of(L); ++l) {
      weight.re.x[l] = val_ld(wt, size_t(l) * S.N);
      if constexpr (!is_real(L)) weight.im.x[l] = -val_ld(wt, size_t(limbs_of(L) + l) * S.N);
    }
    val_norm(weight, e);
    r = c_mul(r, weight);
    val_norm(r, e);
  }
  for (int i = 0; i < int(U.seg); ++i)
    for (int q = 0; q < (1 << U.lgs); ++q) {
      const int w = int(val_ld(S.rec, U.base + 64 * i + (g << U.lgs) + q));
      const int wv = w % M.cols, wd = w / M.cols + (wv != v);
      if (wv == S.n || wd == 0) continue;
      C<L> x = val_get<L>(M.tab, (min(wd, S.tab) - 1) * M.cols + wv);
      int ex = 0;
      if (wd > 1 && !(wd <= S.tab && val_mag(x) >= 0x1p-750 && val_mag(x) <= 0x1p900)) {
        // x^wd is not in the table, or out of range there
        x = val_get<L>(M.tab, wv);
        const double mag = val_mag(x);
        if (mag > 0.0 && mag <= 0x1.fffffffffffffp1023) {
          ex = __builtin_amdgcn_frexp_exp(mag);
          x = bl_ldexp(x, -ex);
          ex *= wd;
        }
        x = c_pow(x, wd);
      }
      val_norm(x, ex);
      r = c_mul(r, x);
      e += ex;
      val_norm(r, e);
    }
  return bl_ldexp(c_mul_d(r, double(d)), e);
}

// Column `col`'s sum over a slice by the calling lane and its Q - 1
// neighbours (the slice's first entries in r): the block's share of J_pv, in
// every one of the Q lanes.  All lanes of the wavefront call it.
template <int L, bool ZERO, bool SMALL>
__device__ __forceinline__ C<L> val_column(const ValView& S, const ValLds<L>& M, const ValBlock& blk, uint32_t e0,
                                           uint32_t e1, int col, int lane, uint32_t (&r)[4]) {
  constexpr int NL = limbs_of(L);
  const uint32_t* ell = S.ell + lane;
  ValSum<NL> re{}, im{};
  const bool at_zero = ZERO && val_mag(val_get<L>(M.tab, col)) == 0.0;  // the column's own variable
  for (uint32_t i0 = e0; i0 < e1; i0 += 4) {
    uint32_t nx[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) nx[i] = i0 + 4 + i < e1 ? val_ld(ell, 64 * size_t(i0 + 4 + i)) : blk.nmon;
    C<L> V[4];
    double d[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = r[i] & 0xffffu;
      V[i] = val_get<L>(M.val, t);
      d[i] = double(r[i] >> 16);
      if constexpr (ZERO) {
        const int z = uint32_t(t) < blk.nmon ? M.zeros[t] : 2;
        if (at_zero ? !(z == 1 && d[i] == 1.0) : z != 0) d[i] = 0.0;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i0 + i < e1) {  // uniform
        val_add<NL>(re, V[i].re, d[i]);
        if constexpr (!is_real(L)) val_add<NL>(im, V[i].im, d[i]);
      }
    }
    val_carry<NL>(re);
    if constexpr (!is_real(L)) val_carry<NL>(im);
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = nx[i];
  }
  C<L> J;
  J.re = val_total<NL>(re);
  if constexpr (!is_real(L)) J.im = val_total<NL>(im);
  for (int m = 1; m < (1 << S.lgQ); m <<= 1) J = c_add(J, shfl_xor_c(J, m));
  if constexpr (SMALL)
    if (!S.inv) {
      const C<L> x = val_get<L>(M.tab, col);
      return val_mag(x) == 0.0 ? J : val_mul(J, val_inverse(x));
    }
  return val_mul(J, val_get<L>(M.tab, S.tab * M.cols + col));
}

// the same by products of all factors
template <int L>
__device__ __forceinline__ C<L> val_column_direct(const ValView& S, const ValLds<L>& M, const ValBlock& blk, uint32_t e0,
                                                  uint32_t e1, int col, int lane, const double* wt) {
  const uint32_t* ell = S.ell + lane;
  C<L> J = c_zero<L>();
  for (uint32_t i = e0; i < e1; ++i) {
    const uint32_t r = val_ld(ell, 64 * size_t(i)), t = r & 0xffffu;
    if (t < blk.nmon) J = c_add(J, val_direct<L>(S, M, blk, t, col, int(r >> 16), wt));
  }
  for (int m = 1; m < (1 << S.lgQ); m <<= 1) J = c_add(J, shfl_xor_c(J, m));
  return J;
}

// F's share of a block by one wavefront, the same in every lane.  Where the
// row takes direct products, so does F: a value stored with its zero factors
// left out is not a term of F beside a factor that is out of range.
template <int L>
__device__ __forceinline__ C<L> val_f(const ValView& S, const ValLds<L>& M, const ValBlock& blk, int lane, bool zero,
                                      bool direct) {
  constexpr int NL = limbs_of(L);
  C<L> f = c_zero<L>();
  if (__builtin_expect(direct, 0)) {
    for (uint32_t t = lane; t < blk.nmon; t += 64) f = c_add(f, val_direct<L>(S, M, blk, t, -1, 1, nullptr));
  } else {
    ValSum<NL> re{}, im{};
    for (uint32_t t = lane; t < blk.nmon; t += 64) {
      if (zero && M.zeros[t] != 0) continue;
      const C<L> V = val_get<L>(M.val, int(t));
      val_add<NL>(re, V.re, 1.0);
      if constexpr (!is_real(L)) val_add<NL>(im, V.im, 1.0);
      if ((t >> 6 & 3) == 3) {
        val_carry<NL>(re);
        if constexpr (!is_real(L)) val_carry<NL>(im);
      }
    }
    f.re = val_total<NL>(re);
    if constexpr (!is_real(L)) f.im = val_total<NL>(im);
  }
#pragma unroll 1
  for (int m = 1; m < 64; m <<= 1) f = c_add(f, shfl_xor_c(f, m));
  return f;
}

// Row p at the point whose table is in M, its prefetch in pre: all threads of
// the workgroup call it (it has barriers; every copy of a workgroup has the
// same number of blocks).  MODE_EVAL: F and J through O; MODE_FONLY: F;
// MODE_ADJ: conj(v_p) J added to M.sum.  inv: the point's first row, which
// forms the reciprocals.
template <int L, int MODE, bool SMALL>
__device__ __forceinline__ void val_row(const ValView& S, const ValLds<L>& M, const OutView& O, int pt, int p, int lv,
                                        int VW, bool live, bool inv, const C<L>& weight, const double* wt,
                                        ValPre<L>& pre) {
  const int lane = lv & 63, w = val_uniform(lv >> 6), nw = VW >> 6;
  const uint32_t b0 = S.multi ? val_ld(S.row_block, p) : uint32_t(p), b1 = S.multi ? val_ld(S.row_block, p + 1) : uint32_t(p) + 1;
  constexpr bool weighted = MODE == MODE_ADJ;
  C<L> F = c_zero<L>();
  const int f0 = val_uniform(M.flag[0]);
  const bool direct0 = (f0 & 2) != 0, zero = (f0 & 1) != 0 && !direct0;
  for (uint32_t b = b0; b < b1; ++b) {
    const ValBlock blk = b == b0 ? pre.blk : val_block(S, b);
    if (__builtin_expect(!direct0 && val_far(S, val_uniform(M.flag[2])), 0))
      for (uint32_t u = blk.unit0 + w; u < blk.unit1; u += nw)
        val_ranges<L, !SMALL>(S, M, val_unit_of(S, blk, u), lane);
    for (uint32_t u = blk.unit0 + w; u < blk.unit1; u += nw) {
      const bool first = b == b0 && u == blk.unit0 + w;
      if (!first) {
        pre.u = val_unit_of(S, blk, u);
        val_records<L>(S, blk, pre.u, lane, pre.r, pre.cf);
      }
      if (SMALL && S.tab < S.emax) {
        // the forms with zero counts hold for every point
        val_unit<L, true, false>(S, M, pre.u, lane, pre.r, pre.cf, direct0, weighted, weight);
      } else if (__builtin_expect(zero, 0)) {
        val_unit<L, true, true>(S, M, pre.u, lane, pre.r, pre.cf, direct0, weighted, weight);
      } else {
        val_unit<L, false, true>(S, M, pre.u, lane, pre.r, pre.cf, direct0, weighted, weight);
      }
    }
    if (MODE != MODE_FONLY && inv && (!SMALL || S.inv) && b == b0) val_inverses(S, M, lv, VW);
    if (lv == 0) val_put(M.val, int(blk.nmon), c_zero<L>());
    __syncthreads();
    const bool direct = direct0 || val_uniform(M.flag[1]) != 0;
    if (MODE != MODE_ADJ && w == nw - 1) {
      const C<L> f = val_f<L>(S, M, blk, lane, zero, direct);
      F = b == b0 ? f : c_add(F, f);
    }
    if (MODE != MODE_FONLY) {
      const int per = 64 >> S.lgQ;
      const uint16_t* perm = S.perm + size_t(p) * S.slices * per;
      const uint32_t* sl = S.slice + blk.slice0;
      for (int c = w; c < S.slices; c += nw) {
        if (b != b0 || c != w) {
          pre.e0 = val_ld(sl, c);
          pre.e1 = val_ld(sl, c + 1);
          pre.col = val_ld(perm, c * per + (lane >> S.lgQ));
          val_entries<L>(S, blk, pre.e0, pre.e1, lane, pre.el);
        }
        C<L> J;
        if (__builtin_expect(direct, 0)) {
          J = val_column_direct<L>(S, M, blk, pre.e0, pre.e1, pre.col, lane, wt);
        } else if (__builtin_expect(zero, 0)) {
          J = val_column<L, true, SMALL>(S, M, blk, pre.e0, pre.e1, pre.col, lane, pre.el);
        } else {
          J = val_column<L, false, SMALL>(S, M, blk, pre.e0, pre.e1, pre.col, lane, pre.el);
        }
        if (pre.col < S.n && (lane & ((1 << S.lgQ) - 1)) == 0) {
          if constexpr (MODE == MODE_ADJ) {
            val_put(M.sum, pre.col, c_add(val_get<L>(M.sum, pre.col), J));
          } else {
            const C<L> T = b == b0 ? J : c_add(val_get<L>(M.sum, pre.col), J);
            if (b + 1 < b1)
              val_put(M.sum, pre.col, T);
            else if (live)
              store_planar(O.J + pt * O.j_pt + int64_t(p) * O.j_row, O.j_plane, pre.col, T);
          }
        }
      }
    }
    __syncthreads();  // the values are free
  }
  if (MODE != MODE_ADJ && lv == VW - 1 && live) {
    if (O.f_sign < 0) F = c_neg(F);
    store_planar(O.F + pt * O.f_pt + int64_t(p) * O.f_row, O.f_plane, 0, F);
  }
}

// ------------------------------------------------------------------ kernels

constexpr int kValThreads = 512;

// Copies of VW threads; copy item c takes rows [R i, R i + R) (in row_order
// when there is one) of point pt, c = pt * groups + i.  Several copies share a
// workgroup when VW is small; systems with rows of several blocks take one
// copy per workgroup.  grid: ceil(P groups / copies)
template <int L, int MODE, bool SMALL>
__global__ __launch_bounds__(kValThreads, limbs_of(L) == 4 ? 2 : 4) void val_rows_kernel(ValView S, OutView O, const double* __restrict__ x,
                                                               int64_t x_pt, int P, int copies, int Rr, int groups,
                                                               int copy_doubles) {
  extern __shared__ __align__(16) double lds[];
  const int VW = 1 << S.lgvw;
  const int cp = val_uniform(int(threadIdx.x) >> S.lgvw);
  const int lv = int(threadIdx.x) & (VW - 1);
  const ValLds<L> M = val_lds<L>(S, lds + copy_doubles * cp, S.multi != 0);
  const int64_t item = int64_t(blockIdx.x) * copies + cp;
  const bool live = item < int64_t(P) * groups;
  const int pt = P == 1 || !live ? 0 : int(item / groups);
  const int i0 = live ? int(item - int64_t(pt) * groups) * Rr : 0;
  const int w = val_uniform(lv >> 6);
  for (int r = 0; r < Rr; ++r) {
    const bool in = live && i0 + r < S.N;
    const int b = min(i0 + r, S.N - 1);
    const int p = S.row_order ? int(S.row_order[b]) : b;
    C<L> x0;
    if (r == 0) x0 = val_first_x<L>(S, x + pt * x_pt, lv);
    ValPre<L> pre;
    val_prefetch<L, MODE>(S, p, w, lv & 63, pre);
    if (r == 0) {
      if (lv == 0) M.flag[0] = M.flag[1] = M.flag[2] = 0;
      __syncthreads();
      val_table<L>(S, M, x + pt * x_pt, lv, VW, x0);
    } else if (lv == 0) {
      M.flag[1] = 0;
    }
    __syncthreads();
    val_row<L, MODE, SMALL>(S, M, O, pt, p, lv, VW, in, r == 0, c_one<L>(), nullptr, pre);
  }
}

// Adjoint: one workgroup (one copy) per point and group of gsize rows; its
// column sums part[(pt NG + gi)][components][n]
template <int L, bool SMALL>
__global__ __launch_bounds__(kValThreads, limbs_of(L) == 4 ? 2 : 4) void val_adjoint_kernel(ValView S, const double* __restrict__ x, int64_t x_pt,
                                                                  const double* __restrict__ v, int64_t v_pt, int NG,
                                                                  int gsize, double* __restrict__ part) {
  extern __shared__ __align__(16) double lds[];
  const int VW = blockDim.x, lv = threadIdx.x;
  const int pt = blockIdx.x / NG, gi = blockIdx.x - pt * NG;
  const ValLds<L> M = val_lds<L>(S, lds, true);
  const int w = val_uniform(lv >> 6);
  const OutView O{};
  for (int p = gi * gsize; p < min(S.N, (gi + 1) * gsize); ++p) {
    C<L> x0;
    if (p == gi * gsize) x0 = val_first_x<L>(S, x + pt * x_pt, lv);
    ValPre<L> pre;
    val_prefetch<L, MODE_ADJ>(S, p, w, lv & 63, pre);
    const C<L> weight = c_conj(load_planar<L>(v + pt * v_pt, S.N, p));
    if (p == gi * gsize) {
      if (lv == 0) M.flag[0] = M.flag[1] = M.flag[2] = 0;
      __syncthreads();
      val_table<L>(S, M, x + pt * x_pt, lv, VW, x0);
      for (int c = lv; c < S.n; c += VW) val_put(M.sum, c, c_zero<L>());
    } else if (lv == 0) {
      M.flag[1] = 0;
    }
    __syncthreads();
    val_row<L, MODE_ADJ, SMALL>(S, M, O, 0, p, lv, VW, true, p == gi * gsize, weight, v + pt * v_pt + p, pre);
  }
  double* out = part + size_t(pt * NG + gi) * width_of(L) * S.n;
  for (int c = lv; c < S.n; c += VW) store_planar(out, S.n, c, val_get<L>(M.sum, c));
}

// g = conj of the groups' sums added in a fixed order: four threads per column
// take every fourth group, their sums are added in order.  grid (ceil(n / 64),
// P), 256 threads
template <int L>
__global__ __launch_bounds__(256) void val_adjoint_reduce_kernel(int n, int NG, const double* __restrict__ part,
                                                                 double* __restrict__ g) {
  __shared__ double red[4 * 64 * width_of(L)];
  const int j = blockIdx.x * 64 + (threadIdx.x & 63), h = threadIdx.x >> 6, pt = blockIdx.y;
  C<L> s = c_zero<L>();
  if (j < n)
#pragma unroll 4
    for (int gi = h; gi < NG; gi += 4)
      s = c_add(s, load_planar<L>(part + size_t(pt * NG + gi) * width_of(L) * n, n, j));
  store_planar(red, 256, threadIdx.x, s);
  __syncthreads();
  if (h == 0 && j < n) {
    for (int q = 1; q < 4; ++q) s = c_add(s, load_planar<L>(red, 256, q * 64 + (threadIdx.x & 63)));
    store_planar(g + size_t(pt) * width_of(L) * n, n, j, c_conj(s));
  }
}

// Persistent: workgroups take (system, row) items from a device counter in
// decreasing cost and evaluate each at all P points, as many points at once
// as the workgroup has copies of the system's width (systems of several blocks
// per row have kValThreads).  Every workgroup reaches the exit test after
// every item, so the grid drains.
template <int L, int MODE, bool SMALL>
__global__ __launch_bounds__(kValThreads, limbs_of(L) == 4 ? 2 : 4) void val_batch_kernel(const ValView* __restrict__ views,
                                                                const uint64_t* __restrict__ items, int64_t nitems,
                                                                int* counter, int P, const double* __restrict__ x,
                                                                const int64_t* __restrict__ x_off, BatchOut out) {
  extern __shared__ __align__(16) double lds[];
  __shared__ __align__(16) int64_t item_sh[2];  // 16 bytes: the numbers behind it are read in 16-byte words
  for (;;) {
    if (threadIdx.x == 0) item_sh[0] = atomicAdd(counter, 1);
    __syncthreads();
    const int64_t it = item_sh[0];
    if (it >= nitems) break;
    const uint64_t w = items[it];
    const int s = int(w >> 32), p = int(w & 0xffffffffu);
    const ValView S = views[s];
    const int VW = 1 << S.lgvw, copies = S.multi ? 1 : kValThreads >> S.lgvw;
    const int cp = val_uniform(int(threadIdx.x) >> S.lgvw);
    const int lv = int(threadIdx.x) & (VW - 1);
    const OutView O = batch_out_view<L>(out, s, S.n, S.N, P);
    const ValLds<L> M =
        val_lds<L>(S, lds + val_copy_doubles<L>(S.n, S.tab + S.inv, S.max_mon, S.multi != 0) * cp, S.multi != 0);
    const double* xs = x + x_off[s] * P;
    for (int pt0 = 0; pt0 < P; pt0 += copies) {
      const int pt = pt0 + cp;
      const bool live = pt < P;
      const double* xpt = xs + int64_t(live ? pt : 0) * width_of(L) * S.n;
      const C<L> x0 = val_first_x<L>(S, xpt, lv);
      ValPre<L> pre;
      val_prefetch<L, MODE>(S, p, val_uniform(lv >> 6), lv & 63, pre);
      if (lv == 0) M.flag[0] = M.flag[1] = M.flag[2] = 0;
      __syncthreads();
      val_table<L>(S, M, xpt, lv, VW, x0);
      __syncthreads();
      val_row<L, MODE, SMALL>(S, M, O, pt, p, lv, VW, live, true, c_one<L>(), nullptr, pre);
    }
  }
}

}  // namespace pe
