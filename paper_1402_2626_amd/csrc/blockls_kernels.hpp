// Least-squares solve of A x = b by Gram-Schmidt on the augmented matrix
// [A b] (Sec. 3, Fig. 4, eq. (2)) in panels of B columns, with the long
// contractions on the int8 matrix cores, for any number of problems at once.
//
// Per panel (columns k0 .. k0 + B - 1 of the working copy W, already updated
// by the panels before it):
//   1. bl_gram_kernel: the Gram matrix of the panel;
//   2. bl_chol_kernel: its factor U^H D U, one workgroup per problem, so that
//      the serial chain of a panel is B small steps in LDS instead of B inner
//      products over all rows and B launches (the method of the Cholesky
//      factor of A^H A, with what it leaves corrected below);
//   3. bl_solve_kernel: X = A U^-1 D^-1/2 by forward substitution, row by row
//      (backward stable in each row), X overwriting the panel;
//   4. bl_dot_kernel: S = X^H [X | trailing columns].  E = X^H X - I is
//      what rounding left (bounds per level at bl_fin_kernel), and its
//      first order is folded into everything
//      that follows: Q = X (I - F), R = (I + F) D^1/2 U, F the upper
//      triangle of E with half its diagonal, so that Q^H Q = I + O(E^2);
//   5. bl_fin_kernel: the rows of R, and T = (I - E) S;
//   6. bl_update_kernel: trailing columns -= X T.
// The trailing columns see the exact projector of the panel's span, panels in
// order: the right-looking sweep of Fig. 4 with its columns in blocks.  A
// panel too ill-conditioned for its Gram matrix is orthogonalised by plain
// modified Gram-Schmidt in step 3 instead (bl_mgs_panel; repeated where one
// sweep would leave E too large), so every matrix the one-column-at-a-time
// algorithm takes is taken.  Problems of a few unknowns are one wavefront's
// work (smallls_kernels.hpp).
//
// Contractions.  A multi-double is cut into ND signed base-256 digits
// (fixed point against a power of two: the column's largest entry for the
// contraction over rows, the row's largest entry of X and the column's
// largest entry of T for the update), and a product is the sum over the digit
// pairs i + j < ND of int8 matrix products with 32-bit sums, which are exact:
// |digit product| <= 2^14, at most ND pairs and 4096 rows (10240 rows at
// ND = 10).  What is dropped is below 2^(-8 ND + 4) of the operands'
// largest products: ND = 16 (128 bits) for double double, 30 (240) for quad
// double, 10 (80) for double, each beyond the arithmetic of mdarith.hpp with
// bits to spare for rows of very uneven size.
// The FP64 pipes spend about 62 instructions on a complex double-double
// multiply-add and reach at most 0.63e12 of them a second; ND = 16 takes
// 544 int8 multiply-adds, of which the matrix cores do 2.5e15 a second.
// Against the column-by-column sweep that this replaces (a launch and two
// workgroup reductions per pivot, FP64 throughout) a Gauss-Newton step went
// from 2.08 to 0.73 ms (complex double double, n = 256), 53.6 to 12.6 ms
// (n = 2048), 35.1 to 6.5 ms (real quad double, n = 1016), and the batched
// step over 96 system-points of n = 32 .. 256 from 39.8 to 1.9 ms.  Where all
// panels are too ill-conditioned (columns that agree to 1e-8 or better) the
// sweep is ahead: 1.3 to 1.8 times in double double at 1e-8, 2.3 to 3.3 at
// 1e-13, 2.7 to 4 in double.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "eval_kernels.hpp"
#include "mdarith.hpp"
#include "newton_kernels.hpp"

namespace pe {

typedef int bl_v4i __attribute__((ext_vector_type(4)));

template <int L>
struct Bl {
  static constexpr int NL = limbs_of(L);
  static constexpr int CX = is_real(L) ? 1 : 2;    // real numbers per number
  static constexpr int B = 64 / CX;                // panel columns: 64 real ones
  static constexpr int ND = NL == 1 ? 10 : (NL == 2 ? 16 : 30);
  static constexpr int NW = (8 * ND + 31) / 32;    // 32-bit words of a fixed-point number
  static constexpr int W = CX * NL;                // doubles per number
  static constexpr int NT = NL == 4 ? 1 : 2;       // tiles of 16 real columns per workgroup of the contraction
  // level code of the Gram matrix and its factor: double works in double double
  static constexpr int LC = NL == 1 ? L + 1 : L;
  static constexpr int WC = CX * limbs_of(LC);
};

constexpr int kBlRows = 64;     // rows of a chunk: the K of a matrix instruction
constexpr int kBlBs = 256;      // rows of a back-substitution block
constexpr int kBlMaxSplit = 4;  // row splits of a contraction
constexpr int kBlGramSplit = 16;  // and of the Gram matrix's
// Row splits of a problem's Gram matrix (per panel) and of its contraction with
// `ncols` real columns in tiles of NT x 16: by the problem's own size, never by
// how many problems a launch holds, since the partial sums are rounded and the
// results of a problem are to be the same in every company.  As many as give a
// single problem two workgroups on every CU; 96 problems of 32 .. 256 rows in a
// launch would do with fewer (a batched step takes 1.87 ms against 1.78 with
// splits by the launch), 1 to 64 problems of 128 .. 256 rows lose or gain up to
// 3 %.
__host__ __device__ inline int bl_chunks(int N) { return (N + kBlRows - 1) / kBlRows; }
__host__ __device__ inline int bl_gram_splits(int N) {
  const int nc = bl_chunks(N);
  return nc < kBlGramSplit ? nc : kBlGramSplit;
}
template <int L>
__host__ __device__ inline int bl_dot_splits(int N, int ncols) {
  const int tiles = (ncols + 16 * Bl<L>::NT - 1) / (16 * Bl<L>::NT), nc = bl_chunks(N);
  const int want = (512 + tiles - 1) / tiles, most = nc < kBlMaxSplit ? nc : kBlMaxSplit;
  return want < most ? want : most;
}

constexpr int kExpOne = 1022;   // biased exponent field E of v: |v| < 2^(E - 1022)

// the problems of one launch group; per-slot strides in bytes
struct BlView {
  const BatchNewtonDesc* desc;  // batch: system's sizes and offsets, or null
  const int* order;
  int P, q0;          // batch: problem q0 + slot is point (q % P) of system order[q / P]
  int N, n;           // uniform problems (desc null): slot s is point q0 + s
  const double* A;    // augmented matrices, row-major planar
  int64_t a_pt, a_plane, ld;
  double* X;
  int64_t x_pt;
  int add;
  double* resid;
  double* Rout;
  double* Qout;
  char* ws;
  size_t slot;        // bytes of a slot
  // byte offsets inside a slot
  size_t oW, oR, oInv, oY, oU, oRp, oF, oS, oXD, oXU, oXr, oSD, oSe, oCe, oMisc, oPiv;
  size_t s_split;     // bytes of one split's contraction output
  size_t g_split;     // and of one split's Gram matrix
  int nmax;           // stride of the two column-exponent arrays
};

struct BlMisc {
  double rmax;   // largest |r_ii| so far
  int flag;      // panel + 1 in which a pivot was numerically zero, and the problem done; 0: none
  int mgs;       // 1: the current panel is orthogonalised by plain MGS
  int ticket;    // its next column
};

// columns of a panel under plain MGS, per sweep: 0 open, 1 orthonormal, 2 given up
struct BlPivots {
  int state[2][64];
  double rmax[64];  // largest |r_ii| so far
  double loss[64];  // bound of |q_i^H q_c| for i < c
};

// Offsets of a slot's regions for problems of at most N rows and n unknowns
// (bytes, each 256-byte aligned): W [components][n + 1][N] the working copy
// by columns, R [components][n + 1][n] by columns (column n is y = Q^H b),
// 1 / r_jj, y, the panel's U and D^1/2 U, F of every panel, S per row split,
// the digits of X in two orders with its row exponents, the digits of T with
// its column exponents, two sets of column exponents, the state, the pivots of
// a panel under plain MGS.
template <int L>
inline void bl_layout(int N, int n, BlView& V) {
  using K = Bl<L>;
  const size_t NC = size_t(N + kBlRows - 1) / kBlRows, B = K::B;
  const size_t panels = (size_t(n) + B - 1) / B;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) & ~size_t(255);
    return at;
  };
  V.nmax = n + 1;
  V.oW = take(size_t(K::W) * (n + 1) * N * 8);
  V.oR = take(size_t(K::W) * (n + 1) * n * 8);
  V.oInv = take(size_t(n) * K::NL * 8);
  V.oY = take(size_t(n) * K::W * 8);
  V.oU = take((B * B * K::W + B * K::NL) * 8);
  V.oRp = take(B * B * K::W * 8 + B * 4);
  V.oF = take(panels * B * B * K::CX * 8);
  V.g_split = B * B * K::WC * 8;
  V.s_split = size_t(n + 1) * B * K::W * 8;
  const size_t gs = std::min<size_t>(NC, kBlGramSplit), ds = std::min<size_t>(NC, kBlMaxSplit);
  V.oS = take(std::max(gs * V.g_split, ds * V.s_split));
  V.oXD = take(NC * K::ND * 4096);
  V.oXU = take(NC * K::ND * 4096);
  V.oXr = take(NC * kBlRows * 4);
  V.oSD = take((size_t(n + 1) * K::CX + 15) / 16 * K::ND * 1024);
  V.oSe = take(size_t(n + 1) * 4);
  V.oCe = take(size_t(n + 1) * 2 * 4);
  V.oMisc = take(sizeof(BlMisc));
  V.oPiv = take(sizeof(BlPivots));
  V.slot = off;
}


struct BlProb {
  int N, n;
  const double* A;
  int64_t a_plane, ld;
  double* x;
  double* resid;
  char* base;
};

template <int L>
__device__ __forceinline__ BlProb bl_prob(const BlView& V, int slot) {
  BlProb p;
  p.base = V.ws + size_t(slot) * V.slot;
  if (V.desc) {
    const int q = V.q0 + slot;
    const int s = V.order[q / V.P], pt = q - (q / V.P) * V.P;
    const BatchNewtonDesc d = V.desc[s];
    p.N = d.N;
    p.n = d.n;
    p.ld = d.n + 1;
    p.a_plane = int64_t(d.N) * p.ld;
    p.A = V.A + d.w_off * V.P + pt * (int64_t(width_of(L)) * p.a_plane);
    p.x = V.X + d.x_off * V.P + pt * (int64_t(width_of(L)) * d.n);
    p.resid = V.resid ? V.resid + (int64_t(s) * V.P + pt) * 2 : nullptr;
  } else {
    const int64_t pt = V.q0 + slot;
    p.N = V.N;
    p.n = V.n;
    p.ld = V.ld;
    p.a_plane = V.a_plane;
    p.A = V.A + pt * V.a_pt;
    p.x = V.X + pt * V.x_pt;
    p.resid = V.resid ? V.resid + 2 * pt : nullptr;
  }
  return p;
}

template <typename T>
__device__ __forceinline__ T* bl_at(const BlProb& p, size_t off) {
  return reinterpret_cast<T*>(p.base + off);
}

__device__ __forceinline__ int bl_exp(double v) {
  return int((__double_as_longlong(v) >> 52) & 0x7ff);
}

// ------------------------------------------------------------------ fixed point

// The ND leading balanced base-256 digits of v = sum of the limbs, |v| <= 2^e,
// as bytes: digit d (weight 2^(e - 6 - 8 d)) is byte 3 - d % 4 of w[d / 4].
// Every limb is cut into signed 32-bit words, each rounded to nearest (adding
// 1.5 2^52 leaves the integer in the low bits, and the remainder is exact),
// the words are added with carries as integers, and the bias of 0x80 per byte
// turns two's complement into digits of -128 .. 127.
template <int NL, int ND>
__device__ __forceinline__ void bl_digits(const double (&x)[NL], int e, uint32_t* w) {
  constexpr int NW = (8 * ND + 31) / 32;
  constexpr double kMagic = 6755399441055744.0;           // 1.5 2^52
  constexpr int64_t kMagicBits = 0x4338000000000000LL;  // its representation
  int64_t acc[NW];
#pragma unroll
  for (int q = 0; q < NW; ++q) acc[q] = 0x80808080LL;
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const int s0 = 53 * l / 32;  // the first word a limb can reach
    double y = __builtin_ldexp(x[l], 30 + 32 * s0 - e);
#pragma unroll
    for (int q = s0; q < NW; ++q) {
      const double t = y + kMagic;
      int64_t bits;
      __builtin_memcpy(&bits, &t, 8);
      acc[q] += bits - kMagicBits;
      y = (y - (t - kMagic)) * 4294967296.0;
    }
  }
  int64_t carry = 0;
#pragma unroll
  for (int q = NW - 1; q >= 0; --q) {
    const int64_t a = acc[q] + carry;
    w[q] = uint32_t(a) ^ 0x80808080u;
    carry = a >> 32;
  }
}

// bytes of four words regrouped: out[s] holds byte 3 - s of each, word 0's lowest
__device__ __forceinline__ void bl_transpose4(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t* out) {
  const uint32_t x = __builtin_amdgcn_perm(a1, a0, 0x05010400u), y = __builtin_amdgcn_perm(a1, a0, 0x07030602u);
  const uint32_t u = __builtin_amdgcn_perm(a3, a2, 0x05010400u), v = __builtin_amdgcn_perm(a3, a2, 0x07030602u);
  out[0] = __builtin_amdgcn_perm(v, y, 0x07060302u);
  out[1] = __builtin_amdgcn_perm(v, y, 0x05040100u);
  out[2] = __builtin_amdgcn_perm(u, x, 0x07060302u);
  out[3] = __builtin_amdgcn_perm(u, x, 0x05040100u);
}

// digits of four numbers (the limbs of number r in v[r]), packed four to a
// word, written to dst[d * stride] for digit d
template <int NL, int ND>
__device__ __forceinline__ void bl_put4(const double (&v)[4][NL], const int (&e)[4], uint32_t* dst, int stride) {
  constexpr int NW = (8 * ND + 31) / 32;
  uint32_t w[4][NW];
#pragma unroll
  for (int r = 0; r < 4; ++r) bl_digits<NL, ND>(v[r], e[r], w[r]);
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    uint32_t o[4];
    bl_transpose4(w[0][q], w[1][q], w[2][q], w[3][q], o);
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (4 * q + s < ND) dst[(4 * q + s) * stride] = o[s];
  }
}

// sum over t of a[t] 2^(-8 t) times 2^e: groups of three sums are exact in a
// double, the groups are added by an error-free chain
template <int NL, int ND>
__device__ __forceinline__ R<NL> bl_value(const int (&a)[ND], int e) {
  constexpr int NG = (ND + 2) / 3;
  double g[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    double s = double(a[3 * q]) * 65536.0;
    if (3 * q + 1 < ND) s = PE_FMA(double(a[3 * q + 1 < ND ? 3 * q + 1 : 0]), 256.0, s);
    if (3 * q + 2 < ND) s += double(a[3 * q + 2 < ND ? 3 * q + 2 : 0]);
    g[q] = __builtin_ldexp(s, -24 * q - 16);
  }
  R<NL> r;
  if constexpr (NL == 1) {
    double s = g[NG - 1];
#pragma unroll
    for (int q = NG - 2; q >= 0; --q) s += g[q];
    r.x[0] = s;
  } else if constexpr (NL == 2) {
    double h = g[0], l = 0.0;
#pragma unroll
    for (int q = 1; q < NG; ++q) {
      double s, t;
      two_sum(h, g[q], s, t);
      h = s;
      l += t;
    }
    fast_two_sum(h, l, r.x[0], r.x[1]);
  } else {
    double x0 = g[0], x1 = 0.0, x2 = 0.0, x3 = 0.0;
#pragma unroll
    for (int q = 1; q < NG; ++q) {
      double s, t, u, v;
      two_sum(x0, g[q], s, t);
      x0 = s;
      two_sum(x1, t, u, v);
      x1 = u;
      two_sum(x2, v, s, t);
      x2 = s;
      x3 += t;
    }
    r = renorm4(x0, x1, x2, x3);
  }
#pragma unroll
  for (int l = 0; l < NL; ++l) r.x[l] = __builtin_ldexp(r.x[l], e);
  return r;
}

template <int L>
__device__ __forceinline__ C<L> bl_ldexp(C<L> a, int e) {
#pragma unroll
  for (int l = 0; l < limbs_of(L); ++l) {
    a.re.x[l] = __builtin_ldexp(a.re.x[l], e);
    if constexpr (!is_real(L)) a.im.x[l] = __builtin_ldexp(a.im.x[l], e);
  }
  return a;
}

template <int LO, int L>
__device__ __forceinline__ C<LO> bl_narrow(const C<L>& a) {
  C<LO> r;
#pragma unroll
  for (int l = 0; l < limbs_of(LO); ++l) {
    r.re.x[l] = a.re.x[l];
    if constexpr (!is_real(L)) r.im.x[l] = a.im.x[l];
  }
  return r;
}

// sum over the row splits of a contraction's output, four loads in flight
template <int L>
__device__ __forceinline__ C<L> bl_sum_splits(const char* base, size_t stride, int ns) {
  C<L> s = load_aos<L>(reinterpret_cast<const double*>(base));
  for (int t = 1; t < ns; t += 3) {
    C<L> v[3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
      v[q] = load_aos<L>(reinterpret_cast<const double*>(base + size_t(min(t + q, ns - 1)) * stride));
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (t + q < ns) s = c_add(s, v[q]);
  }
  return s;
}

// ------------------------------------------------------------------ set up

// Per problem: state cleared, |b|_2 (leading limbs) into resid[0].  grid
// (slots), 256 threads
template <int L>
__global__ __launch_bounds__(256) void bl_init_kernel(BlView V) {
  __shared__ double red[256];
  const BlProb p = bl_prob<L>(V, blockIdx.x);
  const int tid = threadIdx.x;
  int* ce = bl_at<int>(p, V.oCe);
  for (int j = tid; j <= p.n; j += 256) ce[j] = ce[V.nmax + j] = 0;
  if (tid == 0) {
    BlMisc* m = bl_at<BlMisc>(p, V.oMisc);
    m->rmax = 0.0;
    m->flag = 0;
    m->mgs = 0;
  }
  double s = 0.0;
  for (int i = tid; i < p.N; i += 256) {
    const double re = p.A[int64_t(i) * p.ld + p.n];
    const double im = is_real(L) ? 0.0 : p.A[int64_t(limbs_of(L)) * p.a_plane + int64_t(i) * p.ld + p.n];
    s += re * re + im * im;
  }
  red[tid] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (tid < k) red[tid] += red[tid + k];
    __syncthreads();
  }
  if (tid == 0 && p.resid) p.resid[0] = sqrt(red[0]);
}

// [A b] (row-major) -> column-major W, and every column's largest exponent.
// Tiles of 64 rows x 64 columns through LDS, both sides coalesced; grid
// (tiles, components, slots), 256 threads
template <int L>
__global__ __launch_bounds__(256) void bl_copy_in_kernel(BlView V) {
  __shared__ double tile[64][65];
  const BlProb p = bl_prob<L>(V, blockIdx.z);
  const int ncol = p.n + 1, tc = (ncol + 63) / 64;
  const int bt = blockIdx.x;
  const int c0 = (bt % tc) * 64, r0 = (bt / tc) * 64;
  if (r0 >= p.N) return;
  const int comp = blockIdx.y;
  const double* src = p.A + comp * p.a_plane;
  double* dst = bl_at<double>(p, V.oW) + int64_t(comp) * ncol * p.N;
  int* ce = bl_at<int>(p, V.oCe);
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int r = ty; r < 64; r += 4) {
    const int row = r0 + r, col = c0 + tx;
    tile[r][tx] = (row < p.N && col < ncol) ? src[int64_t(row) * p.ld + col] : 0.0;
  }
  __syncthreads();
  for (int c = ty; c < 64; c += 4) {
    const int col = c0 + c, row = r0 + tx;
    const double v = tile[tx][c];
    if (row < p.N && col < ncol) dst[int64_t(col) * p.N + row] = v;
    if (comp % limbs_of(L) == 0) {
      int e = bl_exp(v);
#pragma unroll
      for (int m = 1; m < 64; m <<= 1) e = max(e, __shfl_xor(e, m));
      if (tx == 0 && col < ncol) atomicMax(ce + col, e);
    }
  }
}

// ------------------------------------------------------------------ contractions over rows

// the 4 values of a lane's accumulator tile (16 rows of X's real columns from
// row m on, one real column of the other side) into S at column `col`:
// complex numbers join across neighbouring lanes, which hold the real and
// imaginary part of one column: re = Xr.Ar + Xi.Ai, im = Xr.Ai - Xi.Ar
template <int L, int LO, int ND>
__device__ __forceinline__ void bl_store_s(double* Sp, const bl_v4i (&av)[ND], int e, int col, int m, int comp, bool in) {
  constexpr int NO = limbs_of(LO), B = Bl<L>::B;
  R<NO> val[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    int t[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) t[d] = av[d][r];
    val[r] = bl_value<NO, ND>(t, e);
  }
  if constexpr (is_real(L)) {
    if (in)
#pragma unroll
      for (int r = 0; r < 4; ++r) r_store_aos(Sp + (size_t(col) * B + m + r) * width_of(LO), val[r]);
  } else {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const R<NO> mine = val[2 * h + 1];
      R<NO> other;
#pragma unroll
      for (int l = 0; l < NO; ++l) other.x[l] = __shfl_xor(mine.x[l], 1);
      const R<NO> s = r_add(val[2 * h], comp ? r_neg(other) : other);
      if (in) r_store_aos(Sp + (size_t(col) * B + m / 2 + h) * width_of(LO) + comp * NO, s);
    }
  }
}

// Pairs of rows of a column of W: columns start at any row of an odd N, so the
// 16-byte accesses are aligned to 8 bytes only (global memory asks for 4).
// Against one limb of one row per access, which touched every 128-byte line
// four times: update 60 -> 52 us a panel, contraction 51 -> 48 us (complex
// double double, n = 2048).
typedef double bl_v2d __attribute__((ext_vector_type(2), aligned(8)));

// four rows of a real column of W as limbs (zero outside)
template <int NL>
__device__ __forceinline__ void bl_load4(const double* src, int64_t plane, int row, int N, bool in, double (&v)[4][NL]) {
  if (in && row + 4 <= N) {
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      const bl_v2d* q = reinterpret_cast<const bl_v2d*>(src + l * plane + row);
      const bl_v2d a = q[0], b = q[1];
      v[0][l] = a.x;
      v[1][l] = a.y;
      v[2][l] = b.x;
      v[3][l] = b.y;
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int l = 0; l < NL; ++l) v[r][l] = in && row + r < N ? src[l * plane + row + r] : 0.0;
  }
}

template <int NL>
__device__ __forceinline__ void bl_store4(double* dst, int64_t plane, int row, int N, const double (&v)[4][NL]) {
  if (row + 4 <= N) {
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      bl_v2d* q = reinterpret_cast<bl_v2d*>(dst + l * plane + row);
      q[0] = bl_v2d{v[0][l], v[1][l]};
      q[1] = bl_v2d{v[2][l], v[3][l]};
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int l = 0; l < NL; ++l)
        if (row + r < N) dst[l * plane + row + r] = v[r][l];
  }
}

// Gram matrix of the panel's columns, each scaled by its exponent: per chunk
// of 64 rows the digits of all 64 real columns are cut into LDS once, and
// each of the four wavefronts multiplies 16 of them with the workgroup's NT
// tiles of 16.  Row ranges are summed by bl_chol_kernel.  S is [split][column]
// [B] numbers of the factor's level.  grid (4 / NT, splits, slots), 256 threads
template <int L>
__global__ __launch_bounds__(256, limbs_of(L) == 4 ? 1 : 2) void bl_gram_kernel(BlView V, int panel, int cur) {
  using K = Bl<L>;
  constexpr int NL = K::NL, ND = K::ND, NT = K::NT, CX = K::CX;
  extern __shared__ double lds[];
  bl_v4i* dig = reinterpret_cast<bl_v4i*>(lds);  // [digit][64 real columns][64 rows]
  const BlProb p = bl_prob<L>(V, blockIdx.z);
  const int k0 = panel * K::B;
  if (k0 >= p.n) return;
  const int flag = bl_at<BlMisc>(p, V.oMisc)->flag;  // tested where nothing waits for it
  const int bcur = min(K::B, p.n - k0);
  const int rc0 = blockIdx.x * NT * 16;
  const int NC = (p.N + kBlRows - 1) / kBlRows;
  const int ns = bl_gram_splits(p.N), split = blockIdx.y;
  if (rc0 >= bcur * CX || split >= ns) return;
  const int per = (NC + ns - 1) / ns;
  const int ch0 = split * per, ch1 = min(NC, ch0 + per);
  const double* Wp = bl_at<double>(p, V.oW);
  const int64_t plane = int64_t(p.n + 1) * p.N;
  const int* ce = bl_at<int>(p, V.oCe) + cur * V.nmax + k0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k4 = tid & 15, c16 = tid >> 4;
  bl_v4i av[NT][ND];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int d = 0; d < ND; ++d) av[t][d] = bl_v4i{0, 0, 0, 0};
  for (int ch = ch0; ch < ch1; ++ch) {
    if (ch > ch0) __syncthreads();  // the previous chunk's digits are read
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int m = u * 16 + c16, c = m / CX;
      const bool in = c < bcur;
      double v[4][NL];
      bl_load4<NL>(Wp + int64_t(m % CX) * NL * plane + int64_t(k0 + (in ? c : 0)) * p.N, plane, ch * kBlRows + k4 * 4,
                   p.N, in, v);
      const int ex = in ? ce[c] - kExpOne : 0;
      const int e[4] = {ex, ex, ex, ex};
      bl_put4<NL, ND>(v, e, reinterpret_cast<uint32_t*>(dig) + m * 16 + k4, 1024);
    }
    __syncthreads();
    bl_v4i a[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) a[i] = dig[(i * 64 + 16 * wave + (lane & 15)) * 4 + (lane >> 4)];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        const bl_v4i b = dig[(j * 64 + rc0 + u * 16 + (lane & 15)) * 4 + (lane >> 4)];
#pragma unroll
        for (int i = 0; i < ND; ++i)
          if (i + j < ND) av[u][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b, av[u][i + j], 0, 0, 0);
      }
  }
  if (flag) return;
  double* Sp = reinterpret_cast<double*>(p.base + V.oS + split * V.g_split);
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int rc = rc0 + u * 16 + (lane & 15);
    bl_store_s<L, K::LC, ND>(Sp, av[u], -12, rc / CX, 16 * wave + 4 * (lane >> 4), rc % CX, rc < bcur * CX);
  }
}

template <int L>
__host__ __device__ inline size_t bl_gram_lds() {
  return size_t(Bl<L>::ND) * 4096;
}

// S = X^H C for the orthonormal panel X and the columns C of W from k0 on
// (the panel itself, all later columns, the right-hand side).  One workgroup
// takes NT tiles of 16 real columns and a range of rows: per chunk of 64 rows
// it cuts its columns into digits in LDS once, and each of its four wavefronts
// multiplies them by the digits of 16 of X's 64 real columns.  Row ranges are
// summed by bl_fin_kernel.  S is [split][column][B] numbers.  grid (column
// tiles, splits, slots), 256 threads
template <int L>
__global__ __launch_bounds__(256, limbs_of(L) == 4 ? 1 : 2) void bl_dot_kernel(BlView V, int panel, int cur) {
  using K = Bl<L>;
  constexpr int NL = K::NL, ND = K::ND, NT = K::NT, CX = K::CX;
  __shared__ bl_v4i dig[NT * ND * 64];
  const BlProb p = bl_prob<L>(V, blockIdx.z);
  const int k0 = panel * K::B;
  if (k0 >= p.n) return;
  const int flag = bl_at<BlMisc>(p, V.oMisc)->flag;
  const int bcur = min(K::B, p.n - k0);
  const int ncols = (p.n + 1 - k0) * CX;  // real columns
  const int rc0 = blockIdx.x * NT * 16;
  const int NC = (p.N + kBlRows - 1) / kBlRows;
  const int ns = bl_dot_splits<L>(p.N, ncols), split = blockIdx.y;
  if (rc0 >= ncols || split >= ns) return;
  const int per = (NC + ns - 1) / ns;
  const int ch0 = split * per, ch1 = min(NC, ch0 + per);
  const double* Wp = bl_at<double>(p, V.oW);
  const int64_t plane = int64_t(p.n + 1) * p.N;
  const int* ce = bl_at<int>(p, V.oCe) + cur * V.nmax;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k4 = tid & 15, c16 = tid >> 4;
  // power of two of column c (from the panel's first): X itself is at most 1
  auto col_exp = [&](int c) { return c < bcur ? 0 : ce[k0 + c] - kExpOne; };
  int ex[NT];
  const double* src[NT];
  bl_v4i av[NT][ND];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int rc = min(rc0 + u * 16 + c16, ncols - 1);
    ex[u] = col_exp(rc / CX);
    src[u] = Wp + int64_t(rc % CX) * NL * plane + int64_t(k0 + rc / CX) * p.N;
#pragma unroll
    for (int d = 0; d < ND; ++d) av[u][d] = bl_v4i{0, 0, 0, 0};
  }
  // quad double, alone on its SIMD, loads a chunk's entries while the chunk
  // before is multiplied (38 -> 36 us; double double has no registers for it)
  constexpr bool kAhead = NL == 4;
  double v[NT][4][NL];
  auto fetch = [&](int ch) {
#pragma unroll
    for (int u = 0; u < NT; ++u)
      bl_load4<NL>(src[u], plane, ch * kBlRows + k4 * 4, p.N, rc0 + u * 16 + c16 < ncols, v[u]);
  };
  for (int ch = ch0; ch < ch1; ++ch) {
    const bl_v4i* xd = bl_at<bl_v4i>(p, V.oXD) + size_t(ch) * ND * 256 + (16 * wave + (lane & 15)) * 4 + (lane >> 4);
    bl_v4i a[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) a[i] = xd[i * 256];
    if (!kAhead || ch == ch0) fetch(ch);
    __syncthreads();  // the previous chunk's digits are read
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      const int e[4] = {ex[u], ex[u], ex[u], ex[u]};
      bl_put4<NL, ND>(v[u], e, reinterpret_cast<uint32_t*>(dig) + (u * ND * 16 + c16) * 16 + k4, 256);
    }
    __syncthreads();
    if (kAhead && ch + 1 < ch1) fetch(ch + 1);
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        const bl_v4i b = dig[((u * ND + j) * 16 + (lane & 15)) * 4 + (lane >> 4)];
#pragma unroll
        for (int i = 0; i < ND; ++i)
          if (i + j < ND) av[u][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b, av[u][i + j], 0, 0, 0);
      }
  }
  if (flag) return;
  double* Sp = reinterpret_cast<double*>(p.base + V.oS + split * V.s_split);
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int rc = rc0 + u * 16 + (lane & 15);
    bl_store_s<L, L, ND>(Sp, av[u], col_exp(min(rc, ncols - 1) / CX) - 12, rc / CX, 16 * wave + 4 * (lane >> 4), rc % CX,
                         rc < ncols);
  }
}

// ------------------------------------------------------------------ the panel's factor

// threads of the factor's workgroup and upper-triangle entries per thread
template <int L>
struct BlChol {
  static constexpr int T = Bl<L>::NL == 4 ? (is_real(L) ? 512 : 320) : (is_real(L) ? 704 : 576);
  static constexpr int ENTRIES = Bl<L>::B * (Bl<L>::B + 1) / 2;
  static constexpr int EPT = (ENTRIES + T - 1) / T;
};

// 1 / a to the level's precision: a double estimate corrected by its
// residual, for quad double once more
template <int NLV>
__device__ __forceinline__ R<NLV> bl_recip(const R<NLV>& a) {
  // two Newton steps on the hardware's estimate: within about one unit in the
  // last place for pivots far from the ends of the exponent range
  double y = __builtin_amdgcn_rcp(a.x[0]);
  y = PE_FMA(y, PE_FMA(-a.x[0], y, 1.0), y);
  y = PE_FMA(y, PE_FMA(-a.x[0], y, 1.0), y);
  if constexpr (NLV == 1) {
    return r_from_double<1>(y);
  } else {
    const double r = PE_FMA(-a.x[1], y, PE_FMA(-a.x[0], y, 1.0));
    R<2> z;
    fast_two_sum(y, y * r, z.x[0], z.x[1]);
    if constexpr (NLV == 2) {
      return z;
    } else {
      const R<4> z4{{z.x[0], z.x[1], 0.0, 0.0}};
      const R<4> t = r_sub(r_from_double<4>(1.0), r_mul(a, z4));
      const R<2> c = r_mul(z, R<2>{{t.x[0], t.x[1]}});
      return r_add(z4, R<4>{{c.x[0], c.x[1], 0.0, 0.0}});
    }
  }
}

// Factor of the panel's Gram matrix G (of the columns scaled by their
// exponents): G = U^H D U, U unit upper triangular.  A thread keeps entries
// of the upper triangle in registers; a row is published in LDS when the
// pivots above it are done, and step k's threads subtract
// conj(g_ki) g_kj / d_k, every thread forming the reciprocal of the pivot
// itself, so that a step has one barrier (quad double: the row over its pivot
// once, and two).  Square roots wait for the end.  A pivot below kPivot of its
// column's squared norm would leave E = X^H X - I too large for its first order
// (E is about u_C / pivot ratio, u_C the unit roundoff of the factor's level):
// then the panel is left to plain modified Gram-Schmidt (bl_mgs_panel, in the
// next kernel).  One workgroup per problem: it is bound by the chain of B
// pivots.
template <int L>
__global__ __launch_bounds__(BlChol<L>::T) void bl_chol_kernel(BlView V, int panel, int cur) {
  using K = Bl<L>;
  constexpr int LC = K::LC, NC_ = limbs_of(LC), WC = K::WC, B = K::B, NL = K::NL;
  constexpr int T = BlChol<L>::T, EPT = BlChol<L>::EPT;
  using RC = R<NC_>;
  extern __shared__ double lds[];
  const BlProb p = bl_prob<L>(V, blockIdx.x);
  BlMisc* misc = bl_at<BlMisc>(p, V.oMisc);
  const int k0 = panel * B;
  if (k0 >= p.n) return;
  const int flag = misc->flag;  // tested once the loads are on their way
  const int bcur = min(B, p.n - k0);
  const int tid = threadIdx.x;
  double* G = lds;                    // [B][B] numbers, rows published when final
  double* g0 = G + size_t(B) * B * WC;  // [B] diagonal before the factorisation
  double* dinv = g0 + B;              // [B][NC_] 1 / d
  double* sq = dinv + B * NC_;        // [B][NC_] sqrt(d)
  double* frow = sq + B * NC_;        // [B] numbers (quad double)
  int* ex = reinterpret_cast<int*>(frow + B * WC);  // [B] column exponents
  (void)frow;
  const int ns = bl_gram_splits(p.N);
  const int* ce = bl_at<int>(p, V.oCe) + cur * V.nmax;
  if (tid < B) ex[tid] = tid < bcur ? ce[k0 + tid] - kExpOne : 0;
  // entries in row order, so that whole wavefronts fall idle as rows finish;
  // S holds column j as [j][i]
  int ei[EPT], ej[EPT];
  C<LC> g[EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    int rest = tid + q * T, i = 0;
    // rows above row i hold i B - i (i - 1) / 2 entries
    i = int((2.0f * B + 1.0f - sqrtf((2.0f * B + 1.0f) * (2.0f * B + 1.0f) - 8.0f * float(rest))) * 0.5f);
    i = max(0, min(B - 1, i));
    while (i > 0 && i * B - i * (i - 1) / 2 > rest) --i;
    while (i + 1 < B && (i + 1) * B - (i + 1) * i / 2 <= rest) ++i;
    const int j = i + rest - (i * B - i * (i - 1) / 2);
    const bool in = rest < BlChol<L>::ENTRIES && j < bcur;
    ei[q] = in ? i : -1;
    ej[q] = j;
    g[q] = c_zero<LC>();
    if (in) {
      g[q] = bl_sum_splits<LC>(p.base + V.oS + (size_t(j) * B + i) * WC * 8, V.g_split, ns);
      if (i == j) g0[i] = g[q].re.x[0];
      if (i == 0) store_planar(G, B, j, g[q]);
    }
  }
  if (flag) return;
  constexpr double kPivot = NL == 1 ? 0x1p-26 : 0x1p-46;
  bool bad = false, nonfinite = false;
  for (int k = 0; k < bcur; ++k) {
    __syncthreads();
    nonfinite |= ex[k] == 0x7ff - kExpOne;
    const double* Gk = G + size_t(k) * B * WC;  // row k, planar
    const RC d = load_planar<LC>(Gk, B, k).re;
    bad |= !(d.x[0] > kPivot * g0[k]);
    if constexpr (NC_ < 4) {
      // the product does not wait for the reciprocal
      C<LC> t[EPT];
#pragma unroll
      for (int q = 0; q < EPT; ++q)
        if (ei[q] > k) t[q] = c_mul_conj_a(load_planar<LC>(Gk, B, ei[q]), load_planar<LC>(Gk, B, ej[q]));
      const RC inv = bl_recip<NC_>(d);
      if (tid == 0) r_store_aos(dinv + k * NC_, inv);
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        if (ei[q] <= k) continue;
        g[q] = c_sub(g[q], c_mul_r(t[q], inv));
        if (ei[q] == k + 1) store_planar(G + size_t(k + 1) * B * WC, B, ej[q], g[q]);
      }
    } else {
      // quad double: the row over its pivot once, by the first B threads
      if (tid < B) {
        const RC inv = bl_recip<NC_>(d);
        if (tid == 0) r_store_aos(dinv + k * NC_, inv);
        store_planar(frow, B, tid, c_mul_r(load_planar<LC>(Gk, B, tid), inv));
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < EPT; ++q) {
        if (ei[q] <= k) continue;
        g[q] = c_sub(g[q], c_mul_conj_a(load_planar<LC>(Gk, B, ei[q]), load_planar<LC>(frow, B, ej[q])));
        if (ei[q] == k + 1) store_planar(G + size_t(k + 1) * B * WC, B, ej[q], g[q]);
      }
    }
  }
  if (nonfinite) {
    if (tid == 0) misc->flag = panel + 1;
    return;
  }
  __syncthreads();
  const double thresh = double(p.n) * level_unit<L>();
  double* U = bl_at<double>(p, V.oU);    // [B][B] then [B][NL] 1 / sqrt(d)
  double* Rp = bl_at<double>(p, V.oRp);  // [B][B], then B column exponents
  int* rexp = reinterpret_cast<int*>(Rp + size_t(B) * B * K::W);
  double rmax = misc->rmax;
  if (!bad) {
    double* is = U + size_t(B) * B * K::W;
    if (tid < B) {
      const RC d = tid < bcur ? load_planar<LC>(G + size_t(tid) * B * WC, B, tid).re : r_from_double<NC_>(1.0);
      const RC s = r_sqrt(d);
      r_store_aos(sq + tid * NC_, s);
      const RC q = r_recip(s);
#pragma unroll
      for (int l = 0; l < NL; ++l) is[tid * NL + l] = q.x[l];
      rexp[tid] = ex[tid];
    }
    __syncthreads();
    bool singular = false;
    for (int j = 0; j < bcur; ++j) {
      const double r = __builtin_ldexp(sq[j * NC_], ex[j]);
      rmax = fmax(rmax, r);
      if (!(r > thresh * rmax)) singular = true;
    }
    if (singular) {
      if (tid == 0) misc->flag = panel + 1;
      return;
    }
    for (int idx = tid; idx < B * B; idx += T) {
      const int i = idx / B, j = idx % B;
      C<LC> u = c_zero<LC>();
      C<LC> r = u;
      const RC s = r_load_aos<NC_>(sq + i * NC_);
      if (i == j) {
        r = c_from_r<LC>(s);
      } else if (i < j && j < bcur) {
        u = c_mul_r(load_planar<LC>(G + size_t(i) * B * WC, B, j), r_load_aos<NC_>(dinv + i * NC_));
        // the factor as the substitution takes it (rounded to the level)
        const C<L> un = bl_narrow<L>(u);
        C<LC> w = c_zero<LC>();
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          w.re.x[l] = un.re.x[l];
          if constexpr (!is_real(L)) w.im.x[l] = un.im.x[l];
        }
        r = c_mul_r(w, s);
      }
      store_aos(U + size_t(idx) * K::W, bl_narrow<L>(u));
      store_aos(Rp + size_t(idx) * K::W, bl_narrow<L>(r));
    }
    if (tid == 0) {
      misc->rmax = rmax;
      misc->mgs = 0;
    }
    return;
  }
  // too ill-conditioned: modified Gram-Schmidt, column by column
  for (int idx = tid; idx < B * B; idx += T) {
    store_aos(Rp + size_t(idx) * K::W, c_zero<L>());
    store_aos(U + size_t(idx) * K::W, c_zero<L>());
  }
  if (tid < B) rexp[tid] = 0;
  BlPivots* piv = bl_at<BlPivots>(p, V.oPiv);
  if (tid < 128) piv->state[tid >> 6][tid & 63] = 0;
  if (tid == 0) {
    misc->mgs = 1;
    misc->ticket = 0;
  }
}

template <int L>
__host__ __device__ inline size_t bl_chol_lds() {
  using K = Bl<L>;
  return (size_t(K::B) * K::B * K::WC + K::B * (1 + 2 * limbs_of(K::LC) + K::WC)) * sizeof(double) + K::B * sizeof(int);
}

// ------------------------------------------------------------------ X = A U^-1 D^-1/2

// Rows of X by forward substitution: a wavefront holds one or two rows, its
// lanes the 64 real columns (complex: lane l the real part of column l,
// l < 32, or the imaginary part of column l - 32); step i broadcasts entry i
// through scalar registers, which the lanes of later columns multiply by
// their u_ij.  X replaces the panel in W; its digits are written in the two
// orders the products read: XD (rows contiguous, fixed point against 1) for
// the contraction and XU ([chunk][digit][row][64 real columns], against the
// row's largest entry, so that a small row keeps its relative precision) for
// the update.  Bound by the chain of B steps: few rows per workgroup, so that
// it spreads over the chip.  grid (64-row chunks * 64 / rows per workgroup,
// slots), 256 threads
template <int L>
constexpr int bl_solve_rows() {
  return limbs_of(L) == 4 ? 1 : 2;
}

__device__ __forceinline__ double bl_readlane(double v, int lane) {
  const int64_t b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(int(b), lane), hi = __builtin_amdgcn_readlane(int(b >> 32), lane);
  return __longlong_as_double((int64_t(hi) << 32) | uint32_t(lo));
}

template <int L>
__host__ __device__ inline size_t bl_solve_lds() {
  using K = Bl<L>;
  return (size_t(K::B) * K::B * (is_real(L) ? K::NL : 4 * K::NL) + 4 * bl_solve_rows<L>() * 64 * K::NL) * sizeof(double) + 4 * bl_solve_rows<L>() * sizeof(int);
}

// ------------------------------------------------------------------ plain MGS

__device__ __forceinline__ int bl_load_state(const int* s) {
  return __hip_atomic_load(s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// State of column c once it is no longer open, the same in all 256 threads, with
// the column's memory visible to them.  Bounded: a wait of some seconds gives
// the panel up.
__device__ __forceinline__ int bl_await(const int* state, int* sh) {
  __syncthreads();  // the word is free
  if (threadIdx.x == 0) {
    int s = 0;
    for (int n = 0; n < (1 << 21) && (s = bl_load_state(state)) == 0; ++n) __builtin_amdgcn_s_sleep(8);
    *sh = s == 0 ? 2 : s;
  }
  __syncthreads();
  __threadfence();
  return *sh;
}

// sum of a number over 256 threads, in a fixed order; red: 4 numbers
template <int L>
__device__ __forceinline__ C<L> bl_wg_sum(C<L> v, double* red) {
#pragma unroll 1
  for (int m = 1; m < 64; m <<= 1) v = c_add(v, shfl_xor_c(v, m));
  __syncthreads();  // the numbers are free
  if ((threadIdx.x & 63) == 0) store_aos(red + (threadIdx.x >> 6) * width_of(L), v);
  __syncthreads();
  C<L> s = load_aos<L>(red);
  for (int q = 1; q < 4; ++q) s = c_add(s, load_aos<L>(red + q * width_of(L)));
  return s;
}

// Column j of the panel in one sweep: off with the columns before it as they
// become orthonormal, in order, then normalised; column j of the sweep's R into
// Rr.  The column is kept in LDS (rows from `cap` on in its place in W).  The
// first sweep tests the pivot and bounds what is left of the columns before it
// (piv->loss).  Returns false when the panel is given up (a zero pivot).
template <int L>
__device__ bool bl_mgs_column(const BlProb& p, const BlMisc* misc, BlPivots* piv, int sweep, double* Wp, double* Rr,
                              int k0, int j, double* red, int* sh, double* la, int cap) {
  using K = Bl<L>;
  constexpr int NL = K::NL;
  const int tid = threadIdx.x;
  const int64_t plane = int64_t(p.n + 1) * p.N;
  double* col = Wp + int64_t(k0 + j) * p.N;
  // a thread only ever touches its own rows (the address space is spelled out:
  // the compiler would join the two sides in flat accesses)
  auto* const lc = (__attribute__((address_space(3))) double*)la;
  auto get = [&](int i) {
    if (i >= cap) return load_planar<L>(col, plane, i);
    C<L> v;
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      v.re.x[l] = lc[l * cap + i];
      if constexpr (!is_real(L)) v.im.x[l] = lc[(NL + l) * cap + i];
    }
    return v;
  };
  auto put = [&](int i, const C<L>& v) {
    if (i >= cap) return store_planar(col, plane, i, v);
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      lc[l * cap + i] = v.re.x[l];
      if constexpr (!is_real(L)) lc[(NL + l) * cap + i] = v.im.x[l];
    }
  };
  C<L> s = c_zero<L>();
  for (int i = tid; i < p.N; i += 256) {
    const C<L> v = load_planar<L>(col, plane, i);
    s.re = r_add(s.re, c_norm2(v));
    put(i, v);
  }
  s = bl_wg_sum<L>(s, red);
  const double size = r_sqrt(s.re).x[0];
  double lost = 0.0;
  for (int c = 0; c < j; ++c) {
    if (bl_await(piv->state[sweep] + c, sh) == 2) return false;
    const double* q = Wp + int64_t(k0 + c) * p.N;
    C<L> d = c_zero<L>();
    for (int i = tid; i < p.N; i += 256) d = c_add(d, c_mul_conj_a(load_planar<L>(q, plane, i), get(i)));
    d = bl_wg_sum<L>(d, red);
    const C<L> nd = c_neg(d);
    s = c_zero<L>();
    for (int i = tid; i < p.N; i += 256) {
      const C<L> v = c_add(get(i), c_mul(nd, load_planar<L>(q, plane, i)));
      put(i, v);
      if (c + 1 == j) s.re = r_add(s.re, c_norm2(v));
    }
    if (c + 1 == j) s = bl_wg_sum<L>(s, red);
    lost += piv->loss[c] * (fabs(d.re.x[0]) + fabs(im_lead(d)));
    if (tid == 0) store_aos(Rr + (size_t(c) * K::B + j) * K::W, d);
  }
  const R<NL> r = r_sqrt(s.re);
  if (sweep == 0) {
    const double rmax = fmax(j == 0 ? misc->rmax : piv->rmax[j - 1], r.x[0]);
    if (!(r.x[0] > double(p.n) * level_unit<L>() * rmax)) return false;
    if (tid == 0) {
      piv->rmax[j] = rmax;
      piv->loss[j] = (lost + level_unit<L>() * size) / r.x[0];
    }
  } else if (!(r.x[0] > 0.0)) {
    return false;
  }
  const R<NL> ir = r_recip(r);
  for (int i = tid; i < p.N; i += 256) store_planar(col, plane, i, c_mul_r(get(i), ir));
  if (tid == 0) store_aos(Rr + (size_t(j) * K::B + j) * K::W, c_from_r<L>(r));
  return true;
}

// A panel that is too ill-conditioned for its Gram matrix, by plain modified
// Gram-Schmidt: the workgroups of bl_solve_kernel (256 threads each) take its
// columns by ticket, each subtracts the columns before its own as they are
// published and publishes its own.  A workgroup only ever waits for columns with
// smaller tickets, whose workgroups are running, so it makes progress however
// many of them fit on the chip.  A second sweep where the first leaves too much
// of a column in another one: E's first order has to do, so the loss has to be
// below 2^-33, 2^-64 or 2^-162, whose square and whose product with double's
// roundoff are below the level's.  R = R2 R1 then.  False: the panel was given
// up.  Bound by the chain of pivots (a wait, two passes over a column, its
// publication): 17 us each at 2048 rows in complex double double, 7 at 256,
// where one workgroup for the panel took 90 and 12.
template <int L>
__device__ bool bl_mgs_panel(const BlView& V, const BlProb& p, BlMisc* misc, int panel, int bcur, double* lds) {
  using K = Bl<L>;
  constexpr double kLoss = K::NL == 1 ? 0x1p-33 : (K::NL == 2 ? 0x1p-64 : 0x1p-162);
  const int k0 = panel * K::B, tid = threadIdx.x;
  BlPivots* piv = bl_at<BlPivots>(p, V.oPiv);
  double* Wp = bl_at<double>(p, V.oW);
  double* R1 = bl_at<double>(p, V.oRp);
  double* R2 = bl_at<double>(p, V.oU);
  double* red = lds;
  int* sh = reinterpret_cast<int*>(red + 4 * width_of(L));
  double* la = red + 4 * width_of(L) + 2;
  const int cap = min(p.N, int((bl_solve_lds<L>() / 8 - 4 * width_of(L) - 2) / width_of(L)));
  int j;  // a ticket taken in one sweep may be one of the next
  auto take = [&]() {
    __syncthreads();
    if (tid == 0) *sh = atomicAdd(&misc->ticket, 1);
    __syncthreads();
    j = *sh;
  };
  take();
  for (int sweep = 0; sweep < 2; ++sweep) {
    for (; j < (sweep + 1) * bcur; take()) {
      const int c = j - sweep * bcur;
      const bool ok = bl_mgs_column<L>(p, misc, piv, sweep, Wp, sweep ? R2 : R1, k0, c, red, sh, la, cap);
      if (tid == 0) {
        if (!ok) misc->flag = panel + 1;
        else if (sweep == 0 && c + 1 == bcur) misc->rmax = piv->rmax[c];
      }
      __threadfence();
      __syncthreads();
      if (tid == 0)
        __hip_atomic_store(piv->state[sweep] + c, ok ? 1 : 2, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      if (ok && sweep == 1) {
        // entry (i, c) = sum over m = i .. c of R2[i][m] R1[m][c]
        C<L> s = c_zero<L>();
        for (int m = tid; m <= c; ++m)
          s = c_add(s, c_mul(load_aos<L>(R2 + (size_t(tid) * K::B + m) * K::W), load_aos<L>(R1 + (size_t(m) * K::B + c) * K::W)));
        __syncthreads();
        if (tid <= c) store_aos(R1 + (size_t(tid) * K::B + c) * K::W, s);
      }
    }
    if (bl_await(piv->state[sweep] + bcur - 1, sh) == 2) return false;
    bool again = false;
    for (int c = 0; c < bcur; ++c) again = again || !(piv->loss[c] <= kLoss);
    if (!again) break;
  }
  return true;
}

template <int L>
__global__ __launch_bounds__(256) void bl_solve_kernel(BlView V, int panel, int cur) {
  using K = Bl<L>;
  constexpr int B = K::B, NL = K::NL, ND = K::ND, CX = K::CX, NR = bl_solve_rows<L>(), RPW = 4 * NR;
  using RL = R<NL>;
  extern __shared__ double lds[];
  const BlProb p = bl_prob<L>(V, blockIdx.y);
  BlMisc* misc = bl_at<BlMisc>(p, V.oMisc);
  const int k0 = panel * B, r0 = blockIdx.x * RPW;
  const int NC = (p.N + kBlRows - 1) / kBlRows;
  if (k0 >= p.n || r0 >= NC * kBlRows) return;
  const int flag = misc->flag, mgs = misc->mgs;  // tested once the loads are on their way
  const int bcur = min(B, p.n - k0);
  constexpr int UP = is_real(L) ? NL : 4 * NL;  // planes of a row of U in LDS
  double* Us = lds;                             // [B][planes][B]
  double* xs = lds + size_t(B) * B * UP;        // [RPW][64][NL] results
  int* er = reinterpret_cast<int*>(xs + RPW * 64 * NL);  // [RPW] row exponents
  const double* U = bl_at<double>(p, V.oU);
  double* Wp = bl_at<double>(p, V.oW);
  const int64_t plane = int64_t(p.n + 1) * p.N;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane % B, comp = lane / B;
  RL a[NR];
  auto load_rows = [&]() {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int row = r0 + wave * NR + r;
      const bool live = row < p.N && j < bcur;
#pragma unroll
      for (int l = 0; l < NL; ++l)
        a[r].x[l] = live ? Wp[(comp * NL + l) * plane + int64_t(k0 + j) * p.N + row] : 0.0;
    }
  };
  load_rows();
  // entry (i, j) of plane k at [i][k][j]: the lanes of a row read consecutive
  // words; planes: real limbs, imaginary limbs, their negatives, real limbs
  // again, so that a lane's two factors sit at fixed offsets
#pragma unroll 16
  for (int q = 0; q < B * B * K::W / 256; ++q) {
    const int idx = tid + q * 256, k = idx % K::W, ij = idx / K::W;
    const double u = U[idx];
    double* at = Us + size_t(ij / B) * UP * B + ij % B;
    if constexpr (is_real(L)) {
      at[k * B] = u;
    } else {
      at[k * B] = u;
      at[(k + 2 * NL) * B] = k < NL ? u : -u;
    }
  }
  if (flag) return;
  if (__builtin_expect(mgs, 0)) {
    if (!bl_mgs_panel<L>(V, p, misc, panel, bcur, lds)) return;
    load_rows();
    __syncthreads();  // the words of the waits are free
  } else {
    const double* is = U + size_t(B) * B * K::W;
    RL inv;
#pragma unroll
    for (int l = 0; l < NL; ++l) inv.x[l] = is[j * NL + l];
    const int ex = j < bcur ? -(bl_at<int>(p, V.oCe)[cur * V.nmax + k0 + j] - kExpOne) : 0;
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int l = 0; l < NL; ++l) a[r].x[l] = __builtin_ldexp(a[r].x[l], ex);
    __syncthreads();
    // a_i u_ij = re: ar ur + ai (-ui), im: ar ui + ai ur
    const double* ux = Us + comp * NL * B + j;
    const double* uy = Us + (comp ? 2 * NL : 3 * NL) * B + j;
    auto load_u = [&](int i, RL& x, RL& y) {
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        x.x[l] = ux[(size_t(i) * UP + l) * B];
        if constexpr (!is_real(L)) y.x[l] = uy[(size_t(i) * UP + l) * B];
      }
    };
    RL x, y, xn, yn;
    load_u(0, xn, yn);
    for (int i = 0; i + 1 < bcur; ++i) {
      x = xn;
      y = yn;
      load_u(i + 1, xn, yn);
      // the factors of columns up to i are zero: nothing to branch on
      RL t[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        C<L> ai;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          ai.re.x[l] = bl_readlane(a[r].x[l], i);
          if constexpr (!is_real(L)) ai.im.x[l] = bl_readlane(a[r].x[l], B + i);
        }
        if constexpr (is_real(L))
          t[r] = r_mul(ai.re, x);
        else if constexpr (NL == 1)
          t[r].x[0] = PE_FMA(ai.re.x[0], x.x[0], ai.im.x[0] * y.x[0]);
        else if constexpr (NL == 2)
          t[r] = dd_dot2(ai.re, x, ai.im, y, 1.0);
        else
          t[r] = qd_dot2(ai.re, x, ai.im, y);
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) a[r] = r_sub(a[r], t[r]);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int row = r0 + wave * NR + r;
      a[r] = r_mul(a[r], inv);
      if (row < p.N && j < bcur)
#pragma unroll
        for (int l = 0; l < NL; ++l)
          Wp[(comp * NL + l) * plane + int64_t(k0 + j) * p.N + row] = a[r].x[l];
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int rr = wave * NR + r;
    int e = bl_exp(a[r].x[0]);  // zero for rows and columns past the end
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) e = max(e, __shfl_xor(e, m));
#pragma unroll
    for (int l = 0; l < NL; ++l) xs[(rr * 64 + j * CX + comp) * NL + l] = a[r].x[l];
    if (lane == 0) {
      er[rr] = e - kExpOne;
      bl_at<int>(p, V.oXr)[r0 + rr] = e - kExpOne;
    }
  }
  __syncthreads();
  const int ch = r0 / kBlRows, rin = r0 % kBlRows;
  uint32_t* xd = bl_at<uint32_t>(p, V.oXD) + size_t(ch) * ND * 1024;
  uint32_t* xu = bl_at<uint32_t>(p, V.oXU) + size_t(ch) * ND * 1024;
  for (int t = tid; t < 64 * (RPW / 4) + RPW * 16; t += 256) {
    double v[4][NL];
    int ev[4];
    uint32_t* dst;
    if (t < 64 * (RPW / 4)) {
      const int m = t & 63, g = t >> 6;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ev[r] = 0;
#pragma unroll
        for (int l = 0; l < NL; ++l) v[r][l] = xs[((4 * g + r) * 64 + m) * NL + l];
      }
      dst = xd + m * 16 + (rin / 4 + g);
    } else {
      const int q = t - 64 * (RPW / 4), m4 = q & 15, r2 = q >> 4;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ev[r] = er[r2];
#pragma unroll
        for (int l = 0; l < NL; ++l) v[r][l] = xs[(r2 * 64 + m4 * 4 + r) * NL + l];
      }
      dst = xu + (rin + r2) * 16 + m4;
    }
    bl_put4<NL, ND>(v, ev, dst, 1024);
  }
}

// ------------------------------------------------------------------ R and T

// Columns of S summed over the row splits; the panel's rows of R; T = (I - E) S
// in digits ([tile][digit][16 real columns][64] bytes, real column 2 c
// holding (Tr, -Ti) and 2 c + 1 (Ti, Tr) of the B pairs, so that the update
// is one real product); the exponents of the next panel's columns cleared.
// For the panel's own columns R = (I + F) D^1/2 U instead.  E is about u_C over
// the smallest pivot ratio from the Gram matrix (double double 2^-104 / 2^-46 =
// 2^-58, quad double 2^-160; double, factored in double double, has the rounding
// of X itself, 2^-53 over the root of 2^-26, as its largest part, 2^-35 with a
// panel's 32 columns) and below bl_mgs_panel's kLoss from modified Gram-Schmidt
// (2^-33, 2^-64, 2^-162).  E^2 and E times double's roundoff are below the
// level's roundoff (2^-53, 2^-104, 2^-206) in each case, so its first order
// does and its products need no more than double arithmetic.  grid (column
// groups, slots), 256 threads: B lanes per column
template <int L>
__global__ __launch_bounds__(256) void bl_fin_kernel(BlView V, int panel, int cur) {
  using K = Bl<L>;
  constexpr int B = K::B, NL = K::NL, ND = K::ND, NW = K::NW, CX = K::CX, W = K::W, CPW = 256 / B;
  __shared__ double E[B * B * CX];    // [i][j]
  __shared__ double sl[CPW * B * CX];  // leading limbs of the columns of S
  const BlProb p = bl_prob<L>(V, blockIdx.y);
  const int k0 = panel * B;
  if (k0 >= p.n) return;
  const int flag = bl_at<BlMisc>(p, V.oMisc)->flag;
  const int bcur = min(B, p.n - k0);
  const int c0 = blockIdx.x * CPW;
  if (k0 + c0 > p.n) return;
  const int ns = bl_dot_splits<L>(p.N, (p.n + 1 - k0) * CX);
  const int tid = threadIdx.x;
  auto sum = [&](int c, int i) {
    return bl_sum_splits<L>(p.base + V.oS + (size_t(c) * B + i) * W * 8, V.s_split, ns);
  };
#pragma unroll 4
  for (int q = 0; q < B * B / 256; ++q) {
    const int idx = tid + q * 256, j = idx / B, i = idx % B;
    double re = 0.0, im = 0.0;
    if (i < bcur && j < bcur) {
      C<L> s = sum(j, i);
      if (i == j) s.re = r_sub(s.re, r_from_double<NL>(1.0));
      re = s.re.x[0];
      im = im_lead(s);
    }
    E[(i * B + j) * CX] = re;
    if (CX == 2) E[(i * B + j) * CX + 1] = im;
  }
  const int cl = tid / B, i = tid % B;
  const int c = c0 + cl, col = k0 + c;
  const bool in = col <= p.n;
  const bool own = in && c < bcur;
  C<L> s = in ? (own ? c_zero<L>() : sum(c, i)) : c_zero<L>();
  sl[tid * CX] = s.re.x[0];
  if (CX == 2) sl[tid * CX + 1] = im_lead(s);
  if (flag) return;
  __syncthreads();
  if (blockIdx.x == 0)
    for (int idx = tid; idx < B * B * CX; idx += 256) bl_at<double>(p, V.oF)[size_t(panel) * B * B * CX + idx] = E[idx];
  double* R = bl_at<double>(p, V.oR);
  const int64_t rplane = int64_t(p.n + 1) * p.n;
  int* ce = bl_at<int>(p, V.oCe);
  auto e_at = [&](int a, int b, double& re, double& im) {
    re = E[(a * B + b) * CX];
    im = CX == 2 ? E[(a * B + b) * CX + 1] : 0.0;
  };
  if (own) {
    if (i <= c) {
      const double* Rp = bl_at<double>(p, V.oRp);
      const int* rexp = reinterpret_cast<const int*>(Rp + size_t(B) * B * W);
      C<L> r = load_aos<L>(Rp + (size_t(i) * B + c) * W);
      double fr = 0.0, fi = 0.0;
      for (int m = i; m <= c; ++m) {
        const double* q = Rp + (size_t(m) * B + c) * W;
        const double qr = q[0], qi = CX == 2 ? q[(CX - 1) * NL] : 0.0;
        double er, ei;
        e_at(i, m, er, ei);
        if (m == i) {
          er *= 0.5;
          ei = 0.0;
        }
        fr += er * qr - ei * qi;
        fi += er * qi + ei * qr;
      }
      C<L> f = c_zero<L>();
      f.re.x[0] = fr;
      if constexpr (!is_real(L)) f.im.x[0] = i == c ? 0.0 : fi;
      r = bl_ldexp(c_add(r, f), rexp[c]);
      store_planar(R + int64_t(col) * p.n, rplane, k0 + i, r);
      if (i == c) {
        const auto inv = r_recip(r.re);
        r_store_aos(bl_at<double>(p, V.oInv) + size_t(col) * NL, inv);
      }
    }
    return;
  }
  if (!in) return;
  // lanes of one column are neighbours: B of them
  double lr = 0.0, li = 0.0, hr = 0.0, hi = 0.0;  // sums over j < i (with half of j = i) and over all j
  for (int j = 0; j < bcur; ++j) {
    // E is Hermitian: E_ij read as conj(E_ji), consecutive over the lanes
    double er, ei;
    e_at(j, i, er, ei);
    ei = -ei;
    const double sr = sl[(cl * B + j) * CX], si = CX == 2 ? sl[(cl * B + j) * CX + 1] : 0.0;
    const double tr = er * sr - ei * si, ti = er * si + ei * sr;
    hr += tr;
    hi += ti;
    if (j < i) {
      lr += tr;
      li += ti;
    } else if (j == i) {
      lr += 0.5 * tr;
      li += 0.5 * ti;
    }
  }
  auto minus = [](const C<L>& v, double re, double im) {
    C<L> f = c_zero<L>();
    f.re.x[0] = -re;
    if constexpr (!is_real(L)) f.im.x[0] = -im;
    return c_add(v, f);
  };
  C<L> r = minus(s, lr, li);
  if (ce[cur * V.nmax + col] == 0x7ff) {
    // a column with a value that is not finite has no projection
    const double nan = __builtin_nan("");
    for (int l = 0; l < NL; ++l) {
      r.re.x[l] = nan;
      if constexpr (!is_real(L)) r.im.x[l] = nan;
    }
  }
  if (i < bcur) store_planar(R + int64_t(col) * p.n, rplane, k0 + i, r);
  const C<L> t = minus(s, hr, hi);
  int e = max(bl_exp(t.re.x[0]), bl_exp(im_lead(t)));
#pragma unroll
  for (int m = 1; m < B; m <<= 1) e = max(e, __shfl_xor(e, m));
  if (i == 0) {
    bl_at<int>(p, V.oSe)[c] = e - kExpOne;
    ce[(1 - cur) * V.nmax + col] = 0;
  }
  uint32_t wr[NW], wi[NW], wn[NW];
  bl_digits<NL, ND>(t.re.x, e - kExpOne, wr);
  char* sd = bl_at<char>(p, V.oSD);
  if constexpr (is_real(L)) {
    char* dst = sd + size_t(c / 16) * ND * 1024 + (c % 16) * 64 + i;
#pragma unroll
    for (int d = 0; d < ND; ++d) dst[d * 1024] = char(wr[d / 4] >> (8 * (3 - d % 4)));
  } else {
    bl_digits<NL, ND>(t.im.x, e - kExpOne, wi);
    bl_digits<NL, ND>(r_neg(t.im).x, e - kExpOne, wn);
    const int rc = 2 * c;
    char* dst = sd + size_t(rc / 16) * ND * 1024 + (rc % 16) * 64 + 2 * i;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      const int sh = 8 * (3 - d % 4);
      const uint32_t a = (wr[d / 4] >> sh) & 255u, b = (wi[d / 4] >> sh) & 255u, n = (wn[d / 4] >> sh) & 255u;
      *reinterpret_cast<uint16_t*>(dst + d * 1024) = uint16_t(a | (n << 8));
      *reinterpret_cast<uint16_t*>(dst + d * 1024 + 64) = uint16_t(b | (a << 8));
    }
  }
}

// ------------------------------------------------------------------ trailing update

// Columns behind the panel -= X T.  A workgroup keeps the digits of 64 rows of
// X (16 per wavefront) in registers and walks column tiles of 16 real
// columns, whose digits of T it reads from the cache; K is the panel's 64
// real columns, one matrix instruction.  Also the largest exponent of every
// updated column.  grid (chunks, column groups, slots), 256 threads
template <int L>
__global__ __launch_bounds__(256, limbs_of(L) == 4 ? 1 : 2) void bl_update_kernel(BlView V, int panel, int cur, int tiles_per) {
  using K = Bl<L>;
  constexpr int NL = K::NL, ND = K::ND, CX = K::CX, B = K::B;
  const BlProb p = bl_prob<L>(V, blockIdx.z);
  const int k0 = panel * B, k1 = k0 + B;
  const int ch = blockIdx.x;
  if (k1 >= p.n || ch * kBlRows >= p.N) return;
  const int flag = bl_at<BlMisc>(p, V.oMisc)->flag;
  // tiles count from the panel's first column; its own 64 real columns are 4 tiles
  const int ntiles = ((p.n + 1 - k0) * CX + 15) / 16;
  const int t0 = 4 + blockIdx.y * tiles_per, t1 = min(ntiles, t0 + tiles_per);
  if (t0 >= t1) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t plane = int64_t(p.n + 1) * p.N;
  double* Wp = bl_at<double>(p, V.oW);
  int* ce = bl_at<int>(p, V.oCe) + (1 - cur) * V.nmax;
  const int* se = bl_at<int>(p, V.oSe);
  const bl_v4i* xu = bl_at<bl_v4i>(p, V.oXU) + size_t(ch) * ND * 256 + (16 * wave + (lane & 15)) * 4 + (lane >> 4);
  bl_v4i a[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) a[i] = xu[i * 256];
  const int row0 = ch * kBlRows + 16 * wave + 4 * (lane >> 4);
  int er[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) er[r] = bl_at<int>(p, V.oXr)[row0 + r] - 12;
  if (flag) return;
  for (int t = t0; t < t1; ++t) {
    const bl_v4i* sd = bl_at<bl_v4i>(p, V.oSD) + size_t(t) * ND * 64 + (lane & 15) * 4 + (lane >> 4);
    const int rc = t * 16 + (lane & 15);
    const int c = rc / CX, col = k0 + c;
    const bool in = col <= p.n;
    double* dst = Wp + int64_t(rc % CX) * NL * plane + int64_t(in ? col : p.n) * p.N;
    double old[4][NL];
    bl_load4<NL>(dst, plane, row0, p.N, in, old);
    bl_v4i av[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) av[d] = bl_v4i{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < ND; ++j) {
      const bl_v4i b = sd[j * 64];
#pragma unroll
      for (int i = 0; i < ND; ++i)
        if (i + j < ND) av[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b, av[i + j], 0, 0, 0);
    }
    const int es = in ? se[c] : 0;
    int emax = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int tt[ND];
#pragma unroll
      for (int d = 0; d < ND; ++d) tt[d] = av[d][r];
      const R<NL> v = bl_value<NL, ND>(tt, es + er[r]);
      R<NL> o;
#pragma unroll
      for (int l = 0; l < NL; ++l) o.x[l] = old[r][l];
      const R<NL> w = r_sub(o, v);
#pragma unroll
      for (int l = 0; l < NL; ++l) old[r][l] = w.x[l];
      if (in && row0 + r < p.N) emax = max(emax, bl_exp(w.x[0]));
    }
    if (in) bl_store4<NL>(dst, plane, row0, p.N, old);
    emax = max(emax, __shfl_xor(emax, 16));
    emax = max(emax, __shfl_xor(emax, 32));
    if (CX == 2) emax = max(emax, __shfl_xor(emax, 1));
    if (in && lane < 16 && (CX == 1 || (lane & 1) == 0)) atomicMax(ce + col, emax);
  }
}

// ------------------------------------------------------------------ back substitution

constexpr int kBlBsThreads = 512;

// Diagonal block `stage` (of kBlBs rows, from the bottom) of R x = y, in
// sub-blocks of 32 rows, the columns of their triangles over their pivots so
// that a step of the chain is one product and one sum.  Wavefront 0 solves a
// sub-block, its lanes the rows (complex: real parts in the lower, imaginary
// parts in the upper half), x_j broadcast through scalar registers, the
// triangle staged in LDS.  Meanwhile the other wavefronts subtract the columns
// of the sub-block before from the rows above this one; the rows of the next
// sub-block take this one's columns first, 16 threads a row.  256 rows:
// 88 -> 70 us (complex double double), 228 -> 152 us (real quad double).
// grid (slots), 512 threads
template <int L>
__global__ __launch_bounds__(kBlBsThreads) void bl_bs_diag_kernel(BlView V, int stage) {
  constexpr int NL = limbs_of(L), W = width_of(L), SB = 32, PT = SB * SB / kBlBsThreads;
  static_assert(kBlBsThreads == 16 * SB && kBlBsThreads - 64 >= 2 * (kBlBs - 2 * SB), "threads of the updates");
  using RL = R<NL>;
  constexpr int TP = is_real(L) ? NL : 4 * NL;  // planes: re, im, re, -im
  __shared__ double tri[SB * TP * SB];          // [column][plane][row]
  __shared__ double y[kBlBs * W];
  __shared__ double dinv[kBlBs * NL];
  const BlProb p = bl_prob<L>(V, blockIdx.x);
  const int flag = bl_at<BlMisc>(p, V.oMisc)->flag;
  const int e = p.n - stage * kBlBs;
  if (e <= 0) return;
  const int s = max(0, e - kBlBs);
  const int tid = threadIdx.x;
  const int64_t rplane = int64_t(p.n + 1) * p.n;
  const double* Rm = bl_at<double>(p, V.oR);
  double* yw = bl_at<double>(p, V.oY);
  const double* inv = bl_at<double>(p, V.oInv);
  if (tid < e - s) {
    const C<L> v =
        stage == 0 ? load_planar<L>(Rm + int64_t(p.n) * p.n, rplane, s + tid) : load_planar<L>(yw, p.n, s + tid);
    store_planar(y, kBlBs, tid, v);
    r_store_aos(dinv + tid * NL, r_load_aos<NL>(inv + size_t(s + tid) * NL));
  }
  C<L> next[PT];  // the thread's entries of the next triangle and 1 / their column's pivot
  RL scale[PT];
  auto fetch = [&](int se) {
    const int ss = max(s, se - SB), sb = se - ss;
#pragma unroll
    for (int q = 0; q < PT; ++q) {
      const int idx = tid + q * kBlBsThreads, jj = idx / SB, ii = idx % SB;
      next[q] = (jj < sb && ii < jj) ? load_planar<L>(Rm + int64_t(ss + jj) * p.n, rplane, ss + ii) : c_zero<L>();
      scale[q] = r_load_aos<NL>(inv + size_t(ss + min(jj, sb - 1)) * NL);
    }
  };
  fetch(e);
  if (flag) return;
  for (int se = e; se > s; se -= SB) {
    const int ss = max(s, se - SB), sb = se - ss;
#pragma unroll
    for (int q = 0; q < PT; ++q) {
      const int idx = tid + q * kBlBsThreads;
      next[q] = c_mul_r(next[q], scale[q]);
      store_planar(tri + (idx / SB) * TP * SB, SB, idx % SB, next[q]);
      if constexpr (!is_real(L)) store_planar(tri + ((idx / SB) * TP + 2 * NL) * SB, SB, idx % SB, c_conj(next[q]));
    }
    __syncthreads();
    if (ss > s) fetch(ss);
    // the rows of the next sub-block: row sn + tid / 16, columns tid % 16 and
    // 16 further on, whose entries of R arrive while wavefront 0 solves
    const int sn = max(s, ss - SB), un = tid >> 4, uc = tid & 15;
    C<L> up[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
      up[q] = (sn + un < ss && uc + 16 * q < sb)
                  ? load_planar<L>(Rm + int64_t(ss + uc + 16 * q) * p.n, rplane, sn + un)
                  : c_zero<L>();
    if (tid < 64) {
      const int ii = is_real(L) ? (tid & (SB - 1)) : tid % SB, comp = is_real(L) ? 0 : tid / SB;
      RL v = r_zero<NL>(), dv = v;
      if (ii < sb) {
#pragma unroll
        for (int l = 0; l < NL; ++l) v.x[l] = y[(comp * NL + l) * kBlBs + ss - s + ii];
        dv = r_load_aos<NL>(dinv + (ss - s + ii) * NL);
      }
      const double* fx = tri + comp * NL * SB + ii;
      const double* fy = tri + (comp ? 2 * NL : 3 * NL) * SB + ii;
      auto load_r = [&](int jj, RL& f, RL& g) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          f.x[l] = fx[(jj * TP + l) * SB];
          if constexpr (!is_real(L)) g.x[l] = fy[(jj * TP + l) * SB];
        }
      };
      RL f, g, fn, gn, res = v;
      load_r(sb - 1, fn, gn);
      for (int jj = sb - 1; jj >= 0; --jj) {
        f = fn;
        g = gn;
        load_r(max(jj - 1, 0), fn, gn);
        C<L> xj;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          xj.re.x[l] = bl_readlane(v.x[l], jj);
          if constexpr (!is_real(L)) xj.im.x[l] = bl_readlane(v.x[l], SB + jj);
        }
        RL t;
        if constexpr (is_real(L))
          t = r_mul(xj.re, f);
        else if constexpr (NL == 1)
          t.x[0] = PE_FMA(xj.re.x[0], f.x[0], xj.im.x[0] * g.x[0]);
        else if constexpr (NL == 2)
          t = dd_dot2(xj.re, f, xj.im, g, 1.0);
        else
          t = qd_dot2(xj.re, f, xj.im, g);
        if (ii == jj) res = v;
        v = r_sub(v, t);  // the entries of rows from jj on are zero
      }
      res = r_mul(res, dv);
      if (ii < sb && (!is_real(L) || tid < SB)) {
#pragma unroll
        for (int l = 0; l < NL; ++l) y[(comp * NL + l) * kBlBs + ss - s + ii] = res.x[l];
      }
    } else if (se < e) {
      // the columns of the sub-block before (full: [se, se + 32)) from the
      // rows above this one: two threads per row, even and odd columns
      const int rows = ss - s, i = (tid - 64) >> 1, h = tid & 1;
      if (i < rows) {
        const int64_t at = int64_t(se + h) * p.n + s + i;
        constexpr int UN = W <= 4 ? 8 : 2;  // loads in flight: they would outlast the solve one by one
        C<L> acc = c_zero<L>();
#pragma unroll 1
        for (int q0 = 0; q0 < SB / 2; q0 += UN) {
          C<L> r[UN];
#pragma unroll
          for (int q = 0; q < UN; ++q) r[q] = load_planar<L>(Rm + at + int64_t(2 * (q0 + q)) * p.n, rplane, 0);
#pragma unroll
          for (int q = 0; q < UN; ++q)
            acc = c_add(acc, c_mul(r[q], load_planar<L>(y, kBlBs, se - s + h + 2 * (q0 + q))));
        }
        acc = c_add(acc, shfl_xor_c(acc, 1));
        if (h == 0) store_planar(y, kBlBs, i, c_sub(load_planar<L>(y, kBlBs, i), acc));
      }
    }
    __syncthreads();
    if (ss > s) {
      C<L> acc = c_zero<L>();
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (uc + 16 * q < sb) acc = c_add(acc, c_mul(up[q], load_planar<L>(y, kBlBs, ss - s + uc + 16 * q)));
#pragma unroll 1
      for (int m = 1; m < 16; m <<= 1) acc = c_add(acc, shfl_xor_c(acc, m));
      if (uc == 0 && sn + un < ss)
        store_planar(y, kBlBs, sn - s + un, c_sub(load_planar<L>(y, kBlBs, sn - s + un), acc));
    }
  }
  __syncthreads();
  if (tid < e - s) store_planar(yw, p.n, s + tid, load_planar<L>(y, kBlBs, tid));
}

// y[0, s) -= R[0:s, s:e] x[s:e] for the block `stage` just solved: eight
// lanes per row, their sums added in order.  grid (row blocks of 32,
// slots), 256 threads
template <int L>
__global__ __launch_bounds__(256) void bl_bs_update_kernel(BlView V, int stage) {
  __shared__ double xs[kBlBs * width_of(L)];
  const BlProb p = bl_prob<L>(V, blockIdx.y);
  if (bl_at<BlMisc>(p, V.oMisc)->flag) return;
  const int e = p.n - stage * kBlBs;
  const int s = e - kBlBs;
  const int r0 = blockIdx.x * 32;
  if (s <= 0 || r0 >= s) return;
  const int tid = threadIdx.x;
  const int64_t rplane = int64_t(p.n + 1) * p.n;
  const double* R = bl_at<double>(p, V.oR);
  double* yw = bl_at<double>(p, V.oY);
  store_planar(xs, kBlBs, tid, load_planar<L>(yw, p.n, s + tid));
  __syncthreads();
  // lanes of a wavefront: 32 rows x 2 column halves; the wavefronts take
  // quarters of the columns
  const int i = r0 + (tid & 31), part = tid >> 5;
  C<L> acc = c_zero<L>();
  if (i < s)
#pragma unroll 8
    for (int j = part * (kBlBs / 8); j < (part + 1) * (kBlBs / 8); ++j)
      acc = c_add(acc, c_mul(load_planar<L>(R + int64_t(s + j) * p.n, rplane, i), load_planar<L>(xs, kBlBs, j)));
  __syncthreads();
  double* red = xs;  // [8][32] numbers
  store_planar(red, kBlBs, tid, acc);
  __syncthreads();
  if (tid < 32 && i < s) {
    C<L> t = load_planar<L>(red, kBlBs, tid);
    for (int q = 1; q < 8; ++q) t = c_add(t, load_planar<L>(red, kBlBs, q * 32 + tid));
    const C<L> old =
        stage == 0 ? load_planar<L>(R + int64_t(p.n) * p.n, rplane, i) : load_planar<L>(yw, p.n, i);
    store_planar(yw, p.n, i, c_sub(old, t));
  }
}

// x (+)= dx, dx = 0 when a pivot was zero; resid[1] = |dx|_inf or -1.  grid
// (slots), 256 threads
template <int L>
__global__ __launch_bounds__(256) void bl_finish_kernel(BlView V) {
  __shared__ double red[256];
  const BlProb p = bl_prob<L>(V, blockIdx.x);
  const int tid = threadIdx.x;
  const bool singular = bl_at<BlMisc>(p, V.oMisc)->flag != 0;
  double dmax = 0.0;
  for (int j = tid; j < p.n; j += 256) {
    const C<L> d = singular ? c_zero<L>() : load_planar<L>(bl_at<double>(p, V.oY), p.n, j);
    if (!(singular && V.add)) store_planar(p.x, p.n, j, V.add ? c_add(load_planar<L>(p.x, p.n, j), d) : d);
    dmax = fmax(dmax, fmax(fabs(d.re.x[0]), fabs(im_lead(d))));
  }
  red[tid] = dmax;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (tid < k) red[tid] = fmax(red[tid], red[tid + k]);
    __syncthreads();
  }
  if (tid == 0 && p.resid) p.resid[1] = singular ? -1.0 : red[0];
}

// R (row-major [P][components][n][n + 1], zeros below the diagonal) and
// Q = X (I - F) ([P][components][N][n]); zeros from the panel of a zero pivot
// on, which has neither.  A group of lanes takes a row of a panel of Q.  grid
// (blocks, slots), 256 threads
template <int L>
__global__ __launch_bounds__(256) void bl_export_kernel(BlView V) {
  using K = Bl<L>;
  constexpr int B = K::B, CX = K::CX, NL = K::NL;
  const BlProb p = bl_prob<L>(V, blockIdx.y);
  const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t pt = V.q0 + blockIdx.y;
  const int ncol = p.n + 1;
  const int64_t rplane = int64_t(ncol) * p.n;
  const int flag = bl_at<BlMisc>(p, V.oMisc)->flag;
  const int done = flag ? (flag - 1) * B : p.n;
  if (V.Rout && idx < rplane) {
    const int i = int(idx / ncol), j = int(idx - int64_t(i) * ncol);
    const C<L> r =
        i <= j && i < done ? load_planar<L>(bl_at<double>(p, V.oR) + int64_t(j) * p.n, rplane, i) : c_zero<L>();
    store_planar(V.Rout + pt * (int64_t(K::W) * rplane), rplane, idx, r);
  }
  if (V.Qout && idx < int64_t(p.N) * p.n) {
    // consecutive threads take consecutive columns of a row of Q
    const int i = int(idx / p.n), c = int(idx - int64_t(i) * p.n);
    const int k0 = c / B * B, cc = c - k0;
    const int64_t plane = int64_t(ncol) * p.N;
    if (c >= done) {
      store_planar(V.Qout + pt * (int64_t(K::W) * p.N * p.n), int64_t(p.N) * p.n, idx, c_zero<L>());
      return;
    }
    const double* X = bl_at<double>(p, V.oW) + i;
    const double* F = bl_at<double>(p, V.oF) + size_t(c / B) * B * B * CX;
    double fr = 0.0, fi = 0.0;
    for (int m = 0; m <= cc; ++m) {
      const double xr = X[int64_t(k0 + m) * p.N], xi = CX == 2 ? X[(CX - 1) * NL * plane + int64_t(k0 + m) * p.N] : 0.0;
      double er = F[(m * B + cc) * CX], ei = CX == 2 ? F[(m * B + cc) * CX + CX - 1] : 0.0;
      if (m == cc) {
        er *= 0.5;
        ei = 0.0;
      }
      fr += xr * er - xi * ei;
      fi += xr * ei + xi * er;
    }
    C<L> f = c_zero<L>();
    f.re.x[0] = -fr;
    if constexpr (!is_real(L)) f.im.x[0] = -fi;
    const C<L> q = c_add(load_planar<L>(X + int64_t(c) * p.N, plane, 0), f);
    store_planar(V.Qout + pt * (int64_t(K::W) * p.N * p.n), int64_t(p.N) * p.n, idx, q);
  }
}

}  // namespace pe
