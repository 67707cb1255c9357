// Least-squares solve of small problems by modified Gram-Schmidt on the
// augmented matrix [A b] (Sec. 3, Fig. 4 and eq. (2)) and back substitution
// R x = y, one wavefront per problem.  The panels of blockls_kernels.hpp are
// padded to 64 rows and 64 real columns and take nine launches: for a few
// unknowns that is many times the work, and the whole solve in one launch is
// ahead (small_solve in polyeval.hip has the line and the times).
//
// Lane t owns column t of [A b].  As in the paper's delayed normalisation, the
// pivot column is never normalised in memory: the projection coefficient of
// column j is (a_k^H a_j) / |a_k|^2 and r_kj = (a_k^H a_j) / |a_k|.  Step k first
// updates column k + 1 with pivot k, all lanes together, and stages it in LDS
// beside pivot k; then every later column is updated with pivot k and, in the
// same pass over its rows, its inner product with column k + 1 (the next pivot)
// is accumulated, so a column is read and written once per pivot.  Bound by the
// chain of n pivots of N rows each; many problems share a CU.
#pragma once
#include <hip/hip_runtime.h>

#include "blockls_kernels.hpp"
#include "eval_kernels.hpp"
#include "mdarith.hpp"
#include "newton_kernels.hpp"

namespace pe {

constexpr int kSmallCols = 64;  // columns of [A b], one per lane

// slot of a problem of at most N rows and n unknowns: R [n][n + 1] and y [n],
// numbers of consecutive limbs, and for the callers that keep A a copy of [A b]
template <int L>
inline void small_layout(int N, int n, bool keep, BlView& V) {
  constexpr size_t W = width_of(L);
  size_t off = 0;
  auto take = [&](size_t doubles) {
    const size_t at = off;
    off += (doubles * 8 + 255) & ~size_t(255);
    return at;
  };
  V.oR = take(W * n * (n + 1));
  V.oY = take(W * n);
  V.oW = take(keep ? W * N * (n + 1) : 0);
  V.slot = off;
}

// LDS of a workgroup: pivot k and column k + 1 of N numbers each
template <int L>
inline size_t small_lds(int N) {
  return (2 * size_t(N) + 1) * width_of(L) * sizeof(double);
}

// grid (slots), 64 threads
template <int L>
__global__ __launch_bounds__(64) void small_solve_kernel(BlView V) {
  using RL = R<limbs_of(L)>;
  constexpr int W = width_of(L), NL = limbs_of(L);
  extern __shared__ double lds[];
  const BlProb p = bl_prob<L>(V, blockIdx.x);
  const int N = p.N, n = p.n, ld = n + 1, t = threadIdx.x;
  double* Rm = bl_at<double>(p, V.oR);
  double* Y = bl_at<double>(p, V.oY);
  double* colk = lds;                 // N numbers: pivot k
  double* coln = colk + size_t(N) * W;  // N numbers: column k + 1
  double* dpub = coln + size_t(N) * W;  // a_k^H a_{k+1}
  // a Newton step's matrix is workspace; elsewhere it is the caller's
  double* A = const_cast<double*>(p.A);
  int64_t plane = p.a_plane, row = p.ld;
  if (!V.add) {
    A = bl_at<double>(p, V.oW);
    plane = int64_t(N) * ld;
    row = ld;
    for (int c = 0; c < W; ++c)
      for (int i = t; i < N * ld; i += 64) A[c * plane + i] = p.A[c * p.a_plane + int64_t(i / ld) * p.ld + i % ld];
  }
  __syncthreads();
  auto wave_sum = [](RL s) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
      RL o;
#pragma unroll
      for (int l = 0; l < NL; ++l) o.x[l] = __shfl_xor(s.x[l], m);
      s = r_add(s, o);
    }
    return s;
  };
  // |b|_2 from the leading limbs, |a_0|^2, column 0 staged
  double fs = 0.0;
  RL nk = r_zero<NL>();
  for (int i = t; i < N; i += 64) {
    const double re = A[int64_t(i) * row + n], im = is_real(L) ? 0.0 : A[int64_t(NL) * plane + int64_t(i) * row + n];
    fs += re * re + im * im;
    const C<L> a = load_planar<L>(A, plane, int64_t(i) * row);
    store_aos(colk + size_t(i) * W, a);
    nk = r_add(nk, c_norm2(a));
  }
  nk = wave_sum(nk);
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) fs += __shfl_xor(fs, m);
  __syncthreads();
  // inner products of the pivot with the later columns, unscaled in R's row 0
  if (t >= 1 && t <= n) {
    C<L> d = c_zero<L>();
    for (int i = 0; i < N; ++i)
      d = c_add(d, c_mul_conj_a(load_aos<L>(colk + size_t(i) * W), load_planar<L>(A, plane, int64_t(i) * row + t)));
    store_aos(Rm + size_t(t) * W, d);
    if (t == 1) store_aos(dpub, d);
  }
  __syncthreads();
  double rmax = 0.0;
  int done = n;  // pivots taken
  for (int k = 0; k < n; ++k) {
    const RL rkk = r_sqrt(nk);
    rmax = fmax(rmax, rkk.x[0]);
    if (!(rkk.x[0] > double(n) * level_unit<L>() * rmax)) {
      done = k;
      break;  // uniform: every lane has the same sums
    }
    const RL inv_n = r_recip(nk), inv_r = r_recip(rkk);
    // column k + 1 (the next pivot; the right-hand side when k + 1 = n)
    const C<L> d1 = load_aos<L>(dpub);
    const C<L> cr1 = c_neg(c_mul_r(d1, inv_n));
    RL s2 = r_zero<NL>();
    for (int i = t; i < N; i += 64) {
      C<L> a = load_planar<L>(A, plane, int64_t(i) * row + k + 1);
      a = c_add(a, c_mul(cr1, load_aos<L>(colk + size_t(i) * W)));
      store_planar(A, plane, int64_t(i) * row + k + 1, a);
      store_aos(coln + size_t(i) * W, a);
      s2 = r_add(s2, c_norm2(a));
    }
    nk = wave_sum(s2);
    if (t == 0) {
      store_aos(Rm + (size_t(k) * ld + k) * W, c_from_r<L>(rkk));
      store_aos(Rm + (size_t(k) * ld + k + 1) * W, c_mul_r(d1, inv_r));
    }
    __syncthreads();  // column k + 1 staged, dpub read
    if (t >= k + 2 && t <= n) {
      double* rkj = Rm + (size_t(k) * ld + t) * W;
      const C<L> d = load_aos<L>(rkj);
      store_aos(rkj, c_mul_r(d, inv_r));
      const C<L> cr = c_neg(c_mul_r(d, inv_n));
      C<L> dn = c_zero<L>();
      for (int i = 0; i < N; ++i) {
        C<L> a = load_planar<L>(A, plane, int64_t(i) * row + t);
        a = c_add(a, c_mul(cr, load_aos<L>(colk + size_t(i) * W)));
        store_planar(A, plane, int64_t(i) * row + t, a);
        dn = c_add(dn, c_mul_conj_a(load_aos<L>(coln + size_t(i) * W), a));
      }
      store_aos(Rm + (size_t(k + 1) * ld + t) * W, dn);
      if (t == k + 2) store_aos(dpub, dn);
    }
    __syncthreads();
    double* s = colk;
    colk = coln;
    coln = s;
  }
  const bool singular = done < n;
  // R x = y, y = column n of R; x overwrites Y
  if (!singular) {
    if (t < n) store_aos(Y + size_t(t) * W, load_aos<L>(Rm + (size_t(t) * ld + n) * W));
    __syncthreads();
    for (int k = n - 1; k >= 0; --k) {
      if (t == 0) {
        const RL rkk = load_aos<L>(Rm + (size_t(k) * ld + k) * W).re;
        store_aos(Y + size_t(k) * W, c_mul_r(load_aos<L>(Y + size_t(k) * W), r_recip(rkk)));
      }
      __syncthreads();
      const C<L> dk = load_aos<L>(Y + size_t(k) * W);
      if (t < k) {
        const C<L> s = c_mul(load_aos<L>(Rm + (size_t(t) * ld + k) * W), dk);
        store_aos(Y + size_t(t) * W, c_sub(load_aos<L>(Y + size_t(t) * W), s));
      }
      __syncthreads();
    }
  }
  double dmax = 0.0;
  if (t < n) {
    const C<L> d = singular ? c_zero<L>() : load_aos<L>(Y + size_t(t) * W);
    if (!(singular && V.add)) store_planar(p.x, n, t, V.add ? c_add(load_planar<L>(p.x, n, t), d) : d);
    dmax = fmax(fabs(d.re.x[0]), fabs(im_lead(d)));
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) dmax = fmax(dmax, __shfl_xor(dmax, m));
  if (t == 0 && p.resid) {
    p.resid[0] = sqrt(fs);
    p.resid[1] = singular ? -1.0 : dmax;
  }
  // R (row-major planar, zeros below the diagonal) and the normalised pivots;
  // nothing behind a zero pivot
  const int64_t pt = V.q0 + int64_t(blockIdx.x);
  if (V.Rout)
    for (int i = t; i < n * ld; i += 64)
      store_planar(V.Rout + pt * (int64_t(W) * n * ld), int64_t(n) * ld, i,
                   i / ld <= i % ld && i / ld < done ? load_aos<L>(Rm + size_t(i) * W) : c_zero<L>());
  if (V.Qout)
    for (int i = t; i < N * n; i += 64) {
      const int k = i % n;
      C<L> q = c_zero<L>();
      if (k < done)
        q = c_mul_r(load_planar<L>(A, plane, int64_t(i / n) * row + k), r_recip(load_aos<L>(Rm + (size_t(k) * ld + k) * W).re));
      store_planar(V.Qout + pt * (int64_t(W) * N * n), int64_t(N) * n, i, q);
    }
}

}  // namespace pe
