// Gauss-Newton step on the device (Sec. 4): number helpers of the solve, the
// sizes of a batched step, and the right-hand side of the Newton homotopy.
// The least-squares solve itself is in blockls_kernels.hpp and, for a few
// unknowns, smallls_kernels.hpp.
#pragma once
#include <hip/hip_runtime.h>

#include "eval_kernels.hpp"
#include "mdarith.hpp"

namespace pe {

template <int L>
__device__ __forceinline__ R<L> r_load_aos(const double* p) {
  R<L> r;
#pragma unroll
  for (int l = 0; l < L; ++l) r.x[l] = p[l];
  return r;
}

template <int L>
__device__ __forceinline__ void r_store_aos(double* p, const R<L>& v) {
#pragma unroll
  for (int l = 0; l < L; ++l) p[l] = v.x[l];
}

template <int L>
__device__ __forceinline__ C<L> c_mul_conj_a(const C<L>& a, const C<L>& b) {
  return c_mul(c_conj(a), b);
}

// leading limb of the imaginary part (0 for a real number)
template <int L>
__device__ __forceinline__ double im_lead(const C<L>& a) {
  if constexpr (is_real(L))
    return 0.0;
  else
    return a.im.x[0];
}

// a real level-L number as a complex (or real) one
template <int L>
__device__ __forceinline__ C<L> c_from_r(const R<limbs_of(L)>& r) {
  C<L> d = c_zero<L>();
  d.re = r;
  return d;
}

// unit roundoff of the level: 2^-53, 2^-104, 2^-206 for 1, 2, 4 limbs
template <int L>
__host__ __device__ constexpr double level_unit() {
  return limbs_of(L) == 1 ? 0x1p-53 : (limbs_of(L) == 2 ? 0x1p-104 : 0x1p-206);
}

// Per-system description of a batched Newton step (offsets in doubles for
// one point; a system's block for P points starts at P times its offset).
struct BatchNewtonDesc {
  int N, n;
  int64_t w_off, x_off;
};

// Right-hand side of a Newton step on the homotopy h(x, t) = f(x) - t c
// (Sec. 5.3: c = f(z), so z solves h at t = 1).  The evaluation has written
// b = -f(x) into column n of the augmented matrices (row-major planar, point
// stride w_pt, plane stride plane, row stride ld); this replaces it by
// wF b + wc c_p with wF in {0, 1}: (1, t) is the corrector at t, (0, dt) the
// Euler predictor J dx = c dt.  c is [P][components][N]; grid over P * N.
template <int L>
__global__ void rhs_shift_kernel(double* __restrict__ W, int64_t w_pt, int64_t plane, int64_t ld, int N, int n, int P,
                                 const double* __restrict__ c, double wF, double wc) {
  const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= int64_t(P) * N) return;
  const int p = int(idx / N), i = int(idx - int64_t(p) * N);
  double* b = W + p * w_pt + int64_t(i) * ld + n;
  const C<L> sc = c_mul_d(load_planar<L>(c + int64_t(p) * width_of(L) * N, N, i), wc);
  store_planar(b, plane, 0, wF == 0.0 ? sc : c_add(load_planar<L>(b, plane, 0), sc));
}

}  // namespace pe
