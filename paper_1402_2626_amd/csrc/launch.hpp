// Host-side launchers of the device kernels.  Each launcher is a template
// over the level L; its instances for one (level, kind) are compiled in their
// own translation unit (instances.hip built with PE_LEVEL and PE_KIND), so the
// library builds in parallel.  polyeval.hip only sees the declarations.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "blockls_kernels.hpp"
#include "eval_kernels.hpp"
#include "newton_kernels.hpp"
#include "smallls_kernels.hpp"
#include "value_kernels.hpp"

namespace pe {

// The compiled launch shapes (level, segment length, chunks per workgroup).
// A workgroup of G chunks has G * 256 threads; G > 1 is compiled for up to
// 512 columns only.  Double double with segments of 16 and quad double with
// segments of 8 exist for monomials too wide for the shorter segments (up to
// 1024 and 512 variables in one wavefront); they hold many registers per lane.
#define PE_SHAPES(X) \
  X(1, 8, 1)         \
  X(1, 8, 4)         \
  X(1, 16, 1)        \
  X(1, 16, 2)        \
  X(2, 4, 1)         \
  X(2, 4, 4)         \
  X(2, 6, 1)         \
  X(2, 6, 2)         \
  X(2, 8, 1)         \
  X(2, 8, 2)         \
  X(2, 16, 1)        \
  X(4, 4, 1)         \
  X(4, 2, 1)         \
  X(4, 8, 1)

inline bool shape_compiled(int L, int seg, int G) {
#define PE_X(L_, S_, G_) \
  if (L == L_ && seg == S_ && G == G_) return true;
  PE_SHAPES(PE_X)
#undef PE_X
  return false;
}

// what a launch over one system needs to know about its plan
struct EvalShape {
  SysView view;
  int seg = 4, G = 1, cpl = 1;
  size_t lds = 0;   // dynamic LDS of a workgroup of G chunks
  size_t lds1 = 0;  // dynamic LDS of a one-chunk workgroup
  int64_t n_chunks = 0;  // chunks of the system (per-monomial output)
};

// one persistent launch over the items of a batch class
struct BatchShape {
  int seg = 4, G = 1, cpl = 1;
  int vw = 0;  // copy width of batch_small_kernel, 0: batch_rows_kernel
  size_t lds = 0;
  int64_t nitems = 0;
  const uint64_t* items = nullptr;
  const SysView* views = nullptr;
  const int64_t* x_off = nullptr;
  int* counter = nullptr;
};

template <int L>
hipError_t launch_rows(const EvalShape& sh, int P, const double* x, const OutView& O, int mode, hipStream_t st);

// per-monomial output (terms_waves_kernel)
template <int L>
hipError_t launch_terms(const EvalShape& sh, int P, const double* x, const OutView& O, hipStream_t st);
template <int L>
hipError_t launch_adjoint(const EvalShape& sh, int P, const double* x, const double* v, int NG, int gsize,
                          double* part, double* g, hipStream_t st);
template <int L>
hipError_t launch_batch(const BatchShape& b, int P, const double* x, const BatchOut& out, int mode,
                        hipStream_t st);
template <int L>
hipError_t launch_rhs_shift(double* W, int64_t w_pt, int64_t plane, int64_t ld, int N, int n, int P, const double* c,
                            double wF, double wc, hipStream_t st);

// evaluation through monomial values (value_kernels.hpp); lds: bytes of a
// workgroup of one copy
template <int L>
hipError_t launch_val_rows(const ValView& V, int P, const double* x, const OutView& O, int mode, hipStream_t st);
template <int L>
hipError_t launch_val_adjoint(const ValView& V, int P, const double* x, const double* v, int NG, int gsize, double* part,
                              double* g, hipStream_t st);

// a batch's items whose systems evaluate through monomial values
struct ValBatchShape {
  size_t lds = 0;
  bool small = false;  // a system's table holds x alone
  int64_t nitems = 0;
  const uint64_t* items = nullptr;
  const ValView* views = nullptr;
  const int64_t* x_off = nullptr;
  int* counter = nullptr;
};
template <int L>
hipError_t launch_val_batch(const ValBatchShape& b, int P, const double* x, const BatchOut& out, int mode,
                            hipStream_t st);

// Least-squares solve (blockls_kernels.hpp) of `slots` problems of at most
// Nm rows and nm unknowns, whose workspace slots V.ws holds.
constexpr int kLsMaxRows = 4096;  // N limit of the solve beyond 127 unknowns

template <int L>
hipError_t launch_blockls(const BlView& V, int slots, int Nm, int nm, hipStream_t st);

// The same for small problems (smallls_kernels.hpp), nm < kSmallCols.
template <int L>
hipError_t launch_small_solve(const BlView& V, int slots, int Nm, hipStream_t st);

#ifdef PE_LAUNCH_DEFINITIONS

template <typename K>
hipError_t allow_lds(K kern, size_t lds) {
  if (lds <= 65536) return hipSuccess;
  return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
}

template <int L, int SEG, int CPL, int G, int MODE>
hipError_t launch_rows_t(const EvalShape& sh, int P, const double* x, const OutView& O, hipStream_t st) {
  auto kern = eval_rows_kernel<L, SEG, CPL, G, MODE>;
  hipError_t e = allow_lds(kern, sh.lds);
  if (e != hipSuccess) return e;
  // F alone needs no column tiles (no owners): one workgroup per row-point
  SysView view = sh.view;
  if (MODE == MODE_FONLY) view.col_tiles = 1;
  const int64_t blocks = int64_t(P) * view.N * view.col_tiles;
  hipLaunchKernelGGL(kern, dim3(unsigned(blocks)), dim3(G * kSub), sh.lds, st, view, O, x,
                     int64_t(width_of(L)) * sh.view.n);
  return hipGetLastError();
}

template <int L, int SEG, int G>
hipError_t rows_lsg(const EvalShape& sh, int P, const double* x, const OutView& O, int mode, hipStream_t st) {
  const int cpl = sh.cpl;
  if (mode == MODE_EVAL) {
    if (cpl == 1) return launch_rows_t<L, SEG, 1, G, MODE_EVAL>(sh, P, x, O, st);
    if (cpl == 2) return launch_rows_t<L, SEG, 2, G, MODE_EVAL>(sh, P, x, O, st);
    if (G == 1 && cpl == 4) return launch_rows_t<L, SEG, 4, 1, MODE_EVAL>(sh, P, x, O, st);
    if (G == 1 && cpl == 8) return launch_rows_t<L, SEG, 8, 1, MODE_EVAL>(sh, P, x, O, st);
  } else {
    if (cpl == 1) return launch_rows_t<L, SEG, 1, G, MODE_FONLY>(sh, P, x, O, st);
    if (cpl == 2) return launch_rows_t<L, SEG, 2, G, MODE_FONLY>(sh, P, x, O, st);
    if (G == 1 && cpl == 4) return launch_rows_t<L, SEG, 4, 1, MODE_FONLY>(sh, P, x, O, st);
    if (G == 1 && cpl == 8) return launch_rows_t<L, SEG, 8, 1, MODE_FONLY>(sh, P, x, O, st);
  }
  return hipErrorInvalidValue;
}

template <int L>
hipError_t launch_rows(const EvalShape& sh, int P, const double* x, const OutView& O, int mode, hipStream_t st) {
#define PE_X(L_, S_, G_) \
  if constexpr (limbs_of(L) == L_) \
    if (sh.seg == S_ && sh.G == G_) return rows_lsg<L, S_, G_>(sh, P, x, O, mode, st);
  PE_SHAPES(PE_X)
#undef PE_X
  return hipErrorInvalidValue;
}

template <int L, int SEG>
hipError_t launch_terms_t(const EvalShape& sh, int P, const double* x, const OutView& O, hipStream_t st) {
  auto kern = terms_waves_kernel<L, SEG>;
  const SysView& V = sh.view;
  const size_t lds = size_t(V.tab_last >= V.tab_first ? V.tab_last - V.tab_first + 1 : 0) * (V.n + 1) *
                     width_of(L) * sizeof(double);
  hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  // about eight chunks per wavefront (the table is built once per
  // workgroup), and at least 2048 workgroups in all when there are chunks
  // enough
  const int64_t quads = (sh.n_chunks + 3) / 4;
  int64_t wpp = std::max<int64_t>((quads + 7) / 8, (2048 + P - 1) / P);
  // (and at most 2^31 - 1 in all: a workgroup then takes more chunks)
  wpp = std::max<int64_t>(1, std::min<int64_t>({wpp, quads, 0x7fffffffLL / std::max(P, 1)}));
  hipLaunchKernelGGL(kern, dim3(unsigned(int64_t(P) * wpp)), dim3(kSub), lds, st, V, O, x,
                     int64_t(width_of(L)) * V.n, int(wpp), uint32_t(sh.n_chunks));
  return hipGetLastError();
}

template <int L>
hipError_t launch_terms(const EvalShape& sh, int P, const double* x, const OutView& O, hipStream_t st) {
#define PE_X(L_, S_, G_) \
  if constexpr (limbs_of(L) == L_ && G_ == 1) \
    if (sh.seg == S_) return launch_terms_t<L, S_>(sh, P, x, O, st);
  PE_SHAPES(PE_X)
#undef PE_X
  return hipErrorInvalidValue;
}

template <int L, int SEG, int CPL, int G>
hipError_t launch_adj_t(const EvalShape& sh, int P, const double* x, const double* v, int NG, int gsize,
                        double* part, double* g, hipStream_t st) {
  auto kern = adjoint_rows_kernel<L, SEG, CPL, G>;
  const size_t lds = G > 1 ? sh.lds : sh.lds1;
  hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  const int n = sh.view.n;
  hipLaunchKernelGGL(kern, dim3(unsigned(int64_t(P) * NG)), dim3(G * kSub), lds, st, sh.view, x,
                     int64_t(width_of(L)) * n, v, int64_t(width_of(L)) * sh.view.N, NG, gsize, part);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t tot = int64_t(P) * n;
  hipLaunchKernelGGL(adjoint_reduce_kernel<L>, dim3(unsigned((tot + 255) / 256)), dim3(256), 0, st, n, NG, P,
                     (const double*)part, g);
  return hipGetLastError();
}

// the adjoint runs with the evaluation plan's chunks per workgroup when that
// is 2 (at most 512 columns), else with one chunk at a time
template <int L, int SEG, int G>
hipError_t adj_lsg(const EvalShape& sh, int P, const double* x, const double* v, int NG, int gsize,
                   double* part, double* g, hipStream_t st) {
  if constexpr (G == 2) {
    switch (sh.cpl) {
      case 1: return launch_adj_t<L, SEG, 1, 2>(sh, P, x, v, NG, gsize, part, g, st);
      case 2: return launch_adj_t<L, SEG, 2, 2>(sh, P, x, v, NG, gsize, part, g, st);
    }
    return hipErrorInvalidValue;
  } else {
    switch (sh.cpl) {
      case 1: return launch_adj_t<L, SEG, 1, 1>(sh, P, x, v, NG, gsize, part, g, st);
      case 2: return launch_adj_t<L, SEG, 2, 1>(sh, P, x, v, NG, gsize, part, g, st);
      case 4: return launch_adj_t<L, SEG, 4, 1>(sh, P, x, v, NG, gsize, part, g, st);
      case 8: return launch_adj_t<L, SEG, 8, 1>(sh, P, x, v, NG, gsize, part, g, st);
    }
    return hipErrorInvalidValue;
  }
}

template <int L>
hipError_t launch_adjoint(const EvalShape& sh, int P, const double* x, const double* v, int NG, int gsize,
                          double* part, double* g, hipStream_t st) {
  const int G = sh.G == 2 ? 2 : 1;
#define PE_X(L_, S_, G_) \
  if constexpr (L == L_ && G_ <= 2) \
    if (sh.seg == S_ && G == G_) return adj_lsg<L, S_, G_>(sh, P, x, v, NG, gsize, part, g, st);
  PE_SHAPES(PE_X)
#undef PE_X
  return hipErrorInvalidValue;
}

// persistent grid: as many workgroups as fit on the device at once, at most
// one per item
template <typename Kern>
hipError_t persistent_grid(Kern kern, int threads, size_t lds, int64_t nitems, int64_t& grid) {
  int per_cu = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, threads, lds);
  if (e != hipSuccess) return e;
  int dev = 0, cus = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  grid = std::max<int64_t>(1, std::min<int64_t>(int64_t(std::max(per_cu, 1)) * cus, nitems));
  return hipSuccess;
}

template <int L, int SEG, int CPL, int G, int MODE>
hipError_t launch_batch_t(const BatchShape& K, int P, const double* x, const BatchOut& out, hipStream_t st) {
  auto kern = batch_rows_kernel<L, SEG, CPL, G, MODE>;
  hipError_t e = allow_lds(kern, K.lds);
  if (e != hipSuccess) return e;
  int64_t grid = 0;
  if ((e = persistent_grid(kern, G * kSub, K.lds, K.nitems, grid)) != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(G * kSub), K.lds, st, K.views, K.items, K.nitems, K.counter,
                     P, x, K.x_off, out);
  return hipGetLastError();
}

template <int L, int SEG, int VW, int MODE>
hipError_t launch_batch_small_t(const BatchShape& K, int P, const double* x, const BatchOut& out, hipStream_t st) {
  auto kern = batch_small_kernel<L, SEG, VW, MODE>;
  hipError_t e = allow_lds(kern, K.lds);
  if (e != hipSuccess) return e;
  int64_t grid = 0;
  if ((e = persistent_grid(kern, kSub, K.lds, K.nitems, grid)) != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(kSub), K.lds, st, K.views, K.items, K.nitems, K.counter, P, x,
                     K.x_off, out);
  return hipGetLastError();
}

template <int L, int SEG>
hipError_t batch_small_ls(const BatchShape& K, int P, const double* x, const BatchOut& out, int mode,
                          hipStream_t st) {
  switch (K.vw * 4 + mode) {
#define PE_CASE(VW, MODE) \
  case VW * 4 + MODE:     \
    return launch_batch_small_t<L, SEG, VW, MODE>(K, P, x, out, st);
    PE_CASE(32, MODE_EVAL)
    PE_CASE(32, MODE_FONLY)
    PE_CASE(64, MODE_EVAL)
    PE_CASE(64, MODE_FONLY)
    PE_CASE(128, MODE_EVAL)
    PE_CASE(128, MODE_FONLY)
    PE_CASE(256, MODE_EVAL)
    PE_CASE(256, MODE_FONLY)
#undef PE_CASE
  }
  return hipErrorInvalidValue;
}

template <int L, int SEG, int G>
hipError_t batch_lsg(const BatchShape& K, int P, const double* x, const BatchOut& out, int mode, hipStream_t st) {
  if constexpr (G == 1)
    if (K.vw > 0) return batch_small_ls<L, SEG>(K, P, x, out, mode, st);
  switch (K.cpl * 4 + mode) {
#define PE_CASE(CPL, MODE) \
  case CPL * 4 + MODE:     \
    return launch_batch_t<L, SEG, CPL, G, MODE>(K, P, x, out, st);
    PE_CASE(1, MODE_EVAL)
    PE_CASE(1, MODE_FONLY)
    PE_CASE(2, MODE_EVAL)
    PE_CASE(2, MODE_FONLY)
    PE_CASE(4, MODE_EVAL)
    PE_CASE(4, MODE_FONLY)
    PE_CASE(8, MODE_EVAL)
    PE_CASE(8, MODE_FONLY)
#undef PE_CASE
  }
  return hipErrorInvalidValue;
}

template <int L>
hipError_t launch_batch(const BatchShape& K, int P, const double* x, const BatchOut& out, int mode,
                        hipStream_t st) {
#define PE_X(L_, S_, G_) \
  if constexpr (L == L_ && G_ <= 2) \
    if (K.seg == S_ && K.G == G_) return batch_lsg<L, S_, G_>(K, P, x, out, mode, st);
  PE_SHAPES(PE_X)
#undef PE_X
  return hipErrorInvalidValue;
}

// Copies per workgroup and rows per copy: one row per workgroup of one copy
// while the rows are fewer than the chip can hold at once (about 1024
// workgroups), then copies of narrow systems side by side (256 threads) and up
// to four rows behind one table.  Rows of uneven cost stay apart, so that the
// longest start first.  A launch of at most 1024 rows leaves wavefront slots
// idle: a copy then has a wavefront for F besides those of the slices (DD, n =
// 128, 64 x 12: 8.9 us against 9.4 at P = 1; at P = 64 the wider copies would
// take 67 us against 48).  No sum depends on the number of wavefronts.
template <int L, int MODE, bool SMALL>
hipError_t launch_val_rows_t(ValView V, int P, const double* x, const OutView& O, hipStream_t st) {
  auto kern = val_rows_kernel<L, MODE, SMALL>;
  const size_t copy = val_copy_doubles<L>(V.n, V.tab + V.inv, V.max_mon, V.multi != 0);
  const int64_t rows = int64_t(P) * V.N;
  if (rows <= 1024)
    while ((1 << V.lgvw) < kValThreads && (1 << V.lgvw) < 64 * std::max(V.max_units, V.slices + 1)) ++V.lgvw;
  const int vw = 1 << V.lgvw;
  int copies = 1;
  if (!V.multi)
    while (vw * copies * 2 <= 256 && rows >= 2048 * copies && copy * copies * 2 * sizeof(double) <= 65536) copies *= 2;
  const int Rr = V.row_order ? 1 : int(std::max<int64_t>(1, std::min<int64_t>({4, rows / (1024 * copies), V.N})));
  const size_t lds = copy * copies * sizeof(double);
  hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  const int groups = (V.N + Rr - 1) / Rr;
  const int64_t items = int64_t(P) * groups;
  hipLaunchKernelGGL(kern, dim3(unsigned((items + copies - 1) / copies)), dim3(unsigned(vw * copies)), lds, st, V, O, x,
                     int64_t(width_of(L)) * V.n, P, copies, Rr, groups, int(copy));
  return hipGetLastError();
}

template <int L>
hipError_t launch_val_rows(const ValView& V, int P, const double* x, const OutView& O, int mode, hipStream_t st) {
  if (V.inv)
    return mode == MODE_EVAL ? launch_val_rows_t<L, MODE_EVAL, false>(V, P, x, O, st)
                             : launch_val_rows_t<L, MODE_FONLY, false>(V, P, x, O, st);
  return mode == MODE_EVAL ? launch_val_rows_t<L, MODE_EVAL, true>(V, P, x, O, st)
                           : launch_val_rows_t<L, MODE_FONLY, true>(V, P, x, O, st);
}

template <int L>
hipError_t launch_val_adjoint(const ValView& V, int P, const double* x, const double* v, int NG, int gsize, double* part,
                              double* g, hipStream_t st) {
  auto kern = V.inv ? val_adjoint_kernel<L, false> : val_adjoint_kernel<L, true>;
  const size_t lds = val_copy_doubles<L>(V.n, V.tab + V.inv, V.max_mon, true) * sizeof(double);
  hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(unsigned(int64_t(P) * NG)), dim3(unsigned(std::max(1 << V.lgvw, 256))), lds, st, V, x,
                     int64_t(width_of(L)) * V.n, v, int64_t(width_of(L)) * V.N, NG, gsize, part);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // grid.y is limited to 65535 points per launch
  for (int p0 = 0; p0 < P; p0 += 65535) {
    const int np = std::min(65535, P - p0);
    const size_t num = size_t(width_of(L)) * V.n;
    hipLaunchKernelGGL(val_adjoint_reduce_kernel<L>, dim3(unsigned((V.n + 63) / 64), unsigned(np)), dim3(256), 0, st, V.n,
                       NG, (const double*)part + p0 * size_t(NG) * num, g + p0 * num);
  }
  return hipGetLastError();
}

template <int L, int MODE, bool SMALL>
hipError_t launch_val_batch_t(const ValBatchShape& K, int P, const double* x, const BatchOut& out, hipStream_t st) {
  auto kern = val_batch_kernel<L, MODE, SMALL>;
  hipError_t e = allow_lds(kern, K.lds);
  if (e != hipSuccess) return e;
  int64_t grid = 0;
  if ((e = persistent_grid(kern, kValThreads, K.lds, K.nitems, grid)) != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(kValThreads), K.lds, st, K.views, K.items, K.nitems, K.counter, P,
                     x, K.x_off, out);
  return hipGetLastError();
}

template <int L>
hipError_t launch_val_batch(const ValBatchShape& K, int P, const double* x, const BatchOut& out, int mode,
                            hipStream_t st) {
  if (!K.small)
    return mode == MODE_EVAL ? launch_val_batch_t<L, MODE_EVAL, false>(K, P, x, out, st)
                             : launch_val_batch_t<L, MODE_FONLY, false>(K, P, x, out, st);
  return mode == MODE_EVAL ? launch_val_batch_t<L, MODE_EVAL, true>(K, P, x, out, st)
                           : launch_val_batch_t<L, MODE_FONLY, true>(K, P, x, out, st);
}

template <int L>
hipError_t launch_rhs_shift(double* W, int64_t w_pt, int64_t plane, int64_t ld, int N, int n, int P, const double* c,
                            double wF, double wc, hipStream_t st) {
  const int64_t tot = int64_t(P) * N;
  hipLaunchKernelGGL(rhs_shift_kernel<L>, dim3(unsigned((tot + 255) / 256)), dim3(256), 0, st, W, w_pt, plane, ld, N, n,
                     P, c, wF, wc);
  return hipGetLastError();
}

template <int L>
hipError_t launch_small_solve(const BlView& V, int slots, int Nm, hipStream_t st) {
  const size_t lds = small_lds<L>(Nm);
  const hipError_t e = allow_lds(small_solve_kernel<L>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(small_solve_kernel<L>, dim3(unsigned(slots)), dim3(64), lds, st, V);
  return hipGetLastError();
}

// One group of problems through all panels.  The launches only depend on the
// largest sizes of the group; workgroups of smaller problems end at once.
template <int L>
hipError_t launch_blockls(const BlView& V, int slots, int Nm, int nm, hipStream_t st) {
  using K = Bl<L>;
  const unsigned S = unsigned(slots);
  const int NC = (Nm + kBlRows - 1) / kBlRows;
  hipError_t e;
  const size_t chol_lds = bl_chol_lds<L>(), solve_lds = bl_solve_lds<L>(), gram_lds = bl_gram_lds<L>();
  if ((e = allow_lds(bl_gram_kernel<L>, gram_lds)) != hipSuccess) return e;
  if ((e = allow_lds(bl_chol_kernel<L>, chol_lds)) != hipSuccess) return e;
  if ((e = allow_lds(bl_solve_kernel<L>, solve_lds)) != hipSuccess) return e;
  hipLaunchKernelGGL(bl_init_kernel<L>, dim3(S), dim3(256), 0, st, V);
  hipLaunchKernelGGL(bl_copy_in_kernel<L>, dim3(unsigned(((nm + 1 + 63) / 64) * NC), unsigned(K::W), S), dim3(256), 0,
                     st, V);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // the update's workgroups hold 256 registers (quad double 512): two (one)
  // fit on a CU, and one round of them leaves no tail (double double, n =
  // 2048: 60 us a panel against 68 with three per CU and 74 with one)
  constexpr int kUpdate = limbs_of(L) == 4 ? 256 : 512;
  // (row splits: each problem has its own, and workgroups beyond them end)
  const unsigned gs = unsigned(bl_gram_splits(Nm)), ds = unsigned(std::min(NC, kBlMaxSplit));
  for (int panel = 0, k0 = 0; k0 < nm; ++panel, k0 += K::B) {
    const int cur = panel & 1;
    const int real_cols = (nm + 1 - k0) * K::CX;
    hipLaunchKernelGGL(bl_gram_kernel<L>, dim3(64 / (16 * K::NT), gs, S), dim3(256), gram_lds, st, V, panel, cur);
    hipLaunchKernelGGL(bl_chol_kernel<L>, dim3(S), dim3(BlChol<L>::T), chol_lds, st, V, panel, cur);
    hipLaunchKernelGGL(bl_solve_kernel<L>, dim3(unsigned(NC * kBlRows / (4 * bl_solve_rows<L>())), S), dim3(256), solve_lds, st, V,
                       panel, cur);
    const int dt = (real_cols + 16 * K::NT - 1) / (16 * K::NT);
    hipLaunchKernelGGL(bl_dot_kernel<L>, dim3(unsigned(dt), ds, S), dim3(256), 0, st, V, panel, cur);
    const int cpw = 256 / K::B;
    hipLaunchKernelGGL(bl_fin_kernel<L>, dim3(unsigned((nm + 1 - k0 + cpw - 1) / cpw), S), dim3(256), 0, st, V, panel,
                       cur);
    if (k0 + K::B < nm) {
      const int tiles = (real_cols + 15) / 16 - 4;
      const int groups = std::max(1, std::min(tiles, (kUpdate + NC * slots - 1) / (NC * slots)));
      const int per = (tiles + groups - 1) / groups;
      hipLaunchKernelGGL(bl_update_kernel<L>, dim3(unsigned(NC), unsigned((tiles + per - 1) / per), S), dim3(256), 0, st,
                         V, panel, cur, per);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  for (int stage = 0; stage * kBlBs < nm; ++stage) {
    hipLaunchKernelGGL(bl_bs_diag_kernel<L>, dim3(S), dim3(kBlBsThreads), 0, st, V, stage);
    const int rest = nm - (stage + 1) * kBlBs;
    if (rest > 0)
      hipLaunchKernelGGL(bl_bs_update_kernel<L>, dim3(unsigned((rest + 31) / 32), S), dim3(256), 0, st, V, stage);
  }
  hipLaunchKernelGGL(bl_finish_kernel<L>, dim3(S), dim3(256), 0, st, V);
  if (V.Rout || V.Qout) {
    const int64_t cnt = std::max(int64_t(Nm) * nm, int64_t(nm) * (nm + 1));
    hipLaunchKernelGGL(bl_export_kernel<L>, dim3(unsigned((cnt + 255) / 256), S), dim3(256), 0, st, V);
  }
  return hipGetLastError();
}

#endif  // PE_LAUNCH_DEFINITIONS

}  // namespace pe
