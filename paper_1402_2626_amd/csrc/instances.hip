// Instances of the kernel launchers of launch.hpp for one level and one kind,
// chosen at compile time: PE_LEVEL (a level code: 1, 2 or 4, or 8 | 1, 2, 4
// for real numbers) and PE_KIND (0 rows, 1 adjoint,
// 2 batch, 3 homotopy right-hand side, 4 least squares, 5 evaluation through monomial
// values).
// The build compiles this file once per pair.
#define PE_LAUNCH_DEFINITIONS
#include "launch.hpp"

#if !defined(PE_LEVEL) || !defined(PE_KIND)
#error "compile with -DPE_LEVEL=<1|2|4> -DPE_KIND=<0..5>"
#endif

namespace pe {

#if PE_KIND == 0
template hipError_t launch_rows<PE_LEVEL>(const EvalShape&, int, const double*, const OutView&, int, hipStream_t);
template hipError_t launch_terms<PE_LEVEL>(const EvalShape&, int, const double*, const OutView&, hipStream_t);
#elif PE_KIND == 1
template hipError_t launch_adjoint<PE_LEVEL>(const EvalShape&, int, const double*, const double*, int, int, double*,
                                             double*, hipStream_t);
#elif PE_KIND == 2
template hipError_t launch_batch<PE_LEVEL>(const BatchShape&, int, const double*, const BatchOut&, int, hipStream_t);
#elif PE_KIND == 3
template hipError_t launch_rhs_shift<PE_LEVEL>(double*, int64_t, int64_t, int64_t, int, int, int, const double*, double,
                                               double, hipStream_t);
#elif PE_KIND == 4
template hipError_t launch_blockls<PE_LEVEL>(const BlView&, int, int, int, hipStream_t);
template hipError_t launch_small_solve<PE_LEVEL>(const BlView&, int, int, hipStream_t);
#elif PE_KIND == 5
template hipError_t launch_val_rows<PE_LEVEL>(const ValView&, int, const double*, const OutView&, int, hipStream_t);
#if PE_LEVEL < 8
template hipError_t launch_val_adjoint<PE_LEVEL>(const ValView&, int, const double*, const double*, int, int, double*,
                                                 double*, hipStream_t);
template hipError_t launch_val_batch<PE_LEVEL>(const ValBatchShape&, int, const double*, const BatchOut&, int,
                                               hipStream_t);
#endif
#endif

}  // namespace pe
