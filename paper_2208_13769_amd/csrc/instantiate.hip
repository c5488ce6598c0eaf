// instantiate.hip -- the kernels and launch helpers of one precision.
//
// Built once per precision with LBM_PREC naming the precision traits
// (PrecF64, PrecF32, PrecF32U64, PrecF16 or PrecBF16), so the five
// precisions' step kernels compile in parallel; the runtime sources only
// declare these instantiations.
#include "host_common.hpp"
#include "window_kernel.hpp"

namespace lbm {

template struct Kernels<LBM_PREC>;
template hipError_t window_step<LBM_PREC>(const GenParams &, WinGrid, int, int, hipStream_t);

}  // namespace lbm
