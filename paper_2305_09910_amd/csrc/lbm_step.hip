// lbm_step.hip -- the AA step with streaming hints (see step_aa.h).
#include "step_aa.h"

namespace lbm {

template hipError_t step_aa<true>(const LatticeArgs &, const HrrArgs &, int, int, int, int, int, hipStream_t);

}  // namespace lbm
