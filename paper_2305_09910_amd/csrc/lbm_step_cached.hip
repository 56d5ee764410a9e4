// lbm_step_cached.hip -- the AA step without streaming hints (see step_aa.h).
#include "step_aa.h"

namespace lbm {

template hipError_t step_aa<false>(const LatticeArgs &, const HrrArgs &, int, int, int, int, int, hipStream_t);

}  // namespace lbm
