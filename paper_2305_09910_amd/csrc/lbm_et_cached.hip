// lbm_et_cached.hip -- the Esoteric Twist step without streaming hints (see step_et.h).
#include "step_et.h"

namespace lbm {

template hipError_t step_et<false>(const LatticeArgs &, int, int, int, int, int, hipStream_t);

}  // namespace lbm
