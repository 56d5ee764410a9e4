// lbm_et.hip -- the Esoteric Twist step with streaming hints (see step_et.h), and
// the choice between it and lbm_et_cached.hip.
#include "step_et.h"

namespace lbm {

template hipError_t step_et<true>(const LatticeArgs &, int, int, int, int, int, hipStream_t);
extern template hipError_t step_et<false>(const LatticeArgs &, int, int, int, int, int, hipStream_t);

hipError_t launch_step_et(const LatticeArgs &a, int q, int st, int cl, int coll, int odd, hipStream_t s)
{
    return (odd & SC_CACHED) && step_without_hints(a, q, st, cl, coll)
               ? step_et<false>(a, q, st, cl, coll, odd, s)
               : step_et<true>(a, q, st, cl, coll, odd, s);
}

}  // namespace lbm
