// Forward kernel instances: plain passes by pairs of wavefronts (rd_pair.h).
#include "rd_fwd_kernel.h"
#include "rd_pair.h"

namespace rd {
StreamFn pair_fn() { return &pair_step_kernel<ModelFHN, kPairCpl, kPairDepth>; }
}  // namespace rd
