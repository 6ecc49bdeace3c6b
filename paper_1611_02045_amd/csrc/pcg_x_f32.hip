// Launches of the PCG iteration's x passes, FP32 fields.
#include "pcg_passes.hpp"

namespace gpe {
GPE_PCG_X_PASSES(GPE_LAUNCH_DEFINE, float)
}  // namespace gpe
