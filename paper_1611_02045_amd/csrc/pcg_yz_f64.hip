// Launches of the PCG iteration's strided (y, z) passes, FP64 fields.
#include "pcg_passes.hpp"

namespace gpe {
GPE_PCG_YZ_PASSES(GPE_LAUNCH_DEFINE, double)
}  // namespace gpe
