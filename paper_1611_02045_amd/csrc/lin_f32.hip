// The linear CG's passes and queueing, FP32 fields.
#include "lin_solve.hpp"

namespace gpe {
template hipError_t lin_solve<float>(LinCtx<float>&, LinS&, int);
}  // namespace gpe
