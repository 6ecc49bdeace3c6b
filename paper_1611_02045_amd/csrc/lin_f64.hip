// The linear CG's passes and queueing, FP64 fields.
#include "lin_solve.hpp"

namespace gpe {
template hipError_t lin_solve<double>(LinCtx<double>&, LinS&, int);
}  // namespace gpe
