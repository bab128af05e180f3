// lbvp_step_f16.hip -- the D2Q9 step kernels for FP16 storage (a translation
// unit per storage type, so that they compile in parallel).
#include "lbvp_step.h"

namespace lbvp {
template struct StepLaunch<_Float16>;
}  // namespace lbvp
