// lbvp_step_f64.hip -- the D2Q9 step kernels for FP64 storage (a translation
// unit per storage type, so that they compile in parallel).
#include "lbvp_step.h"

namespace lbvp {
template struct StepLaunch<double>;
}  // namespace lbvp
