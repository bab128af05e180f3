// lbvp_step_bf16.hip -- the D2Q9 step kernels for BF16 storage (a translation
// unit per storage type, so that they compile in parallel).
#include "lbvp_step.h"

namespace lbvp {
template struct StepLaunch<__bf16>;
}  // namespace lbvp
