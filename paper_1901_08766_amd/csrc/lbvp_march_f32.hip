// lbvp_march_f32.hip -- the two-step D2Q9 kernels for FP32 storage.
#include "lbvp_march.h"

namespace lbvp {
template struct MarchLaunch<float>;
}  // namespace lbvp
