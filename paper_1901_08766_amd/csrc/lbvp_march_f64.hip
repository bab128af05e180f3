// lbvp_march_f64.hip -- the two-step D2Q9 kernels for FP64 storage.
#include "lbvp_march.h"

namespace lbvp {
template struct MarchLaunch<double>;
}  // namespace lbvp
