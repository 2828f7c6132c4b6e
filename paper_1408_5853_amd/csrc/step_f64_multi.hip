// The stepping kernel's launches: FP64 fields, rectangular domain, several steps.
#include "step_kernel.h"

namespace cryo {
CRYO_MULTI_LAUNCH(double, false)
}  // namespace cryo
