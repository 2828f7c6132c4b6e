// The stepping kernel's launches: FP64 fields, stepped domain, several steps.
#include "step_kernel.h"

namespace cryo {
CRYO_MULTI_LAUNCH(double, true)
}  // namespace cryo
