// The stepping kernel's launches: FP32 pair fields, stepped domain, several steps.
#include "step_kernel.h"

namespace cryo {
CRYO_MULTI_LAUNCH(float, true)
}  // namespace cryo
