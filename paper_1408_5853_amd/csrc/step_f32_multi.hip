// The stepping kernel's launches: FP32 pair fields, rectangular domain, several steps.
#include "step_kernel.h"

namespace cryo {
CRYO_MULTI_LAUNCH(float, false)
}  // namespace cryo
