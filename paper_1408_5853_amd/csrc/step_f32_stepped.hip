// The stepping kernel's launches: FP32 pair fields, stepped domain, line blocks of several rounds.
#include "step_kernel.h"

namespace cryo {
CRYO_STEP_LAUNCH(float, true, false)
}  // namespace cryo
