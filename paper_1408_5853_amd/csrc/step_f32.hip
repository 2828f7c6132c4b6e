// The stepping kernel's launches: FP32 pair fields, rectangular domain, line blocks of several rounds.
#include "step_kernel.h"

namespace cryo {
CRYO_STEP_LAUNCH(float, false, false)
}  // namespace cryo
