// The stepping kernel's launches: FP64 fields, rectangular domain, line blocks of several rounds.
#include "step_kernel.h"

namespace cryo {
CRYO_STEP_LAUNCH(double, false, false)
}  // namespace cryo
