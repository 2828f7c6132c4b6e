// The stepping kernel's launches: FP32 pair fields, rectangular domain, one round to a launch (axial fluxes shared).
#include "step_kernel.h"

namespace cryo {
CRYO_STEP_LAUNCH(float, false, true)
}  // namespace cryo
