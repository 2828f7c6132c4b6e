// The stepping kernel's launches: FP32 pair fields, stepped domain, one round to a launch (axial fluxes shared).
#include "step_kernel.h"

namespace cryo {
CRYO_STEP_LAUNCH(float, true, true)
}  // namespace cryo
