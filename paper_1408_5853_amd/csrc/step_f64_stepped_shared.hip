// The stepping kernel's launches: FP64 fields, stepped domain, one round to a launch (axial fluxes shared).
#include "step_kernel.h"

namespace cryo {
CRYO_STEP_LAUNCH(double, true, true)
}  // namespace cryo
