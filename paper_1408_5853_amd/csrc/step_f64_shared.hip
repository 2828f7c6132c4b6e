// The stepping kernel's launches: FP64 fields, rectangular domain, one round to a launch (axial fluxes shared).
#include "step_kernel.h"

namespace cryo {
CRYO_STEP_LAUNCH(double, false, true)
}  // namespace cryo
