// The fp32 variants of the step kernel, as a translation unit of their own (see SPEC_STEP_PART).
#define SPEC_STEP_PART 5
#include "step_kernel.hip"
