// The persistent decode step for workgroups of 4 wavefronts (two workgroups per compute unit: launches that carry several messages), fp32 storage.
#define MDI_STEP_WAVES 4
#define MDI_STEP_TYPE float
#define MDI_STEP_TYPE_NAME _f32
#include "step_kernel.h"
