// The persistent decode step for workgroups of 8 wavefronts (one workgroup per compute unit: launches that carry one message), fp32 storage.
#define MDI_STEP_WAVES 8
#define MDI_STEP_TYPE float
#define MDI_STEP_TYPE_NAME _f32
#include "step_kernel.h"
