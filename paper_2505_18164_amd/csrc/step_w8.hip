// The persistent decode step for workgroups of 8 wavefronts (one workgroup per compute unit: launches that carry one message), bf16 storage.
#define MDI_STEP_WAVES 8
#define MDI_STEP_TYPE bf16_t
#define MDI_STEP_TYPE_NAME _bf16
#include "step_kernel.h"
