// The persistent decode step for workgroups of 4 wavefronts (two workgroups per compute unit: launches that carry several messages), bf16 storage.
#define MDI_STEP_WAVES 4
#define MDI_STEP_TYPE bf16_t
#define MDI_STEP_TYPE_NAME _bf16
#include "step_kernel.h"
