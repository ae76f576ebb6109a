// Decode step of several messages with one pass over the weights, RMSNorm, workgroups of 4 wavefronts.
#define MDI_STEP_WAVES 4
#define MDI_BATCH_LN false
#include "step_batch.h"
