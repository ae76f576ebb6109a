// Decode step of several messages with one pass over the weights, RMSNorm.
#define MDI_STEP_WAVES 8
#define MDI_BATCH_LN false
#include "step_batch.h"
