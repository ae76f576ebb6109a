// Decode step of several messages with one pass over the weights, LayerNorm.
#define MDI_STEP_WAVES 8
#define MDI_BATCH_LN true
#include "step_batch.h"
