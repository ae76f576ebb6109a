// The output layers: for one sample (k_logits), for several with one pass over the vocabulary matrix (k_logits_batch).
#define MDI_STEP_WAVES 8
#include "head_one.h"
#include "step_mfma.h"
#include "head_batch.h"
