// Launches of the attention kernels, a translation unit of their own.
#include <hip/hip_runtime.h>

#include "attention.h"
#include "attention_mfma.h"
#include "attention_simple.h"
