#include <hip/hip_runtime.h>

#include "attention_f32.h"

namespace varuna {

template hipError_t launch_attention_fwd_f32<float>(const float*, float*, float*, int, int, int, int, int, const DropArgs&, hipStream_t);
template hipError_t launch_attention_bwd_f32<float>(const float*, const float*, const float*, const float*, float*, float*, int, int, int, int, int,
                                                  const DropArgs&, hipStream_t);

}  // namespace varuna
