#include "gemm_f32_launch.h"

namespace varuna {

template hipError_t launch_gemm_f32<float>(int, int, const float*, const float*, int64_t, int64_t, int64_t, const EpiArgs<float>&, hipStream_t);

}  // namespace varuna
