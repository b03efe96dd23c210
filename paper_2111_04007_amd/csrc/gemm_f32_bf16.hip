#include "gemm_f32_launch.h"

namespace varuna {

template hipError_t launch_gemm_f32<bf16>(int, int, const bf16*, const bf16*, int64_t, int64_t, int64_t, const EpiArgs<bf16>&, hipStream_t);

}  // namespace varuna
