// Level kernels of scale 2^2 (see ff_level_kernels.h).
#include "ff_level_kernels.h"

namespace ffh {

hipError_t launch_level_scale2(const LevelKArgs &a, const BatchStage *batch, int variant, hipStream_t stream) {
  return launch_n<2>(a, batch, variant, stream);
}

hipError_t launch_level_f32_scale2(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_nf32<2>(a, variant, stream);
}

hipError_t launch_level_r2_scale2(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_n_rx<2, 2>(a, variant, stream);
}

hipError_t launch_level_r4_scale2(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_n_rx<2, 4>(a, variant, stream);
}

hipError_t launch_level_wx_scale2(const LevelKArgs &a, int tile, hipStream_t stream) {
  return launch_wx<2>(a, tile, stream);
}

}  // namespace ffh
