// Level kernels of scale 2^0 (see ff_level_kernels.h).
#include "ff_level_kernels.h"

namespace ffh {

hipError_t launch_level_scale0(const LevelKArgs &a, const BatchStage *batch, int variant, hipStream_t stream) {
  return launch_n<0>(a, batch, variant, stream);
}

hipError_t launch_level_f32_scale0(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_nf32<0>(a, variant, stream);
}

hipError_t launch_level_r2_scale0(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_n_rx<0, 2>(a, variant, stream);
}

hipError_t launch_level_r4_scale0(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_n_rx<0, 4>(a, variant, stream);
}

hipError_t launch_level_wx_scale0(const LevelKArgs &a, int tile, hipStream_t stream) {
  return launch_wx<0>(a, tile, stream);
}

}  // namespace ffh
