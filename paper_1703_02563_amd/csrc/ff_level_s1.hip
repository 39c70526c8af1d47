// Level kernels of scale 2^1 (see ff_level_kernels.h).
#include "ff_level_kernels.h"

namespace ffh {

hipError_t launch_level_scale1(const LevelKArgs &a, const BatchStage *batch, int variant, hipStream_t stream) {
  return launch_n<1>(a, batch, variant, stream);
}

hipError_t launch_level_f32_scale1(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_nf32<1>(a, variant, stream);
}

hipError_t launch_level_r2_scale1(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_n_rx<1, 2>(a, variant, stream);
}

hipError_t launch_level_r4_scale1(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_n_rx<1, 4>(a, variant, stream);
}

hipError_t launch_level_wx_scale1(const LevelKArgs &a, int tile, hipStream_t stream) {
  return launch_wx<1>(a, tile, stream);
}

}  // namespace ffh
