// Level kernels of scale 2^4 (see ff_level_kernels.h).
#include "ff_level_kernels.h"

namespace ffh {

hipError_t launch_level_scale4(const LevelKArgs &a, const BatchStage *batch, int variant, hipStream_t stream) {
  return launch_n<4>(a, batch, variant, stream);
}

hipError_t launch_level_f32_scale4(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_nf32<4>(a, variant, stream);
}

hipError_t launch_level_r2_scale4(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_n_rx<4, 2>(a, variant, stream);
}

hipError_t launch_level_r4_scale4(const LevelKArgs &a, int variant, hipStream_t stream) {
  return launch_n_rx<4, 4>(a, variant, stream);
}

hipError_t launch_level_wx_scale4(const LevelKArgs &a, int tile, hipStream_t stream) {
  return launch_wx<4>(a, tile, stream);
}

}  // namespace ffh
