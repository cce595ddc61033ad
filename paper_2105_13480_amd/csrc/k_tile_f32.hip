// conv_tile instantiations: fp32.
#include "tile_kernel.h"

namespace cnnlib {
CNN_TILE_LAUNCHER(launch_tile_f32, CNN_TILE_F32(CNN_CASET))
}  // namespace cnnlib
