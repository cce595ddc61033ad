// conv_tile instantiations: 3x3, fp32 Out.
#include "tile_kernel.h"

namespace cnnlib {
CNN_TILE_LAUNCHER(launch_tile_3x3_bf16, CNN_TILE_3X3(CNN_CASET, 3100, CNN_BF16))
}  // namespace cnnlib
