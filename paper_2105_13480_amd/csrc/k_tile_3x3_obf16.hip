// conv_tile instantiations: 3x3, bf16 Out.
#include "tile_kernel.h"

namespace cnnlib {
CNN_TILE_LAUNCHER(launch_tile_3x3_obf16, CNN_TILE_3X3(CNN_CASET, 3200, CNN_BF16_OBF16))
}  // namespace cnnlib
